"""The kernels whose registers spill to scratch memory (extended classes of 64 slots
at 32 lanes without observation records, of 256 slots with them, and the fused policy
rollout of more than 8,192 general 16-slot stations), against kernels that do the
same work without scratch: records and state bit for bit the same."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cxm():
    from paper_2507_01522_amd import cx
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return cx


def envs(cxm, spec, n, lanes=None):
    pair = [cxm.Env(spec, n_envs=n, seed=53) for _ in range(2)]
    for e in pair:
        if lanes:
            e.set_packing(0, lanes, 2)
        e.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)   # noon: cars at the ports
    return pair


def test_v2g_64_slots_without_observations(cxm):
    spec = W.fanout4_tree(64, 3).replace(v2g=1, battery_kwh=200.0, battery_kw=50.0, alpha_degrad_cars=0.03)
    a, b = envs(cxm, spec, 37, lanes=32)
    x, y = a.rollout(40, cxm.ACT_RANDOM), b.rollout(40, cxm.ACT_RANDOM, cxm.OUT_ACT_REWARD)
    for k in y:
        assert torch.equal(x[k], y[k]), k
    assert a.get_state() == b.get_state()


def test_v2g_256_slots(cxm):
    spec = W.fanout4_tree(256, 4).replace(v2g=1, battery_kwh=200.0, battery_kw=50.0, alpha_degrad_cars=0.03)
    a, b = envs(cxm, spec, 9, lanes=64)
    x = a.rollout(40, cxm.ACT_RANDOM)
    for t in range(40):
        y = b.step(cxm.ACT_RANDOM)
        for k in y:
            assert torch.equal(x[k][t].reshape(-1), y[k].reshape(-1)), (k, t)
    assert a.get_state() == b.get_state()


@pytest.mark.parametrize("hidden", [64, 128, 256])
def test_fused_policy_of_general_16_slot_stations(cxm, hidden):
    spec = W.two_charger_types().replace(alpha_sat=0.3)
    a, b = envs(cxm, spec, 8193 + 40)
    for e in (a, b):
        e.set_policy(hidden, W.policy_weights(16, hidden=hidden, std=0.2, seed=41))
    x, y = a.rollout(12, cxm.ACT_POLICY), b.rollout_policy_noalloc(12)
    for k in x:
        assert torch.equal(x[k], y[k]), k
    assert a.get_state() == b.get_state()
