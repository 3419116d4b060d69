"""Classes with padding slots at four slots per lane: lanes whose ports are adjacent
store their observations at once, the others one by one.  Every step's records
against the observation kernel's, which reads the state port by port."""
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


def spec_of(ports, kind):
    s = W.fanout4_tree(ports, 2 if ports < 64 else 3)
    if kind == "v2g":
        return s.replace(v2g=1, battery_kwh=80.0, battery_kw=40.0)
    if kind == "users":
        return s.replace(charge_sensitive_share=0.5, alpha_sat1=0.2, beta_sat1=0.3)
    return s


@pytest.mark.parametrize("kind", ["general", "v2g", "users"])
@pytest.mark.parametrize("ports", [13, 15, 29, 31, 61, 121, 200, 255])
def test_observations(cxm, ports, kind):
    spec = spec_of(ports, kind)
    a, b = cxm.Env(spec, n_envs=21, seed=61), cxm.Env(spec, n_envs=21, seed=61)
    for e in (a, b):
        slots = e.class_info(0).slots
        assert slots > ports and slots // 4 <= 64
        e.set_packing(0, slots // 4, 2)
        e.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)   # noon: cars at the ports
    x = a.rollout(9, cxm.ACT_RANDOM)
    for t in range(9):
        b.rollout(1, cxm.ACT_RANDOM, cxm.OUT_REWARD)
        assert torch.equal(x["obs"][t].reshape(-1), b.observe().reshape(-1)), t
