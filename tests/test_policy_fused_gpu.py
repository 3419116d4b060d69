"""The fused policy rollout of classes that are not SIMPLE (padding slots, the
dense layout, uneven port maxima, efficiencies and limits) and of every hidden
size its kernels round up to: records and state bit for bit those of the two
kernels per step (cx_rollout_policy_noalloc on an equal context).  The
standalone policy kernel around its blocks of 32 rows and groups of 16 ports:
logits within FP32 accumulation and one BF16 rounding of every hidden unit of an
FP64 product, logits and levels of a row independent of how many rows the call
has."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import parity as PY

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cxm():
    from paper_2507_01522_amd import cx
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return cx


def uneven_eta(n):
    s = W.fanout4_tree(n, 2)
    return s.replace(port_eta=[0.9 + 0.1 * (i % 3) / 3 for i in range(n)], alpha_sat=0.2, alpha_declined=0.1)


SPECS = {
    "types10x6": lambda: W.two_charger_types(),                   # dense layout, 16 slots
    "types3x2": lambda: W.two_charger_types(3, 2).replace(alpha_sat=0.3),   # 5 ports, odd record lengths
    "fan7": lambda: uneven_eta(7),                                # padding in 8 slots
    "fan12": lambda: uneven_eta(12),                              # padding in 16 slots
    "fan31": lambda: uneven_eta(31).replace(n_levels=4),          # 32 slots, 5 levels per port
    "random5": lambda: W.random_station(5, max_ports=24).replace(n_levels=10),
}


@pytest.mark.parametrize("hidden", [32, 128, 256])
@pytest.mark.parametrize("name", sorted(SPECS))
def test_general_fused_equals_two_kernels(cxm, name, hidden):
    spec = SPECS[name]()
    weights = W.policy_weights(spec.n_ports, hidden=hidden, n_levels=spec.n_levels, std=0.2, seed=17)
    for n, T, out_mode in ((67, 30, cxm.OUT_FULL), (33, 25, cxm.OUT_ACT_REWARD)):
        print(f"fused {name} hidden {hidden}: {n} envs x {T} steps", flush=True)
        a, b = cxm.Env(spec, n_envs=n, seed=23), cxm.Env(spec, n_envs=n, seed=23)
        for e in (a, b):
            e.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)   # noon: cars at the ports
            e.set_policy(hidden, weights)
        for _ in range(2):   # the second continues from the state and clock of the first
            x = PY.to_np(a.rollout(T, cxm.ACT_POLICY, out_mode))
            y = PY.to_np(b.rollout_policy_noalloc(T, out_mode))
            assert set(x) == set(y)
            for k in x:
                assert np.array_equal(x[k], y[k]), k
            assert a.get_state() == b.get_state()


@pytest.mark.parametrize("ports,hidden", [(8, 64), (16, 96), (32, 256), (41, 224), (5, 32)])
def test_policy_kernel_sizes(cxm, ports, hidden):
    """Blocks of 32 observations; logits leave in groups of 16 ports."""
    spec = W.single_transformer(ports, 5.0 * ports)
    env = cxm.Env(spec, n_envs=1, seed=29)
    weights = W.policy_weights(ports, hidden=hidden, std=0.1, seed=31)
    env.set_policy(hidden, weights)
    big = 4096 + 33
    obs = torch.rand((big, spec.obs_dim), device="cuda", generator=torch.Generator("cuda").manual_seed(37))
    z, k = env.policy_logits(obs), env.policy_sample(obs, 11)
    f64 = [torch.tensor((np.asarray(w, np.uint32) << 16).view(np.float32), device="cuda").double() for w in weights]
    h = torch.tanh(obs[:4096].to(torch.bfloat16).double() @ f64[0] + f64[1])
    ref = h.to(torch.bfloat16).double() @ f64[2] + f64[3]
    tol = (2.0 ** -8 * h.abs()) @ f64[2].abs() + 1e-5     # a BF16 rounding flip of every hidden unit
    assert torch.all((z[:4096].double() - ref).abs() <= tol)
    for n in (1, 15, 33, 64, 1000):
        assert torch.equal(env.policy_logits(obs[:n]), z[:n]), n
        assert torch.equal(env.policy_sample(obs[:n], 11), k[:n]), n
    odd = torch.zeros(1000 * ports + 1, dtype=torch.uint8, device="cuda")[1:].view(1000, ports)
    assert torch.equal(env.policy_sample(obs[:1000], 11, odd), k[:1000])   # levels at an odd address


def big_stay():
    # 32 slots with a stay table of 2048 entries: no LDS for the held layout
    return W.policy_station().replace(dwell_max=2048)


def long_day():
    # more steps a day than the LDS day tables hold
    return W.scale_station().replace(steps_per_episode=600)


@pytest.mark.parametrize("make,n", [(W.scale_station, 1), (W.scale_station, 17), (W.scale_station, 4096),
                                    (W.scale_station, 4097), (W.scale_station, 8192), (W.scale_station, 8193),
                                    (W.two_charger_types, 4097), (W.two_charger_types, 8193),
                                    (W.policy_station, 33), (W.policy_station, 8193),
                                    (big_stay, 67), (long_day, 67)])
@pytest.mark.parametrize("hidden", [64, 160])
def test_launch_sizes_equal_two_kernels(cxm, make, n, hidden):
    """Around the sizes where a rollout's blocks change (16 lanes a station and
    held weights while every block has a CU of its own: 256 blocks of 16 or 32
    stations), with the day's tables in LDS (T >= 32) and without: records and state
    bit for bit those of the two kernels per step."""
    spec = make()
    weights = W.policy_weights(spec.n_ports, hidden=hidden, n_levels=spec.n_levels, std=0.2, seed=41)
    print(f"fused {spec.name} {n} envs hidden {hidden}", flush=True)
    a, b = cxm.Env(spec, n_envs=n, seed=43), cxm.Env(spec, n_envs=n, seed=43)
    for e in (a, b):
        e.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)
        e.set_policy(hidden, weights)
    for T, out_mode in ((33, cxm.OUT_FULL), (5, cxm.OUT_ACT_REWARD), (1, cxm.OUT_FULL)):
        x = PY.to_np(a.rollout(T, cxm.ACT_POLICY, out_mode))
        y = PY.to_np(b.rollout_policy_noalloc(T, out_mode))
        for k in x:
            assert np.array_equal(x[k], y[k]), (T, k)
        assert a.get_state() == b.get_state()
