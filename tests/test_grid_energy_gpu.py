"""The rounding of the station sums of classes whose ports differ in efficiency
(general and extended kinds): the grid energy of a step, bit for bit, from the
powers that its observation records.

With one slot per lane every product of a power and its slot's factor is
rounded, and adjacent slots are added pair by pair.  With P = 2 or 4 slots per
lane the P slots L = S / P apart are accumulated in slot order by fused
multiply-adds, and the L sums are then added pair by pair.  The station below
makes the reward the negated grid energy exactly (one hour a step, unit prices,
nothing sold) and a port's observed power its power (1 kW ports), so there is no
tolerance.
"""
import numpy as np
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


def fma32(a, b, c):
    """a b + c of FP32 arrays, rounded once to FP32 (the product is exact in FP64,
    its sum with c rounded to odd there)."""
    p, c = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    even = (s.view(np.int64) & 1) == 0
    s = np.where((err != 0) & even, np.nextafter(s, np.copysign(np.inf, err)), s)
    return s.astype(np.float32)


def pairwise(v):
    while v.shape[-1] > 1:
        v = v[..., 0::2] + v[..., 1::2]
    return v[..., 0]


def grid_energy(p, factor, per_lane):
    """FP32 sum over the last axis (slots) of p * factor, in the kernels' order."""
    if per_lane == 1:
        return pairwise(p * factor)
    q = p.reshape(*p.shape[:-1], per_lane, -1)
    f = factor.reshape(q.shape)
    acc = q[..., 0, :] * f[..., 0, :]
    for k in range(1, per_lane):
        acc = fma32(q[..., k, :], f[..., k, :], acc)
    return pairwise(acc)


KINDS = {"general": {}, "v2g": dict(v2g=1), "users": dict(charge_sensitive_share=0.5)}


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("ports,lanes", [(8, 4), (16, 16), (16, 8), (16, 4), (32, 16), (32, 8), (64, 64), (64, 32),
                                         (64, 16), (128, 64), (128, 32), (256, 64)])
def test_grid_energy_bits(cxm, kind, ports, lanes):
    eta = np.random.default_rng(ports).uniform(0.85, 1.0, ports)
    spec = W.fanout4_tree(ports, 2).replace(
        port_pmax_kw=[1.0] * ports, node_limit_kw=[0.45 * ports] + [2.5] * (ports // 4), port_eta=list(eta),
        dt_hours=1.0, tau=0.01, p_sell=0.0, p_sell_grid=1.0, price_base=1.0, price_amp=0.0, price_sigma=0.0,
        cap_lo=1000.0, cap_hi=2000.0, tgt_lo=1.0, tgt_hi=1.0, dwell_mu=8.0, dwell_sigma=0.01, dwell_max=4096,
        steps_per_episode=2000, arrival_rate=np.full(2000, 8.0), arrival_peak=0.0, **KINDS[kind])
    n, T = 9, 12
    env = cxm.Env(spec, n_envs=n, seed=53)
    assert env.class_info(0).slots == ports   # slot = port
    env.set_packing(0, lanes, 2)
    env.rollout(100, cxm.ACT_RANDOM, cxm.OUT_REWARD)
    out = env.rollout(T, cxm.ACT_RANDOM)
    obs = out["obs"].cpu().numpy().reshape(T, n, spec.obs_dim)
    p = np.ascontiguousarray(obs[:, :, 5 * ports:6 * ports])
    assert (obs[:, :, :ports] == 1.0).mean() > 0.95
    up, down = (1.0 / eta).astype(np.float32), eta.astype(np.float32)
    factor = np.where(p > 0, up, down) if kind == "v2g" else np.broadcast_to(up, p.shape)
    want = -grid_energy(p, factor, ports // lanes)
    got = out["reward"].cpu().numpy().reshape(T, n)
    assert np.array_equal(got, want), np.abs(got - want).max()
