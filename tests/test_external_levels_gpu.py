"""Levels given by the caller, at every byte address and in every packing: clamped
to the class's, recorded, and the same rewards, observations and state as from an
aligned buffer with one slot per lane."""
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


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("ports", [16, 32, 128])
def test_every_address_and_packing(cxm, ports, offset):
    spec = W.fanout4_tree(ports, 2).replace(n_levels=7)
    n, T = 19, 11
    raw = torch.randint(0, 256, (T * n * ports + 4,), dtype=torch.uint8, generator=torch.Generator().manual_seed(3)).cuda()
    levels = raw[offset:offset + T * n * ports].view(T, n * ports)
    ref = None
    for per_lane in (1, 2, 4):
        if ports // per_lane > 64:
            continue
        env = cxm.Env(spec, n_envs=n, seed=71)
        env.set_packing(0, ports // per_lane, 4)
        env.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)
        given = levels.clone() if ref is None else levels
        x = env.rollout(T, cxm.ACT_EXTERNAL, actions=given)
        y = env.step(cxm.ACT_EXTERNAL, actions=given[3])
        assert torch.equal(x["actions"], levels.clamp(max=7))
        got = [x, y, env.get_state()]
        if ref is None:
            ref = got
            continue
        for a, b in zip(ref[:2], got[:2]):
            for k in a:
                assert torch.equal(a[k], b[k]), (per_lane, k)
        assert ref[2] == got[2]
