"""SIMPLE classes whose deepest nodes own fewer ports than a lane holds: a slot's
factor is the product of its nodes' from the deepest up in every packing, so the
records and the state are bit for bit those of one slot per lane, and the fused
policy rollout's (four slots per lane) those of the two kernels per step."""
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


def tree(n, sizes, factor=0.4):
    """n ports under nodes of sizes[0], sizes[1], ... ports (deepest first) and a
    root, every node at `factor` of what its children may draw."""
    parent, limit, level = [-1], [0.0], {}
    for i in reversed(range(len(sizes))):
        for k in range(n // sizes[i]):
            level[i, k] = len(parent)
            parent.append(level[i + 1, k * sizes[i] // sizes[i + 1]] if i + 1 < len(sizes) else 0)
            limit.append(sizes[i] * W.PMAX_KW * factor ** (i + 1))
    limit[0] = n * W.PMAX_KW * factor ** (len(sizes) + 1)
    return W.single_transformer(n).replace(node_parent=parent, node_limit_kw=limit, node_eta=[1.0] * len(parent),
                                           port_parent=[level[0, p // sizes[0]] for p in range(n)], alpha_sat=0.2)


TREES = [(16, (1, 4)), (16, (2, 8)), (32, (1, 2)), (32, (2, 8)), (32, (2, 4, 16)), (64, (1, 2, 8)), (128, (2, 16))]


@pytest.mark.parametrize("n,sizes", TREES)
def test_records_in_every_packing(cxm, n, sizes):
    spec = tree(n, sizes)
    outs = []
    for per_lane in (1, 2, 4):
        if not 4 <= n // per_lane <= 64:
            continue
        env = cxm.Env(spec, n_envs=37, seed=31)
        env.set_packing(0, n // per_lane, 2)
        x = env.rollout(160, cxm.ACT_MAX)
        outs.append((x, env.get_state()))
    assert len(outs) >= 2
    for x, state in outs[1:]:
        for k in x:
            assert torch.equal(x[k], outs[0][0][k]), k
        assert state == outs[0][1]


@pytest.mark.parametrize("n,sizes", [t for t in TREES if t[0] <= 32])
def test_fused_policy_rollout(cxm, n, sizes):
    spec = tree(n, sizes)
    weights = W.policy_weights(n, hidden=64, std=0.2, seed=19)
    a, b = cxm.Env(spec, n_envs=67, seed=29), cxm.Env(spec, n_envs=67, seed=29)
    for e in (a, b):
        e.rollout(120, cxm.ACT_MAX, cxm.OUT_REWARD)
        e.set_policy(64, weights)
    x, y = a.rollout(60, cxm.ACT_POLICY), b.rollout_policy_noalloc(60)
    for k in x:
        assert torch.equal(x[k], y[k]), k
    assert a.get_state() == b.get_state()
