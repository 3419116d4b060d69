"""The policy kernel of few ports (16,384 rows and more: levels of up to 8 ports,
logits of up to 4) against the kernel of blocks, which fewer rows take: the same
levels and logits bit for bit."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

ROWS = 16384


@pytest.fixture(scope="module")
def cxm():
    from paper_2507_01522_amd import cx
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return cx


@pytest.mark.parametrize("hidden", [32, 64, 96, 128, 224, 256])
@pytest.mark.parametrize("ports,n_levels", [(1, 10), (2, 3), (3, 11), (4, 10), (5, 7), (6, 1), (7, 10), (8, 11), (9, 10)])
def test_equals_blocks(cxm, ports, n_levels, hidden):
    spec = W.single_transformer(ports, 9.0 * ports).replace(n_levels=n_levels)
    env = cxm.Env(spec, n_envs=1, seed=73)
    env.set_policy(hidden, W.policy_weights(ports, hidden=hidden, n_levels=n_levels, std=0.3, seed=79))
    n = ROWS + 37
    obs = torch.rand((n, spec.obs_dim), generator=torch.Generator().manual_seed(83)).cuda()
    levels, logits = env.policy_sample(obs, 11), env.policy_logits(obs)
    few = env.policy_sample(obs[:ROWS], 11), env.policy_logits(obs[:ROWS])   # no ragged wave
    for k in (1, 16, 1000, ROWS - 1):
        assert torch.equal(levels[:k], env.policy_sample(obs[:k], 11)), k
        assert torch.equal(logits[:k], env.policy_logits(obs[:k])), k
        assert torch.equal(levels[:k], few[0][:k]) and torch.equal(logits[:k], few[1][:k]), k
    # the last rows, among others' (an infinite feature there does not reach them)
    tail = obs[-64:].clone()
    tail[:32] = float("inf")
    assert torch.equal(logits[-32:], env.policy_logits(tail)[32:])
    odd = torch.zeros(n * ports + 1, dtype=torch.uint8, device="cuda")[1:].view(n, ports)
    assert torch.equal(env.policy_sample(obs, 11, odd), levels)


def test_rollout_of_few_ports(cxm):
    """Two kernels per step on both sides of the size: the first stations of a large
    context take the same levels as a small one's, from the same draws."""
    spec = W.single_transformer(3, 30.0).replace(alpha_sat=0.2)
    weights = W.policy_weights(3, hidden=96, std=0.3, seed=89)
    a, b = cxm.Env(spec, n_envs=ROWS + 5, seed=97), cxm.Env(spec, n_envs=33, seed=97)
    for e in (a, b):
        e.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)
        e.set_policy(96, weights)
    x, y = a.rollout(9, cxm.ACT_POLICY), b.rollout(9, cxm.ACT_POLICY)
    for k in x:
        assert torch.equal(x[k].reshape(9, -1)[:, :y[k].reshape(9, -1).shape[1]], y[k].reshape(9, -1)), k
