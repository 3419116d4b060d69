"""The policy kernel on inputs at the ends of their range, for sizes that are padded
in the kernel (hidden units to 64, 128 or 256, levels to 12): the padding changes
nothing."""
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


def f64(bits):
    return torch.from_numpy((bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64))


@pytest.mark.parametrize("ports", [16, 32])
@pytest.mark.parametrize("hidden", [32, 64, 96, 160, 256])
def test_infinite_observation(cxm, hidden, ports):
    """One infinite feature a row (or one that BF16 rounds to infinity): every hidden
    unit is +-1 and the logits finite.  Tolerance: 1.6e-5 of the absolute products, for
    their FP32 sum of up to 256 (256 x 2^-24 = 1.53e-5 at worst)."""
    spec = W.fanout4_tree(ports, 2)
    weights = W.policy_weights(ports, hidden=hidden, std=0.2, seed=7)
    env = cxm.Env(spec, n_envs=1, seed=3)
    env.set_policy(hidden, weights)
    rng = np.random.default_rng(11)
    n = 77
    obs = torch.from_numpy(rng.uniform(-1, 1, (n, spec.obs_dim)).astype(np.float32))
    col = torch.from_numpy(rng.integers(0, spec.obs_dim, n))
    obs[torch.arange(n), col] = torch.tensor([np.inf, -np.inf, 3.4e38], dtype=torch.float32).repeat(n)[:n]
    w1, b1, w2, b2 = (f64(w) for w in weights)
    w1, w2 = w1.reshape(spec.obs_dim, hidden), w2.reshape(hidden, -1)
    assert (w1 != 0).all()
    h = torch.tanh(obs.bfloat16().double() @ w1 + b1)
    assert (h.abs() == 1).all()
    err = (env.policy_logits(obs.cuda()).cpu().double() - (h @ w2 + b2)).abs()
    assert (err <= 1.6e-5 * (h.abs() @ w2.abs() + b2.abs())).all()


@pytest.mark.parametrize("bias", ["lowest", "-inf"])
@pytest.mark.parametrize("n_levels", [1, 3, 6, 10, 11])
def test_masked_port(cxm, n_levels, bias):
    """A port whose every level has the lowest finite bias: all of its weights
    overflow alike, and the draw takes the last level, as without padding levels (11
    levels and 0).  With biases of -inf no weight is a number, and it takes level 0.
    The other ports draw what they draw without the mask."""
    spec = W.fanout4_tree(16, 2).replace(n_levels=n_levels)
    w1, b1, w2, b2 = W.policy_weights(16, hidden=64, n_levels=n_levels, std=0.2, seed=7)
    env = cxm.Env(spec, n_envs=1, seed=3)
    obs = torch.rand(200, spec.obs_dim, generator=torch.Generator().manual_seed(5)).cuda()
    env.set_policy(64, (w1, b1, w2, b2))
    free = env.policy_sample(obs, 9).cpu().numpy()
    masked = [2, 7]
    b2 = b2.reshape(16, n_levels + 1).copy()
    b2[masked] = {"lowest": 0xFF7F, "-inf": 0xFF80}[bias]   # in BF16
    env.set_policy(64, (w1, b1, w2, b2.reshape(-1)))
    got = env.policy_sample(obs, 9).cpu().numpy()
    assert (got[:, masked] == (n_levels if bias == "lowest" else 0)).all()
    rest = np.setdiff1d(np.arange(16), masked)
    assert np.array_equal(got[:, rest], free[:, rest])
