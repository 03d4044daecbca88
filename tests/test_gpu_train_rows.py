"""The training kernels' row order and their sums at the edges of their split: 64
samples a block, 64 partial rows in flight, the division by a row count through a
reciprocal."""
import math

import numpy as np
import pytest

import oracle.mlp as M
from paper_1811_03510_amd import scenes as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MASK = (1 << 64) - 1


def splitmix(x):
    x = (x + 0x9E3779B97F4A7C15) & MASK
    z = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & MASK
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & MASK
    return x, z ^ (z >> 31)


def permutation(seed, epoch, n):
    """Row order of an epoch: row(position) = (a position + c) mod n, gcd(a, n) = 1."""
    if n <= 1:
        return 1, 0
    x, a = splitmix(seed ^ ((epoch * 0xD1B54A32D192ED03) & MASK))
    a = a % n or 1
    while math.gcd(a, n) != 1:
        a = a + 1 if a + 1 < n else 1
    return a, splitmix(x)[1] % n


@pytest.mark.parametrize("n,batch", [(1, 1), (2, 1), (97, 10), (4096, 4096), (1000003, 8192), (1 << 20, 1000),
                                     (3000017, 400000)])
def test_minibatches_are_those_of_the_permutation(n, batch):
    """One row is labelled: a step's loss is positive exactly where its minibatch holds that row."""
    from paper_1811_03510_amd import ccs
    theta = torch.from_numpy(S.mlp_init()).cuda()
    X = torch.zeros((n, 16), device="cuda")
    per_epoch = max(1, n // batch)
    steps = min(2 * per_epoch + 3, 300)
    for row in sorted({0, n - 1, n // 3, (7 * n) // 11}):
        y = torch.full((n,), ccs.NO_LABEL, dtype=torch.uint8, device="cuda")
        y[row] = 2
        loss = ccs.policy_train(theta.clone(), X, y, steps=steps, batch=batch, seed=9, bf16=False).cpu().numpy()
        want = np.zeros(steps, bool)
        for s in range(steps):
            a, c = permutation(9, s // per_epoch, n)
            pos = ((row - c) * pow(a, -1, n)) % n if n > 1 else 0
            want[s] = (s % per_epoch) * batch <= pos < (s % per_epoch + 1) * batch
        assert np.array_equal(loss > 0, want), (row, np.flatnonzero((loss > 0) != want)[:5])


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 64 * 63 + 1, 64 * 64, 64 * 64 + 5, 64 * 130 + 17])
def test_gradient_sums(n, bf16):
    """Against the FP64 network.  fp32 chains of at most 32 products per unit and 64 + 131 terms per parameter: each
    term within (32 + 32 + 4) u of its value, the sums within (64 + 131) u of the terms' magnitudes, together below
    270 u = 1.7e-5 of the summed magnitudes; against the norm of the gradient, which cancels, 2e-4 (fp32).  A hidden
    value that rounds to the other bfloat16 differs by 2^-8 of itself on a few rows: 1e-2."""
    from paper_1811_03510_amd import ccs
    rng = np.random.default_rng(n)
    X = rng.uniform(-1, 1, (n, 16)).astype(np.float32)
    y = rng.integers(0, 4, n).astype(np.uint8)
    y[rng.random(n) < 0.3] = ccs.NO_LABEL
    if n < 3:
        y[:] = 1
    theta = S.mlp_init()
    loss, grad = ccs.policy_grad(torch.from_numpy(theta).cuda(), torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(),
                                 bf16=bf16)
    lw, gw = M.loss_and_grad(theta.astype(np.float64), X.astype(np.float64), y, bf16=bf16)[:2]
    g = grad.cpu().numpy().astype(np.float64)
    tol = 1e-2 if bf16 else 2e-4
    assert abs(loss - lw) <= tol * abs(lw)
    assert np.linalg.norm(g - gw) <= tol * np.linalg.norm(gw)
