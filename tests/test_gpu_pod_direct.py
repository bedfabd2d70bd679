"""POD through the direct eigensolver at the sizes where its layout changes:
one pair, odd sizes, two / five blocks per thread (126 / 127), exchange in LDS
or in memory (200 / 201), the largest."""
import numpy as np
import pytest

import gen
from test_gpu_parity import case, solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,p", [(2, 1), (3, 2), (5, 2), (126, 8), (127, 16), (200, 32), (201, 32), (256, 32)])
def test_direct_pod_matches_numpy(lib, M, p):
    """Singular values and modes against a 64-bit SVD.  The eigenvalues of the
    Gram are within M eps lambda_1 of the exact ones, so sigma_j within
    M eps sigma_1^2 / (2 sigma_j), and a mode turns by at most M eps lambda_1
    over its gap; r < M - 1 leaves a null space."""
    w = gen.c1_workload(n=31, k=0)
    N = w.op.N
    r = min(M - 1, 2 * p)
    rng = np.random.default_rng(M)
    U = np.linalg.qr(rng.standard_normal((N, r)))[0]
    V = np.linalg.qr(rng.standard_normal((M, r)))[0]
    X = rng.standard_normal((N, 1)) / N ** 0.5 + (U * 0.9 ** np.arange(r)) @ V.T
    case(f"direct pod M={M} p={p}")
    s = solver(lib, w.op, None, "assembled")
    Phi, sigma = s.pod(np.asfortranarray(X), p)
    Phi = Phi.cpu().numpy()
    Ux, sx, _ = np.linalg.svd(X - X.mean(1, keepdims=True), full_matrices=False)
    eps = np.finfo(np.float64).eps
    lam = sx ** 2
    assert np.all(np.abs(sigma - sx[:p]) <= M * eps * lam[0] / sx[:p] + 10 * eps * sx[0])
    gap = np.array([min(abs(lam[j] - lam[q]) for q in (j - 1, j + 1) if 0 <= q < len(lam)) for j in range(p)])
    off = 1.0 - np.abs(np.sum(Phi * Ux[:, :p], axis=0))
    assert np.all(off <= (10 * M * eps * lam[0] / gap) ** 2 + 100 * eps * lam[0] / lam[:p])
    assert np.abs(Phi.T @ Phi - np.eye(p)).max() <= 10 * M * eps * lam[0] / lam[p - 1]


def test_direct_pod_separates_small_modes(lib):
    """Snapshots that hardly differ: one mode and 99 of 1e-7 to 2e-7 of its size.  The
    modes stay orthonormal as far as the Gram's rounding allows: entries of
    eps / M, a matrix of norm 2 eps / sqrt(M), twice for the sums behind them and
    once more for the eigensolver, over lambda_j >= tail^2 (in units of lambda_1)."""
    M, p, tail = 100, 16, 2e-7
    w = gen.c1_workload(n=31, k=0)
    rng = np.random.default_rng(M)
    U = np.linalg.qr(rng.standard_normal((w.op.N, M)))[0]
    V = np.linalg.qr(rng.standard_normal((M, M)))[0]
    X = (U * np.r_[1.0, tail * np.linspace(1.0, 0.5, M - 1)]) @ V.T
    case("direct pod, small modes")
    s = solver(lib, w.op, None, "assembled")
    Phi = s.pod(np.asfortranarray(X), p)[0].cpu().numpy()
    orth = np.abs(Phi.T @ Phi - np.eye(p)).max()
    print(f"   orthonormal to {orth:.2e}", flush=True)
    assert orth <= 5 * np.finfo(np.float64).eps / M ** 0.5 / tail ** 2
