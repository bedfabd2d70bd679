"""Set-up of the coarse space against the oracle: column tiles that are not
full, odd numbers of modes, short last sub-tiles, the stencil forms (5 and 7
diagonals, any other number) and operator scales."""
import numpy as np
import pytest

import gen
import oracle
from test_gpu_parity import case, solver, spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,k,prec", [
    ("cd", 17, 3, "fp64"), ("cd", 31, 23, "mixed"), ("cd", 33, 40, "fp64"), ("cd", 33, 55, "mixed"),
    ("cd13", 31, 16, "fp64"), ("five", 31, 32, "fp64"), ("cube", 9, 64, "fp64"), ("cube", 11, 5, "mixed")])
def test_coarse_matrix_matches_oracle(lib, kind, n, k, prec):
    """E of the orthonormalised restricted modes: its eigenvalues to 1e-9 and the
    condition number to 1e-8 (FP64 sums over at most 1331 rows)."""
    form = "assembled" if kind in ("cd13", "five") else "factored"
    if kind == "cube":
        op, Z = gen.ocp_3d_obstacle(n=n, B=1).op, gen.sine_modes_3d(n, k)[0]
    else:
        op, Z = gen.c2_operator(n)[0], gen.sine_modes_2d(n, k)[0]
        if kind == "five":
            op = gen.Operator(n=n, dim=2, B=gen.c3_operator(n)[1], shift=1e-3, name="five-point")
    mask = (np.random.default_rng(n + k).random(op.N) < 0.2).astype(np.uint8)
    case(f"coarse matrix {prec} {form} {kind} n={n} k={k}")
    s = solver(lib, op, Z, form, precision=lib.FP64 if prec == "fp64" else lib.MIXED_REFINE)
    nI, keff, cond, rc = s.restrict(mask)
    I, _, _ = oracle.compact(mask)
    S = spec(op, form)
    S_II = oracle.restrict_factored(op.A, op.alpha, op.shift, I)[0] if form == "factored" else oracle.restrict(S, I)[0]
    Zo, kept = oracle.restricted_basis(Z, I)
    cs, fb = oracle.coarse_setup(S_II, Zo)
    assert nI == len(I) and keff == len(kept) and rc == 0 and not fb
    E, keptg, _, _ = s.coarse_info()
    np.testing.assert_array_equal(np.flatnonzero(keptg), kept)
    assert abs(cond / cs.cond - 1) < 1e-8, (cond, cs.cond)
    np.testing.assert_allclose(np.linalg.eigvalsh(E), np.linalg.eigvalsh(cs.E), rtol=1e-9)
