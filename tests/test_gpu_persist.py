"""Persistent chunk kernels (one launch runs a chunk of iterations) against the
oracle, at the sizes where their tiling and forms change."""
import threading

import numpy as np
import pytest
import torch

import gen
import oracle
from test_gpu_parity import _xstar, case, solver, spec

pytestmark = pytest.mark.gpu


def _check(lib, w, S, out, prec, which, tol):
    """The bars of the parity tests: e_rel <= max(1e-8, 2 x the oracle's), FP64
    iteration counts within 2, the true residual in the refinement modes."""
    X = out["x"].cpu().numpy()
    for m in which:
        inst = w.instances[m]
        ref = oracle.solve_instance(S, w.Z, inst.mask, inst.b, tol)
        I, xs = _xstar(S, inst.mask, inst.b)
        e = oracle.rel_err(X[m, I], xs)
        print(f"   m={m} iters {out['iters'][m]} (oracle {ref.iters}) e_rel {e:.2e}", flush=True)
        assert out["status"][m] == 0
        assert np.all(X[m, inst.mask == 1] == 0.0)
        assert e <= max(1e-8, 2 * oracle.rel_err(ref.x[I], xs)), (m, e)
        if prec == "fp64":
            assert abs(int(out["iters"][m]) - ref.iters) <= 2
        else:
            assert out["relres_true"][m] <= tol


# one tile that is not full; one full tile and no modes; 13 diagonals; tiles of
# 512 rows, boundary form, several teams; W left out (Z^T S z), tiles of 1024
# rows, every compute unit taken
@pytest.mark.parametrize("n,k,B,prec,form", [
    (15, 8, 1, "fp64", "factored"), (16, 0, 2, "fp64", "factored"), (63, 16, 3, "fp64", "assembled"),
    (63, 24, 2, "mixed", "assembled"), (95, 16, 5, "mixed", "factored"),
    (33, 8, 2, "fp32", "factored"), (47, 0, 1, "fp32", "assembled"), (127, 40, 16, "fp64", "factored")])
def test_chunk_kernel_matches_oracle(lib, n, k, B, prec, form):
    w = gen.c2_workload(n=n, k=k, B=B)
    S = spec(w.op, form)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    case(f"persistent chunk {prec} {form} cd2d n={n} k={k} B={B}")
    s = solver(lib, w.op, w.Z if k else None, form, profile=1,
               precision=dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE, fp32=lib.FP32_REFINE)[prec])
    out = s.solve_batched(masks, bs, 1e-10)
    assert s.stats()["chunk"]["launches"] > 0
    _check(lib, w, S, out, prec, sorted({0, B // 2, B - 1}), 1e-10)


def test_chunk_kernel_3d_exchanges_the_inner_product(lib):
    """7-point operator whose reach (529) is beyond a 256-row tile: A p goes
    through memory instead of LDS."""
    w = gen.c5_workload(n=23, k=8, B=2)
    S = spec(w.op, "factored")
    case("persistent chunk fp64 3d n=23 k=8 B=2")
    s = solver(lib, w.op, w.Z, "factored", profile=1)
    out = s.solve_batched(np.stack([i.mask for i in w.instances]), np.stack([i.b for i in w.instances]), 1e-8)
    assert s.stats()["chunk"]["launches"] > 0
    _check(lib, w, S, out, "fp64", (0, 1), 1e-8)


def test_chunk_kernels_of_two_threads(lib):
    """Two contexts on two streams at once, each launch as large as the GPU:
    neither waits for the other for good and both get their solutions."""
    w = gen.c2_workload(n=127, k=32, B=12)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    case("persistent chunk, two threads, cd2d n=127 k=32 B=12")
    ref = solver(lib, w.op, w.Z, "factored").solve_batched(masks, bs, 1e-10)["x"].cpu().numpy()
    got = [None, None]

    def work(q):
        with torch.cuda.stream(torch.cuda.Stream()):
            s = solver(lib, w.op, w.Z, "factored")
            for _ in range(3):
                got[q] = s.solve_batched(masks, bs, 1e-10)["x"].cpu().numpy()

    ts = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for q in range(2):
        assert got[q] is not None
        assert np.linalg.norm(got[q] - ref) <= 1e-8 * np.linalg.norm(ref)


def test_chunk_kernel_fills_the_xcds_evenly(lib):
    """9 tiles x 56 instances, 504 of the 512 places: every XCD gets 63 of its
    64, so no launch is called off (no kernel of the per-step form runs)."""
    w = gen.c2_workload(n=91, k=8, B=56)
    S = spec(w.op, "factored")
    case("persistent chunk mixed cd2d n=91 k=8 B=56")
    s = solver(lib, w.op, w.Z, "factored", profile=1, precision=lib.MIXED_REFINE)
    out = s.solve_batched(np.stack([i.mask for i in w.instances]), np.stack([i.b for i in w.instances]), 1e-10)
    st = s.stats()
    assert st["chunk"]["launches"] > 0
    assert st["update_tm"]["launches"] == 0 and st["pupdate_tm"]["launches"] == 0
    _check(lib, w, S, out, "mixed", (0, 55), 1e-10)
