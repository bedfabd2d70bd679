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


def _problem(kind, n, k, B):
    """(operator, modes, masks, right-hand sides)."""
    if kind in ("noise", "cube"):
        # every inactive row has an active neighbour; a 7-point factor
        op, Z = (gen.c2_operator(n)[0], gen.c2_workload(n=n, k=k, B=1).Z) if kind == "noise" else \
            (gen.ocp_3d_obstacle(n=n, B=1).op, gen.sine_modes_3d(n, k)[0])
        rng = np.random.default_rng(n + B)
        return op, Z, (rng.random((B, op.N)) < 0.25).astype(np.uint8), rng.standard_normal((B, op.N))
    w = (gen.c3_workload if kind == "het" else gen.c2_workload)(n=n, k=k, B=B)
    if kind == "het":
        w.op = gen.Operator(n=n, dim=2, B=gen.c3_operator(n)[1], shift=w.op.shift, name="five-point")
    return w.op, w.Z, np.stack([i.mask for i in w.instances]), np.stack([i.b for i in w.instances])


# batches whose blocks of one instance are not all resident: groups of 16.  A
# group of 9, 5 steps a tile (8 in registers), last tile short; every row listed
# (more than LDS holds), 10 steps (16); A p through memory, 18 steps (20), modes
# in three column tiles; 64 modes; a 7-point factor; a 5-point operator that
# isn't factored, each instance with its own scale
@pytest.mark.parametrize("kind,n,k,B", [
    ("cd", 91, 8, 57), ("noise", 159, 16, 40), ("cd", 191, 40, 64), ("cd", 95, 64, 60), ("cube", 25, 20, 33),
    ("het", 95, 16, 60)])
def test_group_chunk_kernel_matches_oracle(lib, kind, n, k, B):
    op, Z, masks, bs = _problem(kind, n, k, B)
    form = "assembled" if kind == "het" else "factored"
    case(f"persistent group chunk mixed {kind} n={n} k={k} B={B}")
    tol = 1e-8
    s = solver(lib, op, Z, form, profile=1, precision=lib.MIXED_REFINE)
    scale = np.linspace(0.5, 2.0, B) if kind == "het" else None
    out = s.solve_batched(masks, bs, tol, a=scale, c=None if scale is None else op.shift * scale)
    st = s.stats()
    assert st["chunk"]["launches"] > 0 and st["update_tm"]["launches"] == 0
    X = out["x"].cpu().numpy()
    for m in (0, B // 2, B - 1):
        # (S_m = a_m S_ref + c_m I, and S_ref holds the shift already)
        S = spec(op, form) if scale is None else spec(op, form, a=scale[m], c=2 * op.shift * scale[m])
        ref = oracle.solve_instance(S, Z, masks[m], bs[m], tol)
        I, xs = _xstar(S, masks[m], bs[m])
        e, e0 = oracle.rel_err(X[m, I], xs), oracle.rel_err(ref.x[I], xs)
        print(f"   m={m} iters {out['iters'][m]} (oracle {ref.iters}) e_rel {e:.2e} (oracle {e0:.2e})", flush=True)
        assert out["status"][m] == 0 and out["relres_true"][m] <= tol
        assert np.all(X[m, masks[m] == 1] == 0.0)
        assert e <= max(1e-8, 2 * e0), (m, e)


@pytest.mark.parametrize("prec,n,B", [("fp64", 95, 60), ("fp32", 95, 60), ("mixed", 191, 40)])
def test_instances_left_go_on_in_smaller_launches(lib, prec, n, B):
    """Iteration counts that differ by more than two: a batch too large for the
    chunk kernel starts with a kernel per step (groups of 16 in mixed precision)
    and its last instances go on in chunk launches of their own."""
    w = gen.c3_workload(n=n, k=16, B=B)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    case(f"instances left {prec} het n={n} B={B}")
    s = solver(lib, w.op, w.Z, "factored", profile=1,
               precision=dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE, fp32=lib.FP32_REFINE)[prec])
    scale = np.array([i.a for i in w.instances])
    out = s.solve_batched(masks, bs, 1e-8, a=scale)
    st = s.stats()
    assert out["iters"].max() > 2 * out["iters"].min()
    assert st["chunk"]["launches"] > 0
    if prec != "mixed":
        assert st["pupdate"]["launches"] + st["pupdate_bt"]["launches"] > 0
    X = out["x"].cpu().numpy()
    order = np.argsort(out["iters"])
    for m in (order[0], order[B // 2], order[-1]):
        S = spec(w.op, "factored", a=scale[m], c=scale[m] * w.op.shift)
        I, xs = _xstar(S, masks[m], bs[m])
        ref = oracle.solve_instance(S, w.Z, masks[m], bs[m], 1e-8)
        e, e0 = oracle.rel_err(X[m, I], xs), oracle.rel_err(ref.x[I], xs)
        print(f"   m={m} iters {out['iters'][m]} (oracle {ref.iters}) e_rel {e:.2e} (oracle {e0:.2e})", flush=True)
        assert out["status"][m] == 0
        assert e <= max(1e-8, 2 * e0), (m, e)


def test_breakdown_stays_in_its_instance(lib):
    """Instance 0 of a group overflows in its first iteration: its operator is
    1e-315 times the others' and shifted below a Ritz value of the modes (so that it
    runs without them), alpha = r.r / p.S p is infinite, and so is its z on its
    listed rows, the first of every tile's list. The other instances get the
    solutions they get beside a sound instance 0."""
    n, k, B, tol = 91, 8, 57, 1e-8
    op, Z, masks, bs = _problem("cd", n, k, B)
    bs[0] = np.random.default_rng(3).standard_normal(op.N)
    case(f"breakdown in a group, mixed cd n={n} k={k} B={B}")
    out = []
    for broken in (False, True):
        s = solver(lib, op, Z, "factored", profile=1, precision=lib.MIXED_REFINE, precond=lib.NONE)
        s._check = lambda rc, **kw: rc
        a, c = np.ones(B), np.zeros(B)
        if broken:
            a[0], c[0] = 1e-315, -1.9e-310
        out.append(s.solve_batched(masks, bs, tol, a=a, c=c))
        st = s.stats()
        assert st["chunk"]["launches"] > 0 and st["update_tm"]["launches"] == 0
    sound, broken = out
    assert broken["status"][0] < 0
    assert np.all(sound["status"] == 0)
    assert np.all(broken["status"][1:] == 0), broken["status"]
    assert np.all(broken["relres_true"][1:] <= tol)
    x0, x1 = sound["x"].cpu().numpy(), broken["x"].cpu().numpy()
    for m in range(1, B):
        # both solve to a relative residual of tol, cond(S) <= 3e5
        assert np.linalg.norm(x1[m] - x0[m]) <= 2 * 3e5 * tol * np.linalg.norm(x0[m]), m


# 16 tiles an instance; groups of 16, listed rows through LDS; FP32 vectors
@pytest.mark.parametrize("prec,n,k,B,form", [("fp64", 63, 16, 2, 1), ("mixed", 91, 8, 57, 2), ("fp32", 63, 8, 3, 1)])
def test_a_wait_that_is_given_up_costs_time_only(lib, prec, n, k, B, form):
    """Blocks that give up a wait (for a block that starts 1 ms late) leave instances
    with vectors of different iterations: the solve starts again with a kernel per
    step, and the next one runs chunk launches again."""
    w = gen.c2_workload(n=n, k=k, B=B)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    case(f"waits given up, {prec} cd2d n={n} k={k} B={B}")
    s = solver(lib, w.op, w.Z, "factored",
               precision=dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE, fp32=lib.FP32_REFINE)[prec])
    tol = 1e-8
    S = spec(w.op, "factored")
    for fault, from_launch, lost in ((2, 0, 1), (2, 3, 2), (0, 0, 2)):
        s.fault(fault, from_launch)
        out = s.solve_batched(masks, bs, tol)
        v = s.chunk_variant()
        print(f"   fault {fault} from launch {from_launch}: {v}", flush=True)
        assert v["lost"] == lost and v["called_off"] == 0
        assert v["form"] == (0 if fault else form) and (v["launches"] == 0) == (fault != 0)
        _check(lib, w, S, out, prec, (0, B - 1), tol)


@pytest.mark.parametrize("prec,n,k,B", [("fp64", 63, 16, 2), ("mixed", 91, 8, 57), ("fp32", 63, 8, 3)])
def test_called_off_launches_step_back(lib, prec, n, k, B):
    """A chunk launch that is called off leaves its solve to the kernels per
    step: the tuned ones when it is the first launch, from where the solve is when it
    is a later one. The next solves remember it."""
    w = gen.c2_workload(n=n, k=k, B=B)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    case(f"chunk launches called off, {prec} cd2d n={n} k={k} B={B}")
    tol = 1e-8
    S = spec(w.op, "factored")
    per_step = ("pupdate", "pupdate_bt", "pupdate_tm")
    for from_launch in (0, 3):
        s = solver(lib, w.op, w.Z, "factored", profile=1,
                   precision=dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE, fp32=lib.FP32_REFINE)[prec])
        s.fault(1, from_launch)
        out = s.solve_batched(masks, bs, tol)
        v, st = s.chunk_variant(), s.stats()
        print(f"   from launch {from_launch}: {v}, trial ms {s.variant()[2].max():.2f}", flush=True)
        assert v["called_off"] == 1 and v["lost"] == 0
        assert sum(st[q]["launches"] for q in per_step) > 0
        assert (v["launches"] == 0) == (from_launch == 0)
        assert (s.variant()[2].max() > 0) == (from_launch == 0)      # tuned
        _check(lib, w, S, out, prec, (0, B - 1), tol)
        # two solves without a try, one that tries, then four
        tries = []
        for _ in range(7):
            s.solve_batched(masks, bs, 1e-2)
            tries.append(s.chunk_variant()["called_off"])
        if from_launch == 0:
            assert tries == [1, 1, 2, 2, 2, 2, 2], tries
            # half-way, with the tuned variant standing by
            s.fault(1, 2)
            tuned = s.variant()[:2]
            out = s.solve_batched(masks, bs, tol)
            assert s.chunk_variant()["launches"] > 0 and s.chunk_variant()["called_off"] == 3
            assert s.variant()[:2] == tuned
            _check(lib, w, S, out, prec, (0, B - 1), tol)
        s.fault(0)
        out = s.solve_batched(masks, bs, tol)
        assert s.chunk_variant()["form"] > 0
        _check(lib, w, S, out, prec, (0, B - 1), tol)


@pytest.mark.parametrize("from_launch", [0, 1, 2])
def test_called_off_launches_and_the_iteration_cap(lib, from_launch):
    """The launches queued behind one that is called off are no iterations: a
    refinement solve that reaches its cap says so."""
    w = gen.c2_workload(n=63, k=8, B=3)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    case(f"called off at launch {from_launch}, then the iteration cap")
    s = solver(lib, w.op, w.Z, "factored", precision=lib.MIXED_REFINE, maxit=150, segment_maxit=5)
    s.fault(1, from_launch)
    out = s.solve_batched(masks, bs, 1e-10)
    v = s.chunk_variant()
    print(f"   {v} iters {out['iters']}", flush=True)
    assert v["called_off"] == 1
    assert np.all(out["status"] == lib.W_MAXIT) and np.all(out["iters"] == 150)


@pytest.mark.parametrize("prec,n,k,B,form", [("fp64", 31, 8, 2, 1), ("mixed", 91, 8, 57, 2)])
def test_allocations_that_fail(lib, prec, n, k, B, form):
    """Each allocation of a first solve fails in turn.  The chunk launches' buffers
    are not needed to solve: without them the kernels per step run. After any other
    the solve says E_NOMEM, and the next one finds everything it needs."""
    w = gen.c2_workload(n=n, k=k, B=B)
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    S = spec(w.op, "factored")
    tol = 1e-8
    solved = refused = 0
    s = solver(lib, w.op, w.Z, "factored", precision=dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE)[prec])
    ref = s.solve_batched(masks, bs, tol)
    _check(lib, w, S, ref, prec, (0, B - 1), tol)
    ref = ref["x"].cpu().numpy()
    for at in range(100):
        case(f"allocation {at} fails, {prec} cd2d n={n} B={B}")
        s = solver(lib, w.op, w.Z, "factored", precision=dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE)[prec])
        s.fault(3, at)
        try:
            x = s.solve_batched(masks, bs, tol)["x"].cpu().numpy()
            first = s.chunk_variant()["form"]
            assert np.linalg.norm(x - ref) <= 1e-6 * np.linalg.norm(ref)
            solved += first == 0
        except lib.Adef2Error as e:
            assert e.code == lib.E_NOMEM
            refused += 1
            first = 0
        s.fault()
        x = s.solve_batched(masks, bs, tol)["x"].cpu().numpy()
        assert s.chunk_variant()["form"] == form
        assert np.linalg.norm(x - ref) <= 1e-6 * np.linalg.norm(ref)
        if first == form:                          # fewer allocations than that
            break
    print(f"   {solved} solved without chunk launches, {refused} refused", flush=True)
    assert first == form and solved >= 4 and refused >= 20


def test_chunk_launch_bytes(lib):
    """The bytes of a chunk launch in stats(): 32 iterations read the operator and
    move p, everything else moves once."""
    w = gen.c2_workload(n=63, k=16, B=1)
    mask, b = w.instances[0].mask, w.instances[0].b
    N, nI = mask.size, int((mask == 0).sum())
    case("chunk launch bytes, fp64 63^2, k = 0 and 16")

    def diagonals(A):
        return np.unique(A.indices - np.repeat(np.arange(N), np.diff(A.indptr))).size

    D, D1 = diagonals(w.op.S()), diagonals(w.op.A)
    for form, k, op in (("assembled", 0, nI * D * 8), ("factored", 16, (N * D1 + nI * D1) * 8)):
        s = solver(lib, w.op, w.Z if k else None, form, profile=1, poll_max=1)
        s.solve_batched(mask[None], b[None], 1e-6)
        st = s.stats()["chunk"]
        it = op + N * 8 + nI * 8 + 3 * nI * k * 8          # p read and written; Z twice, W
        assert st["alg_bytes"] / st["launches"] == 32 * it + nI * 9 * 8 + N


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_what_is_bitwise_by_default(lib, prec):
    """Default options, 60 instances that start with a kernel per step (FP64; tuned)
    or in groups of 16 (mixed) and end in smaller chunk launches: a repeated solve is
    bitwise the same. The launches follow the instances left at each poll, so with
    another poll_max or sweep_async the sums have another order, and the solutions
    agree to the bars of the parity tests."""
    w = gen.c2_workload(n=95, k=16, B=60)
    S = spec(w.op, "factored")
    masks = np.stack([i.mask for i in w.instances])
    bs = np.stack([i.b for i in w.instances])
    tol = 1e-8
    case(f"repeated solves, polls and segments, {prec} cd2d n=95 B=60")
    p = dict(fp64=lib.FP64, mixed=lib.MIXED_REFINE)[prec]
    s = solver(lib, w.op, w.Z, "factored", precision=p)
    a, b = s.solve_batched(masks, bs, tol), s.solve_batched(masks, bs, tol)
    np.testing.assert_array_equal(a["iters"], b["iters"])
    np.testing.assert_array_equal(a["x"].cpu().numpy(), b["x"].cpu().numpy())
    assert s.chunk_variant()["launches"] > 0
    if prec == "fp64":
        assert s.variant()[2].max() > 0                # trial times: the tuner ran
    for opts in (dict(poll_max=1), dict(sweep_async=0)):
        s = solver(lib, w.op, w.Z, "factored", precision=p, **opts)
        _check(lib, w, S, s.solve_batched(masks, bs, tol), prec, (0, 29, 59), tol)
