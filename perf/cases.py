"""The workloads whose speed this framework is measured on.

Every case is a call (or the pair of calls) that a program solving
state-constrained control problems makes through paper_2606_17971_amd.binding,
on the operators, modes, masks and right-hand sides that gen builds for the
tests and the benchmark.  A program keeps one Solver per configuration
(operator, modes, precision) and feeds it new masks and right-hand sides, so
the Solver is the handle that prepare() keeps; what changes with the seed is
the inactive set, the right-hand side, the operator scale and the parameters.

Kinds:
  solve      restrict + solve of one instance (B = 1), or solve_batched
  learned    solve_batched with the learned enrichment vectors
  activeset  the primal active-set loop over a batch
  restrict   the coarse set-up of one inactive set alone
  pod        POD of an archive of solutions
  grad       loss and parameter gradient of the enrichment network

The iteration counts and the residual at exit are not among the outputs: they
tell how a solve went, not what it computed, and a change of the order of a
sum moves them by a few.
"""
import functools
import math
import os
import tempfile

import numpy as np
import torch

# reference modes found by an eigensolver are kept between runs
os.environ.setdefault("ADEF2_CACHE", os.path.join(tempfile.gettempdir(), "adef2_modes_%d" % os.getuid()))

import gen  # noqa: E402
from paper_2606_17971_amd import binding  # noqa: E402


def _case(name, kind, **kw):
    return dict(name=name, kind=kind, **kw)


def listed():
    return [
        # the smallest whole solve: the quick-start size, one instance, double
        # precision; a few hundred iterations of very short kernels
        _case("lap63_fp64_b1", "solve", family="lap", n=63, k=16, B=1, precision="FP64", tol=1e-11),
        # the paper's own setting: one optimal-control instance at a time,
        # double precision, 40 closed-form modes
        _case("ocp255_fp64_b1", "solve", family="ocp", n=255, k=40, B=1, precision="FP64", tol=1e-11),
        # a handful of right-hand sides at a size that no tile divides
        _case("cd191_mixed_b5", "solve", family="cd", n=191, k=32, B=5, precision="MIXED_REFINE", tol=1e-10),
        # the benchmark's convection-diffusion batch at half and at three
        # quarters of its grid
        _case("cd255_mixed_b16", "solve", family="cd", n=255, k=32, B=16, precision="MIXED_REFINE", tol=1e-10),
        _case("cd383_mixed_b16", "solve", family="cd", n=383, k=32, B=16, precision="MIXED_REFINE", tol=1e-9),
        # a parameter sweep on the heterogeneous-diffusion operator: many
        # instances, each with its own operator scale and active fraction
        _case("het191_mixed_b48", "solve", family="het", n=191, k=32, B=48, precision="MIXED_REFINE", tol=1e-8),
        # three dimensions, coefficient jumps, modes prolonged from a coarse
        # grid, stopped on the true residual
        _case("inc3d47_fp64r_b8", "solve", family="inc3d", n=47, k=64, B=8, precision="FP64_REFINE", tol=1e-8),
        # the optimal-control suite: the active-set loop of 30 parameters
        _case("activeset100_fp64_b30", "activeset", name_ocp="2d_nonsep", n=100, k=40, B=30, tol=1e-11),
        # learned enrichment in use: a basis of its own for every instance
        _case("learned127_fp64_b16", "learned", n=127, k=32, p=32, B=16, tol=1e-10),
        # set-up of one inactive set on the benchmark's full grid
        _case("restrict511_mixed", "restrict", n=511, k=32, precision="MIXED_REFINE"),
        # the enrichment pool: POD of 200 archived solutions
        _case("pod255_m200", "pod", n=255, M=200, p=32),
        # one full-batch training step's gradient
        _case("grad512", "grad", n=47, k=16, M=512, p=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("lap", "ocp", "cd", "cd", "het", "inc3d", "activeset", "learned", "restrict", "pod", "grad"))
    if kind == "lap":
        precision = rng.choice(("FP64", "MIXED_REFINE", "FP32_REFINE"))
        return dict(kind="solve", family="lap", n=_log_int(rng, 31, 160), k=rng.randint(0, 32),
                    B=rng.choice((1, 1, 2, 3, 7, 8)), precision=precision, tol=1e-11)
    if kind == "ocp":
        return dict(kind="solve", family="ocp", n=_log_int(rng, 63, 300), k=rng.randint(8, 48), B=1,
                    precision="FP64", tol=1e-11)
    if kind == "cd":
        n = rng.randint(95, 300)
        return dict(kind="solve", family="cd", n=n, k=rng.choice((16, 24, 32, 40)), B=rng.randint(1, 16),
                    precision="MIXED_REFINE", tol=1e-10 if n <= 255 else 1e-9)
    if kind == "het":
        return dict(kind="solve", family="het", n=rng.randint(95, 180), k=rng.choice((16, 32)),
                    B=rng.randint(12, 48), precision="MIXED_REFINE", tol=1e-8)
    if kind == "inc3d":
        nc, c = rng.choice(((7, 3), (9, 3), (11, 3), (12, 3), (15, 2), (17, 2), (19, 2)))
        return dict(kind="solve", family="inc3d", n=c * (nc + 1) - 1, nc=nc, k=rng.choice((32, 48, 64)),
                    B=rng.randint(1, 8), precision=rng.choice(("FP64", "FP64_REFINE")), tol=1e-8)
    if kind == "activeset":
        return dict(kind="activeset", name_ocp=rng.choice(gen.OCP_2D), n=_log_int(rng, 40, 100),
                    k=rng.randint(8, 40), B=rng.randint(2, 30), tol=1e-11)
    if kind == "learned":
        return dict(kind="learned", n=rng.randint(63, 127), k=rng.choice((16, 24, 32)), p=rng.choice((16, 32)),
                    B=rng.randint(2, 16), tol=1e-10)
    if kind == "restrict":
        return dict(kind="restrict", n=rng.randint(127, 511), k=rng.choice((16, 32)),
                    precision=rng.choice(("FP64", "MIXED_REFINE")))
    if kind == "pod":
        M = rng.choice((_log_int(rng, 40, 180), rng.randint(300, 600)))    # either eigensolver
        return dict(kind="pod", n=_log_int(rng, 63, 300), M=M, p=rng.choice((8, 16, 32)))
    return dict(kind="grad", n=rng.randint(31, 63), k=rng.choice((8, 16)), M=_log_int(rng, 32, 600),
                p=rng.choice((16, 32, 64)))


# ---------------------------------------------------------------------------
# operators, modes and instances
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=8)
def _operator(family, n):
    if family == "lap":
        return gen.c1_workload(n=n, k=0).op
    if family == "cd":
        return gen.c2_operator(n)[0]
    if family == "het":
        return gen.c3_operator(n)[0]
    if family == "inc3d":
        return gen.c5_operator(n)[0]
    return gen.ocp_2d(family, n=n, B=1).op


def _coarse_n(case):
    return case.get("nc", (case["n"] + 1) // 3 - 1)


@functools.lru_cache(maxsize=8)
def _modes(family, n, k, nc):
    """Reference modes (N x k), or the coarse grid's for three dimensions."""
    if family == "cd":
        return gen.c2_workload(n=n, k=k, B=1).Z
    if family == "het":
        return gen.c3_workload(n=n, k=k, B=1).Z
    if family == "inc3d":
        return gen.c5_workload(n=n, k=k, B=1, nc=nc).meta["Zc"]
    return gen.sine_modes_2d(n, k)[0] if k > 0 else None


def _family(case):
    """The operator's family of a case."""
    return {"solve": lambda: "2d_asym" if case["family"] == "ocp" else case["family"],
            "activeset": lambda: case["name_ocp"], "learned": lambda: "cd", "restrict": lambda: "cd",
            "pod": lambda: "lap", "grad": lambda: "lap"}[case["kind"]]()


@functools.lru_cache(maxsize=None)
def _solver(family, n, k, nc, precision, kind, p):
    """The handle a program keeps for one configuration."""
    s = binding.Solver(precision=getattr(binding, precision))
    Z = _modes(family, n, k, nc)
    if family == "inc3d":
        Z = s.prolong_basis(Z, 3, n, nc)
    s.set_operator(_operator(family, n), Z)
    if kind == "learned":
        # POD modes of earlier solutions of the family and the network's
        # parameters, as a program loads them
        old = [gen.c2_family_instance(n, th) for th in gen.c2_thetas(2 * p, 700)]
        snap = s.solve_batched(np.stack([i.mask for i in old]), np.stack([i.b for i in old]), 1e-8)["x"]
        Phi, _ = s.pod(snap.T, p)
        s.set_enrichment(Phi, gen.mlp_params(3))
    return s


def _instances(case, seed):
    """masks, right-hand sides, operator scales (or None) and parameters, from the seed alone."""
    family, n, B = _family(case), case["n"], case.get("B", case.get("M", 1))
    rng = np.random.default_rng(seed)
    a = c = theta = None
    if family == "cd":
        theta = rng.uniform(0.0, 1.0, size=(B, 4))
        if B > 1:
            theta[:, 0] = np.arange(B) / (B - 1)
        ins = [gen.c2_family_instance(n, th) for th in theta]
        masks, b = [i.mask for i in ins], [i.b for i in ins]
    elif family == "het":
        op = _operator(family, n)
        field = gen.sinusoid_field(n, int(rng.integers(1 << 30)))
        theta = rng.uniform(0.0, 1.0, size=(B, 4))
        ins = [gen.c3_instance(n, th, field, op.shift) for th in theta]
        masks, b = [i.mask for i in ins], [i.b for i in ins]
        a, c = np.array([i.a for i in ins]), np.array([i.c for i in ins])
    elif family == "inc3d":
        masks, b = [], []
        for m in range(B):
            field = gen.sinusoid_field(n, int(rng.integers(1 << 30)), dim=3)
            masks.append(gen.mask_top_fraction(field, 0.15 + 0.20 * m / max(B - 1, 1)))
            b.append(gen.gaussian_bump(n, rng.uniform(0.2, 0.8, size=3), dim=3))
    elif family == "lap":
        masks, b = [], []
        for m in range(B):
            masks.append(gen.mask_top_fraction(gen.sinusoid_field(n, int(rng.integers(1 << 30))),
                                               rng.uniform(0.1, 0.3)))
            b.append(rng.standard_normal(n * n))
        theta = rng.uniform(0.0, 1.0, size=(B, 4))
    else:
        lo, hi = gen.OCP_RANGES[family]
        masks, b = [], []
        for q in rng.uniform(lo, hi, size=B):
            yd = gen.ocp_desired_state(family, n, q)
            masks.append(gen.mask_top_fraction(gen.ocp_unconstrained(n, yd), rng.uniform(0.1, 0.3)))
            b.append(yd)
    return np.stack(masks), np.stack(b), a, c, theta


def _dev(x, dtype=torch.float64):
    return None if x is None else torch.as_tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")


def _scales(case, op, a, c):
    """Scales (a, c) of solve_batched: its c is added to a times the whole
    reference operator, whose own shift is op.shift."""
    return (None, None) if a is None else (a, c - a * op.shift)


def _archive(case, seed):
    """Snapshots for the POD: a mean and combinations of fields of decaying weight."""
    rng = torch.Generator(device="cuda").manual_seed(seed)
    N, M = case["n"] ** 2, case["M"]
    r = min(M - 1, 2 * case["p"])
    U, V, mean = (torch.randn(rows, cols, generator=rng, device="cuda", dtype=torch.float64)
                  for rows, cols in ((N, r), (M, r), (N, 1)))
    weight = 0.9 ** torch.arange(r, device="cuda", dtype=torch.float64)
    return mean / N ** 0.5 + (torch.linalg.qr(U)[0] * weight) @ torch.linalg.qr(V)[0].T


def _states(case, seed):
    """Desired states of random members of an optimal-control family, and the bound."""
    family, n, B = case["name_ocp"], case["n"], case["B"]
    lo, hi = gen.OCP_RANGES[family]
    q = np.random.default_rng(seed).uniform(lo, hi, size=B)
    psi = gen.ocp_2d(family, n=n, B=1).psi
    return _dev(np.stack([gen.ocp_desired_state(family, n, v) for v in q])), _dev(np.repeat(psi, B, axis=0))


def prepare(case, seed):
    kind, family, n = case["kind"], _family(case), case["n"]
    k, p, precision = case.get("k", 0), case.get("p", 0), case.get("precision", "FP64")
    nc = _coarse_n(case) if family == "inc3d" else 0
    s = _solver(family, n, k, nc, precision, kind if kind in ("learned", "grad", "pod") else "solve",
                p if kind in ("learned", "grad") else 0)
    st = {"kind": kind, "solver": s, "tol": case.get("tol")}
    if kind == "pod":
        st["X"], st["p"] = _archive(case, seed), p
        return st
    if kind == "activeset":
        st["yd"], st["psi"] = _states(case, seed)
        return st
    masks, b, a, c, theta = _instances(case, seed)
    st["masks"], st["b"] = _dev(masks, torch.uint8), _dev(b)
    st["a"], st["c"] = _scales(case, _operator(family, n), a, c)
    if kind == "restrict" or (kind == "solve" and case["B"] == 1):
        st["masks"], st["b"] = st["masks"][0], st["b"][0]
    if kind == "learned":
        st["theta"] = _dev(theta, torch.float32)
    if kind == "grad":
        # training samples: members with their solutions, and the pool
        N = n * n
        Phi = np.linalg.qr(np.random.default_rng(11).standard_normal((N, p)))[0]
        s.set_pod_modes(Phi)
        sol = s.solve_batched(st["masks"], st["b"], 1e-9)["x"]
        # the prepared samples live in the handle: one handle for every set of them
        t = st["solver"] = binding.Solver()
        t.set_operator(_operator(family, n), _modes(family, n, k, 0))
        t.set_pod_modes(Phi)
        t.learned_set_params(gen.mlp_params(seed % 1000))
        t.learned_prepare(st["masks"], st["b"], sol, _dev(theta, torch.float32))
    return st


def run(st):
    s, kind = st["solver"], st["kind"]
    if kind == "pod":
        Phi, sigma = s.pod(st["X"], st["p"])
        return {"Phi": Phi, "sigma": sigma}
    if kind == "grad":
        loss, grad = s.learned_loss_grad()
        return {"loss": loss, "grad": grad}
    if kind == "activeset":
        o = s.active_set_batched(st["yd"], st["psi"], tol=st["tol"])
        return {"y": o["y"], "masks": o["masks"], "outer": o["outer"], "status": o["status"]}
    if kind == "restrict":
        n_inactive, k_eff, cond, _ = s.restrict(st["masks"])
        E, kept, _, _ = s.coarse_info()
        return {"n_inactive": n_inactive, "k_eff": k_eff, "cond_E": np.array(cond), "E": E, "kept": kept}
    if kind == "learned":
        o = s.solve_batched(st["masks"], st["b"], st["tol"], theta=st["theta"])
        return {"x": o["x"], "cond_E": o["cond_E"], "n_inactive": o["n_inactive"], "status": o["status"],
                "learned": o["learned"]}
    if st["masks"].dim() == 1:
        n_inactive, _, cond, _ = s.restrict(st["masks"])
        o = s.solve(st["b"], st["tol"])
        return {"x": o.x, "cond_E": np.array(cond), "n_inactive": n_inactive, "status": o.status}
    o = s.solve_batched(st["masks"], st["b"], st["tol"], a=st["a"], c=st["c"])
    return {"x": o["x"], "cond_E": o["cond_E"], "n_inactive": o["n_inactive"], "status": o["status"]}


# conjugate-gradient iterations of a solve over n^2, about (they scale with
# the root of the condition number, that of a squared second-order operator)
ITERATIONS = {"lap": 0.14, "ocp": 0.11, "cd": 0.09, "het": 0.2, "inc3d": 1.5, "activeset": 0.2, "learned": 0.09}


def work(case):
    kind, n = case["kind"], case["n"]
    N = float(n ** 3 if case.get("family") == "inc3d" else n * n)
    k, B, M, p = case.get("k", 0), case.get("B", 1), case.get("M", 0), case.get("p", 0)
    if kind == "pod":
        return {"bytes": 8 * N * (M + p), "flops": N * M * M + 2 * N * M * p}
    if kind == "grad":
        mlp = 2.0 * (4 * 128 + 128 * 128 + 128 * 512)
        return {"bytes": M * 8.0 * (p * p + p + 2) + 8.0 * 83200 + M * 24.0,
                "flops": M * (3 * mlp + 4.0 * 8 * p * p)}
    d = 7 if case.get("family") == "inc3d" else 5
    operand = 8 * N * (k + d)
    if kind == "restrict":
        return {"bytes": operand + N + 8.0 * k * k, "flops": N * (4.0 * d * k + 4.0 * k * k)}
    # masks and right-hand sides in, solutions out, the operator and the modes;
    # an iteration applies both factors, the projection (three panel products)
    # and the vector updates
    its = ITERATIONS[kind if kind in ITERATIONS else case["family"]] * n ** 2
    return {"bytes": operand + B * N * 17.0, "flops": its * B * N * (4.0 * d + 6.0 * k + 14.0)}


# ---------------------------------------------------------------------------
# the same results in 64 bits with torch alone
# ---------------------------------------------------------------------------
def _csr(M):
    M = M.tocsr()
    return torch.sparse_csr_tensor(torch.as_tensor(M.indptr.astype(np.int64)),
                                   torch.as_tensor(M.indices.astype(np.int64)),
                                   torch.as_tensor(M.data), size=M.shape).cuda()


def _lower(R, X):
    """R^-1 X for lower triangular R, a thousand columns at a time (the
    library's workspace for more does not always fit)."""
    return torch.cat([torch.linalg.solve_triangular(R, X[..., q:q + 1024].contiguous(), upper=False)
                      for q in range(0, X.shape[-1], 1024)], -1)


class _Direct:
    """Restricted systems of S = alpha A^T A + shift I by block Cholesky.

    Rows are taken in blocks as long as the operator's reach, so S is block
    tridiagonal; active rows become rows of the identity.  Each solve is
    refined with the residual in the factored form."""

    def __init__(self, op):
        self.N = op.N
        self.A, self.At, self.shift, self.alpha = _csr(op.A), _csr(op.A.T), op.shift, op.alpha
        m = self.m = 2 * op.n ** (op.dim - 1)
        nb = self.nb = -(-op.N // m)
        C = (op.alpha * (op.A.T @ op.A)).tocoo()
        i, j = torch.as_tensor(C.row.astype(np.int64)), torch.as_tensor(C.col.astype(np.int64))
        v = torch.as_tensor(C.data)
        self.D = torch.zeros(nb, m, m, dtype=torch.float64)
        self.L = torch.zeros(nb, m, m, dtype=torch.float64)      # L[q] = S[block q + 1, block q]
        bi, bj = i // m, j // m
        on, low = bi == bj, bi == bj + 1
        self.D[bi[on], i[on] % m, j[on] % m] = v[on]
        self.L[bj[low], i[low] % m, j[low] % m] = v[low]
        self.D, self.L = self.D.cuda(), self.L.cuda()

    def apply(self, x, a, sh):
        return a[:, None] * self.alpha * (self.At @ (self.A @ x.T)).T + sh[:, None] * x

    def solve(self, masks, b, a=None, c=None):
        B = masks.shape[0]
        few = max(1, int(2e7) // self.m ** 2)        # instances factorised together
        if B > few:
            cut = lambda v, q: None if v is None else v[q:q + few]  # noqa: E731
            return torch.cat([self.solve(masks[q:q + few], b[q:q + few], cut(a, q), cut(c, q))
                              for q in range(0, B, few)])
        a = torch.ones(B, dtype=torch.float64, device="cuda") if a is None else _dev(a)
        sh = a * self.shift + (0.0 if c is None else _dev(c))
        act = masks.bool()
        b = torch.where(act, torch.zeros_like(b), b)
        pad = self.nb * self.m - self.N
        on = torch.cat([~act, torch.zeros(B, pad, dtype=torch.bool, device="cuda")], 1)
        on = on.double().reshape(B, self.nb, self.m)
        eye = torch.eye(self.m, dtype=torch.float64, device="cuda")
        R, K = [], []
        for q in range(self.nb):
            w = on[:, q]
            D = (a[:, None, None] * self.D[q] + sh[:, None, None] * eye) * w[:, :, None] * w[:, None, :]
            D = D + torch.diag_embed(1.0 - w)
            if q:
                D = D - K[-1] @ K[-1].transpose(1, 2).contiguous()
            R.append(torch.linalg.cholesky(D))
            if q + 1 < self.nb:
                L = a[:, None, None] * self.L[q] * on[:, q + 1, :, None] * w[:, None, :]
                K.append(_lower(R[-1], L.transpose(1, 2)).transpose(1, 2).contiguous())

        def once(r):
            r = torch.nn.functional.pad(r, (0, pad)).reshape(B, self.nb, self.m, 1)
            y = []
            for q in range(self.nb):
                t = r[:, q] - (K[q - 1] @ y[-1] if q else 0.0)
                y.append(_lower(R[q], t))
            x = [None] * self.nb
            for q in reversed(range(self.nb)):
                t = y[q] - (K[q].transpose(1, 2).contiguous() @ x[q + 1] if q + 1 < self.nb else 0.0)
                x[q] = torch.linalg.solve_triangular(R[q].transpose(1, 2).contiguous(), t, upper=True)
            return torch.stack(x, 1).reshape(B, -1)[:, :self.N]

        x = once(b)
        for _ in range(3):
            res = torch.where(act, torch.zeros_like(b), b - self.apply(x, a, sh))
            x = torch.where(act, torch.zeros_like(x), x + once(res))
        return x


def _exact_grad(case, seed):
    """Loss and gradient of every sample from dense matrices."""
    n, k, p, M = case["n"], case["k"], case["p"], case["M"]
    op = _operator("lap", n)
    masks, b, _, _, theta = _instances(case, seed)
    S = torch.as_tensor(op.S().toarray(), device="cuda")
    Z = _dev(_modes("lap", n, k, 0))
    Phi = _dev(np.linalg.qr(np.random.default_rng(11).standard_normal((n * n, p)))[0])
    V = torch.cat([Z, Phi], 1)
    x = _Direct(op).solve(_dev(masks, torch.uint8), _dev(b))
    H, g, e0, bx = [], [], [], []
    for m in range(M):
        on = _dev(masks[m] == 0)
        Vm, bm = V * on[:, None], _dev(b[m]) * on
        G = Vm.T @ (S @ Vm)
        r = Vm.T @ bm
        Y = torch.linalg.solve(G[:k, :k], torch.cat([G[:k, k:], r[:k, None]], 1))
        Hm = G[k:, k:] - G[k:, :k] @ Y[:, :p]
        H.append(0.5 * (Hm + Hm.T))
        g.append(r[k:] - G[k:, :k] @ Y[:, p])
        e0.append(r[:k] @ Y[:, p])
        bx.append(bm @ x[m])
    H, g, e0, bx = (torch.stack(v) for v in (H, g, e0, bx))
    q, leaves, at = gen.mlp_params(seed % 1000), [], 0
    for l in range(3):
        i, o = gen.MLP_DIMS[l], gen.MLP_DIMS[l + 1]
        W = torch.as_tensor(q[at:at + o * i].reshape(o, i)).to(torch.bfloat16).double().cuda().requires_grad_()
        c = torch.as_tensor(q[at + o * i:at + o * i + o]).double().cuda().requires_grad_()
        leaves += [W, c]
        at += o * i + o
    h = _dev(theta.astype(np.float32))
    for l in range(3):
        h = h @ leaves[2 * l].T + leaves[2 * l + 1]
        h = torch.nn.functional.gelu(h) if l < 2 else h
    C = h.reshape(M, 8, 64)[:, :, :p]
    s = (C * g[:, None, :]).sum(2)
    T = C @ H @ C.transpose(1, 2).contiguous()
    loss = 1.0 - (e0 + (s * torch.linalg.solve(T, s)).sum(1)) / bx
    loss.mean().backward()
    return {"loss": loss.detach(), "grad": torch.cat([v.grad.reshape(-1) for v in leaves])}


def _exact_restrict(case, seed):
    op = _operator("cd", case["n"])
    masks = _dev(_instances(case, seed)[0][0], torch.uint8).bool()
    Z = torch.where(masks[:, None], 0.0, _dev(_modes("cd", case["n"], case["k"], 0)))
    A, At = _csr(op.A), _csr(op.A.T)
    W = op.alpha * (At @ (A @ Z)) + op.shift * Z
    R = torch.linalg.cholesky(Z.T @ Z).T
    E = torch.linalg.solve_triangular(R, Z.T @ W, upper=True, left=False)
    E = torch.linalg.solve_triangular(R.T.contiguous(), E, upper=False)
    E = 0.5 * (E + E.T)
    return {"n_inactive": None, "k_eff": None, "cond_E": torch.linalg.cond(E), "E": E, "kept": None}


def _exact_active_set(case, seed, op):
    yd, psi = _states(case, seed)
    direct, act = _Direct(op), torch.zeros_like(yd, dtype=torch.bool)
    one = torch.ones(yd.shape[0], dtype=torch.float64, device="cuda")
    for _ in range(20):
        known = torch.where(act, psi, 0.0)
        x = direct.solve(act, yd - direct.apply(known, one, op.shift * one))
        y = torch.where(act, psi, x)
        new = y > psi - 1e-10
        if torch.equal(new, act):
            break
        act = new
    return {"y": y}


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "pod":
        X = _archive(case, seed)
        return {"Phi": None, "sigma": torch.linalg.svdvals(X - X.mean(1, keepdim=True))[:case["p"]]}
    if kind == "grad":
        return _exact_grad(case, seed)
    if kind == "restrict":
        return _exact_restrict(case, seed)
    op = _operator(_family(case), n)
    m = 2.0 * n ** (op.dim - 1)
    if case["B"] * op.N * m * m > 2e13:
        return None             # the factorisation takes too long
    if kind == "activeset":
        return _exact_active_set(case, seed, op)
    masks, b, a, c, _ = _instances(case, seed)
    a, c = _scales(case, op, a, c)
    x = _Direct(op).solve(_dev(masks, torch.uint8), _dev(b), a, c)
    return {"x": x[0] if kind == "solve" and case["B"] == 1 else x}
