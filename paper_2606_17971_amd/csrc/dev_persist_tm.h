// Persistent tile-major iteration for modes shared by the batch (gfx950,
// wave64, FP64 matrix cores): one launch runs a whole chunk of A-DEF2
// iterations for groups of 16 instances.
//
// One block owns a tile of rows for the 16 instances of a group.  Lane l of a
// wave holds row 4 s + l / 16 of the wave's rows for instance l % 16, s = 0 ..
// er - 1: the layout of the B and D operands of v_mfma_f64_16x16x4, so z and r
// go from the registers they live in straight into [Z^T z | Z^T r], and Z c
// comes out of the matrix cores in the registers of the rows it belongs to.
// The modes are read once for 16 instances; r, w, p and, while they fit, the
// Jacobi entries and x stay in registers for the chunk.  What neighbouring tiles need
// (p, and A p where it does not stay in LDS) is exchanged in rows of 16
// instances, one 128-byte line each.
//
// Communication, the handshake and the bounded waits are those of
// dev_persist.h.  The sums of p.w (16 values per tile) are added by every block
// itself; the sums of an iteration's update (2 KP + 2 values per instance and
// tile) by one leading block per instance, which runs the stopping test and the
// coarse solve and publishes coordinates, beta, r.y and whether to go on.
//
// Bound: the vector-memory pipes in the stencils (a row of 16 instances takes
// ten loads of 128 bytes, and 26 of the 45 us of an iteration at 255^2 x 16 go
// there and into the four exchanges), not HBM.  An iteration, against a kernel
// per step: 255^2 x 16, k = 32: 70.0 -> 44.7 us; 383^2 x 16: 109 -> 77;
// 191^2 x 48: 73.9 -> 59.7; 127^2 x 40: 72.3 -> 41.5.
#pragma once
#include <type_traits>

#include "dev_persist.h"

namespace adef2 {

constexpr int PT_G = 16;                  // instances per group
constexpr int PT_TB = 512;                // threads per block: half as many waves with twice the
                                          //   registers spend fewer of them on addresses
constexpr int PT_NW = PT_TB / 64;
constexpr int PT_STEP = 4 * PT_NW;        // rows of a block per step

struct PersistTmArgs {
  unsigned* flags;      // [groups][nt] step counters
  double* pw;           // [3][groups][nt][16]
  double* dots;         // [3][nb][nt][2 KP + 2]
  double* pub;          // [3][groups][16][KP + 3]: coordinates, beta, r.y, go on (0) or not
  double* P;            // rows of 16 instances, [groups][N + 2 halo][16]: p,
  double* T;            //   A p (while it goes through memory),
  double* Q;            //   z on the listed rows (when LDS does not hold them),
  double* X;            //   x and the Jacobi entries (while they are not in
  double* D;            //   registers)
  int64_t gs;           // stride of a group in P, T, Q, X, D
  unsigned* shake;
  unsigned seq, base, nblk;
  long long stall;
  int nt, ng;           // tiles, groups
  const int* ids;       // the instances of this launch (those still iterating), nb of them
  int nb;
  int rows, er;         // rows per tile (PT_STEP er) and steps
  int chunk;
  int reach1, reach, fused;
};

// The handshake takes the words of PersistArgs.
__device__ __forceinline__ PersistArgs pt_shake_args(const PersistTmArgs& a) {
  PersistArgs p{};
  p.shake = a.shake; p.seq = a.seq; p.base = a.base; p.nblk = a.nblk; p.stall = a.stall;
  return p;
}

// Value at p once it has arrived (bounded; ok becomes false past the bound).
__device__ __forceinline__ double pt_take(const double* p, unsigned* lost, bool& ok) {
  unsigned long long b = ps_bits(p);
  if (b == PS_EMPTY) {
    const long long c0 = wall_clock64();
    int n = 0;
    while ((b = ps_bits(p)) == PS_EMPTY) {
      if ((++n & 63) == 0 && (ld_agent(lost) != 0u || wall_clock64() - c0 > PS_WAIT_TICKS)) {
        st_agent(lost, 1u);
        ok = false;
        break;
      }
    }
  }
  return __longlong_as_double((long long)b);
}

// threadIdx.x that the compiler takes for a new value each time: address
// arithmetic stays in the phase that uses it
__device__ __forceinline__ int pt_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ unsigned pt_bits(unsigned v) {   // and row masks
  asm volatile("" : "+v"(v));
  return v;
}
// the same for a uniform value
__device__ __forceinline__ int pt_opaque(int n) {
  asm volatile("" : "+v"(n));
  return __builtin_amdgcn_readfirstlane(n);
}

// Sum of every 16th lane, in all of them: lanes of one instance.
__device__ __forceinline__ double pt_inst_sum(double v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// E: steps the registers are laid out for (er <= E).  Dynamic LDS: A p of the
// tile and the outer stencil's reach on both sides (pa.fused), and the waves'
// product tiles (2 x 2 x 256 doubles each) in the same place.
template <int KP, int E>
__global__ void __launch_bounds__(PT_TB) k_persist_tm(IterArgs<double, float> a, PersistTmArgs pa) {
  using M = float;
  constexpr int NV = 2 * KP + 2;
  constexpr int NP = KP + 3;
  constexpr int KS = KP / 4;                         // matrix-core steps over the modes
  constexpr int NQT = (KP + 15) / 16;                // 16-column tiles of the modes
  constexpr bool KEEPD = E <= 16;                    // the Jacobi entries in registers
  constexpr bool KEEPX = E <= 8;                     // x too
  constexpr int ED = KEEPD ? E : 1, EX = KEEPX ? E : 1;
  constexpr int U = 20;                              // tiles a leader polls together
  constexpr int CAP = 2048;                          // listed rows of a block kept in LDS
  extern __shared__ double dyn[];
  __shared__ double cfs[PT_G][KP + 1];
  __shared__ double s_beta[PT_G], s_rho[PT_G], s_alpha[PT_G], s_a[PT_G], s_c[PT_G];
  __shared__ int s_live[PT_G], s_fresh[PT_G], s_defl[PT_G], s_was[PT_G];
  __shared__ double red[PT_NW][PT_G][2];
  __shared__ double absum[PT_G][KP];
  __shared__ double gd[KP];
  __shared__ double Cl[KP <= 40 ? KP * KP : 1];      // C of the instance this block leads (if one)
  __shared__ int e0s[PT_G], e1s[PT_G];
  // the block's listed rows by instance, thread and step: their z and their
  // places in the list of boundary rows (when there are at most CAP)
  __shared__ double zb[CAP];
  __shared__ int zent[CAP];
  __shared__ int zof[PT_G + 1];
  __shared__ int zcn[PT_TB];
  // kept by the leading block of an instance
  __shared__ double s_rr[PT_G], s_pw[PT_G], s_rend[PT_G], s_thr[PT_G];
  __shared__ int s_it[PT_G], s_sw[PT_G], s_stat[PT_G], s_cap[PT_G], s_dir[PT_G], s_done[PT_G];
  __shared__ int s_bad;
  int tile, grp;
  ps_place(pa.ng, tile, grp);
  if (tile >= pa.nt) return;
  const int t0_ = threadIdx.x;
  const int wid = __builtin_amdgcn_readfirstlane(t0_ >> 6);
  const int g0 = grp * PT_G;
  const int G = min(PT_G, pa.nb - g0);
  const int* ids = pa.ids + g0;              // the group's instances
  unsigned* flag = pa.flags + (size_t)grp * pa.nt;
  unsigned* lost = pa.shake + PS_LOST;
  const size_t allpw = (size_t)pa.ng * pa.nt * PT_G, alld = (size_t)pa.nb * pa.nt * NV, allp = (size_t)pa.ng * PT_G * NP;
  // the instances this block leads, spread over the tiles
  unsigned lead = 0u;
  for (int i = 0; i < G; ++i)
    if (i * pa.nt / PT_G == tile) lead |= 1u << i;
  auto leads = [&](int i) { return (lead >> i) & 1u; };
  if (t0_ < PT_G) {
    const int i = t0_;
    s_live[i] = 0; s_fresh[i] = 0; s_defl[i] = 0;
    s_beta[i] = s_rho[i] = s_alpha[i] = s_a[i] = s_c[i] = 0.0;
    s_done[i] = 0;
    e0s[i] = e1s[i] = 0;
    if (i < G) {
      const Inst* S = a.inst + ids[i];
      s_live[i] = !S->done;
      s_fresh[i] = S->fresh;
      s_defl[i] = S->kk > 0;
      s_beta[i] = S->fresh ? 0.0 : S->beta;
      s_rho[i] = S->rho; s_alpha[i] = S->alpha; s_a[i] = S->a; s_c[i] = S->c;
      s_thr[i] = S->thresh2; s_rr[i] = S->rr; s_pw[i] = S->pw; s_rend[i] = S->rho_end;
      s_it[i] = S->iters; s_sw[i] = S->sweep_iters; s_stat[i] = S->status; s_cap[i] = S->capped; s_dir[i] = S->has_dir;
    }
    s_was[i] = s_live[i];
  }
  if (t0_ == 0) s_bad = 0;
  if (KP <= 40 && lead)
    for (int e = t0_; e < KP * KP; e += PT_TB) Cl[e] = a.C[(size_t)ids[__ffs(lead) - 1] * KP * KP + e];
  for (int e = t0_; e < PT_G * KP; e += PT_TB) {
    const int i = e / KP, q = e - i * KP;
    cfs[i][q] = i < G ? a.inst[ids[i]].coef[q] : 0.0;
  }
  // own counters and slots empty before any block is let go
  if (t0_ == 0) st_agent(flag + tile, 0u);
  auto clear = [&](int t, int slot) {
    for (int e = t; e < G * NV; e += PT_TB) {
      const int i = e / NV, v = e - i * NV;
      st_agent((unsigned long long*)(pa.dots + slot * alld + ((size_t)(g0 + i) * pa.nt + tile) * NV + v), PS_EMPTY);
    }
    if (t < PT_G)
      st_agent((unsigned long long*)(pa.pw + slot * allpw + ((size_t)grp * pa.nt + tile) * PT_G + t), PS_EMPTY);
    for (int i = 0; lead >> i; ++i)
      if (leads(i))
        for (int v = t; v < NP; v += PT_TB)
          st_agent((unsigned long long*)(pa.pub + slot * allp + ((size_t)grp * PT_G + i) * NP + v), PS_EMPTY);
  };
  for (int sl = 0; sl < 3; ++sl) clear(t0_, sl);
  if (!ps_handshake(pt_shake_args(pa))) return;
  ps_stall(pt_shake_args(pa), tile);
  const int64_t N = a.op.N;
  const int64_t base = (int64_t)tile * pa.rows;
  const int rows = (int)(N - base < pa.rows ? N - base : pa.rows);
  const int er = pa.er;
  // group's rows of 16; row i of instance j at [i * 16 + j]
  double* Pg = pa.P + grp * pa.gs;
  double* Tg = pa.T ? pa.T + grp * pa.gs : nullptr;
  double* Qg = pa.Q ? pa.Q + grp * pa.gs : nullptr;
  double* Xg = pa.X ? pa.X + grp * pa.gs : nullptr;
  double* Dg = pa.D ? pa.D + grp * pa.gs : nullptr;
  double r[E], w[E], p[E], dv[ED], x[EX];
  unsigned on = 0u, bnd = 0u;                // bit s: row inactive and inside; a listed row
  {
    const int i = t0_ & 15, j0 = wid * 4 * er + ((t0_ >> 4) & 3);
    const int id = ids[i < G ? i : 0];
    const int64_t vi = (int64_t)id * a.vs;
    const size_t mi = (size_t)id * N;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      r[s] = 0.0;
      w[s] = 0.0;
      p[s] = 0.0;
      if constexpr (KEEPD) dv[s] = 0.0;
      if constexpr (KEEPX) x[s] = 0.0;
      const int j = j0 + 4 * s;
      if (s < er && j < rows && s_live[i]) {
        const int64_t gi = base + j;
        double pv = 0.0;
        if (a.mask[mi + gi] == 0) {
          on |= 1u << s;
          r[s] = a.r[vi + gi];
          if (!s_fresh[i]) pv = a.p[vi + gi];
          p[s] = pv;
          if constexpr (KEEPD) dv[s] = a.dinv[mi + gi];
          else Dg[gi * PT_G + i] = a.dinv[mi + gi];
          w[s] = a.dinv[mi + gi] * r[s];   // z, until S p takes its place
          if constexpr (KEEPX) x[s] = a.x[vi + gi];
          else Xg[gi * PT_G + i] = a.x[vi + gi];
          if (a.bnd[mi + gi]) bnd |= 1u << s;
        }
        // the exchange buffers hold 0 on active rows
        st_agent(Pg + gi * PT_G + i, pv);
      }
    }
  }
  {
    // the listed rows of the tile: a run of the instance's list, which is in
    // row order
    if (t0_ < 2 * PT_G && (t0_ >> 1) < G) {
      const int i = t0_ >> 1;
      const int32_t* to = a.btoff + (size_t)ids[i] * (a.ub_ntiles + 1);
      int lo = to[0], hi = to[a.ub_ntiles];
      const int64_t row = (t0_ & 1) ? base + rows : base;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a.bidx[mid] < row) lo = mid + 1; else hi = mid;
      }
      ((t0_ & 1) ? e1s : e0s)[i] = lo;
    }
  }
  int zslot = 0;                             // this thread's first slot in zb
  bool inlds = false;
  {
    zcn[t0_] = __popc(bnd);
    __syncthreads();
    if (t0_ < PT_G) {
      int n = 0;
      for (int q = t0_; q < PT_TB; q += PT_G) n += zcn[q];
      zof[t0_ + 1] = n;
    }
    __syncthreads();
    if (t0_ == 0) {
      zof[0] = 0;
      for (int q = 0; q < PT_G; ++q) zof[q + 1] += zof[q];
    }
    __syncthreads();
    inlds = zof[PT_G] <= CAP;
    const int i = t0_ & 15;
    zslot = zof[i];
    for (int q = i; q < t0_; q += PT_G) zslot += zcn[q];
    if (inlds) {
      int k = zslot;
#pragma unroll
      for (int s = 0; s < E; ++s)
        if ((bnd >> s) & 1u) {
          const int row = (int)base + wid * 4 * er + ((t0_ >> 4) & 3) + 4 * s;
          int lo = e0s[i], hi = e1s[i];
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (a.bidx[mid] < row) lo = mid + 1; else hi = mid;
          }
          zent[k++] = lo;
        }
    }
  }
  __syncthreads();
  bool ok = true;
  unsigned step = 0u;
  auto exchange = [&](int t, int h) {
    ++step;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    wait_mem();
    __syncthreads();
    if (t == 0) st_agent(flag + tile, step);
    const int lo = (int)(base - h < 0 ? 0 : (base - h) / pa.rows);
    const int hi = (int)min((int64_t)pa.nt - 1, (base + rows - 1 + h) / pa.rows);
    bool f = true;
    for (int q = lo + t; q <= hi; q += PT_TB) f = ps_wait_ge(flag + q, step, lost) && f;
    if (!f) s_bad = 1;
    __syncthreads();
    ok = !s_bad;
  };
  // w = the operator's stencils on the inactive rows of v (rows of 16), without
  // the scale and the shift; DC: diagonals of both stencils, the main one in the
  // middle
  auto sweep = [&](auto dc, int64_t Nq, const double* v) {
    constexpr int DC = decltype(dc)::value;
    constexpr int D0 = DC / 2;
    // rows whose loads are in flight together
    constexpr int RB = (E <= 8 ? 8 : 4) / (DC > 5 ? 2 : 1);
    const int t = pt_tid();
    const unsigned m = pt_bits(on);
    const bool live = s_live[t & 15] != 0;
    const int i = t & 15, j0 = wid * 4 * er + ((t >> 4) & 3);
    const M* o = a.dia + base;
    auto combine = [&](const M (&cw)[DC], const double (&vw)[DC]) {
      double acc = (double)cw[D0] * vw[D0];
#pragma unroll
      for (int d = 0; d < DC; ++d)
        if (d != D0) acc += (double)cw[d] * (vw[d] - vw[D0]);
      return acc;
    };
    if (a.op.D1 && pa.fused) {
      exchange(t, pa.reach + pa.reach1);
      if (!ok) return;
      const int64_t lo = base - pa.reach;
      const int jl = lo < 0 ? (int)-lo : 0;                       // rows inside: jl <= j < jh
      const int jh = (int)min((int64_t)(rows + 2 * pa.reach), Nq - lo);
      const int J = rows + 2 * pa.reach;
      if (live)
#pragma unroll 1
        for (int b0 = t >> 4; b0 < J; b0 += RB * (PT_TB / PT_G)) {
          double vw[RB][DC];
          M cw[RB][DC];
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const int j = b0 + u * (PT_TB / PT_G);
            const unsigned jc = j < jl ? jl : j < jh ? j : jh - 1;
#pragma unroll
            for (int d = 0; d < DC; ++d) {
              cw[u][d] = (a.dia1 + lo + (size_t)d * Nq)[jc];
              vw[u][d] = ld_agent(v + (lo + a.op.offs1[d]) * PT_G + (jc * PT_G + i));
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const int j = b0 + u * (PT_TB / PT_G);
            if (j < J) dyn[j * PT_G + i] = j >= jl && j < jh ? combine(cw[u], vw[u]) : 0.0;
          }
        }
      __syncthreads();
#pragma unroll
      for (int s0 = 0; s0 < E; s0 += RB) {
        M cw[RB][DC];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          const int j = j0 + 4 * (s0 + u);
          const unsigned jc = j < rows ? j : rows - 1;
#pragma unroll
          for (int d = 0; d < DC; ++d) cw[u][d] = (o + (size_t)d * Nq)[jc];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          const int s = s0 + u;
          if (s < E && ((m >> s) & 1u)) {
            double vw[DC];
#pragma unroll
            for (int d = 0; d < DC; ++d) vw[d] = dyn[(j0 + 4 * s + pa.reach + a.op.offs[d]) * PT_G + i];
            w[s] = combine(cw[u], vw);
          }
        }
      }
      return;
    }
    // rows of the tile from memory: st(s, value) for each
    auto rowsof = [&](const M* c, const int* offs, const double* src, auto st) {
#pragma unroll
      for (int s0 = 0; s0 < E; s0 += RB) {
        if (s0 >= er) break;
        double vw[RB][DC];
        M cw[RB][DC];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          const int j = j0 + 4 * (s0 + u);
          const unsigned jc = j < rows ? j : rows - 1;
#pragma unroll
          for (int d = 0; d < DC; ++d) {
            cw[u][d] = (c + (size_t)d * Nq)[jc];
            vw[u][d] = ld_agent(src + (base + offs[d]) * PT_G + (jc * PT_G + i));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < RB; ++u)
          if (s0 + u < E) st(s0 + u, combine(cw[u], vw[u]));
      }
    };
    const double* src = v;
    if (a.op.D1) {
      exchange(t, pa.reach1);
      if (!ok) return;
      rowsof(a.dia1 + base, a.op.offs1, v, [&](int s, double x) {
        const int j = j0 + 4 * s;
        if (s < er && j < rows && live) st_agent(Tg + base * PT_G + (unsigned)(j * PT_G + i), x);
      });
      src = Tg;
    }
    exchange(t, pa.reach);
    if (!ok) return;
    rowsof(o, a.op.offs, src, [&](int s, double x) {
      if ((m >> s) & 1u) w[s] = x;
    });
  };
  // element of row s of this thread in a tile's rows of 16
  auto at = [&](int t, int s) { return (unsigned)((wid * 4 * er + ((t >> 4) & 3) + 4 * s) * PT_G + (t & 15)); };
  auto jac = [&](int t, unsigned m, int s) -> double {
    if constexpr (KEEPD) return dv[s];
    else return ((m >> s) & 1u) ? (Dg + base * PT_G)[at(t, s)] : 0.0;
  };

  for (int it = 0; it < pa.chunk; ++it) {
    const int slot = it % 3;
    const int64_t Nq = pt_opaque((int)N);
    double* pws = pa.pw + slot * allpw + (size_t)grp * pa.nt * PT_G;
    double* pub = pa.pub + slot * allp + (size_t)grp * PT_G * NP;
    {
      const int t = pt_tid();
      if (!__any(s_live[t & 15] != 0)) break;  // the same for every wave and block of the group
      if (it >= 2) clear(t, (it + 1) % 3);
    }
    // p = z - Z c + beta p: 16 rows x 16 instances of Z c per matrix-core tile
    {
      const int t = pt_tid();
      const unsigned m = pt_bits(on);
      const int i = t & 15, kk = (t >> 4) & 3, wb = wid * 4 * er;
      const bool live = s_live[i] != 0;
      double cb[KS];
#pragma unroll
      for (int q = 0; q < KS; ++q) cb[q] = s_defl[i] ? cfs[i][kk * KS + q] : 0.0;
      const double beta = s_beta[i];
      const bool fresh = s_fresh[i] != 0;
      constexpr int NS = (E + 3) / 4;
      // the modes of one 16-row slice (z is in w)
      auto load = [&](int S, M (&zf)[KS]) {
        const int64_t gr = base + wb + 16 * S + i;       // operand A: row l % 16
        const unsigned zr = (unsigned)(gr < Nq ? gr : Nq - 1);
#pragma unroll
        for (int q = 0; q < KS; ++q) zf[q] = a.ZT[(size_t)zr * KP + kk * KS + q];
      };
      M zf[2][KS];
      load(0, zf[0]);
#pragma unroll
      for (int S = 0; S < NS; ++S) {
        if (4 * S >= er) break;
        if (S + 1 < NS) load(S + 1, zf[(S + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        tm_d4 d = tm_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < KS; ++q)
          d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)zf[S & 1][q], cb[q], d, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int s = 4 * S + e;
          if (s < E && ((m >> s) & 1u) && live) {
            double pn = w[s] - d[e];
            if (!fresh) pn += beta * p[s];
            p[s] = pn;
            st_agent(Pg + base * PT_G + at(t, s), pn);
          }
        }
      }
    }
    // w = S p, p.w
    if (a.op.D == 5) sweep(std::integral_constant<int, 5>{}, Nq, Pg);
    else sweep(std::integral_constant<int, 7>{}, Nq, Pg);
    if (!ok) break;
    {
      const int t = pt_tid();
      const unsigned m = pt_bits(on);
      const int i = t & 15, lane = t & 63;
      const bool live = s_live[i] != 0;
      const double sa = s_a[i], sc = s_c[i];
      double sum = 0.0;
#pragma unroll
      for (int s = 0; s < E; ++s)
        if ((m >> s) & 1u) {
          w[s] = sa * w[s] + sc * p[s];
          sum += p[s] * w[s];
        }
      sum = pt_inst_sum(sum);
      if (lane < PT_G) red[wid][i][0] = sum;
      __syncthreads();
      if (t < PT_G && live) {
        double b = 0.0;
#pragma unroll
        for (int q = 0; q < PT_NW; ++q) b += red[q][t][0];
        st_agent(pws + (size_t)tile * PT_G + t, b);
      }
      // every block adds the tiles' sums: thread (tile mod 32, instance)
      sum = 0.0;
      if (live) {
        for (int q0 = t >> 4; q0 < pa.nt; q0 += 8 * (PT_TB / PT_G)) {
          unsigned long long b[8];
          bool wait = true;
          int n = 0;
          long long c0 = 0;
#pragma unroll 1
          while (wait) {
            wait = false;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              const int q = q0 + u * (PT_TB / PT_G);
              b[u] = q < pa.nt ? ps_bits(pws + (size_t)q * PT_G + i) : 0ull;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) wait |= b[u] == PS_EMPTY;
            if (wait && (++n & 63) == 0) {
              if (n == 64) c0 = wall_clock64();
              if (ld_agent(lost) != 0u || wall_clock64() - c0 > PS_WAIT_TICKS) {
                st_agent(lost, 1u);
                ok = wait = false;
              }
            }
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) sum += __longlong_as_double((long long)b[u]);
          if (!ok) break;
        }
      }
      sum = pt_inst_sum(sum);
      if (lane < PT_G) red[wid][i][1] = sum;
      if (!ok) s_bad = 1;
      __syncthreads();
      if (s_bad) { ok = false; break; }
    }
    {
      const int t = pt_tid();
      const unsigned m = pt_bits(on), mb = pt_bits(bnd);
      const int i = t & 15, lane = t & 63;
      bool live = s_live[i] != 0;
      double pw = 0.0;
#pragma unroll
      for (int q = 0; q < PT_NW; ++q) pw += red[q][i][1];
      const bool broke = live && (!(pw > 0.0) || !(pw < INFINITY));
      const double alpha = s_rho[i] / pw;
      __syncthreads();                         // every thread has read the live flags and sums
      if (t < PT_G && live) {
        s_pw[t] = pw;
        if (broke) { s_live[t] = 0; s_done[t] = 2; s_stat[t] = -5; }
        else s_alpha[t] = alpha;
      }
      live = live && !broke;
      // x += alpha p, r -= alpha w, z = K r; what is not in registers is loaded
      // UB rows at a time
      double rz = 0.0, rr = 0.0;
      constexpr int UB = KEEPX ? E : 8;
      int k = zslot;
#pragma unroll
      for (int s0 = 0; s0 < E; s0 += UB) {
        double xl[UB], dl[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int s = s0 + u;
          xl[u] = dl[u] = 0.0;
          if (s < E && ((m >> s) & 1u)) {
            if constexpr (!KEEPX) xl[u] = (Xg + base * PT_G)[at(t, s)];
            if constexpr (!KEEPD) dl[u] = jac(t, m, s);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int s = s0 + u;
          if (s < E && ((m >> s) & 1u) && live) {
            double ds;
            if constexpr (KEEPD) ds = dv[s]; else ds = dl[u];
            if constexpr (KEEPX) x[s] += alpha * p[s];
            else (Xg + base * PT_G)[at(t, s)] = xl[u] + alpha * p[s];
            r[s] -= alpha * w[s];
            const double zs = ds * r[s];
            rz += r[s] * zs;
            rr += r[s] * r[s];
            w[s] = zs;
            if ((mb >> s) & 1u) {
              if (inlds) zb[k++] = zs;
              else (Qg + base * PT_G)[at(t, s)] = zs;
            }
          }
        }
      }
      rz = pt_inst_sum(rz);
      rr = pt_inst_sum(rr);
      if (lane < PT_G) { red[wid][i][0] = rz; red[wid][i][1] = rr; }
    }
    __syncthreads();                           // the LDS of A p is free, red is written
    // [Z^T z | Z^T r], two 16-column tiles at a time
#pragma unroll 1
    for (int qp = 0; qp < NQT; qp += 2) {
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        const int qt = qp + qh;
        if (qt < NQT) {
          const int t = pt_tid();
          const unsigned m = pt_bits(on);
          const int i = t & 15, lane = t & 63, j0 = wid * 4 * er + ((t >> 4) & 3);
          tm_d4 dz = tm_d4{0.0, 0.0, 0.0, 0.0}, dr = dz;
          const int q = qt * 16 + i;
          const bool col = KP % 16 == 0 || q < KP;
          constexpr int EC = E <= 16 ? E : (E + 1) / 2;  // rows loaded together
#pragma unroll
          for (int sc = 0; sc < E; sc += EC) {
            M zf[EC];
#pragma unroll
            for (int u = 0; u < EC; ++u) {
              const int64_t gr = base + j0 + 4 * (sc + u);
              const unsigned zr = (unsigned)(gr < Nq ? gr : Nq - 1);
              zf[u] = (M)0;
              if (sc + u < er && col) zf[u] = a.ZT[(size_t)zr * KP + q];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < EC; ++u) {
              const int s = sc + u;
              if (s < E && s < er) {
                const double zs = w[s];
                dz = __builtin_amdgcn_mfma_f64_16x16x4f64((double)zf[u], zs, dz, 0, 0, 0);
                dr = __builtin_amdgcn_mfma_f64_16x16x4f64((double)zf[u], r[s], dr, 0, 0, 0);
              }
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            dyn[(((wid * 2 + qh) * 2 + 0) * 4 + e) * 64 + lane] = dz[e];
            dyn[(((wid * 2 + qh) * 2 + 1) * 4 + e) * 64 + lane] = dr[e];
          }
        }
      }
      if (qp == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        wait_mem();                            // z on the listed rows is in place
      }
      __syncthreads();
      const int t = pt_tid();
      const int i = t & 15, lane = t & 63, kk = lane >> 4;
      {
        if (qp == 0) {
          // the listed rows of instances wid, wid + PT_NW: 64 / KL entries per
          // step, lanes over the columns, in a fixed order
          constexpr int KL = KP <= 32 ? 32 : 64;
          const int bq = lane % KL, sub = lane / KL;
#pragma unroll 1
          for (int li = wid; li < PT_G; li += PT_NW) {
            double ab = 0.0;
            const bool want = s_live[li] && s_defl[li];
            if (inlds) {
              const int k1 = want ? zof[li + 1] : 0;
              for (int k = zof[li] + sub; k < k1; k += 16 * (64 / KL)) {
                M bw[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                  const int q = k + u * (64 / KL);
                  bw[u] = (M)0;
                  if (q < k1 && bq < KP) bw[u] = a.bW[(size_t)zent[q] * KP + bq];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                  const int q = k + u * (64 / KL);
                  // (past the end: slot 0 is another instance's, which may hold Inf)
                  ab += (double)bw[u] * (q < k1 ? zb[q] : 0.0);
                }
              }
            } else {
              const int e1 = want ? e1s[li] : 0;
              for (int e = e0s[li] + sub; e < e1; e += 64 / KL)
                ab += (bq < KP ? (double)a.bW[(size_t)e * KP + bq] : 0.0) * Qg[(int64_t)a.bidx[e] * PT_G + li];
            }
            if (KL == 32) ab += __shfl_down(ab, 32, 64);
            if (sub == 0 && bq < KP) absum[li][bq] = ab;
          }
          __syncthreads();
        }
      }
      // sums over the waves: (column tile, z or r, element, lane of D)
      const bool live = s_live[i] != 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = (t >> 8) & 1, e = (t >> 6) & 3;
        const int q = (qp + h) * 16 + 4 * e + kk;
        if (qp + h < NQT && q < KP && live) {
          double b = 0.0;
#pragma unroll
          for (int v = 0; v < PT_NW; ++v) b += dyn[(((v * 2 + h) * 2 + c) * 4 + e) * 64 + lane];
          if (!s_defl[i]) b = 0.0;
          else if (c == 0) b = (s_a[i] * a.mu[q] + s_c[i]) * b + absum[i][q];
          st_agent(pa.dots + slot * alld + ((size_t)(g0 + i) * pa.nt + tile) * NV + c * KP + q, b);
        }
      }
      if (qp == 0 && t < 2 * PT_G && live) {
        const int c = t >> 4;
        double b = 0.0;
#pragma unroll
        for (int q = 0; q < PT_NW; ++q) b += red[q][i][c];
        st_agent(pa.dots + slot * alld + ((size_t)(g0 + i) * pa.nt + tile) * NV + 2 * KP + c, b);
      }
      if (qp + 2 < NQT) __syncthreads();
    }
    // the leading block of an instance: totals, stopping test, coarse solve
#pragma unroll 1
    for (int li = 0; lead >> li; ++li) {
      if (!leads(li)) continue;
      __syncthreads();
      if (!s_live[li]) continue;
      const int t = pt_tid(), lane = t & 63;
      constexpr int GR = PT_TB / NV;           // thread groups
      const int g = t / NV, v = t - g * NV;
      const double* ds = pa.dots + slot * alld + (size_t)(g0 + li) * pa.nt * NV;
      double sum = 0.0;
      if (g < GR)
#pragma unroll 1
        for (int q0 = g; q0 < pa.nt && ok; q0 += GR * U) {
          unsigned long long b[U];
          bool wait = true;
          int n = 0;
          long long c0 = 0;
#pragma unroll 1
          while (wait) {
            wait = false;
#pragma unroll
            for (int u = 0; u < U; ++u)
              b[u] = q0 + u * GR < pa.nt ? ps_bits(ds + (q0 + u * GR) * NV + v) : 0ull;
#pragma unroll
            for (int u = 0; u < U; ++u) wait |= b[u] == PS_EMPTY;
            if (wait && (++n & 63) == 0) {
              if (n == 64) c0 = wall_clock64();
              if (ld_agent(lost) != 0u || wall_clock64() - c0 > PS_WAIT_TICKS) {
                st_agent(lost, 1u);
                ok = wait = false;
              }
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) sum += __longlong_as_double((long long)b[u]);
        }
      dyn[t] = sum;
      if (!ok) s_bad = 1;
      __syncthreads();
      if (s_bad) { ok = false; break; }
      if (wid == 0) {
        double tz = 0.0, tr = 0.0, rz = 0.0, rr2 = 0.0;
#pragma unroll 4
        for (int q = 0; q < GR; ++q) {
          if (lane < KP) {
            tz += dyn[q * NV + lane];
            tr += dyn[q * NV + KP + lane];
          }
          rz += dyn[q * NV + 2 * KP];
          rr2 += dyn[q * NV + 2 * KP + 1];
        }
        double corr = 0.0, cq = 0.0;
        if (s_defl[li]) {
          if (lane < KP) {
            gd[lane] = tz - tr;
            double c1 = 0.0;
            auto solve = [&](const double* Cm) {
#pragma unroll 8
              for (int l = 0; l < KP; l += 2) {
                cq += Cm[l * KP + lane] * gd[l];
                c1 += Cm[(l + 1) * KP + lane] * gd[l + 1];
              }
            };
            if (KP <= 40 && !(lead & (lead - 1u))) solve(Cl);
            else solve(a.C + (size_t)ids[li] * KP * KP);
            cq += c1;
          }
          corr = ps_wave_sum(lane < KP ? tr * cq : 0.0);
        }
        const double rho = rz - corr, rho_o = s_rho[li];
        const int its = s_it[li] + 1, sw = s_sw[li] + 1;
        int go = 1;
        if (!(rr2 > s_thr[li]) || (a.seg_maxit > 0 && sw >= a.seg_maxit)) go = rr2 < INFINITY ? 2 : 0;
        else if (its >= a.maxit) go = 3;
        double* o = pub + (size_t)li * NP;
        if (lane < KP) st_agent(o + lane, cq);
        if (lane == 0) {
          s_it[li] = its;
          s_sw[li] = sw;
          s_rr[li] = rr2;
          if (go == 2) { s_done[li] = 1; s_cap[li] = rr2 > s_thr[li]; s_rend[li] = rho; s_dir[li] = 1; }
          else if (go == 0) { s_done[li] = 2; s_stat[li] = -5; s_cap[li] = rr2 > s_thr[li]; }
          else if (go == 3) { s_done[li] = 2; s_stat[li] = 2; }
          st_agent(o + KP, go == 1 ? rho / rho_o : s_beta[li]);
          st_agent(o + KP + 1, go == 1 ? rho : rho_o);
          st_agent(o + KP + 2, go == 1 ? 0.0 : 1.0);
        }
      }
    }
    if (!ok) break;
    __syncthreads();
    // the next coordinates, beta and r.y of the group's iterating instances
    {
      const int t = pt_tid();
#pragma unroll 1
      for (int e = t; e < G * NP; e += PT_TB) {
        const int li = e / NP, v = e - li * NP;
        if (!s_live[li]) continue;
        const double b = pt_take(pub + e, lost, ok);
        if (v < KP) cfs[li][v] = b;
        else if (v == KP) s_beta[li] = b;
        else if (v == KP + 1) s_rho[li] = b;
        else s_was[li] = b == 0.0 ? 1 : 2;     // 2: ends here
      }
      if (!ok) s_bad = 1;
      __syncthreads();
      if (s_bad) { ok = false; break; }
      if (t < PT_G && s_live[t]) {
        if (s_was[t] == 2) s_live[t] = 0;
        else s_fresh[t] = 0;
      }
      __syncthreads();
    }
  }
  {
    const int i = t0_ & 15, j0 = wid * 4 * er + ((t0_ >> 4) & 3);
    const int id = ids[i < G ? i : 0];
    const int64_t vi = (int64_t)id * a.vs;
#pragma unroll
    for (int s = 0; s < E; ++s)
      if ((on >> s) & 1u) {
        const int64_t gi = base + j0 + 4 * s;
        double xs, zs;
        if constexpr (KEEPX) xs = x[s]; else xs = Xg[gi * PT_G + i];
        if constexpr (KEEPD) zs = dv[s] * r[s]; else zs = a.dinv[(size_t)id * N + gi] * r[s];
        a.x[vi + gi] = xs;
        a.r[vi + gi] = r[s];
        a.z[vi + gi] = zs;
        a.p[vi + gi] = p[s];
      }
  }
  __syncthreads();
  for (int i = 0; i < G; ++i) {
    if (!leads(i) || !s_was[i]) continue;      // s_was is 0 for instances idle from the start
    Inst* S = a.inst + ids[i];
    for (int q = t0_; q < KP; q += PT_TB) S->coef[q] = cfs[i][q];
    if (t0_ == 0) {
      S->rho = s_rho[i]; S->beta = s_beta[i]; S->alpha = s_alpha[i]; S->rr = s_rr[i]; S->pw = s_pw[i];
      S->rho_end = s_rend[i]; S->iters = s_it[i]; S->sweep_iters = s_sw[i]; S->fresh = s_fresh[i];
      S->capped = s_cap[i]; S->has_dir = s_dir[i]; S->status = s_stat[i];
      if (s_done[i]) S->done = 1;
      if (s_done[i] == 2) S->outer_done = 1;
    }
  }
}

}  // namespace adef2
