// Persistent form of the per-instance iteration (gfx950, wave64): one launch
// runs a whole chunk of A-DEF2 iterations.
//
// One block owns R consecutive rows of one instance and keeps their x, r, z,
// p and Jacobi entries in registers for the whole chunk; the blocks of an
// instance (its team) exchange the search direction p and, for the factored
// operator, t = A p with the neighbouring tiles through memory, and every
// block adds the team's partial sums itself, in tile order, so all of them
// hold the same totals and take the same decisions.  Per iteration this costs
// four waits on other blocks instead of four to five kernel boundaries with a
// reduction tree each, and none of the vector traffic.
//
// All communication is by agent-scope stores and loads, which are coherent
// across the XCDs; a wait polls
//   - one step counter per tile (flags), published after the tile's stores
//     have completed, or
//   - the partial sums themselves: a slot holds a signalling NaN, which no
//     arithmetic produces, until its value arrives.  The slots rotate by three:
//     a block reaches iteration i only after every block of its team has read
//     the sums of iteration i - 2, so it may clear those then.
// What bounds it: the four waits (1 us each with 16 blocks, 1.4-2 us with 64, 3 us
// with 256), then the panel products.  Whole solves, one kernel per step against this:
// 63^2, k = 16, FP64 34.6 / 10.1 ms; 255^2, k = 40, FP64 427 / 182 ms;
// 191^2 x 5, k = 32, mixed 201 / 101 ms; 127^2 x 16 with learned vectors
// (k = 40 per instance), FP64 108 / 60 ms; 100^2 x 30 active-set loop, k = 40,
// FP64 170 / 119 ms.
// Every block must be resident.  The launch has at most as many blocks as fit
// the device, and begins with a handshake: a block that does not see all of
// them arrive in time (other work may hold compute units) calls the launch
// off; nothing has been changed then and the host goes on with one kernel per
// step.  Waits after the handshake are bounded too: when a block gives one up the
// host solves again with one kernel per step.
#pragma once
#include "dev_kernels.h"

namespace adef2 {

constexpr int PS_TB = 512;              // threads per block
constexpr int PS_NW = PS_TB / 64;
constexpr long long PS_SHAKE_TICKS = 2000000;      // 20 ms of the 100 MHz counter
constexpr long long PS_WAIT_TICKS = 400000000;     // 4 s
constexpr unsigned long long PS_EMPTY = 0x7FF4A5A55A5A4321ull;   // signalling NaN

// PS_DECISION: 2 seq of the last launch when it was called off, else 2 seq + 1.
// PS_LOST: 1 when a block gave up a wait (PS_GIVE_UP: none has, but every one is to
// that waits for long).  The host clears the words, and reads these two where it
// reads the instances' states.
enum { PS_ARRIVED = 0, PS_DECISION = 16, PS_LOST = 32, PS_WORDS = 48 };
enum { PS_GIVE_UP = 2 };

struct PersistArgs {
  unsigned* flags;      // [nb][nt] step counters
  double* pw;           // [3][nb][nt] partial sums of p.w
  double* dots;         // [3][nb][nt][2 KP + 2] partial sums of the update
  unsigned* shake;      // PS_WORDS words
  long long stall;      // tests: the first tiles start late by this many ticks
  unsigned seq;         // number of this launch (from 2: 2 seq - 2 is not 0)
  unsigned base;        // arrivals before this launch
  unsigned nblk;        // blocks that arrive
  int nt;               // tiles of an instance
  const int* ids;       // the instances of this launch (those still iterating), nb of them
  int nb;
  int chunk;            // iterations
  int reach1, reach;    // reach of the inner (factored) and of the outer stencil
  int fused;            // the inner product stays in LDS, its halo formed twice
};

template <typename T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tile and instance (or group of instances) of this block, n of them per tile,
// in a grid of 8 * ceil(nt n / 8) blocks (tile >= nt: nothing to do).  Blocks go
// to the 8 XCDs in turn, each XCD owning a contiguous range of (tile, instance):
// every XCD then has the same number of blocks to hold, where whole tiles per
// XCD leave some with more than fit (25 tiles x 20 instances: 80 on an XCD that
// holds 64) and the launch is called off.
__device__ __forceinline__ void ps_place(int n, int& tile, int& which) {
  const int id = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  tile = id / n;
  which = id - tile * n;
}

// Poll until *p reaches v (step counters grow); false when the bound passed.
__device__ __forceinline__ bool ps_wait_ge(const unsigned* p, unsigned v, unsigned* lost) {
  if ((int)(ld_agent(p) - v) >= 0) return true;
  const long long t0 = wall_clock64();
  for (;;) {
    for (int i = 0; i < 64; ++i)
      if ((int)(ld_agent(p) - v) >= 0) return true;
    if (ld_agent(lost) != 0u || wall_clock64() - t0 > PS_WAIT_TICKS) {
      st_agent(lost, 1u);
      return false;
    }
  }
}

__device__ __forceinline__ unsigned long long ps_bits(const double* p) {
  return ld_agent((const unsigned long long*)p);
}

// Every block of the launch calls this once.  True: all blocks are resident
// and every one of them was told so.  False: the launch is called off, at once if
// the one before it was.
__device__ inline bool ps_handshake(const PersistArgs& a) {
  __shared__ int s_go;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  wait_mem();
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned* dec = a.shake + PS_DECISION;
    const unsigned go = 2u * a.seq + 1u, off = 2u * a.seq;
    const unsigned old = __hip_atomic_fetch_add(a.shake + PS_ARRIVED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned cur = ld_agent(dec);
    const bool behind = cur == off - 2u;       // the launch before was called off
    const bool last = old - a.base == a.nblk - 1u && !behind;
    const long long t0 = wall_clock64();
    while (cur != go && cur != off) {
      const bool late = behind || wall_clock64() - t0 > PS_SHAKE_TICKS;
      if (last || late) {
        unsigned want = cur;
        if (__hip_atomic_compare_exchange_strong(dec, &want, last ? go : off, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
          cur = last ? go : off;
        else
          cur = want;
      } else {
        __builtin_amdgcn_s_sleep(1);
        cur = ld_agent(dec);
      }
    }
    s_go = cur == go;
  }
  __syncthreads();
  return s_go != 0;
}

__device__ __forceinline__ void ps_stall(const PersistArgs& a, int tile) {
  if (a.stall == 0 || tile != 0) return;
  const long long t0 = wall_clock64();
  while (wall_clock64() - t0 < a.stall) __builtin_amdgcn_s_sleep(8);
}

// Sum over the 64 lanes, in every lane: four DPP steps add the 16 lanes of a
// row (quad swaps, then mirrored halves and rows; each step is symmetric, so
// all lanes hold the same bits), the four row sums come over scalar registers.
// About 150 cycles; the shuffle tree through LDS takes about 900.
template <int CTRL>
__device__ __forceinline__ double ps_dpp(double v) {
  union { double d; int i[2]; } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, 0xf, 0xf, true);
  return b.d;
}
__device__ __forceinline__ double ps_row_sum(double v) {
  v += ps_dpp<0xB1>(v);     // quad_perm [1, 0, 3, 2]
  v += ps_dpp<0x4E>(v);     // quad_perm [2, 3, 0, 1]
  v += ps_dpp<0x141>(v);    // row_half_mirror
  v += ps_dpp<0x140>(v);    // row_mirror
  return v;
}
__device__ __forceinline__ double ps_lane(double v, int lane) {
  union { double d; int i[2]; } a;
  a.d = v;
  a.i[0] = __builtin_amdgcn_readlane(a.i[0], lane);
  a.i[1] = __builtin_amdgcn_readlane(a.i[1], lane);
  return a.d;
}
__device__ __forceinline__ double ps_wave_sum(double v) {
  v = ps_row_sum(v);
  return (ps_lane(v, 0) + ps_lane(v, 16)) + (ps_lane(v, 32) + ps_lane(v, 48));
}

// Sums over the lanes of PG values (at most 16): lane g < PG holds value g.
template <int PG>
__device__ __forceinline__ double ps_lane_sums(double (&v)[PG], int lane) {
  double s = 0.0;
#pragma unroll
  for (int g = 0; g < PG; ++g) {
    const double r = ps_row_sum(v[g]);
    s = (lane & 15) == g ? r : s;
  }
  s += __shfl_xor(s, 16, 64);
  s += __shfl_xor(s, 32, 64);
  return s;
}

// out[q] = sum over the tile's rows of col(q)[row] * vec(q)[row], q < NQ;
// wave w takes the columns w, w + PS_NW, ...; PG columns are loaded before any
// is used, 32 loads per lane at the most
template <typename M, int R, int NQ, typename ColF, typename VecF>
__device__ __forceinline__ void ps_panel_dots(int rows, ColF col, VecF vec, double* out) {
  constexpr int RL = R / 64;                          // rows per lane
  constexpr int NQW = (NQ + PS_NW - 1) / PS_NW;       // columns per wave
  constexpr int PM = RL >= 32 ? 1 : RL >= 16 ? 2 : RL >= 8 ? 4 : 8;
  constexpr int PG = PM < NQW ? PM : NQW;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll 1
  for (int s0 = 0; s0 < NQW; s0 += PG) {
    M c[PG][RL];
#pragma unroll
    for (int g = 0; g < PG; ++g) {
      const int q = wid + (s0 + g) * PS_NW;
      const M* cp = col(q < NQ ? q : 0);
#pragma unroll
      for (int u = 0; u < RL; ++u) {
        const unsigned j = lane + 64 * u;
        c[g][u] = cp[j < (unsigned)rows ? j : 0u];
      }
    }
    __builtin_amdgcn_sched_barrier(0);                // every load before the first use
    double acc[PG];
#pragma unroll
    for (int g = 0; g < PG; ++g) {
      const int q = wid + (s0 + g) * PS_NW;
      const double* v = vec(q < NQ ? q : 0);
      acc[g] = 0.0;
#pragma unroll
      for (int u = 0; u < RL; ++u) acc[g] += (double)c[g][u] * v[lane + 64 * u];
    }
    const double tot = ps_lane_sums<PG>(acc, lane);
    const int s = s0 + lane, q = wid + s * PS_NW;
    if (lane < PG && s < NQW && q < NQ) out[q] = tot;
  }
}

// The same for one panel and two vectors: out[q] = col(q).v0, out[NQ + q] = col(q).v1
template <typename M, int R, int NQ, typename ColF>
__device__ __forceinline__ void ps_panel_dots2(int rows, ColF col, const double* v0, const double* v1, double* out) {
  constexpr int RL = R / 64;
  constexpr int NQW = (NQ + PS_NW - 1) / PS_NW;
  constexpr int PM = RL >= 32 ? 1 : RL >= 16 ? 2 : RL >= 8 ? 4 : 8;
  constexpr int PG = PM < NQW ? PM : NQW;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll 1
  for (int s0 = 0; s0 < NQW; s0 += PG) {
    M c[PG][RL];
#pragma unroll
    for (int g = 0; g < PG; ++g) {
      const int q = wid + (s0 + g) * PS_NW;
      const M* cp = col(q < NQ ? q : 0);
#pragma unroll
      for (int u = 0; u < RL; ++u) {
        const unsigned j = lane + 64 * u;
        c[g][u] = cp[j < (unsigned)rows ? j : 0u];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    double acc[2 * PG];
#pragma unroll
    for (int g = 0; g < 2 * PG; ++g) acc[g] = 0.0;
#pragma unroll
    for (int u = 0; u < RL; ++u) {
      const double a0 = v0[lane + 64 * u], a1 = v1[lane + 64 * u];
#pragma unroll
      for (int g = 0; g < PG; ++g) {
        acc[2 * g] += (double)c[g][u] * a0;
        acc[2 * g + 1] += (double)c[g][u] * a1;
      }
    }
    const double tot = ps_lane_sums<2 * PG>(acc, lane);
    const int s = s0 + lane / 2, q = wid + s * PS_NW;
    if (lane < 2 * PG && s < NQW && q < NQ) out[(lane & 1) * NQ + q] = tot;
  }
}

// This thread's share of the sums of NV values over the nt tiles of a team:
// thread (g, v) adds slot[tile][v] over the tiles g, g + G, ... in that order,
// each polled until it has arrived (PS_U polled together, and no more groups G
// than that leaves work for).  ok becomes false when a wait passed its bound.
constexpr int PS_U = 8;
template <int NV>
__device__ __forceinline__ int ps_groups(int nt) {
  constexpr int most = PS_TB / NV;
  const int g = NV == 1 ? PS_TB : (nt + PS_U - 1) / PS_U;
  return g < most ? g : most;
}
template <int NV>
__device__ __forceinline__ double ps_gather(const double* slot, int nt, unsigned* lost, bool& ok) {
  constexpr int U = PS_U;
  const int G = ps_groups<NV>(nt);
  static_assert(NV <= PS_TB, "one thread per value");
  const int t = threadIdx.x;
  const int g = t / NV, v = t - g * NV;
  double s = 0.0;
  if (g < G) {
    for (int t0 = g; t0 < nt && ok; t0 += G * U) {
      unsigned long long b[U];
      const double* p = slot + (size_t)t0 * NV + v;
      bool wait = true;
      int n = 0;
      long long c0 = 0;
#pragma unroll 1
      while (wait) {
        wait = false;
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = t0 + u * G < nt ? ps_bits(p + (size_t)u * G * NV) : 0ull;
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
      for (int u = 0; u < U; ++u) s += __longlong_as_double((long long)b[u]);
    }
  }
  return s;
}

// One row of a stencil of DC diagonals, the main one in the middle:
// coefficients at db[d N + j], sources src(d); the arithmetic and order of
// stencil_row.
template <int DC, typename M, typename SrcF>
__device__ __forceinline__ double ps_row(const M* db, int64_t N, unsigned j, SrcF src) {
  constexpr int D0 = DC / 2;
  double vw[DC];
  M cw[DC];
#pragma unroll
  for (int d = 0; d < DC; ++d) {
    cw[d] = (db + (size_t)d * N)[j];
    vw[d] = src(d);
  }
  __builtin_amdgcn_sched_barrier(0);
  double acc = 0.0;
  if constexpr (sizeof(M) == 4) {
    acc = (double)cw[D0] * vw[D0];
#pragma unroll
    for (int d = 0; d < DC; ++d)
      if (d != D0) acc += (double)cw[d] * (vw[d] - vw[D0]);
  } else {
#pragma unroll
    for (int d = 0; d < DC; ++d) acc += (double)cw[d] * vw[d];
  }
  return acc;
}
// the same for any number of diagonals
template <typename M, typename SrcF>
__device__ __forceinline__ double ps_row_any(const M* db, int64_t N, unsigned j, int D, int d0, SrcF src) {
  double acc = 0.0;
  if (sizeof(M) == 4 && d0 >= 0) {
    const double vi = src(d0);
    acc = (double)(db + (size_t)d0 * N)[j] * vi;
#pragma unroll 4
    for (int d = 0; d < D; ++d)
      if (d != d0) acc += (double)(db + (size_t)d * N)[j] * (src(d) - vi);
    return acc;
  }
#pragma unroll 4
  for (int d = 0; d < D; ++d) acc += (double)(db + (size_t)d * N)[j] * src(d);
  return acc;
}

template <typename M, typename SrcF>
__device__ __forceinline__ double ps_stencil(const M* db, int64_t N, unsigned j, int D, int d0, SrcF src) {
  if (D == 5 && d0 == 2) return ps_row<5>(db, N, j, src);
  if (D == 7 && d0 == 3) return ps_row<7>(db, N, j, src);
  return ps_row_any(db, N, j, D, d0, src);
}

// Forms of W^T z: the stored panel W; SPEC, the boundary form of W (FP32
// panels, modes shared by the instances); FREE, Z^T (S z) with no panel W (FP64
// only), which costs one more exchange and saves the instance's panel.
enum { PS_STORED = 0, PS_SPEC = 1, PS_FREE = 2 };

// Dynamic LDS: C (KP x KP), then t = A p for the tile and the outer stencil's
// reach on both sides (pa.fused).
template <typename V, typename M, int KP, int R, int FORM>
__global__ void __launch_bounds__(PS_TB) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_persist(IterArgs<V, M> a, PersistArgs pa) {
  constexpr int RPT = R > PS_TB ? R / PS_TB : 1;
  constexpr int NV = 2 * KP + 2;
  constexpr int K1 = KP > 0 ? KP : 1;
  constexpr bool SPEC = FORM == PS_SPEC;
  extern __shared__ double dyn[];
  double* Cl = dyn;
  double* tl = dyn + KP * KP;
  __shared__ double zl[R], rl[R];
  __shared__ double gl[PS_TB];
  __shared__ double bv[NV];
  __shared__ double cf[K1], gd[K1];
  __shared__ double red[PS_NW][2];           // wave sums
  __shared__ double redp[2][PS_NW];          // wave sums of p.w, own and the team's
  __shared__ int s_bad[2];
  __shared__ double s_tot[2];                // r.y, r.r
  __shared__ short blist[SPEC ? R : 1];
  __shared__ int bcnt[SPEC ? R / 64 + 1 : 1];
  int tile, place;
  ps_place(pa.nb, tile, place);
  if (tile >= pa.nt) return;
  const int t0_ = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(t0_ >> 6);
  const int m = pa.ids[place];
  Inst* S = a.inst + m;
  const bool idle = S->done;
  unsigned* flag = pa.flags + (size_t)place * pa.nt;
  unsigned* lost = pa.shake + PS_LOST;
  const size_t team = (size_t)place * pa.nt, all = (size_t)pa.nb * pa.nt;
  double rho = S->rho, beta = S->fresh ? 0.0 : S->beta;
  double rr_last = S->rr, pw_last = S->pw, rho_end = S->rho_end;
  const double thresh2 = S->thresh2, sa = S->a, sc = S->c;
  int iters = S->iters, sweep_iters = S->sweep_iters;
  int done = 0, outer_done = 0, status = S->status, capped = S->capped, has_dir = S->has_dir, fresh = S->fresh;
  double alpha = S->alpha;
  const bool defl = KP > 0 && S->kk > 0;
  for (int q = t0_; q < KP; q += PS_TB) cf[q] = S->coef[q];
  for (int e = t0_; e < KP * KP; e += PS_TB) Cl[e] = a.C[(size_t)m * KP * KP + e];
  if (t0_ < 2) s_bad[t0_] = 0;
  // own counter and slots empty before any block of the team is let go
  if (t0_ == 0) st_agent(flag + tile, 0u);
  for (int e = t0_; e < 3 * (NV + 1); e += PS_TB) {
    const int sl = e / (NV + 1), v = e - sl * (NV + 1);
    double* p = v < NV ? pa.dots + (sl * all + team + tile) * NV + v : pa.pw + sl * all + team + tile;
    st_agent((unsigned long long*)p, PS_EMPTY);
  }
  // (S->off: for a reader of the states; the host goes by the words.  Without the
  // two marks the compiler spills other registers: 100^2 x 30, k = 40 111 -> 113 ms)
  if (!ps_handshake(pa)) {
    if (tile == 0 && t0_ == 0) S->off = 1;
    return;
  }
  if (idle) return;
  ps_stall(pa, tile);

  const int64_t N = a.op.N;
  const int64_t base = (int64_t)tile * R;
  const int rows = (int)(N - base < R ? N - base : R);
  V* zv = a.z + m * a.vs;
  V* pv = a.p + m * a.vs;
  V* tv = a.op.D1 ? a.t + m * a.vs : nullptr;
  V x[RPT], r[RPT], z[RPT], p[RPT], w[RPT], dv[RPT];
  unsigned on = 0u;                          // bit rr: row inactive and inside
#pragma unroll
  for (int rr = 0; rr < RPT; ++rr) {
    const int j = rr * PS_TB + t0_;
    x[rr] = r[rr] = z[rr] = p[rr] = w[rr] = dv[rr] = (V)0;
    if (j < rows && j < R && a.mask[(size_t)m * N + base + j] == 0) {
      on |= 1u << rr;
      x[rr] = (a.x + m * a.vs + base)[j];
      r[rr] = (a.r + m * a.vs + base)[j];
      z[rr] = (zv + base)[j];
      dv[rr] = (a.dinv + (size_t)m * N + base)[j];
      if (!fresh) p[rr] = (pv + base)[j];
    }
  }
  int nb = 0;
  if constexpr (SPEC) {
    // the tile's boundary rows, in row order
    const uint8_t* bm = a.bnd + (size_t)m * N + base;
    const int lane = t0_ & 63;
    for (int c = wid; c < R / 64; c += PS_NW) {
      const int j = 64 * c + lane;
      const unsigned long long bal = __ballot(j < rows && bm[j] != 0);
      if (lane == 0) bcnt[c + 1] = __popcll(bal);
    }
    __syncthreads();
    if (t0_ == 0) {
      bcnt[0] = 0;
      for (int c = 0; c < R / 64; ++c) bcnt[c + 1] += bcnt[c];
    }
    __syncthreads();
    for (int c = wid; c < R / 64; c += PS_NW) {
      const int j = 64 * c + lane;
      const bool f = j < rows && bm[j] != 0;
      const unsigned long long bal = __ballot(f);
      if (f) blist[bcnt[c] + __popcll(bal & ((1ull << lane) - 1ull))] = (short)j;
    }
    nb = bcnt[R / 64];
  }
  // the tile's rows of column q of the basis (with a per-instance basis the
  // first kb columns are the shared ones) and of W
  const M* Zb = a.Z + (size_t)m * a.zs + base;
  const M* Zs = a.Zsh + base;
  const M* Wb = a.W + (size_t)m * KP * N + base;
  auto Zcol = [&](int q, int64_t n) { return (q < a.kb ? Zs : Zb) + (size_t)q * n; };
  __syncthreads();
  bool ok = true;
  unsigned step = 0u;
  // this tile's stores are done; go on when those of the tiles within h rows are
  auto exchange = [&](int t, int h) {
    ++step;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    wait_mem();
    __syncthreads();
    if (t == 0) st_agent(flag + tile, step);
    const int lo = (int)(base - h < 0 ? 0 : (base - h) / R);
    const int hi = (int)min((int64_t)pa.nt - 1, (base + rows - 1 + h) / R);
    bool f = true;
    for (int q = lo + t; q <= hi; q += PS_TB) f = ps_wait_ge(flag + q, step, lost) && f;
    if (!f) s_bad[0] = 1;
    __syncthreads();
    ok = !s_bad[0];
  };
  // acc = the operator's stencils on the inactive rows of v, whose tile this
  // block has stored (without the scale and the shift)
  auto apply = [&](int t, int64_t Nq, const V* v, double (&acc)[RPT]) {
    const M* o = a.dia + base;
    if (!a.op.D1) {
      exchange(t, pa.reach);
      if (!ok) return;
#pragma unroll
      for (int rr = 0; rr < RPT; ++rr) {
        const unsigned j = rr * PS_TB + t;
        if ((on >> rr) & 1u)
          acc[rr] = ps_stencil(o, Nq, j, a.op.D, a.op.d0,
                               [&](int d) { return (double)ld_agent(v + base + a.op.offs[d] + j); });
      }
      return;
    }
    if (pa.fused) {
      // the inner stencil for the tile and the outer one's reach, kept in LDS
      exchange(t, pa.reach + pa.reach1);
      if (!ok) return;
      const int64_t lo = base - pa.reach;
      for (int e = t; e < rows + 2 * pa.reach; e += PS_TB) {
        const int64_t i = lo + e;
        double s = 0.0;
        if (i >= 0 && i < Nq)
          s = (double)(V)ps_stencil(a.dia1 + lo, Nq, (unsigned)e, a.op.D1, a.op.d01,
                                    [&](int d) { return (double)ld_agent(v + lo + a.op.offs1[d] + (unsigned)e); });
        tl[e] = s;
      }
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < RPT; ++rr) {
        const unsigned j = rr * PS_TB + t;
        if ((on >> rr) & 1u)
          acc[rr] = ps_stencil(o, Nq, j, a.op.D, a.op.d0,
                               [&](int d) { return tl[(int)j + pa.reach + a.op.offs[d]]; });
      }
      return;
    }
    exchange(t, pa.reach1);
    if (!ok) return;
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
      const unsigned j = rr * PS_TB + t;
      if (j < (unsigned)rows)
        st_agent(tv + base + j,
                 (V)ps_stencil(a.dia1 + base, Nq, j, a.op.D1, a.op.d01,
                               [&](int d) { return (double)ld_agent(v + base + a.op.offs1[d] + j); }));
    }
    exchange(t, pa.reach);
    if (!ok) return;
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
      const unsigned j = rr * PS_TB + t;
      if ((on >> rr) & 1u)
        acc[rr] = ps_stencil(o, Nq, j, a.op.D, a.op.d0,
                             [&](int d) { return (double)ld_agent(tv + base + a.op.offs[d] + j); });
    }
  };

  for (int it = 0; it < pa.chunk && !done; ++it) {
    const int slot = it % 3;
    // keeps the address arithmetic of an iteration in the iteration: hoisted,
    // it would take most of the registers
    int64_t Nq = N;
    int t = threadIdx.x;
    asm volatile("" : "+s"(Nq), "+v"(t));
    const int lane = t & 63;
    double* dots = pa.dots + (slot * all + team) * NV;
    double* pws = pa.pw + slot * all + team;
    if (it >= 2) {
      const int ns = (it + 1) % 3;
      for (int v = t; v <= NV; v += PS_TB) {
        double* q = v < NV ? pa.dots + (ns * all + team + tile) * NV + v : pa.pw + ns * all + team + tile;
        st_agent((unsigned long long*)q, PS_EMPTY);
      }
    }
    // p = z - Z c + beta p
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
      const unsigned j = rr * PS_TB + t;
      if ((on >> rr) & 1u) {
        double s = (double)z[rr];
        if (defl) {
          constexpr int CH = KP > 32 ? KP / 2 : K1;      // columns loaded together
#pragma unroll 1
          for (int q0 = 0; q0 < KP; q0 += CH) {
            M zq[CH];
#pragma unroll
            for (int q = 0; q < CH; ++q) zq[q] = Zcol(q0 + q, Nq)[j];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < CH; ++q) s -= (double)zq[q] * cf[q0 + q];
          }
        }
        if (!fresh) s += beta * (double)p[rr];
        p[rr] = (V)s;
        st_agent(pv + base + j, p[rr]);
      }
    }
    // w = S p on the inactive rows, p.w
    double acc[RPT];
    apply(t, Nq, pv, acc);
    if (!ok) break;
    double s = 0.0;
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr)
      if ((on >> rr) & 1u) {
        w[rr] = (V)(sa * acc[rr] + sc * (double)p[rr]);
        s += (double)p[rr] * (double)w[rr];
      }
    s = ps_wave_sum(s);
    if (lane == 0) redp[0][wid] = s;
    __syncthreads();
    if (t == 0) {
      double b = 0.0;
#pragma unroll
      for (int q = 0; q < PS_NW; ++q) b += redp[0][q];
      st_agent(pws + tile, b);
    }
    ok = true;
    s = ps_wave_sum(ps_gather<1>(pws, pa.nt, lost, ok));
    if (lane == 0) redp[1][wid] = s;
    if (!ok) s_bad[1] = 1;
    __syncthreads();
    if (s_bad[1]) { ok = false; break; }
    pw_last = 0.0;
#pragma unroll
    for (int q = 0; q < PS_NW; ++q) pw_last += redp[1][q];
    if (!(pw_last > 0.0) || !(pw_last < INFINITY)) {
      done = outer_done = 1;
      status = -5;
      break;
    }
    alpha = rho / pw_last;
    // x += alpha p, r -= alpha w, z = K r
    double v2[2] = {0.0, 0.0};
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
      const unsigned j = rr * PS_TB + t;
      if ((on >> rr) & 1u) {
        x[rr] = (V)((double)x[rr] + alpha * (double)p[rr]);
        r[rr] = (V)((double)r[rr] - alpha * (double)w[rr]);
        z[rr] = (V)((double)dv[rr] * (double)r[rr]);
        v2[0] += (double)r[rr] * (double)z[rr];
        v2[1] += (double)r[rr] * (double)r[rr];
        if (FORM == PS_FREE) st_agent(zv + base + j, z[rr]);
      }
      if (R >= PS_TB || j < R) {
        zl[j] = (double)z[rr];
        rl[j] = (double)r[rr];
      }
    }
    v2[0] = ps_wave_sum(v2[0]);
    v2[1] = ps_wave_sum(v2[1]);
    if (lane == 0) { red[wid][0] = v2[0]; red[wid][1] = v2[1]; }
    if constexpr (FORM == PS_FREE) {
      // u = S z takes z's place in the products
      apply(t, Nq, zv, acc);
      if (!ok) break;
#pragma unroll
      for (int rr = 0; rr < RPT; ++rr) {
        const unsigned j = rr * PS_TB + t;
        if ((on >> rr) & 1u) zl[j] = sa * acc[rr] + sc * (double)z[rr];
      }
    }
    __syncthreads();
    if constexpr (KP > 0) {
      if (!defl) {
        for (int q = t; q < 2 * KP; q += PS_TB) bv[q] = 0.0;
      } else if constexpr (FORM == PS_STORED) {
        ps_panel_dots<M, R, 2 * KP>(rows, [&](int q) { return q < KP ? Wb + (size_t)q * Nq : Zcol(q - KP, Nq); },
                                    [&](int q) { return q < KP ? (const double*)zl : (const double*)rl; }, bv);
      } else {
        ps_panel_dots2<M, R, KP>(rows, [&](int q) { return Zcol(q, Nq); }, zl, rl, bv);
        if constexpr (SPEC) {
          // W^T z = Lambda Z^T z + the listed rows of W - Lambda Z
          __syncthreads();
          for (int q = wid; q < KP; q += PS_NW) {
            const M* wc = Wb + (size_t)q * Nq;
            double aw = 0.0;
            for (int e = lane; e < nb; e += 64) aw += (double)wc[blist[e]] * zl[blist[e]];
            aw = ps_wave_sum(aw);
            if (lane == 0) bv[q] = (q < a.ne && a.eig[q] ? (sa * a.mu[q] + sc) * bv[q] : 0.0) + aw;
          }
        }
      }
      __syncthreads();
    }
    for (int v = t; v < NV; v += PS_TB) {
      double b = 0.0;
      if (v < 2 * KP) b = bv[v];
      else
#pragma unroll
        for (int q = 0; q < PS_NW; ++q) b += red[q][v - 2 * KP];
      st_agent(dots + (size_t)tile * NV + v, b);
    }
    gl[t] = ps_gather<NV>(dots, pa.nt, lost, ok);
    if (!ok) s_bad[1] = 1;
    __syncthreads();
    if (s_bad[1]) { ok = false; break; }
    // totals, then c = C (W^T z - Z^T r) and r.y = r.z - c.(Z^T r), by one wave
    // (C is symmetric; lane q holds coordinate q)
    if (wid == 0) {
      const int G = ps_groups<NV>(pa.nt);
      double tz = 0.0, tr = 0.0, rz = 0.0, rr2 = 0.0;
#pragma unroll 4
      for (int g = 0; g < G; ++g) {
        if (lane < KP) {
          tz += gl[g * NV + lane];
          tr += gl[g * NV + KP + lane];
        }
        rz += gl[g * NV + 2 * KP];
        rr2 += gl[g * NV + 2 * KP + 1];
      }
      double corr = 0.0;
      if (defl) {
        if (lane < KP) gd[lane] = tz - tr;
        double c0 = 0.0, c1 = 0.0;
        if (lane < KP) {
#pragma unroll 8
          for (int l = 0; l < KP; l += 2) {
            c0 += Cl[l * KP + lane] * gd[l];
            c1 += Cl[(l + 1) * KP + lane] * gd[l + 1];
          }
          c0 += c1;
          gl[lane] = c0;
        }
        corr = ps_wave_sum(lane < KP ? tr * c0 : 0.0);
      }
      if (lane == 0) { s_tot[0] = rz - corr; s_tot[1] = rr2; }
    }
    __syncthreads();
    // stopping tests, next coarse coordinates and beta (every block alike)
    const double rrt = s_tot[1], rho_n = s_tot[0];
    iters += 1;
    sweep_iters += 1;
    rr_last = rrt;
    int go = 1;
    if (!(rrt > thresh2) || (a.seg_maxit > 0 && sweep_iters >= a.seg_maxit)) {
      done = 1;
      capped = rrt > thresh2;
      go = 2;
      if (!(rrt < INFINITY)) { outer_done = 1; status = -5; go = 0; }
    } else if (iters >= a.maxit) {
      done = outer_done = 1;
      status = 2;
      go = 0;
    }
    if (go && defl && t < KP) cf[t] = gl[t];
    if (go == 1) {
      beta = rho_n / rho;
      rho = rho_n;
      fresh = 0;
    } else if (go == 2) {
      rho_end = rho_n;
      has_dir = 1;
    }
    __syncthreads();
  }
#pragma unroll
  for (int rr = 0; rr < RPT; ++rr)
    if ((on >> rr) & 1u) {
      const int j = rr * PS_TB + t0_;
      (a.x + m * a.vs + base)[j] = x[rr];
      (a.r + m * a.vs + base)[j] = r[rr];
      (zv + base)[j] = z[rr];
    }
  if (tile == 0) {
    for (int q = t0_; q < KP; q += PS_TB) S->coef[q] = cf[q];
    if (t0_ == 0) {
      S->rho = rho; S->beta = beta; S->alpha = alpha; S->rr = rr_last; S->pw = pw_last; S->rho_end = rho_end;
      S->iters = iters; S->sweep_iters = sweep_iters; S->fresh = fresh; S->capped = capped; S->has_dir = has_dir;
      S->status = status;
      if (done) S->done = 1;
      if (outer_done) S->outer_done = 1;
      if (!ok) S->off = 2;
    }
  }
}

}  // namespace adef2
