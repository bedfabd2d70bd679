// Kernels of the learned coarse-space enrichment: POD of solution snapshots,
// per-sample loss data, the MLP theta -> C (BF16 weights, FP32 accumulation),
// its loss gradient, backward pass and Adam, and the basis expansion
// V = Phi C^T appended to the shared reference modes.
#pragma once
#include "dev_setup.h"

namespace adef2 {

// ---------------------------------------------------------------------------
// Tall-skinny Gram  out[m] = X_m^T Y_m  (FP64), optional row mask (rows with
// mask != 0 skipped).  X_m = X + m*sx (N x nx column-major), Y_m likewise.
// Grid (row blocks, output tiles, B); partial sums per row block are written
// to part[m][rb][nx][ny] and summed by k_gram_finish in a fixed order.
// ---------------------------------------------------------------------------
constexpr int GT = 64;    // output tile edge
constexpr int GROWS = 32; // rows staged per step

__global__ void __launch_bounds__(TPB) k_gram_ts(int64_t N, int nx, int ny, const double* X, int64_t sx,
                                                 const double* Y, int64_t sy, const uint8_t* mask,
                                                 int64_t smask, int rows_per_block, double* part) {
  __shared__ double xs[GROWS][GT];
  __shared__ double ys[GROWS][GT];
  const int m = blockIdx.z;
  const int ntx = (nx + GT - 1) / GT;
  const int tx = blockIdx.y % ntx, ty = blockIdx.y / ntx;
  const double* Xm = X + (size_t)m * sx;
  const double* Ym = Y + (size_t)m * sy;
  const uint8_t* mk = mask ? mask + (size_t)m * smask : nullptr;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = min(N, r0 + rows_per_block);
  double acc[GT * GT / TPB];
#pragma unroll
  for (int o = 0; o < GT * GT / TPB; ++o) acc[o] = 0.0;
  for (int64_t rb = r0; rb < r1; rb += GROWS) {
    for (int e = threadIdx.x; e < GROWS * GT; e += TPB) {
      const int rr = e / GT, cc = e % GT;
      const int64_t i = rb + rr;
      const bool on = i < r1 && (!mk || mk[i] == 0);
      const int cx = tx * GT + cc, cy = ty * GT + cc;
      xs[rr][cc] = (on && cx < nx) ? Xm[(size_t)cx * N + i] : 0.0;
      ys[rr][cc] = (on && cy < ny) ? Ym[(size_t)cy * N + i] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int o = 0; o < GT * GT / TPB; ++o) {
      const int idx = threadIdx.x + o * TPB;
      const int a = idx / GT, b = idx % GT;
      double s = 0.0;
      for (int rr = 0; rr < GROWS; ++rr) s += xs[rr][a] * ys[rr][b];
      acc[o] += s;
    }
    __syncthreads();
  }
  const int nrb = gridDim.x;
#pragma unroll
  for (int o = 0; o < GT * GT / TPB; ++o) {
    const int idx = threadIdx.x + o * TPB;
    const int a = tx * GT + idx / GT, b = ty * GT + idx % GT;
    if (a < nx && b < ny) part[(((size_t)m * nrb + blockIdx.x) * nx + a) * ny + b] = acc[o];
  }
}

__global__ void k_gram_finish(int nrb, int nx, int ny, const double* part, double* out) {
  const int m = blockIdx.y;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nx * ny) return;
  double s = 0.0;
  for (int r = 0; r < nrb; ++r) s += part[((size_t)m * nrb + r) * nx * ny + e];
  out[(size_t)m * nx * ny + e] = s;
}

// row means of X (N x M) and centred copy Xc = X - mean
__global__ void k_center(int64_t N, int M, const double* X, double* Xc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  double s = 0.0;
  for (int j = 0; j < M; ++j) s += X[(size_t)j * N + i];
  const double mu = s / M;
  for (int j = 0; j < M; ++j) Xc[(size_t)j * N + i] = X[(size_t)j * N + i] - mu;
}

// ---------------------------------------------------------------------------
// Cyclic Jacobi eigen-decomposition of a symmetric n x n matrix A (n <= JMAX,
// row-major): rotations of the n / 2 pairs of a round at once, the pairs of the
// following rounds by the circle method (the same pairs in the same order for
// every n: they settle the signs of the vectors).
//
// One workgroup.  A stays in registers, a thread holding the 2 x 2 blocks (pair
// i, pair j), i <= j, of the places tid, tid + 1024, ...; a round rotates every
// block from both sides and moves the entries to their places of the next round
// through LDS (through memory when it doesn't fit, n > 200).  The moves are the
// same in every round, so their addresses are held too.  The rotations are
// logged for the eigenvectors, whose rows don't depend on each other
// (k_jacobi_vecs, a wave per row).  Bound: LDS instructions and the serial chain
// of a rotation.  At n = 200 (rank 64) 6.1 ms and 0.3 ms for the vectors; with A
// and V in memory, read and written column by column, 346 ms, and 1.2 s where
// rounding in the null space kept the sweeps going.  n = 256: 50 ms (2.7 s).
// ---------------------------------------------------------------------------
constexpr int JMAX = 256;
constexpr int JSWEEPS = 60;
constexpr int JTB = 1024;

// pairs, rounds of a sweep and 2 x 2 blocks of an n x n matrix
struct JacGeom {
  int np, rounds, nblk;
};
__host__ __device__ inline JacGeom jac_geom(int n) {
  const int np = (n + 1) / 2;
  return JacGeom{np, 2 * np - 1, np * (np + 1) / 2};
}
__device__ __forceinline__ int jac_block(int np, int i, int j) {   // i <= j; diagonal blocks first
  return i == j ? i : np + i * (np - 1) - i * (i - 1) / 2 + (j - i - 1);
}
// where the entry at position p (pair p / 2, first or second of it) of the next
// round is now: the first entries move up, the second ones down, entry 0 stays
__device__ __forceinline__ int jac_from(int np, int p) {
  const int i = p >> 1;
  if (np == 1 || p == 0) return p;
  if (p & 1) return i == np - 1 ? 2 * i : p + 2;
  return i == 1 ? 1 : p - 2;
}

// (p, q) by the rotation (s, h = tan of half the angle): p - s (q + h p) instead
// of c p - s q, whose c^2 + s^2 is off 1 by a rounding each time
__device__ __forceinline__ void jac_rotate(const double2& sh, double& p, double& q) {
  const double p0 = p, q0 = q;
  p = p0 - sh.x * (q0 + sh.y * p0);
  q = q0 + sh.x * (p0 - sh.y * q0);
}

// the index whose entry starts at position p: pair t of round r holds the indices
// r - t and r + t mod 2 np - 1, pair 0 the last index and r
__device__ __forceinline__ int jac_index(int np, int p) {
  return p & 1 ? p >> 1 : 2 * np - 1 - (p >> 1);
}

// S: blocks per thread; LDSX: the exchange goes through LDS (4 nblk doubles after
// the np rotations), else through xg, and LDS holds the addresses.  log: [JSWEEPS (2 np - 1)][np] rotations, nrounds: how many
// rounds were done.
template <int S, bool LDSX>
__global__ void __launch_bounds__(JTB) k_jacobi_rot(int n, const double* A, double2* log, int* nrounds, double* xg,
                                                    double* evals) {
  extern __shared__ double2 jcs[];
  __shared__ double red[2][JTB / 64];
  const JacGeom g = jac_geom(n);
  const int np = g.np, nblk = g.nblk, tid = threadIdx.x;
  double* xl = (double*)(jcs + np);                    // LDSX: the exchange;
  uint2* lfrom = (uint2*)(jcs + np);                   //   else the addresses and pairs of the blocks
  int* lij = (int*)(lfrom + nblk);
  double m[S][4];
  uint2 from[LDSX ? S : 1];
  int ij[LDSX ? S : 1];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    int e = tid + u * JTB, i = 0, j;
    if (e >= nblk) e = 0;                              // a copy of block 0, never stored
    if (e < np) i = j = e;
    else {
      e -= np;
      while (e >= np - 1 - i) e -= np - 1 - i++;
      j = i + 1 + e;
    }
    unsigned at[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      int p = 2 * i + (k >> 1), q = 2 * j + (k & 1);
      const int lo = min(jac_index(np, p), jac_index(np, q)), hi = max(jac_index(np, p), jac_index(np, q));
      m[u][k] = hi < n ? A[(size_t)lo * n + hi] : 0.0;
      p = jac_from(np, p);
      q = jac_from(np, q);
      if ((p >> 1) > (q >> 1)) { const int t = p; p = q; q = t; }
      at[k] = ((p & 1) * 2 + (q & 1)) * nblk + jac_block(np, p >> 1, q >> 1);
    }
    const uint2 f{at[0] | at[1] << 16, at[2] | at[3] << 16};
    if constexpr (LDSX) { from[u] = f; ij[u] = i | j << 16; }
    else if (tid + u * JTB < nblk) { lfrom[tid + u * JTB] = f; lij[tid + u * JTB] = i | j << 16; }
  }
  int done = 0;
  double prev = INFINITY;
  for (int sweep = 0; sweep < JSWEEPS; ++sweep) {
    double off = 0.0, dia = 0.0;
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int e = tid + u * JTB;
      if (e < np) {
        off += 2.0 * m[u][1] * m[u][1];
        dia += m[u][0] * m[u][0] + m[u][3] * m[u][3];
      } else if (e < nblk) {
#pragma unroll
        for (int k = 0; k < 4; ++k) off += 2.0 * m[u][k] * m[u][k];
      }
    }
    off = wave_sum(off);
    dia = wave_sum(dia);
    if ((tid & 63) == 0) { red[0][tid >> 6] = off; red[1][tid >> 6] = dia; }
    __syncthreads();
    off = dia = 0.0;
    for (int w = 0; w < JTB / 64; ++w) { off += red[0][w]; dia += red[1][w]; }
    // diagonal, or at rounding level and no longer shrinking (the null space of
    // a rank-deficient Gram; eigenvalues 1e-14 of the largest are still being
    // separated at this level, by a factor of 3 to 10 a sweep)
    if (!(off > 1e-30 * dia) || (off <= 1e-27 * dia && off > 0.9 * prev)) break;
    prev = off;
    for (int rnd = 0; rnd < g.rounds; ++rnd, ++done) {
      if (tid < np) {
        const double apq = m[0][1], app = m[0][0], aqq = m[0][3];
        double s = 0.0, h = 0.0;
        if (fabs(apq) > 1e-300) {
          const double tau = (aqq - app) / (2.0 * apq);
          // equal diagonal entries: by the order of the indices
          int i0 = tid ? rnd - tid : g.rounds, i1 = rnd + tid;
          if (i0 < 0) i0 += g.rounds;
          if (i1 >= g.rounds) i1 -= g.rounds;
          const bool pos = i0 < i1 ? tau >= 0.0 : tau > 0.0;
          const double t = (pos ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
          const double c = 1.0 / sqrt(1.0 + t * t);
          s = t * c;
          h = s / (1.0 + c);
          m[0][0] = app - t * apq;
          m[0][3] = aqq + t * apq;
          m[0][1] = m[0][2] = 0.0;
        }
        jcs[tid] = double2{s, h};
        log[(size_t)done * np + tid] = double2{s, h};
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const int e = tid + u * JTB;
        if (e >= nblk) continue;
        if (u > 0 || e >= np) {
          int w;
          if constexpr (LDSX) w = ij[u]; else w = lij[e];
          const double2 ci = jcs[w & 0xffff], cj = jcs[w >> 16];
#pragma unroll
          for (int k = 0; k < 2; ++k) jac_rotate(ci, m[u][k], m[u][2 + k]);       // rows of pair i
#pragma unroll
          for (int k = 0; k < 4; k += 2) jac_rotate(cj, m[u][k], m[u][k + 1]);    // columns of pair j
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if constexpr (LDSX) xl[k * nblk + e] = m[u][k];
          else xg[k * nblk + e] = m[u][k];
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < S; ++u)
        if (tid + u * JTB < nblk) {
          uint2 f;
          if constexpr (LDSX) f = from[u]; else f = lfrom[tid + u * JTB];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const unsigned at = ((k & 2 ? f.y : f.x) >> (16 * (k & 1))) & 0xffffu;
            if constexpr (LDSX) m[u][k] = xl[at];
            else m[u][k] = xg[at];
          }
        }
    }
  }
  // every sweep ends with the entries at their own places
  if (tid < np) {
    const int i0 = jac_index(np, 2 * tid), i1 = jac_index(np, 2 * tid + 1);
    if (i0 < n) evals[i0] = m[0][0];
    if (i1 < n) evals[i1] = m[0][3];
  }
  if (tid == 0) *nrounds = done;
}

// lane + 1's / lane - 1's value (0 beyond the wave)
__device__ __forceinline__ double jac_shift(double v, bool up) {
  union { double d; int i[2]; } a, b;
  a.d = v;
#pragma unroll
  for (int h = 0; h < 2; ++h)
    b.i[h] = up ? __builtin_amdgcn_update_dpp(0, a.i[h], 0x138, 0xf, 0xf, true)     // wave_shr:1
                : __builtin_amdgcn_update_dpp(0, a.i[h], 0x130, 0xf, 0xf, true);    // wave_shl:1
  return b.d;
}

// Row i of the eigenvectors (V[i][j] = entry i of eigenvector j): row i of the
// identity through the logged rotations, one wave per row, two pairs per lane.
__global__ void __launch_bounds__(256) k_jacobi_vecs(int n, const double2* log, const int* nrounds, double* V) {
  constexpr int PF = 8;                                // rounds whose rotations are loaded together
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  const int np = jac_geom(n).np, R = *nrounds;
  const int k0 = min(2 * lane, np - 1), k1 = min(2 * lane + 1, np - 1);
  double v[4];                                         // pairs 2 lane and 2 lane + 1
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = jac_index(np, 4 * lane + k) == i && 2 * lane + (k >> 1) < np ? 1.0 : 0.0;
  double2 cs[2][PF][2];
  auto load = [&](int r0, double2 (&b)[PF][2]) {
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      const size_t r = (size_t)min(r0 + q, R - 1) * np;
      b[q][0] = log[r + k0];
      b[q][1] = log[r + k1];
    }
  };
  auto round = [&](const double2 (&b)[2]) {
    double t0 = v[0], b0 = v[1], t1 = v[2], b1 = v[3];
    jac_rotate(b[0], t0, b0);
    jac_rotate(b[1], t1, b1);
    if (np == 1) { v[0] = t0; v[1] = b0; return; }
    const double tl = jac_shift(t1, true), br = jac_shift(b0, false);
    v[0] = lane == 0 ? t0 : tl;                        // first entries move up, entry 0 stays
    v[2] = lane == 0 ? b0 : t0;
    v[1] = 2 * lane == np - 1 ? t0 : b1;               // second entries move down
    v[3] = 2 * lane + 1 == np - 1 ? t1 : br;
  };
  if (R > 0) load(0, cs[0]);
  for (int r0 = 0; r0 < R; r0 += 2 * PF) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      load(r0 + (h + 1) * PF, cs[(h + 1) & 1]);
#pragma unroll
      for (int q = 0; q < PF; ++q)
        if (r0 + h * PF + q < R) round(cs[h][q]);
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int j = jac_index(np, 4 * lane + k);
    if (2 * lane + (k >> 1) < np && j < n) V[(size_t)i * n + j] = v[k];
  }
}

// Phi[:, j] = Xc v_c / sqrt(lambda_c), c = sel[j] (eigenvalue order,
// descending; identity when sel is null); entry m of eigenvector c at
// V[m * vsm + c * vsc]
__global__ void k_pod_modes(int64_t N, int M, int p, const double* Xc, const double* V, int64_t vsm,
                            int64_t vsc, const int* sel, const double* evals, double* Phi) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (i >= N || j >= p) return;
  const int c = sel ? sel[j] : j;
  double s = 0.0;
  for (int m = 0; m < M; ++m) s += Xc[(size_t)m * N + i] * V[(size_t)m * vsm + (size_t)c * vsc];
  const double lam = evals[c];
  Phi[(size_t)j * N + i] = lam > 0.0 ? s / sqrt(lam) : 0.0;
}

// ---------------------------------------------------------------------------
// Subspace iteration for the leading eigenpairs of a large snapshot Gram
// (M > JMAX): blocks of L orthonormal columns are multiplied by G, rotated
// by the Rayleigh-Ritz eigenvectors of Q^T G Q and re-orthonormalised
// (scaled Gram + eigen-decomposition, "SVQB"), until the residuals of the
// wanted Ritz pairs are small.
// ---------------------------------------------------------------------------
constexpr int SYB = 8;   // columns per thread in k_symm_block

// Y[:, j] = G Q[:, j], G symmetric M x M (row-major: row i is column i, so
// the loads along m are coalesced across threads); Q, Y column-major M x L.
__global__ void __launch_bounds__(256) k_symm_block(int M, int L, const double* G, const double* Q,
                                                    double* Y) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j0 = blockIdx.y * SYB;
  if (i >= M) return;
  double s[SYB];
#pragma unroll
  for (int c = 0; c < SYB; ++c) s[c] = 0.0;
  for (int m = 0; m < M; ++m) {
    const double g = G[(size_t)m * M + i];
#pragma unroll
    for (int c = 0; c < SYB; ++c)
      if (j0 + c < L) s[c] += g * Q[(size_t)(j0 + c) * M + m];
  }
#pragma unroll
  for (int c = 0; c < SYB; ++c)
    if (j0 + c < L) Y[(size_t)(j0 + c) * M + i] = s[c];
}

// out[:, c] = scale[c] * sum_l A[:, l] pre[l] W[l][col(c)], col(c) = sel[c]
// (or c); A, out column-major M x L, W row-major L x L (entry l of column j
// at W[l * L + j]).  pre / scale / sel may be null (ones / identity).
__global__ void k_comb_cols(int M, int L, const double* A, const double* pre, const double* W,
                            const int* sel, const double* scale, double* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int c = blockIdx.y;
  if (i >= M) return;
  const int col = sel ? sel[c] : c;
  double s = 0.0;
  for (int l = 0; l < L; ++l) s += A[(size_t)l * M + i] * (pre ? pre[l] : 1.0) * W[(size_t)l * L + col];
  out[(size_t)c * M + i] = scale ? s * scale[c] : s;
}

// SVQB pre-scaling: dsc[l] = C[l][l]^-1/2 (0 for a zero column) and
// C <- D C D, symmetrised.  One workgroup.
__global__ void k_svqb_scale(int L, double* C, double* dsc) {
  for (int l = threadIdx.x; l < L; l += blockDim.x) {
    const double d = C[(size_t)l * L + l];
    dsc[l] = d > 0.0 ? 1.0 / sqrt(d) : 0.0;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < L * L; e += blockDim.x) {
    const int a = e / L, b = e % L;
    if (a > b) continue;
    const double v = 0.5 * (C[(size_t)a * L + b] + C[(size_t)b * L + a]) * dsc[a] * dsc[b];
    C[(size_t)a * L + b] = v;
    C[(size_t)b * L + a] = v;
  }
}

// SVQB post-scaling: inv[c] = d[c]^-1/2 for eigenvalues above drop * max(d),
// else 0 (the direction is dropped: a zero column).  One workgroup.
__global__ void k_svqb_inv(int L, const double* d, double drop, double* inv) {
  __shared__ double mx;
  if (threadIdx.x == 0) {
    double m = 0.0;
    for (int l = 0; l < L; ++l) m = fmax(m, d[l]);
    mx = m;
  }
  __syncthreads();
  for (int l = threadIdx.x; l < L; l += blockDim.x) inv[l] = d[l] > drop * mx ? 1.0 / sqrt(d[l]) : 0.0;
}

// H <- (H + H^T) / 2 (L x L).  One workgroup.
__global__ void k_symmetrize(int L, double* H) {
  for (int e = threadIdx.x; e < L * L; e += blockDim.x) {
    const int a = e / L, b = e % L;
    if (a >= b) continue;
    const double v = 0.5 * (H[(size_t)a * L + b] + H[(size_t)b * L + a]);
    H[(size_t)a * L + b] = v;
    H[(size_t)b * L + a] = v;
  }
}

// res[c] = || YW[:, c] - th[c] QW[:, c] ||_2 (one workgroup per column)
__global__ void __launch_bounds__(256) k_ritz_resid(int M, const double* QW, const double* YW,
                                                    const double* th, double* res) {
  __shared__ double red[4];
  const int c = blockIdx.x;
  double s = 0.0;
  for (int i = threadIdx.x; i < M; i += blockDim.x) {
    const double r = YW[(size_t)c * M + i] - th[c] * QW[(size_t)c * M + i];
    s += r * r;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) res[c] = sqrt(red[0] + red[1] + red[2] + red[3]);
}

// deterministic start block: entries uniform in [-1, 1) from a 64-bit mix
// of the entry index (splitmix64 finaliser)
__global__ void k_start_block(int64_t n, double* Q) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  uint64_t z = (uint64_t)e + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  Q[e] = (double)(z >> 11) * 0x1.0p-52 - 1.0;
}

// ---------------------------------------------------------------------------
// Per-sample loss data from the Grams of [Z | Phi] (one workgroup per sample):
//   G = [Z|P]^T S [Z|P]  ((k+p) x (k+p)),  bZP = [Z|P]^T b,
//   H = Gpp - Gpz Gzz^-1 Gzp, g = bP - Gpz Gzz^-1 bZ, e0 = bZ^T Gzz^-1 bZ.
// Gzz is factorised by Cholesky (with the same column dropping as the coarse
// setup: dependent columns contribute nothing).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024) k_loss_data(int k, int p, const double* G, const double* bzp,
                                                    double* H, double* gv, double* e0v, double drop_rel,
                                                    const double* Gd, double* Nout) {
  extern __shared__ double sm[];
  double* L = sm;                 // k x k Cholesky (lower)
  double* A = L + k * k;          // k x (p+1): Gzz^-1 [Gzp | bZ]
  double* GA = A + k * (p + 1);   // k x p: Dzz Gzz^-1 Gzp (with Gd only)
  __shared__ int s_keep[64];
  __shared__ double s_d;
  const int m = blockIdx.x;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int n = k + p;
  const double* Gm = G + (size_t)m * n * n;
  const double* bm = bzp + (size_t)m * n;
  for (int e = tid; e < k * k; e += nt) L[e] = Gm[(e / k) * n + e % k];
  __syncthreads();
  for (int j = 0; j < k; ++j) {
    if (tid == 0) {
      const double d = L[j * k + j];
      const double g0 = Gm[j * n + j];
      s_keep[j] = (g0 > 0.0) && (d > drop_rel * drop_rel * g0);
      s_d = s_keep[j] ? sqrt(d) : 0.0;
    }
    __syncthreads();
    if (s_keep[j]) {
      for (int l = j + 1 + tid; l < k; l += nt) L[l * k + j] /= s_d;
      if (tid == 0) L[j * k + j] = s_d;
      __syncthreads();
      const int rem = k - j - 1;
      for (int e = tid; e < rem * rem; e += nt) {
        const int l = j + 1 + e / rem, q = j + 1 + e % rem;
        if (q <= l) L[l * k + q] -= L[l * k + j] * L[q * k + j];
      }
    } else {
      for (int l = tid; l < k; l += nt) { L[l * k + j] = 0.0; L[j * k + l] = 0.0; }
    }
    __syncthreads();
  }
  // A[:, c] = Gzz^-1 rhs_c  (forward then backward substitution, one column per thread)
  for (int c = tid; c < p + 1; c += nt) {
    for (int i = 0; i < k; ++i) {
      double s = (c < p) ? Gm[i * n + k + c] : bm[i];
      for (int q = 0; q < i; ++q) s -= L[i * k + q] * A[q * (p + 1) + c];
      A[i * (p + 1) + c] = s_keep[i] ? s / L[i * k + i] : 0.0;
    }
    for (int i = k - 1; i >= 0; --i) {
      double s = A[i * (p + 1) + c];
      for (int q = i + 1; q < k; ++q) s -= L[q * k + i] * A[q * (p + 1) + c];
      A[i * (p + 1) + c] = s_keep[i] ? s / L[i * k + i] : 0.0;
    }
  }
  __syncthreads();
  double* Hm = H + (size_t)m * p * p;
  for (int e = tid; e < p * p; e += nt) {
    const int a = e / p, b = e % p;
    double s = 0.0;
    for (int q = 0; q < k; ++q) s += Gm[q * n + k + a] * A[q * (p + 1) + b];
    const double h1 = Gm[(k + a) * n + k + b] - s;
    double s2 = 0.0;
    for (int q = 0; q < k; ++q) s2 += Gm[q * n + k + b] * A[q * (p + 1) + a];
    const double h2 = Gm[(k + b) * n + k + a] - s2;
    Hm[e] = 0.5 * (h1 + h2);
  }
  for (int a = tid; a < p; a += nt) {
    double s = 0.0;
    for (int q = 0; q < k; ++q) s += Gm[q * n + k + a] * A[q * (p + 1) + p];
    gv[(size_t)m * p + a] = bm[k + a] - s;
  }
  if (tid == 0) {
    double s = 0.0;
    for (int q = 0; q < k; ++q) s += bm[q] * A[q * (p + 1) + p];
    e0v[m] = s;
  }
  if (!Gd) return;
  // N = P~^T D P~ with P~ = P - Z Gzz^-1 Gzp (the candidates made
  // S-orthogonal to Z) from the D-weighted Gram Gd of [Z | P]:
  //   N = Dpp - Dpz A - A^T Dzp + A^T Dzz A,  A = Gzz^-1 Gzp
  const double* Dm = Gd + (size_t)m * n * n;
  for (int e = tid; e < k * p; e += nt) {
    const int q = e / p, b = e % p;
    double s = 0.0;
    for (int r = 0; r < k; ++r) s += Dm[q * n + r] * A[r * (p + 1) + b];
    GA[e] = s;
  }
  __syncthreads();
  double* Nm = Nout + (size_t)m * p * p;
  for (int e = tid; e < p * p; e += nt) {
    const int a = e / p, b = e % p;
    double s1 = Dm[(k + a) * n + k + b], s2 = Dm[(k + b) * n + k + a];
    for (int q = 0; q < k; ++q) {
      const double aqa = A[q * (p + 1) + a], aqb = A[q * (p + 1) + b];
      s1 += aqa * GA[q * p + b] - Dm[(k + a) * n + q] * aqb - aqa * Dm[q * n + k + b];
      s2 += aqb * GA[q * p + a] - Dm[(k + b) * n + q] * aqa - aqb * Dm[q * n + k + a];
    }
    Nm[e] = 0.5 * (s1 + s2);
  }
}

// DV[q] = D V[q] on inactive rows (0 on active ones), D = diag(S_II) =
// a diag + c of the instance (one->a, one->c)
__global__ void k_dscale_cols(int64_t N, const double* Vb, const double* diag, const uint8_t* mask,
                              const Inst* one, double* DV) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  if (i >= N) return;
  DV[(size_t)q * N + i] = mask[i] ? 0.0 : (one->a * diag[i] + one->c) * Vb[(size_t)q * N + i];
}

// ---------------------------------------------------------------------------
// MLP 4 -> 128 -> 128 -> (NV x P) with exact erf-GELU.  Weights in BF16
// (row-major [out][in]), biases FP32, FP32 accumulation.  One block per
// sample; activations kept for the backward pass.
// ---------------------------------------------------------------------------
constexpr int MD0 = 4, MD1 = 128, MD2 = 128, MD3 = 512;
constexpr int MLP_NV = 8, MLP_P = 64;

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {    // round to nearest even
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * expf(-0.5f * x * x) * 0.3989422804014327f;
}

struct MLPW {            // BF16 compute copies and FP32 biases (device)
  const uint16_t* W1; const float* b1;
  const uint16_t* W2; const float* b2;
  const uint16_t* W3; const float* b3;
};

// a + row . h, in order; the row is loaded 8 weights at a time (rows of W2 and W3
// start at multiples of 256 bytes from W1, whose 512 weights and 128 biases come
// first: 16-byte aligned)
template <int K>
__device__ __forceinline__ float mlp_dot(const uint16_t* row, const float* h, float a) {
  uint4 q[K / 8];
#pragma unroll
  for (int k = 0; k < K / 8; ++k) q[k] = ((const uint4*)row)[k];
#pragma unroll
  for (int k = 0; k < K / 8; ++k) {
    const uint32_t w[4] = {q[k].x, q[k].y, q[k].z, q[k].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) a += bf2f((uint16_t)(w[e >> 1] >> (16 * (e & 1)))) * h[8 * k + e];
  }
  return a;
}

// theta: [B][4]; act: [B][A1 128 | H1 128 | A2 128 | H2 128]; out: [B][512]
__global__ void __launch_bounds__(512) k_mlp_fwd(int B, const float* theta, MLPW w, float* act, float* out) {
  __shared__ float x0[MD0], h1[MD1], h2[MD2];
  const int s = blockIdx.x;
  const int t = threadIdx.x;
  if (s >= B) return;
  if (t < MD0) x0[t] = theta[s * MD0 + t];
  __syncthreads();
  float* as = act + (size_t)s * 4 * MD1;
  if (t < MD1) {
    float a = w.b1[t];
    for (int k = 0; k < MD0; ++k) a += bf2f(w.W1[t * MD0 + k]) * x0[k];
    as[t] = a;
    h1[t] = gelu_f(a);
    as[MD1 + t] = h1[t];
  }
  __syncthreads();
  if (t < MD2) {
    float a = w.b2[t];
    a = mlp_dot<MD1>(w.W2 + t * MD1, h1, a);
    as[2 * MD1 + t] = a;
    h2[t] = gelu_f(a);
    as[3 * MD1 + t] = h2[t];
  }
  __syncthreads();
  if (t < MD3) {
    float a = w.b3[t];
    a = mlp_dot<MD2>(w.W3 + t * MD2, h2, a);
    out[(size_t)s * MD3 + t] = a;
  }
}

// Loss and dL/dC of one sample.  C (NV x p) is the leading p columns of
// out reshaped NV x 64 (row-major); H is p x p and g has p entries:
//   s = C g, T = C H C^T + eps I, u = T^-1 s,
//   L = 1 - (e0 + s.u) / bx,  dL/dC = -(2 u g^T - 2 u u^T C H) / bx.
// Output columns p..63 get zero gradient.  dout is scaled by wscale
// (1 / batch size).
__global__ void __launch_bounds__(512) k_loss_grad(int B, int p, const float* out, const double* H,
                                                   const double* gv, const double* e0v, const double* bxv,
                                                   double eps, float wscale, float* dout, double* lossv) {
  __shared__ double Hs[MLP_P * MLP_P];
  __shared__ double C[MLP_NV * MLP_P], CH[MLP_NV * MLP_P];
  __shared__ double T[MLP_NV * MLP_NV], sv[MLP_NV], u[MLP_NV], gs[MLP_P];
  const int smp = blockIdx.x, t = threadIdx.x;
  if (smp >= B) return;
  const double* Hm = H + (size_t)smp * p * p;
  for (int e = t; e < p * p; e += blockDim.x) Hs[e] = Hm[e];
  for (int e = t; e < MLP_NV * p; e += blockDim.x) C[e] = out[(size_t)smp * MD3 + (e / p) * MLP_P + e % p];
  for (int e = t; e < p; e += blockDim.x) gs[e] = gv[(size_t)smp * p + e];
  __syncthreads();
  for (int e = t; e < MLP_NV * p; e += blockDim.x) {
    const int i = e / p, j = e % p;
    double s = 0.0;
    for (int q = 0; q < p; ++q) s += C[i * p + q] * Hs[q * p + j];
    CH[e] = s;
  }
  if (t < MLP_NV) {
    double s = 0.0;
    for (int q = 0; q < p; ++q) s += C[t * p + q] * gs[q];
    sv[t] = s;
  }
  __syncthreads();
  if (t < MLP_NV * MLP_NV) {
    const int i = t / MLP_NV, j = t % MLP_NV;
    double s = 0.0;
    for (int q = 0; q < p; ++q) s += CH[i * p + q] * C[j * p + q];
    T[t] = s + (i == j ? eps : 0.0);
  }
  __syncthreads();
  if (t == 0) {      // 8 x 8 Cholesky solve T u = s (symmetrised T)
    double Lc[MLP_NV * MLP_NV];
    bool ok = true;
    for (int j = 0; j < MLP_NV && ok; ++j) {
      double d = T[j * MLP_NV + j];
      for (int q = 0; q < j; ++q) d -= Lc[j * MLP_NV + q] * Lc[j * MLP_NV + q];
      if (!(d > 0.0)) { ok = false; break; }
      Lc[j * MLP_NV + j] = sqrt(d);
      for (int l = j + 1; l < MLP_NV; ++l) {
        double v = 0.5 * (T[l * MLP_NV + j] + T[j * MLP_NV + l]);
        for (int q = 0; q < j; ++q) v -= Lc[l * MLP_NV + q] * Lc[j * MLP_NV + q];
        Lc[l * MLP_NV + j] = v / Lc[j * MLP_NV + j];
      }
    }
    double y[MLP_NV];
    for (int i = 0; i < MLP_NV; ++i) {
      double v = sv[i];
      for (int q = 0; q < i && ok; ++q) v -= Lc[i * MLP_NV + q] * y[q];
      y[i] = ok ? v / Lc[i * MLP_NV + i] : 0.0;
    }
    for (int i = MLP_NV - 1; i >= 0; --i) {
      double v = y[i];
      for (int q = i + 1; q < MLP_NV && ok; ++q) v -= Lc[q * MLP_NV + i] * u[q];
      u[i] = ok ? v / Lc[i * MLP_NV + i] : 0.0;
    }
    double su = 0.0;
    for (int i = 0; i < MLP_NV; ++i) su += sv[i] * u[i];
    lossv[smp] = 1.0 - (e0v[smp] + su) / bxv[smp];
  }
  __syncthreads();
  const double ib = 1.0 / bxv[smp];
  for (int e = t; e < MLP_NV * MLP_P; e += blockDim.x) {
    const int i = e / MLP_P, j = e % MLP_P;
    double gr = 0.0;
    if (j < p) {
      double uCH = 0.0;
      for (int q = 0; q < MLP_NV; ++q) uCH += u[q] * CH[q * p + j];
      gr = -(2.0 * u[i] * gs[j] - 2.0 * u[i] * uCH) * ib;
    }
    dout[(size_t)smp * MD3 + e] = (float)(gr * wscale);
  }
}

// Deflated-spectrum loss of one sample and its gradient.  C (NV x p) as in
// k_loss_grad; H and N (p x p) are the S_II- and D-weighted Grams of the
// candidates made S_II-orthogonal to the reference modes.  With
// T = C H C^T and U = C N C^T, R = tr(U^-1 T) is the sum of the Ritz values
// of the Jacobi-preconditioned deflated operator on the span of the NV
// enrichment vectors:
//   L = log R,  dL/dC = 2 (U^-1 C H - U^-1 T U^-1 C N) / R.
// A sample whose U is not positive definite (rank-deficient C) gets a NaN
// loss and zero gradient.
__global__ void __launch_bounds__(512) k_loss_grad_spec(int B, int p, const float* out, const double* H,
                                                        const double* Nv, float wscale, float* dout,
                                                        double* lossv) {
  __shared__ double buf[MLP_P * MLP_P];
  __shared__ double C[MLP_NV * MLP_P], CH[MLP_NV * MLP_P], CN[MLP_NV * MLP_P];
  __shared__ double T[MLP_NV * MLP_NV], U[MLP_NV * MLP_NV], X[MLP_NV * MLP_NV], P[MLP_NV * MLP_NV];
  __shared__ double s_r;
  const int smp = blockIdx.x, t = threadIdx.x;
  if (smp >= B) return;
  for (int e = t; e < MLP_NV * p; e += blockDim.x) C[e] = out[(size_t)smp * MD3 + (e / p) * MLP_P + e % p];
  for (int pass = 0; pass < 2; ++pass) {
    const double* src = (pass == 0 ? H : Nv) + (size_t)smp * p * p;
    double* dst = pass == 0 ? CH : CN;
    __syncthreads();
    for (int e = t; e < p * p; e += blockDim.x) buf[e] = src[e];
    __syncthreads();
    for (int e = t; e < MLP_NV * p; e += blockDim.x) {
      const int i = e / p, j = e % p;
      double s = 0.0;
      for (int q = 0; q < p; ++q) s += C[i * p + q] * buf[q * p + j];
      dst[e] = s;
    }
  }
  __syncthreads();
  if (t < 2 * MLP_NV * MLP_NV) {
    const int w = t / (MLP_NV * MLP_NV), o = t % (MLP_NV * MLP_NV);
    const int i = o / MLP_NV, j = o % MLP_NV;
    const double* src = w == 0 ? CH : CN;
    double s = 0.0;
    for (int q = 0; q < p; ++q) s += src[i * p + q] * C[j * p + q];
    (w == 0 ? T : U)[o] = s;
  }
  __syncthreads();
  if (t == 0) {      // X = U^-1 by Cholesky (symmetrised U), R = tr(X T), P = X T X
    double Lc[MLP_NV * MLP_NV];
    bool ok = true;
    for (int j = 0; j < MLP_NV && ok; ++j) {
      double d = U[j * MLP_NV + j];
      for (int q = 0; q < j; ++q) d -= Lc[j * MLP_NV + q] * Lc[j * MLP_NV + q];
      if (!(d > 0.0)) { ok = false; break; }
      Lc[j * MLP_NV + j] = sqrt(d);
      for (int l = j + 1; l < MLP_NV; ++l) {
        double v = 0.5 * (U[l * MLP_NV + j] + U[j * MLP_NV + l]);
        for (int q = 0; q < j; ++q) v -= Lc[l * MLP_NV + q] * Lc[j * MLP_NV + q];
        Lc[l * MLP_NV + j] = v / Lc[j * MLP_NV + j];
      }
    }
    for (int c = 0; c < MLP_NV; ++c) {
      double y[MLP_NV];
      for (int i = 0; i < MLP_NV; ++i) {
        double v = (i == c) ? 1.0 : 0.0;
        for (int q = 0; q < i && ok; ++q) v -= Lc[i * MLP_NV + q] * y[q];
        y[i] = ok ? v / Lc[i * MLP_NV + i] : 0.0;
      }
      for (int i = MLP_NV - 1; i >= 0; --i) {
        double v = y[i];
        for (int q = i + 1; q < MLP_NV && ok; ++q) v -= Lc[q * MLP_NV + i] * X[q * MLP_NV + c];
        X[i * MLP_NV + c] = ok ? v / Lc[i * MLP_NV + i] : 0.0;
      }
    }
    double r = 0.0;
    for (int i = 0; i < MLP_NV; ++i)
      for (int j = 0; j < MLP_NV; ++j) r += X[i * MLP_NV + j] * 0.5 * (T[j * MLP_NV + i] + T[i * MLP_NV + j]);
    double XT[MLP_NV * MLP_NV];
    for (int i = 0; i < MLP_NV; ++i)
      for (int j = 0; j < MLP_NV; ++j) {
        double v = 0.0;
        for (int q = 0; q < MLP_NV; ++q) v += X[i * MLP_NV + q] * 0.5 * (T[q * MLP_NV + j] + T[j * MLP_NV + q]);
        XT[i * MLP_NV + j] = v;
      }
    for (int i = 0; i < MLP_NV; ++i)
      for (int j = 0; j < MLP_NV; ++j) {
        double v = 0.0;
        for (int q = 0; q < MLP_NV; ++q) v += XT[i * MLP_NV + q] * X[q * MLP_NV + j];
        P[i * MLP_NV + j] = v;
      }
    ok = ok && r > 0.0 && isfinite(r);
    s_r = ok ? r : 0.0;
    lossv[smp] = ok ? log(r) : __builtin_nan("");
  }
  __syncthreads();
  const double r = s_r;
  for (int e = t; e < MLP_NV * MLP_P; e += blockDim.x) {
    const int i = e / MLP_P, j = e % MLP_P;
    double gr = 0.0;
    if (j < p && r > 0.0) {
      double v = 0.0;
      for (int q = 0; q < MLP_NV; ++q) v += X[i * MLP_NV + q] * CH[q * p + j] - P[i * MLP_NV + q] * CN[q * p + j];
      gr = 2.0 * v / r;
    }
    dout[(size_t)smp * MD3 + e] = (float)(gr * wscale);
  }
}

// per-sample backward through the activations: dA2 (128), dA1 (128).  Thread
// (t, part) sums a quarter of the outputs for input t (512 samples: 9.2 us; 20
// with one thread per input).
__global__ void __launch_bounds__(512) k_mlp_bwd_act(int B, MLPW w, const float* act, const float* dout,
                                                     float* dA2, float* dA1) {
  __shared__ float ds[MD3], d2[MD2], part[4][MD2];
  const int s = blockIdx.x, t = threadIdx.x & 127, h = threadIdx.x >> 7;
  if (s >= B) return;
  const float* as = act + (size_t)s * 4 * MD1;
  ds[threadIdx.x] = dout[(size_t)s * MD3 + threadIdx.x];
  __syncthreads();
  float g = 0.0f;
#pragma unroll 16
  for (int j = h * (MD3 / 4); j < (h + 1) * (MD3 / 4); ++j) g += ds[j] * bf2f(w.W3[j * MD2 + t]);
  part[h][t] = g;
  __syncthreads();
  if (h == 0) {
    d2[t] = ((part[0][t] + part[1][t]) + (part[2][t] + part[3][t])) * gelu_d(as[2 * MD1 + t]);
    dA2[(size_t)s * MD2 + t] = d2[t];
  }
  __syncthreads();
  g = 0.0f;
#pragma unroll 16
  for (int j = h * (MD2 / 4); j < (h + 1) * (MD2 / 4); ++j) g += d2[j] * bf2f(w.W2[j * MD1 + t]);
  part[h][t] = g;
  __syncthreads();
  if (h == 0)
    dA1[(size_t)s * MD1 + t] = ((part[0][t] + part[1][t]) + (part[2][t] + part[3][t])) * gelu_d(as[t]);
}

// Weight / bias gradients summed over the batch, all three layers at once:
//   dW[o][i] = sum_s dA[s][o] X[s][i],  db[o] = sum_s dA[s][o]
// One block per (64 x 64 tile of a layer's weights, slice of the samples): the
// tile's operands of 32 samples are staged in LDS, 4 x 4 entries per thread;
// part[slice] holds the sums of a slice in the layout of the parameters, added
// in order by k_mlp_wsum.  At 512 samples 12 us and 3 us; a thread per weight
// that walked all samples took 550 us, one load latency per sample.
struct MLPGrad {
  const float *dout, *dA2, *dA1, *act, *theta;
  int ow[3], ob[3], np;    // offsets of the layers' weights and biases, parameters
};
constexpr int WGT = 64, WGS = 32;                       // tile edge, samples per step
constexpr int WG3 = (MD3 / WGT) * (MD2 / WGT), WG2 = (MD2 / WGT) * (MD1 / WGT), WG1 = MD1 / WGT;
constexpr int WG_SLICES = 16;                           // slices at the most

__global__ void __launch_bounds__(256) k_mlp_wgrad(int B, int per, MLPGrad g, float* part) {
  __shared__ float as[WGS][WGT], xs[WGS][WGT];
  int tile = blockIdx.x, nin, ldA, ldX, layer, ntx;
  const float *A, *X;
  if (tile < WG3) { layer = 2; nin = MD2; A = g.dout; ldA = MD3; X = g.act + 3 * MD1; ldX = 4 * MD1; ntx = MD2 / WGT; }
  else if (tile < WG3 + WG2) { tile -= WG3; layer = 1; nin = MD1; A = g.dA2; ldA = MD2; X = g.act + MD1; ldX = 4 * MD1; ntx = MD1 / WGT; }
  else { tile -= WG3 + WG2; layer = 0; nin = MD0; A = g.dA1; ldA = MD1; X = g.theta; ldX = MD0; ntx = 1; }
  const int o0 = tile / ntx * WGT, i0 = tile % ntx * WGT;
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
  float acc[4][4] = {}, ab[4] = {};
  const int s1 = min(B, ((int)blockIdx.y + 1) * per);
  for (int s0 = blockIdx.y * per; s0 < s1; s0 += WGS) {
#pragma unroll
    for (int u = 0; u < WGS * WGT / 256; ++u) {
      const int e = t + u * 256, r = e / WGT, c = e % WGT;
      const bool on = s0 + r < s1;
      as[r][c] = on ? A[(size_t)(s0 + r) * ldA + o0 + c] : 0.0f;
      xs[r][c] = on && i0 + c < nin ? X[(size_t)(s0 + r) * ldX + i0 + c] : 0.0f;
    }
    __syncthreads();
#pragma unroll 8
    for (int r = 0; r < WGS; ++r) {
      float a[4], x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { a[q] = as[r][ty * 4 + q]; x[q] = xs[r][tx * 4 + q]; }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        ab[q] += a[q];
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[q][v] += a[q] * x[v];
      }
    }
    __syncthreads();
  }
  float* out = part + (size_t)blockIdx.y * g.np;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int o = o0 + ty * 4 + q;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (i0 + tx * 4 + v < nin) out[g.ow[layer] + o * nin + i0 + tx * 4 + v] = acc[q][v];
    if (tx == 0 && i0 == 0) out[g.ob[layer] + o] = ab[q];
  }
}

__global__ void k_mlp_wsum(int n, int slices, const float* part, float* grad) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  float v[WG_SLICES];
#pragma unroll
  for (int q = 0; q < WG_SLICES; ++q) v[q] = q < slices ? part[(size_t)q * n + e] : 0.0f;
  float s = 0.0f;
#pragma unroll
  for (int q = 0; q < WG_SLICES; ++q) s += v[q];
  grad[e] = s;
}

// Adam (Kingma & Ba 2015) on FP32 master parameters; refreshes the BF16 copy
__global__ void k_adam(int n, float* p, const float* g, float* mo, float* ve, uint16_t* bf, float lr,
                       float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float m = b1 * mo[i] + (1.0f - b1) * gi;
  const float v = b2 * ve[i] + (1.0f - b2) * gi * gi;
  mo[i] = m;
  ve[i] = v;
  const float pn = p[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
  p[i] = pn;
  if (bf) bf[i] = f2bf(pn);
}

__global__ void k_to_bf16(int n, const float* p, uint16_t* bf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) bf[i] = f2bf(p[i]);
}

// Per-instance basis [Z | V_m], V_m = Phi C_m^T  (column-major, KP columns,
// FP64 and FP32), C_m = out[m] reshaped NV x P.
__global__ void k_expand_basis(int64_t N, int k, int KP, int p, const double* Z, const double* Phi,
                               const float* out, double* Zb64, float* Zb32) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  const int m = blockIdx.z;
  if (i >= N) return;
  double v = 0.0;
  if (q < k) {
    v = Z[(size_t)q * N + i];
  } else if (q < k + MLP_NV) {
    const float* Cm = out + (size_t)m * MD3 + (size_t)(q - k) * MLP_P;
    for (int j = 0; j < p; ++j) v += (double)Cm[j] * Phi[(size_t)j * N + i];
  }
  Zb64[((size_t)m * KP + q) * N + i] = v;
  Zb32[((size_t)m * KP + q) * N + i] = (float)v;
}

// W[:, q] = a A^T T[:, q] + c Vtilde[:, q] on inactive rows (0 on active
// rows): S_II applied to the columns of V (factored operator, FP64).
__global__ void k_outer_cols(OpGeom op, const double* AT64, const double* T, const double* Vb,
                             const uint8_t* mask, const Inst* one, double* Wv) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  const int64_t N = op.N;
  if (i >= N) return;
  double v = 0.0;
  if (mask[i] == 0) {
    const double* Tq = T + (size_t)q * N;
    double acc = 0.0;
    for (int d = 0; d < op.D; ++d) {
      const int64_t j = i + op.offs[d];
      if (j >= 0 && j < N) acc += AT64[(size_t)d * N + i] * Tq[j];
    }
    v = one->a * acc + one->c * Vb[(size_t)q * N + i];
  }
  Wv[(size_t)q * N + i] = v;
}

}  // namespace adef2
