// Sparse coarse factorisation, numeric phase (see amsp_tree.h): multifrontal
// Cholesky of A0 = R0 A R0^T over a nested-dissection tree of supernodes, and
// the coarse solve through it.
//
// A front of T x T tiles (64x64, row-major inside a tile) keeps only its
// lower tiles, packed: tile (I, J), J <= I, at fbase + I(I+1)/2 + J.  Its
// first K tile rows are its own coarse dofs, the rest its update dofs.  The
// right-looking tile Cholesky runs over the own columns k < K; afterwards the
// trailing tiles hold the Schur complement that the parent adds in.
// X (T x K tiles, full) is formed by a right-looking solve of
// [L11 0; L21 I] X = [I; 0], so X = [inv(L11); -L21 inv(L11)].
// Kernels of one step take a 2D grid: y = front (inside a level's range), x =
// work item of that front; items past a front's work return at once.
#include "amsp_tree.h"
#include "k_common.h"

namespace amsp {

__device__ __forceinline__ double *ftile(double *F, const TreeDev &t, int f, int I, int J) {
  return F + ((size_t)t.fbase[f] + (size_t)I * (I + 1) / 2 + J) * TE;
}
__device__ __forceinline__ const double *ftile(const double *F, const TreeDev &t, int f, int I,
                                               int J) {
  return F + ((size_t)t.fbase[f] + (size_t)I * (I + 1) / 2 + J) * TE;
}
__device__ __forceinline__ double &fentry(double *F, const TreeDev &t, int f, int R, int C) {
  return ftile(F, t, f, R >> 6, C >> 6)[(R & 63) * TS + (C & 63)];
}
template <typename T>
__device__ __forceinline__ T *xtile(T *X, const TreeDev &t, int f, int I, int J) {
  return X + ((size_t)t.xbase[f] + (size_t)I * t.K[f] + J) * TE;
}

// (ii, jj), jj <= ii, of packed lower-triangle index b
__device__ __forceinline__ void tri_index(int b, int &ii, int &jj) {
  ii = (int)((sqrt(8.0 * b + 1.0) - 1.0) * 0.5);
  while ((ii + 1) * (ii + 2) / 2 <= b) ++ii;
  while (ii * (ii + 1) / 2 > b) --ii;
  jj = b - ii * (ii + 1) / 2;
}

// ------------------------------------------------------------ assembly ---
// Block (i, j) of A0 for every coupled pair: Phi_i^T (A Phi_j) summed over the
// pair's overlap list in fixed segments, into pb[pair][a][b] (nev x nev).
__global__ void __launch_bounds__(WG) k_pair_blocks(Plan p, CoarsePlan c,
                                                    const double *__restrict__ phi,
                                                    const double *__restrict__ W,
                                                    double *__restrict__ pb) {
  const int pr = blockIdx.x;
  const int i = c.pair_i[pr], j = c.pair_j[pr];
  const int nev = p.nev, nn = nev * nev, nseg = WG / nn;
  const int mi = p.mi[i], mj = p.mi[j];
  __shared__ double part[WG];
  const int t = threadIdx.x, ab = t % nn, seg = t / nn;
  const int a = ab / nev, b = ab % nev;
  double s = 0.0;
  if (seg < nseg && a < mi && b < mj) {
    const int q0 = c.pair_ptr[pr], len = c.pair_ptr[pr + 1] - q0;
    const int s0 = q0 + (int)(((long long)len * seg) / nseg);
    const int s1 = q0 + (int)(((long long)len * (seg + 1)) / nseg);
    const int ri = p.sd_ptr[i];
    for (int q = s0; q < s1; ++q)
      s = fma(phi[(size_t)(ri + c.pair_l[q]) * nev + a],
              W[(size_t)(c.ext_ptr[j] + c.pair_e[q]) * nev + b], s);
  }
  part[t] = s;
  __syncthreads();
  if (t < nn) {
    double tot = 0.0;
    for (int g = 0; g < nseg; ++g) tot += part[g * nn + t];
    pb[(size_t)pr * nn + t] = (a < mi && b < mj) ? tot : 0.0;
  }
}

// Unit diagonal on the own padding rows of every front and the identity in
// X's own diagonal tiles (F and X zero-filled before).
__global__ void __launch_bounds__(WG) k_tree_diag_init(TreeDev t, double *__restrict__ F,
                                                       double *__restrict__ X) {
  const int f = blockIdx.x;
  const int K = t.K[f], kd = t.kdof[f];
  for (int r = threadIdx.x; r < K * TS; r += WG) {
    if (r >= kd) fentry(F, t, f, r, r) = 1.0;
    xtile(X, t, f, r >> 6, r >> 6)[(r & 63) * TS + (r & 63)] = 1.0;
  }
}

// Lower entries of the pair blocks that land in fronts, symmetrised:
// 0.5 (B_ij[a][b] + B_ji[b][a]).
__global__ void __launch_bounds__(WG) k_tree_assemble(Plan p, TreeDev t,
                                                      const double *__restrict__ pb,
                                                      double *__restrict__ F) {
  const int e = blockIdx.x;
  const int pr = t.as_pair[e], rv = t.as_rev[e], f = t.as_front[e];
  const int i = t.pair_i[pr], j = t.pair_j[pr];
  const int nev = p.nev, nn = nev * nev;
  const int a = threadIdx.x / nev, b = threadIdx.x % nev;
  if ((int)threadIdx.x >= nn || a >= p.mi[i] || b >= p.mi[j]) return;
  const int R = t.as_ri[e] + a, C = t.as_rj[e] + b;
  if (R < C) return;  // diagonal block: its upper half is the transpose
  fentry(F, t, f, R, C) = 0.5 * (pb[(size_t)pr * nn + a * nev + b] + pb[(size_t)rv * nn + b * nev + a]);
}

// Children's Schur complements into their parents: one workgroup per lower
// tile of a child's update block; each child of the launch has its own
// parent, and a child's update rows map to distinct parent rows (increasing),
// so no two workgroups add into the same entry.
__global__ void __launch_bounds__(WG) k_tree_extend_add(TreeDev t, const int *__restrict__ children,
                                                        double *__restrict__ F) {
  const int c = children[blockIdx.y];
  const int Kc = t.K[c], U = t.T[c] - Kc, ud = t.udof[c];
  const int b = blockIdx.x;
  if (b >= U * (U + 1) / 2) return;
  int ii, jj;
  tri_index(b, ii, jj);
  const double *src = ftile(F, t, c, Kc + ii, Kc + jj);
  const int pf = t.parent[c];
  const int *ea = t.ea_row + t.vbase[c];
  for (int e = threadIdx.x; e < TE; e += WG) {
    const int r = e >> 6, cc = e & 63;
    const int t1 = TS * ii + r, t2 = TS * jj + cc;
    if (t1 >= ud || t2 >= ud || (ii == jj && cc > r)) continue;
    fentry(F, t, pf, ea[t1], ea[t2]) += src[e];
  }
}

// --------------------------------------------------- factor, step k -------
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_tree_potrf(TreeDev t, int f0, int k, double *F, double *dinv, int *status) {
  extern __shared__ double lds[];
  double *A = lds, *Y = lds + TS * LDT;
  __shared__ int fail;
  const int f = f0 + blockIdx.y;
  if (k >= t.K[f]) return;
  if (threadIdx.x == 0) fail = 0;
  double *a = ftile(F, t, f, k, k);
  tile_to_lds(a, A);
  __syncthreads();
  lds_potrf_trtri(A, Y, &fail);
  lds_to_tile(A, a);
  lds_to_tile(Y, dinv + (size_t)(t.dbase[f] + k) * TE);
  __syncthreads();
  if (threadIdx.x == 0 && fail) atomicOr(status, 1);
}

// L_ik = A_ik inv(L_kk)^T, k < i < T (in place: each wavefront reads only
// its own rows of A_ik before writing them)
__global__ void __launch_bounds__(WG) k_tree_trsm(TreeDev t, int f0, int k, double *F,
                                                  const double *dinv) {
  const int f = f0 + blockIdx.y, i = k + 1 + blockIdx.x;
  if (k >= t.K[f] || i >= t.T[f]) return;
  double *a = ftile(F, t, f, i, k);
  Acc4 o;
  acc_zero(o);
  acc_mma_abt(o, a, TS, dinv + (size_t)(t.dbase[f] + k) * TE, TS, 1.0);
  acc_store(o, a);
}

// A_ij -= L_ik L_jk^T, k < j <= i < T
__global__ void __launch_bounds__(WG) k_tree_syrk(TreeDev t, int f0, int k, double *F) {
  const int f = f0 + blockIdx.y;
  const int T = t.T[f];
  if (k >= t.K[f]) return;
  const int m = T - k - 1;
  if ((int)blockIdx.x >= m * (m + 1) / 2) return;
  int ii, jj;
  tri_index(blockIdx.x, ii, jj);
  const int i = k + 1 + ii, j = k + 1 + jj;
  __shared__ double Ly[TS * LDT];  // every wavefront multiplies by the whole L_jk
  tile_to_lds(ftile(F, t, f, j, k), Ly);
  double *c = ftile(F, t, f, i, j);
  Acc4 o;
  acc_load(o, c);
  __syncthreads();
  acc_mma_abt(o, ftile(F, t, f, i, k), TS, Ly, LDT, -1.0);
  acc_store(o, c);
}

// X_kj <- inv(L_kk) X_kj, j <= k
__global__ void __launch_bounds__(WG) k_tree_inv_row(TreeDev t, int f0, int k, double *X,
                                                     const double *dinv) {
  extern __shared__ double lds[];
  const int f = f0 + blockIdx.y, j = blockIdx.x;
  if (k >= t.K[f] || j > k) return;
  double *w = xtile(X, t, f, k, j);
  tile_to_lds(w, lds);
  __syncthreads();
  Acc4 o;
  acc_zero(o);
  acc_mma_ab(o, dinv + (size_t)(t.dbase[f] + k) * TE, TS, lds, LDT, 1.0);
  acc_store(o, w);
}

// X_ij -= L_ik X_kj, k < i < T, j <= k
__global__ void __launch_bounds__(WG) k_tree_inv_update(TreeDev t, int f0, int k,
                                                        const double *F, double *X) {
  const int f = f0 + blockIdx.y;
  if (k >= t.K[f]) return;
  const int i = k + 1 + (int)blockIdx.x / (k + 1), j = (int)blockIdx.x % (k + 1);
  if (i >= t.T[f]) return;
  __shared__ double Xk[TS * LDT];
  tile_to_lds(xtile(X, t, f, k, j), Xk);
  double *c = xtile(X, t, f, i, j);
  Acc4 o;
  acc_load(o, c);
  __syncthreads();
  acc_mma_ab(o, ftile(F, t, f, i, k), TS, Xk, LDT, -1.0);
  acc_store(o, c);
}

__global__ void k_x_to_f32(const double *__restrict__ src, float *__restrict__ dst, size_t n) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (size_t)gridDim.x * blockDim.x)
    dst[e] = (float)src[e];
}

// ----------------------------------------------------------- the solve ---
// One launch per level and direction.  A level costs its dependent memory
// round trips (gather, tiles, store), so each is taken once for as much as
// possible: a thread gathers up to four rows with their loads together, and a
// wavefront (b, j) of the 4 NJ loads its 16-row quarter b of every NJ-th tile,
// four tiles at a time, as contiguous 16-byte pieces.
// Measured (three-dimensional tree of 13824 coarse dofs in 8 levels, float32,
// both directions): 255 us with each lane walking 64-byte pieces of one tile
// after the other, 151 us so.
// A level whose fronts sum up to four tiles (SMALL) is latency alone: it loads just
// those tiles, ahead of the gather, gathers a row per thread, and adds shares in LDS
// without lane exchanges.  1024 coarse dofs of 256 regions (fronts of one to four
// tiles, float32): the coarse part of an application takes 50.4 us, 54.5 without (four
// tiles loaded behind the gather whatever their number).

// v[k][e] = entry (16 b + 4k + (l >> 4), 4 (l & 15) + e) of a tile, lane l
template <typename TX>
__device__ __forceinline__ void quarter_load(TX (&v)[4][4], const TX *__restrict__ g, int b) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[k][e] = g[(16 * b + 4 * k + (l >> 4)) * TS + 4 * (l & 15) + e];
}

// cs[r] = c + the children's contributions to front row r (in order), r < rows
// (U rows per thread with their loads together)
template <int U>
__device__ __forceinline__ void tree_gather(const TreeDev &t, int rb, int rows, int nthreads,
                                            const double *__restrict__ c,
                                            const double *v, double *cs) {
  for (int r0 = threadIdx.x; r0 < rows; r0 += U * nthreads) {
    int rc[U], g0[U], g1[U];
    double s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = rb + min(r0 + u * nthreads, rows - 1);
      rc[u] = t.row_coarse[r];
      g0[u] = t.gptr[r];
      g1[u] = t.gptr[r + 1];
    }
    int most = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double x = c[max(rc[u], 0)];
      s[u] = rc[u] >= 0 ? x : 0.0;
      most = max(most, g1[u] - g0[u]);
    }
    for (int k = 0; k < most; ++k) {
      int src[U];
      double x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) src[u] = g0[u] + k < g1[u] ? t.gsrc[g0[u] + k] : -1;
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = src[u] >= 0 ? v[src[u]] : 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u) s[u] = src[u] >= 0 ? s[u] + x[u] : s[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r0 + u * nthreads < rows) cs[r0 + u * nthreads] = s[u];
  }
}

// z[r] = y (own rows, r < own) or x (update rows) of front row r, a <= r < rows
template <int U>
__device__ __forceinline__ void tree_rows(const TreeDev &t, int rb, int a, int own, int rows,
                                          int nthreads, const double *y, const double *x,
                                          double *z) {
  for (int r0 = a + threadIdx.x; r0 < rows; r0 += U * nthreads) {
    int rc[U];
    double s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) rc[u] = t.row_coarse[rb + min(r0 + u * nthreads, rows - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = (r0 + u * nthreads < own ? y : x)[max(rc[u], 0)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r0 + u * nthreads < rows) z[r0 + u * nthreads] = rc[u] < 0 ? 0.0 : s[u];
  }
}

// Forward, one level: workgroup (front f, row tile I) forms the front's own
// input cs = c + the children's contributions, then rows 64I.. of X cs:
// own rows give y (by coarse index), update rows give the front's update
// vector v_f = (X cs) + the children's contributions to those rows.
template <typename TX, int NJ, int NB, int B, bool SMALL>
__global__ void __launch_bounds__(64 * NB * NJ) k_tree_fwd(TreeDev t, int f0, const TX *__restrict__ X,
                                                       const double *__restrict__ c,
                                                       double *__restrict__ y, double *v,
                                                       const int *__restrict__ done) {
  if (done && *done) return;
  extern __shared__ double cs[];  // 64 K
  constexpr int NQ = 4 / NB;  // workgroups per row tile
  const int f = f0 + blockIdx.y, I = blockIdx.x / NQ;
  const int K = t.K[f];
  if (I >= t.T[f]) return;
  const int rb = t.rbase[f], jn = I < K ? I + 1 : K;  // inv(L11) is lower triangular
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, j = w / NB;
  const int b0 = NB * (blockIdx.x % NQ), b = b0 + w % NB;
  TX x[B][4][4];
  auto load = [&](int J0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < B; ++u)  // (past the last tile: the last one again, unused)
      quarter_load(x[u], xtile(X, t, f, I, min(J0 + u * NJ, jn - 1)), b);
  };
  if (SMALL) load(j);
  tree_gather<SMALL ? 1 : 4>(t, rb, jn * TS, 64 * NB * NJ, c, v, cs);
  __syncthreads();
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int J0 = j; J0 < jn; J0 += B * NJ) {
    if (!SMALL) load(J0);
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (J0 + u * NJ < jn) {
        double cc[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) cc[e] = cs[(J0 + u * NJ) * TS + 4 * (l & 15) + e];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) a[k] = fma((double)x[u][k][e], cc[e], a[k]);
      }
  }
  // the 16 lanes of a row group add their shares of four rows: two steps halve
  // the rows a lane carries (lane's row 16b + 4 ((l >> 2) & 3) + (l >> 4)), two
  // add the last four lanes
#pragma unroll
  for (int o = 2; o > 0; o >>= 1)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (k < o) {
        const bool up = (l & (4 * o)) != 0;
        const double mine = up ? a[k + o] : a[k], other = up ? a[k] : a[k + o];
        a[k] = mine + __shfl_xor(other, 4 * o, 64);
      }
  const double sum = quad_sum(a[0]);
  const int rq = 4 * ((l >> 2) & 3) + (l >> 4);  // the lane's row of the quarter
  auto out = [&](int R, double s) {
    if (I < K) {
      const int rc = t.row_coarse[rb + R];
      if (rc >= 0) y[rc] = s;
    } else {
      const int u = R - K * TS;
      if (u < t.udof[f]) {
        for (int g = t.gptr[rb + R]; g < t.gptr[rb + R + 1]; ++g) s += v[t.gsrc[g]];
        v[t.vbase[f] + u] = s;
      }
    }
  };
  if constexpr (NJ == 1) {
    if ((l & 3) == 0) out(I * TS + 16 * b + rq, sum);
  } else {
    __shared__ double red[NJ][16 * NB];
    if ((l & 3) == 0) red[j][16 * (b - b0) + rq] = sum;
    __syncthreads();
    if (w != 0 || l >= 16 * NB) return;
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < NJ; ++u) s += red[u][l];
    out(I * TS + 16 * b0 + l, s);
  }
}

// Backward, one level: workgroup (front f, column tile J) forms
// z = [y on the own rows; x on the update rows (ancestors, solved)] and
// x[own rows 64J..] = (X^T z) restricted to those columns.
template <typename TX, int NJ, int B, bool SMALL>
__global__ void __launch_bounds__(256 * NJ) k_tree_bwd(TreeDev t, int f0, const TX *__restrict__ X,
                                                       const double *__restrict__ y, double *x,
                                                       const int *__restrict__ done) {
  if (done && *done) return;
  extern __shared__ double z[];  // 64 T
  // the shares of the wavefronts, or of their four row groups
  constexpr int NR = SMALL ? 16 * NJ : 4 * NJ;
  __shared__ __align__(16) double red[NR][TS];
  const int f = f0 + blockIdx.y, J = blockIdx.x;
  const int K = t.K[f], T = t.T[f];
  if (J >= K) return;
  const int rb = t.rbase[f];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, b = w & 3, j = w >> 2;
  TX xt[B][4][4];
  auto load = [&](int I0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < B; ++u)
      quarter_load(xt[u], xtile(X, t, f, min(I0 + u * NJ, T - 1), J), b);
  };
  if (SMALL) load(J + j);
  tree_rows<SMALL ? 1 : 4>(t, rb, J * TS, K * TS, T * TS, 256 * NJ, y, x, z);
  __syncthreads();
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int I0 = J + j; I0 < T; I0 += B * NJ) {
    if (!SMALL) load(I0);
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (I0 + u * NJ < T) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double zz = z[(I0 + u * NJ) * TS + 16 * b + 4 * k + (l >> 4)];
#pragma unroll
          for (int e = 0; e < 4; ++e) a[e] = fma((double)xt[u][k][e], zz, a[e]);
        }
      }
  }
  if (SMALL) {
#pragma unroll
    for (int e = 0; e < 4; ++e) red[4 * w + (l >> 4)][4 * (l & 15) + e] = a[e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      a[e] += __shfl_xor(a[e], 16, 64);
      a[e] += __shfl_xor(a[e], 32, 64);
      if (l < 16) red[w][4 * l + e] = a[e];
    }
  }
  __syncthreads();
  if (w != 0) return;
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < NR; ++u) s += red[u][l];
  const int rc = t.row_coarse[rb + J * TS + l];
  if (rc >= 0) x[rc] = s;
}

// The same for a quarter of a column tile per workgroup (columns 16b .. of
// tile J): sixteen wavefronts, each loading 64 rows x 16 columns of every
// sixteenth tile (64-byte pieces).
template <typename TX>
__global__ void __launch_bounds__(1024) k_tree_bwd_quarter(TreeDev t, int f0,
                                                           const TX *__restrict__ X,
                                                           const double *__restrict__ y, double *x,
                                                           const int *__restrict__ done) {
  if (done && *done) return;
  extern __shared__ double z[];  // 64 T
  __shared__ double red[16][16];
  const int f = f0 + blockIdx.y, J = blockIdx.x >> 2, b = blockIdx.x & 3;
  const int K = t.K[f], T = t.T[f];
  if (J >= K) return;
  const int rb = t.rbase[f];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  tree_rows<4>(t, rb, J * TS, K * TS, T * TS, 1024, y, x, z);
  __syncthreads();
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int I0 = J + w; I0 < T; I0 += 16 * 2) {
    TX xt[2][4][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const TX *g = xtile(X, t, f, min(I0 + 16 * u, T - 1), J) + (l >> 2) * TS + 16 * b + 4 * (l & 3);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) xt[u][k][e] = g[16 * k * TS + e];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (I0 + 16 * u < T) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double zz = z[(I0 + 16 * u) * TS + 16 * k + (l >> 2)];
#pragma unroll
          for (int e = 0; e < 4; ++e) a[e] = fma((double)xt[u][k][e], zz, a[e]);
        }
      }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) a[e] += __shfl_xor(a[e], o, 64);
    if (l < 4) red[w][4 * l + e] = a[e];
  }
  __syncthreads();
  if (threadIdx.x >= 16) return;
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) s += red[u][l];
  const int rc = t.row_coarse[rb + J * TS + 16 * b + l];
  if (rc >= 0) x[rc] = s;
}

// ---- the same for EIGP columns at once -----------------------------------
// c, y, v and x hold rows of EIGP values (columns nr .. of c read as zero).
// The products run on the matrix cores: wavefront (b, j) of NW = 4 NJ owns
// rows (forward; columns backward) 16b .. of the output tile and every NJ-th
// tile of the sum; MFMA step (g, u), lane quarter q stands for entry
// 16g + 4q + u of the summed index.  The input rows are staged CH tiles at a
// time.  (One column after the other, two launches per level each, was 416 us
// of a batched step of 32 problems and eight columns; so it is
// 92 us.)
constexpr int LVM = EIGP + 4;  // staged rows 4 apart fall into different banks
constexpr int TREE_CH = 4;     // tiles staged per pass

template <typename F>
__device__ __forceinline__ void tree_stage(double *cs, int rows, int nthreads, F &&value) {
  for (int e = threadIdx.x; e < rows * EIGP; e += nthreads)
    cs[(e / EIGP) * LVM + e % EIGP] = value(e / EIGP, e % EIGP);
}

// acc += A B over one tile: a[4g + u] = entry (., 16g + 4q + u) of the lane's
// output row, B from the staged rows at cs
template <typename TX>
__device__ __forceinline__ void tree_mma(d4 &acc, const TX (&a)[16], const double *cs, int mi,
                                         int mq) {
#pragma unroll
  for (int e = 0; e < 16; ++e)
    acc = mfma16x16x4((double)a[e], cs[(16 * (e >> 2) + 4 * mq + (e & 3)) * LVM + mi], acc);
}

// The NJ wavefronts' shares of the output tile added in order; out(row, col, s)
// for every entry.
template <int NJ, typename F>
__device__ __forceinline__ void tree_out(const d4 &acc, double *red, int b, int j, int mi, int mq,
                                         F &&out) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
    red[(j * TS + 16 * b + mq + 4 * r) * EIGP + mi] = acc[r];
  __syncthreads();
  for (int e = threadIdx.x; e < TS * EIGP; e += 256 * NJ) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < NJ; ++u) s += red[u * TS * EIGP + e];
    out(e / EIGP, e % EIGP, s);
  }
}

template <typename TX, int NJ>
__global__ void __launch_bounds__(256 * NJ) k_tree_fwd_multi(TreeDev t, int f0, int nr,
                                                             const TX *__restrict__ X,
                                                             const double *__restrict__ c,
                                                             double *__restrict__ y,
                                                             double *__restrict__ v) {
  __shared__ double cs[TREE_CH * TS * LVM], red[NJ * TS * EIGP];
  const int f = f0 + blockIdx.y, I = blockIdx.x;
  const int K = t.K[f];
  if (I >= t.T[f]) return;
  const int rb = t.rbase[f], jn = I < K ? I + 1 : K;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, mi = l & 15, mq = l >> 4;
  const int b = w & 3, j = w >> 2;
  auto children = [&](int r, int k) {
    double s = 0.0;
    for (int g = t.gptr[r]; g < t.gptr[r + 1]; ++g) s += v[(size_t)t.gsrc[g] * EIGP + k];
    return s;
  };
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int c0 = 0; c0 < jn; c0 += TREE_CH) {
    const int nt = min(TREE_CH, jn - c0);
    __syncthreads();  // the last pass's reads of cs done
    tree_stage(cs, nt * TS, 256 * NJ, [&](int r, int k) {
      const int row = rb + c0 * TS + r, rc = t.row_coarse[row];
      return (rc >= 0 && k < nr ? c[(size_t)rc * EIGP + k] : 0.0) + children(row, k);
    });
    __syncthreads();
    for (int J = j; J < nt; J += NJ) {
      const TX *x = xtile(X, t, f, I, c0 + J) + (16 * b + mi) * TS + 4 * mq;
      TX a[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) a[e] = x[16 * (e >> 2) + (e & 3)];
      tree_mma(acc, a, cs + J * TS * LVM, mi, mq);
    }
  }
  tree_out<NJ>(acc, red, b, j, mi, mq, [&](int r, int k, double s) {
    const int R = I * TS + r;
    if (I < K) {
      const int rc = t.row_coarse[rb + R];
      if (rc >= 0) y[(size_t)rc * EIGP + k] = s;
    } else if (R - K * TS < t.udof[f]) {
      v[(size_t)(t.vbase[f] + R - K * TS) * EIGP + k] = s + children(rb + R, k);
    }
  });
}

template <typename TX, int NJ>
__global__ void __launch_bounds__(256 * NJ) k_tree_bwd_multi(TreeDev t, int f0,
                                                             const TX *__restrict__ X,
                                                             const double *__restrict__ y,
                                                             double *__restrict__ x) {
  __shared__ double zs[TREE_CH * TS * LVM], red[NJ * TS * EIGP];
  const int f = f0 + blockIdx.y, J = blockIdx.x;
  const int K = t.K[f], T = t.T[f];
  if (J >= K) return;
  const int rb = t.rbase[f];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, mi = l & 15, mq = l >> 4;
  const int b = w & 3, j = w >> 2;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int c0 = J; c0 < T; c0 += TREE_CH) {
    const int nt = min(TREE_CH, T - c0);
    __syncthreads();
    tree_stage(zs, nt * TS, 256 * NJ, [&](int r, int k) {
      const int R = c0 * TS + r, rc = t.row_coarse[rb + R];
      return rc < 0 ? 0.0 : (R < K * TS ? y : x)[(size_t)rc * EIGP + k];
    });
    __syncthreads();
    for (int I = j; I < nt; I += NJ) {
      const TX *xt = xtile(X, t, f, c0 + I, J) + 4 * mq * TS + 16 * b + mi;
      TX a[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) a[e] = xt[(16 * (e >> 2) + (e & 3)) * TS];
      tree_mma(acc, a, zs + I * TS * LVM, mi, mq);
    }
  }
  tree_out<NJ>(acc, red, b, j, mi, mq, [&](int r, int k, double s) {
    const int rc = t.row_coarse[rb + J * TS + r];
    if (rc >= 0) x[(size_t)rc * EIGP + k] = s;
  });
}

// ------------------------------------------------------------- launchers ---
static size_t two_tiles() { return (size_t)(2 * TS * LDT) * sizeof(double); }
static size_t one_tile() { return (size_t)(TS * LDT) * sizeof(double); }

void launch_pair_blocks(hipStream_t s, const Plan &p, const CoarsePlan &c, const double *phi,
                        const double *W, double *pb) {
  if (c.npairs == 0) return;
  hipLaunchKernelGGL(k_pair_blocks, dim3(c.npairs), dim3(WG), 0, s, p, c, phi, W, pb);
}

void launch_tree_init(hipStream_t s, const TreeDev &t, int nfront, int, double *F, double *X) {
  if (nfront == 0) return;
  hipLaunchKernelGGL(k_tree_diag_init, dim3(nfront), dim3(WG), 0, s, t, F, X);
}

void launch_tree_assemble(hipStream_t s, const Plan &p, const TreeDev &t, int nas, const double *pb,
                          double *F) {
  if (nas == 0) return;
  hipLaunchKernelGGL(k_tree_assemble, dim3(nas), dim3(WG), 0, s, p, t, pb, F);
}

void launch_tree_extend_add(hipStream_t s, const TreeDev &t, const int *children, int nchild,
                            int maxU, double *F) {
  if (nchild == 0 || maxU == 0) return;
  hipLaunchKernelGGL(k_tree_extend_add, dim3(maxU, nchild), dim3(WG), 0, s, t, children, F);
}

void launch_tree_factor_step(hipStream_t s, const TreeDev &t, int f0, int f1, int maxT, int k,
                             double *F, double *dinv, int *status) {
  const int nf = f1 - f0, m = maxT - k - 1;
  if (nf <= 0) return;
  allow_lds(k_tree_potrf, two_tiles());
  hipLaunchKernelGGL(k_tree_potrf, dim3(1, nf), dim3(WG), two_tiles(), s, t, f0, k, F, dinv, status);
  if (m <= 0) return;
  hipLaunchKernelGGL(k_tree_trsm, dim3(m, nf), dim3(WG), 0, s, t, f0, k, F, dinv);
  hipLaunchKernelGGL(k_tree_syrk, dim3(m * (m + 1) / 2, nf), dim3(WG), 0, s, t, f0, k, F);
}

void launch_tree_inverse_step(hipStream_t s, const TreeDev &t, int f0, int f1, int maxT, int k,
                              const double *F, const double *dinv, double *X) {
  const int nf = f1 - f0, m = maxT - k - 1;
  if (nf <= 0) return;
  hipLaunchKernelGGL(k_tree_inv_row, dim3(k + 1, nf), dim3(WG), one_tile(), s, t, f0, k, X, dinv);
  if (m <= 0) return;
  hipLaunchKernelGGL(k_tree_inv_update, dim3(m * (k + 1), nf), dim3(WG), 0, s, t, f0, k, F, X);
}

void launch_tree_x_to_f32(hipStream_t s, const double *X, float *Xf, long long ntiles) {
  const size_t n = (size_t)ntiles * TE;
  if (n == 0) return;
  size_t b = (n + WG - 1) / WG;
  if (b > 65535) b = 65535;
  hipLaunchKernelGGL(k_x_to_f32, dim3((unsigned)b), dim3(WG), 0, s, X, Xf, n);
}

// Workgroups of a level: a whole tile each, four wavefronts, or sixteen where a
// front has more than four tiles to sum (a front whose vector leaves no LDS
// for their sums: four).  Few large fronts (at most 512 such workgroups):
// sixteen wavefronts per quarter of a tile, so that a row's or column's tiles
// arrive at more compute units.  Forward that pays from more than sixteen
// tiles (one front of 34 tiles 17.0 -> 10.4 us; eight of 35 rows by 5 columns
// 9.1 -> 15.5, their gathers being repeated), backward from more than four
// (10.2 -> 8.4, 11.2 -> 8.4).
static bool tree_wide(int sum_tiles) { return sum_tiles > 4 && sum_tiles <= 300; }
static bool tree_quarter(int out_tiles, int nf, int sum_tiles, int from) {
  return tree_wide(sum_tiles) && sum_tiles > from && (long long)out_tiles * nf <= 512;
}

template <typename TX>
void launch_tree_solve(hipStream_t s, const TreeDev &t, const std::vector<int> &lvl_ptr,
                       const std::vector<int> &lvl_maxT, const std::vector<int> &lvl_maxK,
                       int maxK, int maxT, const TX *X, const double *c, double *y, double *v,
                       double *x, const int *done) {
  const int nl = (int)lvl_ptr.size() - 1;
  const size_t smk = (size_t)maxK * TS * sizeof(double), smt = (size_t)maxT * TS * sizeof(double);
  allow_lds(k_tree_fwd<TX, 1, 4, 4, false>, smk);
  allow_lds(k_tree_fwd<TX, 4, 4, 4, false>, smk);
  allow_lds(k_tree_fwd<TX, 16, 1, 4, false>, smk);
  allow_lds(k_tree_bwd<TX, 1, 4, false>, smt);
  allow_lds(k_tree_bwd<TX, 4, 4, false>, smt);
  allow_lds(k_tree_bwd_quarter<TX>, smt);
  // tiles per batch of the four-wavefront form, and whether one holds all
  auto batch = [](int sum_tiles, auto &&go) {
    constexpr std::true_type small{};
    if (sum_tiles <= 1)
      go(std::integral_constant<int, 1>{}, small);
    else if (sum_tiles <= 2)
      go(std::integral_constant<int, 2>{}, small);
    else if (sum_tiles <= 4)
      go(std::integral_constant<int, 4>{}, small);
    else
      go(std::integral_constant<int, 4>{}, std::false_type{});
  };
  for (int h = 0; h < nl; ++h) {
    const int f0 = lvl_ptr[h], nf = lvl_ptr[h + 1] - f0, nt = lvl_maxT[h], nk = lvl_maxK[h];
    const size_t sm = (size_t)nk * TS * sizeof(double);
    if (tree_quarter(nt, nf, nk, 16))
      hipLaunchKernelGGL((k_tree_fwd<TX, 16, 1, 4, false>), dim3(4 * nt, nf), dim3(1024), sm, s, t, f0, X,
                         c, y, v, done);
    else if (tree_wide(nk))
      hipLaunchKernelGGL((k_tree_fwd<TX, 4, 4, 4, false>), dim3(nt, nf), dim3(1024), sm, s, t, f0, X, c, y,
                         v, done);
    else
      batch(nk, [&](auto b, auto small) {
        hipLaunchKernelGGL((k_tree_fwd<TX, 1, 4, decltype(b)::value, decltype(small)::value>),
                           dim3(nt, nf), dim3(256), sm, s, t, f0, X, c, y, v, done);
      });
  }
  for (int h = nl - 1; h >= 0; --h) {
    const int f0 = lvl_ptr[h], nf = lvl_ptr[h + 1] - f0, nt = lvl_maxT[h], nk = lvl_maxK[h];
    const size_t sm = (size_t)nt * TS * sizeof(double);
    if (tree_quarter(nk, nf, nt, 4))
      hipLaunchKernelGGL((k_tree_bwd_quarter<TX>), dim3(4 * nk, nf), dim3(1024), sm, s, t, f0, X, y,
                         x, done);
    else if (tree_wide(nt))
      hipLaunchKernelGGL((k_tree_bwd<TX, 4, 4, false>), dim3(nk, nf), dim3(1024), sm, s, t, f0, X, y, x,
                         done);
    else
      batch(nt, [&](auto b, auto small) {
        hipLaunchKernelGGL((k_tree_bwd<TX, 1, decltype(b)::value, decltype(small)::value>),
                           dim3(nk, nf), dim3(256), sm, s, t, f0, X, y, x, done);
      });
  }
}

template <typename TX>
void launch_tree_solve_multi(hipStream_t s, const TreeDev &t, const std::vector<int> &lvl_ptr,
                             const std::vector<int> &lvl_maxT, const std::vector<int> &lvl_maxK,
                             int nr, const TX *X, const double *c, double *y, double *v,
                             double *x) {
  const int nl = (int)lvl_ptr.size() - 1;
  for (int h = 0; h < nl; ++h) {
    const int f0 = lvl_ptr[h];
    const dim3 grid(lvl_maxT[h], lvl_ptr[h + 1] - f0);
    if (lvl_maxK[h] > 1)
      hipLaunchKernelGGL((k_tree_fwd_multi<TX, 4>), grid, dim3(1024), 0, s, t, f0, nr, X, c, y, v);
    else
      hipLaunchKernelGGL((k_tree_fwd_multi<TX, 1>), grid, dim3(256), 0, s, t, f0, nr, X, c, y, v);
  }
  for (int h = nl - 1; h >= 0; --h) {
    const int f0 = lvl_ptr[h];
    const dim3 grid(lvl_maxK[h], lvl_ptr[h + 1] - f0);
    if (lvl_maxT[h] > 1)
      hipLaunchKernelGGL((k_tree_bwd_multi<TX, 4>), grid, dim3(1024), 0, s, t, f0, X, y, x);
    else
      hipLaunchKernelGGL((k_tree_bwd_multi<TX, 1>), grid, dim3(256), 0, s, t, f0, X, y, x);
  }
}

#define AMSP_TREE_INST(TX)                                                                      \
  template void launch_tree_solve<TX>(hipStream_t, const TreeDev &, const std::vector<int> &,   \
                                      const std::vector<int> &, const std::vector<int> &, int,  \
                                      int, const TX *, const double *, double *, double *,      \
                                      double *, const int *);                                   \
  template void launch_tree_solve_multi<TX>(hipStream_t, const TreeDev &,                       \
                                            const std::vector<int> &, const std::vector<int> &, \
                                            const std::vector<int> &, int, const TX *,          \
                                            const double *, double *, double *, double *);
AMSP_TREE_INST(double)
AMSP_TREE_INST(float)
#undef AMSP_TREE_INST

}  // namespace amsp
