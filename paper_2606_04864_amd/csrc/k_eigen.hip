// Batched local eigensolver and coarse-basis construction.
//
// For every region the lowest eigenpairs of the local eigenproblem
// hat A_i psi = lambda S_i psi (Section 3.2) are computed through the
// standard form B_i z = lambda z with B_i = S^{-1/2} hat A_i S^{-1/2} and
// psi = S^{-1/2} z (Section 5, parameter test).  Method: block shift-invert
// subspace iteration (Bathe-Wilson) with EIGP columns: Y = (B_i + sigma I)^{-1} X
// (Cholesky solves, k_env_solve_block), then a Rayleigh-Ritz
// step here through the Gram matrices: G = Y^T Y = L L^T, K = Y^T B_i Y with
// the sparse B_i, H = inv(L) K inv(L)^T, cyclic Jacobi on the EIGP x EIGP
// matrix H, X = Y inv(L)^T V sorted ascending, and residuals
// ||B_i x - theta x|| for the m_i + 1 lowest pairs.  Regions
// with n_i <= EIGP are solved directly by Jacobi on the dense B_i.
#include "k_common.h"
#include "k_solve.h"

namespace amsp {

constexpr int HP = EIGP + 1;  // padded row stride of the small matrices
constexpr int GR = EIG_GRAM_ROWS;
static_assert(WG == EIGP * EIGP, "one thread per entry of the EIGP x EIGP Gram matrices");

__device__ __forceinline__ double hash_uniform(unsigned a, unsigned b) {
  // SplitMix-style integer hash of (a, b) mapped to (-1, 1)
  unsigned long long x = ((unsigned long long)a << 32) ^ (unsigned long long)b;
  x += 0x9E3779B97F4A7C15ULL;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ULL;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBULL;
  x ^= x >> 31;
  return ((double)(x >> 11) * (1.0 / 9007199254740992.0)) * 2.0 - 1.0;
}

// X: column 0 = S^{1/2} 1 (the exact null vector of B_i), others pseudo-random
// functions of (global dof, column); padding rows zero.
__global__ void __launch_bounds__(WG) k_eig_init(Plan p, const double *__restrict__ sdiag,
                                                 double *__restrict__ X) {
  const int i = blockIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  const int npad = p.vp_ptr[i + 1] - p.vp_ptr[i];
  double *Xi = X + (size_t)p.vp_ptr[i] * EIGP;
  for (int e = threadIdx.x; e < npad * EIGP; e += WG) {
    const int l = e / EIGP, c = e % EIGP;
    double v = 0.0;
    if (l < ni) v = (c == 0) ? sqrt(sdiag[r0 + l]) : hash_uniform((unsigned)p.sd_dofs[r0 + l], (unsigned)c);
    Xi[e] = v;
  }
}

// Cyclic Jacobi on the symmetric EIGP x EIGP matrix H (LDS, stride HS) by one
// wavefront; V (EIGP rows) accumulates the rotations.  Round-robin ordering:
// EIGP/2 disjoint pairs per round, EIGP-1 rounds per sweep.  The index pairs of
// a round sit in the slots (2k, 2k + 1) of H and of V's columns, and every round
// writes its results to the next round's slots, a fixed permutation that a sweep
// closes: all addresses are constants of the lane.  Lane (i, j) = (t / 8, t % 8)
// forms the rotations of pairs i and j itself (the same arithmetic in every lane
// that needs them) and rotates the 2 x 2 block of H at the rows of pair i and the
// columns of pair j, rows first (J^T H) then columns (H J), and rows 2i, 2i + 1
// of V at the columns of pair j.  LDS operations of a wavefront are in order,
// so one buffer is enough.
constexpr int HS = EIGP + 2;  // row stride of H and V (16-byte pieces)

// Slot of index p at the start and the end of a sweep, and the index in slot s.
__device__ __forceinline__ int jacobi_slot(int p) { return p < 8 ? 2 * p : 2 * (EIGP - 1 - p) + 1; }
__device__ __forceinline__ int jacobi_index(int s) { return s & 1 ? EIGP - 1 - s / 2 : s / 2; }

// Rotation (c, s) that clears the entry b2 / 2 between diagonals differing by a:
// tan from tau = a / b2, formed as c^2 = (1 + |a| / r) / 2, s = b2 / (2 r c) with
// r^2 = a^2 + b2^2 (two inverse roots, no divisions), a and b2 scaled by a
// common power of two.
__device__ __forceinline__ void jacobi_rotation(double a, double b2, double &c, double &s) {
  const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(a), fabs(b2)));
  const double as = ldexp(a, e), bs = ldexp(b2, e);
  const double ri = rsqrt_d(fma(as, as, bs * bs));
  const double x = 0.5 * fma(fabs(as), ri, 1.0);
  const double xi = rsqrt_d(x);
  const double sv = 0.5 * bs * ri * xi;
  c = b2 != 0.0 ? x * xi : 1.0;
  s = b2 != 0.0 ? (a < 0.0 ? -sv : sv) : 0.0;
}

__device__ void jacobi16(double *H, double *V, double off_rel2) {
  static_assert(EIGP == 16, "lane (i, j) of one wavefront per pair of pairs");
  const int t = threadIdx.x, i = t >> 3, j = t & 7;
  for (int e = t; e < EIGP * EIGP; e += 64)
    V[(e / EIGP) * HS + jacobi_slot(e % EIGP)] = (e / EIGP == e % EIGP) ? 1.0 : 0.0;
  // slots of pair k's indices in the next round
  auto next = [](int k, int &s0, int &s1) {
    s0 = k == 0 ? 3 : 2 * k - 2;
    s1 = k == 0 ? 1 : k == 7 ? 14 : 2 * k + 3;
  };
  int r0, r1, c0, c1;
  next(i, r0, r1);
  next(j, c0, c1);
  const double *const hi = H + 2 * i * HS + 2 * i, *const hj = H + 2 * j * HS + 2 * j;
  const double *const hb = H + 2 * i * HS + 2 * j, *const vb = V + 2 * i * HS + 2 * j;
  wave_sync();
  for (int sweep = 0; sweep < 30; ++sweep) {
    // stop once the off-diagonal part is below sqrt(off_rel2) relative
    // (never below 1e-14: rounding keeps it near 1e-16 relative)
    double off = 0.0, tot = 0.0;
#pragma unroll
    for (int e = t; e < EIGP * EIGP; e += 64) {
      const int a = e / EIGP, b = e % EIGP;
      const double h2 = H[a * HS + b] * H[a * HS + b];
      tot += h2;
      off += a != b ? h2 : 0.0;
    }
    off = wave_sum(off);
    tot = wave_sum(tot);
    if (__all(off <= off_rel2 * tot)) break;
#pragma unroll 1
    for (int rnd = 0; rnd < EIGP - 1; ++rnd) {
      const d2 di = *reinterpret_cast<const d2 *>(hi), dj = *reinterpret_cast<const d2 *>(hj);
      const double ei = hi[HS + 1], ej = hj[HS + 1];
      const d2 hp = *reinterpret_cast<const d2 *>(hb), hq = *reinterpret_cast<const d2 *>(hb + HS);
      const d2 vp = *reinterpret_cast<const d2 *>(vb), vq = *reinterpret_cast<const d2 *>(vb + HS);
      double ci, si, cj, sj;
      jacobi_rotation(ei - di[0], 2.0 * di[1], ci, si);
      jacobi_rotation(ej - dj[0], 2.0 * dj[1], cj, sj);
      // rows of pair i's rotation, columns of pair j
      const double rpp = ci * hp[0] - si * hq[0], rqp = si * hp[0] + ci * hq[0];
      const double rpq = ci * hp[1] - si * hq[1], rqq = si * hp[1] + ci * hq[1];
      wave_sync();
      H[r0 * HS + c0] = cj * rpp - sj * rpq;
      H[r0 * HS + c1] = sj * rpp + cj * rpq;
      H[r1 * HS + c0] = cj * rqp - sj * rqq;
      H[r1 * HS + c1] = sj * rqp + cj * rqq;
      V[2 * i * HS + c0] = cj * vp[0] - sj * vp[1];
      V[2 * i * HS + c1] = sj * vp[0] + cj * vp[1];
      V[(2 * i + 1) * HS + c0] = cj * vq[0] - sj * vq[1];
      V[(2 * i + 1) * HS + c1] = sj * vq[0] + cj * vq[1];
      wave_sync();
    }
  }
}

// Rayleigh-Ritz on the span of the solve output Y (n_i x EIGP), without
// forming an orthonormal basis: with G = Y^T Y = L L^T and K = Y^T B Y, the
// Ritz problem is H = L^{-1} K L^{-T}, H V = V Theta, and the Ritz vectors
// are X = Y C with C = L^{-T} V.  Per sweep: BY = B Y (sparse
// product) with G and K (MFMA), the small Ritz problems, then X = Y C and
// the residuals (BY) C - X Theta (MFMA again).

// Off-diagonal entries of B_i = S^{-1/2} hat A_i S^{-1/2} for every local CSR
// entry; 0 on the diagonal (B_i has a unit diagonal).  Once per setup.
__global__ void __launch_bounds__(WG) k_eig_bval(Plan p, const double *__restrict__ val,
                                                 const double *__restrict__ sdiag,
                                                 double *__restrict__ bval) {
  const int i = blockIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  for (int l = threadIdx.x; l < ni; l += WG) {
    const double sl = sdiag[r0 + l];
    for (int e = p.loc_rowptr[r0 + l]; e < p.loc_rowptr[r0 + l + 1]; ++e) {
      const int c = p.loc_col[e];
      bval[e] = (c == l) ? 0.0 : val[p.loc_src[e]] / sqrt(sl * sdiag[r0 + c]);
    }
  }
}

// Region i's part b of the Gram matrices (its parts start at its padded rows'
// share, one spare per region for the remainders).
__device__ __forceinline__ size_t gram_part(const Plan &p, int i, int b) {
  return (size_t)(p.vp_ptr[i] / GR + i + b) * 2 * EIGP * EIGP;
}

// BY = B Y for the real rows of every unconverged region and, in the same pass,
// the Gram matrices G = Y^T Y and K = Y^T (B Y): workgroup (b, i) takes rows
// GR b .. of region i and leaves its part of both at gram_part(i, b).  Four lanes per
// row, four columns each (32-byte pieces of each neighbour row; a row's entry
// indices and values are loaded by four lanes); a wavefront's 16 rows of Y and BY
// then go through LDS to the matrix cores' layout (four rows per MFMA, lane l
// row l / 16 and column l % 16 as both operands).
// Bound by memory.  64 regions of 1284 rows take 12 us, 1024 of them 153; with
// the Gram matrices as a pass of their own over Y and BY 10 + 20 and 119 + 60.
// (GR: 64 rows 13 and 176, 256 rows 14 and 172.)
// Regions with n_i <= EIGP store G = I and K = dense B_i padded with a diagonal
// above [0, 2].
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4))) k_eig_spmm(Plan p, const double *__restrict__ val,
                                                 const double *__restrict__ sdiag,
                                                 const double *__restrict__ bval,
                                                 const double *__restrict__ Y,
                                                 double *__restrict__ BY,
                                                 double *__restrict__ GK,
                                                 const int *__restrict__ conv) {
  const int i = blockIdx.y;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  if (conv[i] || (int)blockIdx.x * GR >= ni) return;
  __shared__ __attribute__((aligned(32))) double sh[WG / 64][2][EIGP * EIGP];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int a = 4 * (t & 3);
  const size_t base = (size_t)p.vp_ptr[i] * EIGP;
  double *out = GK + gram_part(p, i, blockIdx.x);
  d4 g = {0.0, 0.0, 0.0, 0.0}, k = {0.0, 0.0, 0.0, 0.0};
  for (int rb = (int)blockIdx.x * GR; rb < min(ni, (int)(blockIdx.x + 1) * GR); rb += WG / 4) {
    const int row = rb + (t >> 2), l = min(row, ni - 1);
    const d4 y0 = *reinterpret_cast<const d4 *>(Y + base + (size_t)l * EIGP + a);
    double acc[4] = {y0[0], y0[1], y0[2], y0[3]};
    const int e0 = p.loc_rowptr[r0 + l], e1 = p.loc_rowptr[r0 + l + 1];
    // the first SU entries (a row has at least its diagonal): all index and
    // value loads, then all row loads, then the products in entry order;
    // longer rows continue one by one
    constexpr int SU = 8;
    int c[SU];
    double b[SU];
    d4 y[SU];
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int e = min(e0 + u, e1 - 1);
      c[u] = p.loc_col[e];
      b[u] = bval[e];
    }
#pragma unroll
    for (int u = 0; u < SU; ++u) y[u] = *reinterpret_cast<const d4 *>(Y + base + (size_t)c[u] * EIGP + a);
#pragma unroll
    for (int u = 0; u < SU; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double f = fma(b[u], y[u][j], acc[j]);
        acc[j] = e0 + u < e1 ? f : acc[j];
      }
    for (int e = e0 + SU; e < e1; ++e) {
      const double be = bval[e];
      const d4 ye = *reinterpret_cast<const d4 *>(Y + base + (size_t)p.loc_col[e] * EIGP + a);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = fma(be, ye[j], acc[j]);
    }
    const bool real = row < ni;
    const d4 zero = {0.0, 0.0, 0.0, 0.0}, by = {acc[0], acc[1], acc[2], acc[3]};
    if (real) *reinterpret_cast<d4 *>(BY + base + (size_t)l * EIGP + a) = by;
    *reinterpret_cast<d4 *>(&sh[w][0][(lane >> 2) * EIGP + a]) = real ? y0 : zero;
    *reinterpret_cast<d4 *>(&sh[w][1][(lane >> 2) * EIGP + a]) = real ? by : zero;
    wave_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double ys = sh[w][0][64 * s + lane], bs = sh[w][1][64 * s + lane];
      g = mfma16x16x4(ys, ys, g);
      k = mfma16x16x4(ys, bs, k);
    }
    wave_sync();
  }
  if (ni <= EIGP) {
    const int ra = t / EIGP, rc = t % EIGP;
    out[t] = (ra == rc) ? 1.0 : 0.0;
    double h = (ra == rc) ? (ra < ni ? 1.0 : 3.0 + ra) : 0.0;
    if (ra < ni && rc < ni && ra != rc) {
      const double sa = sdiag[r0 + ra];
      for (int e = p.loc_rowptr[r0 + ra]; e < p.loc_rowptr[r0 + ra + 1]; ++e)
        if (p.loc_col[e] == rc) h = val[p.loc_src[e]] / sqrt(sa * sdiag[r0 + rc]);
    }
    out[EIGP * EIGP + t] = h;
    return;
  }
  // D register q holds entry (lane/16 + 4q, lane%16); wavefronts added in order
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = ((lane >> 4) + 4 * q) * EIGP + (lane & 15);
    sh[w][0][e] = g[q];
    sh[w][1][e] = k[q];
  }
  __syncthreads();
  double sg = 0.0, sk = 0.0;
#pragma unroll
  for (int ww = 0; ww < WG / 64; ++ww) {
    sg += sh[ww][0][t];
    sk += sh[ww][1][t];
  }
  out[t] = sg;
  out[EIGP * EIGP + t] = sk;
}

// The small Ritz problems: L L^T = G, H = L^{-1} K L^{-T} (symmetrised), Jacobi,
// C = L^{-T} V with columns sorted by ascending Ritz value.  One wavefront per
// region; a serial chain bounds it (16 pivots, then 15 rounds a Jacobi sweep).
// CC[i] holds C (row-major EIGP x EIGP) then the Ritz values.
// 64 regions take 24 us, 59 before: the pivots are eliminated in registers
// (block_factor), the products run on the matrix cores, and a Jacobi round
// reads and writes fixed LDS addresses and forms its rotations without divisions.
__global__ void __launch_bounds__(64) k_eig_ritz(Plan p, double off_rel2,
                                                 const double *__restrict__ GK,
                                                 double *__restrict__ CC,
                                                 const int *__restrict__ conv) {
  const int i = blockIdx.x;
  if (conv[i]) return;
  __shared__ double G[EIGP * HP], K[EIGP * HP], Li[EIGP * HP];
  __shared__ __attribute__((aligned(16))) double H[EIGP * HS], V[EIGP * HS];
  __shared__ int perm[EIGP];
  __shared__ double theta[EIGP];
  const int t = threadIdx.x, q = t >> 4, c = t & 15;
  const int np = (p.sd_ptr[i + 1] - p.sd_ptr[i] + GR - 1) / GR;
  const double *in = GK + gram_part(p, i, 0);
  d4 g = {0.0, 0.0, 0.0, 0.0}, k = {0.0, 0.0, 0.0, 0.0};
  for (int b = 0; b < np; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      g[r] += in[(size_t)b * 2 * EIGP * EIGP + 64 * r + t];
      k[r] += in[(size_t)b * 2 * EIGP * EIGP + EIGP * EIGP + 64 * r + t];
    }
  block_store<HP>(G, g);  // (entry 64 r + t is row q + 4 r, column c)
  block_store<HP>(K, k);
  double tr = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) tr += (q + 4 * r == c) ? g[r] : 0.0;
  tr = wave_sum(tr);
  const double lo = 1e-26 * (tr > 0.0 ? tr : 1.0);  // smallest pivot
  wave_sync();
  block_factor<HP>(G, Li, lo, 1.0 / sqrt(lo));
  wave_sync();
  const d4 zero = {0.0, 0.0, 0.0, 0.0};
  const d4 lk = block_mma<false, HP>(Li, K, zero, 1.0);
  wave_sync();
  block_store<HP>(K, lk);
  wave_sync();
  const d4 h = block_mma<true, HP>(K, Li, zero, 1.0);  // (Li K) Li^T
  block_store<HP>(G, h);
  wave_sync();
#pragma unroll
  for (int r = 0; r < 4; ++r)
    H[jacobi_slot(q + 4 * r) * HS + jacobi_slot(c)] = 0.5 * (h[r] + G[c * HP + q + 4 * r]);
  wave_sync();
  jacobi16(H, V, off_rel2);
  if (t < EIGP) {  // ascending order, ties by index (a stable sort): lane a places slot a's value
    auto key = [&](int a) {
      const double x = H[a * HS + a];
      return x == x ? x : INFINITY;  // a NaN sorts last (the result is then unused)
    };
    const double th = key(t);
    int rank = 0;
#pragma unroll
    for (int b = 0; b < EIGP; ++b) {
      const double x = key(b);
      rank += (x < th || (x == th && jacobi_index(b) < jacobi_index(t))) ? 1 : 0;
    }
    perm[rank] = t;
    theta[rank] = H[t * HS + t];
  }
  wave_sync();
  double *out = CC + (size_t)i * (EIGP * EIGP + EIGP);
  d4 cc = zero;  // C = Li^T V (sorted columns)
  const int pc = perm[c];
#pragma unroll
  for (int s = 0; s < 4; ++s)
    cc = mfma16x16x4(Li[(q + 4 * s) * HP + c], V[(q + 4 * s) * HS + pc], cc);
#pragma unroll
  for (int r = 0; r < 4; ++r) out[(q + 4 * r) * EIGP + c] = cc[r];
  if (t < EIGP) out[EIGP * EIGP + t] = theta[t];
}

// X = Y C and residuals ||B x_j - theta_j x_j|| = ||(BY) C - X Theta||_j for
// the m_i + 1 lowest pairs, convergence flags and eigenvalues.  MFMA over
// 16-row blocks with the K slots permuted (slot q of step s stands for
// k = 4q + s), so a lane reads four contiguous entries of one row of Y and
// of BY and holds C[4q + s][l%16] in registers.  Y and X are distinct
// buffers; padded rows of X are zeroed (they feed the next block solve).
// Bound by memory, with few regions by the latency of a wavefront's steps, so
// their loads do not wait on each other (rows past the region are clamped, not
// branched over): 64 regions of 1284 rows 15 us (25 before), 1024 of them 93 (106).
constexpr int NW = 8;  // wavefronts
__global__ void __launch_bounds__(64 * NW) k_eig_finish(Plan p, const double *__restrict__ Y,
                                                   const double *__restrict__ BY,
                                                   double *__restrict__ X,
                                                   const double *__restrict__ CC, double tol,
                                                   int *__restrict__ conv,
                                                   double *__restrict__ lam, int ntest_extra) {
  const int i = blockIdx.x;
  if (conv[i]) return;
  __shared__ double C[EIGP * EIGP], theta[EIGP];
  __shared__ double res[NW][EIGP];
  const int t = threadIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  const int npad = p.vp_ptr[i + 1] - p.vp_ptr[i];
  const int m = p.mi[i];
  const double *in = CC + (size_t)i * (EIGP * EIGP + EIGP);
  if (t < EIGP * EIGP) C[t] = in[t];
  if (t < EIGP) theta[t] = in[EIGP * EIGP + t];
  __syncthreads();
  const size_t base = (size_t)p.vp_ptr[i] * EIGP;
  const bool small = ni <= EIGP;
  const int nchk = (m + 1 < ni ? m + 1 : ni);
  const int ntest = m + ntest_extra;  // pairs whose residuals decide convergence
  const int w = t >> 6, lane = t & 63, q = lane >> 4, col = lane & 15;
  double rs = 0.0;  // this lane's sum of squared residuals of column col
  if (small) {
    for (int e = t; e < npad * EIGP; e += 64 * NW) {
      const int l = e / EIGP, j = e % EIGP;
      X[base + e] = (l < ni) ? C[l * EIGP + j] : 0.0;
    }
  } else {
    double cb[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) cb[st] = C[(4 * q + st) * EIGP + col];
    const double th = theta[col];
    for (int rb = 16 * w; rb < npad; rb += 16 * NW) {
      const int ra = rb + col;  // A operand row: lane%16
      d4 x = {0.0, 0.0, 0.0, 0.0}, bx = {0.0, 0.0, 0.0, 0.0};
      if (rb < ni) {
        // (a row past the region is read at its last one and dropped below)
        const size_t at = base + (size_t)min(ra, ni - 1) * EIGP + 4 * q;
        const d4 ya = *reinterpret_cast<const d4 *>(Y + at);
        const d4 ba = *reinterpret_cast<const d4 *>(BY + at);
#pragma unroll
        for (int st = 0; st < 4; ++st) {
          x = mfma16x16x4(ya[st], cb[st], x);
          bx = mfma16x16x4(ba[st], cb[st], bx);
        }
      }
      // D register u holds row rb + q + 4u, column col
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = rb + q + 4 * u;
        const bool real = row < ni;
        X[base + (size_t)row * EIGP + col] = real ? x[u] : 0.0;
        const double rr = real ? bx[u] - th * x[u] : 0.0;
        rs = fma(rr, rr, rs);
      }
    }
  }
  // column sums: lanes col, col+16, col+32, col+48, then wavefronts in order
  rs += __shfl_xor(rs, 16, 64);
  rs += __shfl_xor(rs, 32, 64);
  if (lane < EIGP) res[w][lane] = rs;
  __syncthreads();
  if (t >= 64) return;
  double s = 0.0;
  if (!small && t < min(ntest, nchk)) {
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) s += res[ww][t];
    s = sqrt(s);
  }
  const bool met = __all(s <= tol);  // (false for a NaN)
  if (t == 0) conv[i] = met ? 1 : 0;
  const int ld = p.nev + 1;
  if (t < ld) lam[(size_t)i * ld + t] = (t < nchk) ? theta[t] : __builtin_nan("");
}

// psi = S^{-1/2} z for the m_i kept columns, sign: largest |psi| entry
// positive (ties: lowest global dof), Phi = psi / multiplicity (pou == 0).
__global__ void __launch_bounds__(WG) k_build_basis(Plan p, const double *__restrict__ sdiag,
                                                    const double *__restrict__ X,
                                                    double *__restrict__ phi, int pou) {
  const int i = blockIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  const int m = p.mi[i], nev = p.nev;
  const double *Xi = X + (size_t)p.vp_ptr[i] * EIGP;
  __shared__ double bestv[EIGP][WG / 64], bests[EIGP][WG / 64];
  __shared__ int bestg[EIGP][WG / 64];
  __shared__ double sgn[EIGP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // one pass over the rows for all kept columns: each thread's largest
  // |psi| per column (ties: lowest global dof) and its sign, then the
  // wavefronts' and the workgroup's (the order of comparison does not
  // matter: (|psi|, -dof) is a total order)
  double bv[EIGP], bs[EIGP];
  int bg[EIGP];
#pragma unroll
  for (int k = 0; k < EIGP; ++k) {
    bv[k] = -1.0;
    bg[k] = 0x7fffffff;
    bs[k] = 1.0;
  }
  for (int l = threadIdx.x; l < ni; l += WG) {
    const double sq = sqrt(sdiag[r0 + l]);
    const int g = p.sd_dofs[r0 + l];
    const double *xr = Xi + (size_t)l * EIGP;
    double xv[EIGP];
#pragma unroll
    for (int k = 0; k < EIGP; ++k) xv[k] = xr[k];
#pragma unroll
    for (int k = 0; k < EIGP; ++k) {
      const double ps = xv[k] / sq;
      const double a = fabs(ps);
      if (a > bv[k] || (a == bv[k] && g < bg[k])) {
        bv[k] = a;
        bg[k] = g;
        bs[k] = ps < 0.0 ? -1.0 : 1.0;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < EIGP; ++k) {
    if (k < m) {  // uniform
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(bv[k], o, 64);
        const int og = __shfl_xor(bg[k], o, 64);
        const double os = __shfl_xor(bs[k], o, 64);
        if (ov > bv[k] || (ov == bv[k] && og < bg[k])) {
          bv[k] = ov;
          bg[k] = og;
          bs[k] = os;
        }
      }
      if (lane == 0) {
        bestv[k][w] = bv[k];
        bestg[k][w] = bg[k];
        bests[k][w] = bs[k];
      }
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < m) {
    const int k = threadIdx.x;
    double v = bestv[k][0];
    int g = bestg[k][0];
    double sg = bests[k][0];
    for (int u = 1; u < WG / 64; ++u)
      if (bestv[k][u] > v || (bestv[k][u] == v && bestg[k][u] < g)) {
        v = bestv[k][u];
        g = bestg[k][u];
        sg = bests[k][u];
      }
    sgn[k] = sg;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < ni * nev; e += WG) {
    const int l = e / nev, k = e % nev;
    double v = 0.0;
    if (k < m) {
      v = sgn[k] * Xi[(size_t)l * EIGP + k] / sqrt(sdiag[r0 + l]);
      if (pou == 0) v /= (double)p.mult[p.sd_dofs[r0 + l]];
    }
    phi[(size_t)(r0 + l) * nev + k] = v;
  }
}

__global__ void k_basis_convert(const double *__restrict__ src, void *__restrict__ dst,
                                size_t count, int bf16) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (size_t)gridDim.x * blockDim.x) {
    if (bf16)
      reinterpret_cast<__hip_bfloat16 *>(dst)[e] = __float2bfloat16((float)src[e]);
    else
      reinterpret_cast<float *>(dst)[e] = (float)src[e];
  }
}

// The mixed forms store the basis in float32 or bfloat16; rounding the FP64
// basis in place first makes A0 = R0 A R0^T the Galerkin matrix of the basis
// the apply actually uses, with the products still accumulated in FP64.
__global__ void k_basis_round(double *__restrict__ phi, size_t count, int bf16) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (size_t)gridDim.x * blockDim.x) {
    const float f = (float)phi[e];
    phi[e] = bf16 ? (double)__bfloat162float(__float2bfloat16(f)) : (double)f;
  }
}

// ------------------------------------------------------------- launchers ---
// ------------------------------------------- block solve (EIGP rhs) -------
// Y = (L L^T)^{-1} X on the row-major padded blocks X[rows][EIGP] of every
// region that skip[] does not flag (env_solve, k_solve.h).
struct BlockIO {
  struct Idx {};
  struct Aux {};
  const double *in;  // the region's rows
  double *out;
  int col, rb;  // this lane's column and first row of a block
  template <typename F>
  __device__ __forceinline__ Idx idx(F, int) const {
    return {};
  }
  template <typename F>
  __device__ __forceinline__ Aux aux(F, int) const {
    return {};
  }
  template <typename F>
  __device__ __forceinline__ void load(F, int r0, Idx, d4 &x) const {
    const double *src = F::value ? in : out;  // backward: this lane's own stores
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = src[(size_t)(r0 + rb + 4 * r) * EIGP + col];
  }
  template <typename F>
  __device__ __forceinline__ void store(F, int r0, const d4 &y, Aux) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(size_t)(r0 + rb + 4 * r) * EIGP + col] = y[r];
  }
  __device__ __forceinline__ double row(int r) const { return out[(size_t)r * EIGP + col]; }
};

template <typename T, int EVU, int PF>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(EVU <= 4 && PF == 1 ? 4 : 2)))
k_env_solve_block(Plan p, const T *__restrict__ diag, const T *__restrict__ erow,
                  const T *__restrict__ ecol, const double *Xin, double *X,
                  const int *__restrict__ skip) {
  const int i = blockIdx.x;
  if (skip && skip[i]) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const size_t base = (size_t)p.vp_ptr[i] * EIGP;
  BlockIO io{Xin + base, X + base, l & 15, 16 * w + (l >> 4)};
  env_solve<EVU, PF>(p, i, diag, erow, ecol, io);
}

// Entries staged per thread: the regions of a plane grid have some 300
// envelope entries per block (four per thread cover 1024); where blocks
// average more than 700, as in three dimensions, sixteen.  Blocks in flight:
// two for a float64 factor (64 regions of 21 blocks: 79 us with one, 75 with two;
// 256: 90 / 84; 1024: 310 / 296), one for a float32 factor, whose third and fourth
// workgroup per unit are worth more where there are regions for them (1024: 215 / 235;
// 256: 83 / 80, 64: 78 / 76), and where the staged entries already fill the registers
// (regions of 16 blocks in three dimensions, 512 with a float64 factor: 165 / 169, 1728
// with a float32 one: 396 / 456).
template <typename T>
void launch_env_solve_block(hipStream_t s, const Plan &p, const T *diag, const T *erow,
                            const T *ecol, const double *X, double *Y, const int *skip) {
  if (p.env_mean <= 700)
    hipLaunchKernelGGL((k_env_solve_block<T, 4, sizeof(T) == 8 ? 2 : 1>), dim3(p.N), dim3(WG), 0,
                       s, p, diag, erow, ecol, X, Y, skip);
  else
    hipLaunchKernelGGL((k_env_solve_block<T, 16, 1>), dim3(p.N), dim3(WG), 0, s, p, diag, erow,
                       ecol, X, Y, skip);
}
template void launch_env_solve_block<double>(hipStream_t, const Plan &, const double *,
                                             const double *, const double *, const double *,
                                             double *, const int *);
template void launch_env_solve_block<float>(hipStream_t, const Plan &, const float *,
                                            const float *, const float *, const double *, double *,
                                            const int *);

void launch_eig_init(hipStream_t s, const Plan &p, const double *sdiag, double *X) {
  hipLaunchKernelGGL(k_eig_init, dim3(p.N), dim3(WG), 0, s, p, sdiag, X);
}

void launch_eig_bval(hipStream_t s, const Plan &p, const double *val, const double *sdiag,
                     double *bval) {
  hipLaunchKernelGGL(k_eig_bval, dim3(p.N), dim3(WG), 0, s, p, val, sdiag, bval);
}

void launch_eig_rr(hipStream_t s, const Plan &p, int max_ni, const double *val,
                   const double *sdiag, const double *bval, const double *Y, double *BY, double *X,
                   double *GK, double *CC, double tol, int *conv, double *lam, bool test_next) {
  hipLaunchKernelGGL(k_eig_spmm, dim3((max_ni + GR - 1) / GR, p.N), dim3(WG), 0, s, p, val, sdiag,
                     bval, Y, BY, GK, conv);
  // the small eigenproblems are diagonalised to 1e-2 tol relative: their
  // Ritz vectors then carry errors far below the residual bound the sweep
  // tests (on the vectors themselves), so this only saves Jacobi sweeps
  const double rel = fmax(1e-14, 1e-2 * tol);
  hipLaunchKernelGGL(k_eig_ritz, dim3(p.N), dim3(64), 0, s, p, rel * rel, GK, CC, conv);
  hipLaunchKernelGGL(k_eig_finish, dim3(p.N), dim3(64 * NW), 0, s, p, Y, BY, X, CC, tol, conv, lam,
                     test_next ? 1 : 0);
}

void launch_build_basis(hipStream_t s, const Plan &p, const double *sdiag, const double *X,
                        double *phi, int pou) {
  hipLaunchKernelGGL(k_build_basis, dim3(p.N), dim3(WG), 0, s, p, sdiag, X, phi, pou);
}

void launch_basis_convert(hipStream_t s, const double *phi, void *dst, size_t count, int bf16) {
  if (count == 0) return;
  size_t b = (count + WG - 1) / WG;
  if (b > 65535) b = 65535;
  hipLaunchKernelGGL(k_basis_convert, dim3((unsigned)b), dim3(WG), 0, s, phi, dst, count, bf16);
}

void launch_basis_round(hipStream_t s, double *phi, size_t count, int bf16) {
  if (count == 0) return;
  size_t b = (count + WG - 1) / WG;
  if (b > 65535) b = 65535;
  hipLaunchKernelGGL(k_basis_round, dim3((unsigned)b), dim3(WG), 0, s, phi, count, bf16);
}

}  // namespace amsp
