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

// Cyclic Jacobi on the symmetric EIGP x EIGP matrix H (LDS, stride HP) by
// one wavefront; V accumulates the rotations.  Round-robin ordering: EIGP/2
// disjoint pairs per round, EIGP-1 rounds per sweep.  Lane (i, j) = (t / 8,
// t % 8) forms the rotations of pairs i and j itself (the same arithmetic in
// every lane that needs them) and rotates the 2 x 2 block of H at the rows
// of pair i and the columns of pair j, rows first (J^T H) then columns (H J),
// and the same block of V by columns, into the other buffer of each pair
// (Hs, Vs): one barrier per round.  H and V end up pointing at the result.
__device__ void jacobi16(double *&H, double *&V, double *Hs, double *Vs, int *flag,
                         double off_rel2) {
  static_assert(EIGP == 16, "lane (i, j) of one wavefront per pair of pairs");
  const int t = threadIdx.x;
  for (int e = t; e < EIGP * EIGP; e += 64) V[(e / EIGP) * HP + e % EIGP] = (e / EIGP == e % EIGP) ? 1.0 : 0.0;
  __syncthreads();
  const int i = t >> 3, j = t & 7;
  for (int sweep = 0; sweep < 30; ++sweep) {
    {  // off-diagonal and total Frobenius norms
      double off = 0.0, tot = 0.0;
      for (int e = t; e < EIGP * EIGP; e += 64) {
        const int a = e / EIGP, b = e % EIGP;
        const double h2 = H[a * HP + b] * H[a * HP + b];
        tot += h2;
        if (a != b) off += h2;
      }
      off = wave_sum(off);
      tot = wave_sum(tot);
      // stop once the off-diagonal part is below sqrt(off_rel2) relative
      // (never below 1e-14: rounding keeps it near 1e-16 relative)
      if (t == 0) *flag = (off <= off_rel2 * tot) ? 1 : 0;
    }
    __syncthreads();
    if (*flag) break;
    for (int rnd = 0; rnd < EIGP - 1; ++rnd) {
      auto pair = [&](int k, int &pp, int &qq) {
        if (k == 0) {
          pp = rnd;
          qq = EIGP - 1;
        } else {
          pp = (rnd + k) % (EIGP - 1);
          qq = (rnd - k + (EIGP - 1)) % (EIGP - 1);
        }
        if (pp > qq) {
          const int tmp = pp;
          pp = qq;
          qq = tmp;
        }
      };
      auto rotation = [&](int pp, int qq, double &c, double &s) {
        const double apq = H[pp * HP + qq];
        c = 1.0;
        s = 0.0;
        if (apq != 0.0) {
          const double tau = (H[qq * HP + qq] - H[pp * HP + pp]) / (2.0 * apq);
          const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
          c = 1.0 / sqrt(1.0 + tt * tt);
          s = tt * c;
        }
      };
      int pi, qi, pj, qj;
      pair(i, pi, qi);
      pair(j, pj, qj);
      double ci, si, cj, sj;
      rotation(pi, qi, ci, si);
      rotation(pj, qj, cj, sj);
      const double hpp = H[pi * HP + pj], hpq = H[pi * HP + qj];
      const double hqp = H[qi * HP + pj], hqq = H[qi * HP + qj];
      const double vpp = V[pi * HP + pj], vpq = V[pi * HP + qj];
      const double vqp = V[qi * HP + pj], vqq = V[qi * HP + qj];
      // rows pi, qi (pair i's rotation), columns pj and qj
      const double rpp = ci * hpp - si * hqp, rqp = si * hpp + ci * hqp;
      const double rpq = ci * hpq - si * hqq, rqq = si * hpq + ci * hqq;
      // then columns pj, qj (pair j's rotation)
      Hs[pi * HP + pj] = cj * rpp - sj * rpq;
      Hs[pi * HP + qj] = sj * rpp + cj * rpq;
      Hs[qi * HP + pj] = cj * rqp - sj * rqq;
      Hs[qi * HP + qj] = sj * rqp + cj * rqq;
      Vs[pi * HP + pj] = cj * vpp - sj * vpq;
      Vs[pi * HP + qj] = sj * vpp + cj * vpq;
      Vs[qi * HP + pj] = cj * vqp - sj * vqq;
      Vs[qi * HP + qj] = sj * vqp + cj * vqq;
      __syncthreads();
      double *x = H;
      H = Hs;
      Hs = x;
      x = V;
      V = Vs;
      Vs = x;
    }
  }
}

// Rayleigh-Ritz on the span of the solve output Y (n_i x EIGP), without
// forming an orthonormal basis: with G = Y^T Y = L L^T and K = Y^T B Y, the
// Ritz problem is H = L^{-1} K L^{-T}, H V = V Theta, and the Ritz vectors
// are X = Y C with C = L^{-T} V.  Per sweep: BY = B Y (flat sparse product),
// G and K (MFMA over Y and BY), the small Ritz problems, then X = Y C and
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

// BY = B Y for the real rows of every unconverged region: grid (row block,
// region), 16 rows per workgroup, thread = (row, column); 16 consecutive
// threads share a row and read 128 contiguous bytes of each neighbour row.
__global__ void __launch_bounds__(WG) k_eig_spmm(Plan p, const double *__restrict__ bval,
                                                 const double *__restrict__ Y,
                                                 double *__restrict__ BY,
                                                 const int *__restrict__ conv) {
  const int i = blockIdx.y;
  if (conv[i]) return;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  // four lanes per row, four columns each (32-byte row pieces): a row's
  // entry indices and values are loaded by four lanes instead of sixteen
  const int l = blockIdx.x * (WG / 4) + (threadIdx.x >> 2), a = 4 * (threadIdx.x & 3);
  if (l >= ni) return;
  const size_t base = (size_t)p.vp_ptr[i] * EIGP;
  const d4 y0 = *reinterpret_cast<const d4 *>(Y + base + (size_t)l * EIGP + a);
  double acc[4] = {y0[0], y0[1], y0[2], y0[3]};
  const int e0 = p.loc_rowptr[r0 + l], e1 = p.loc_rowptr[r0 + l + 1];
  // the first SU entries: all index and value loads, then all row loads,
  // then the products in entry order; longer rows continue one by one
  constexpr int SU = 8;
  int c[SU];
  double b[SU];
  d4 y[SU];
#pragma unroll
  for (int u = 0; u < SU; ++u) {
    const bool in = e0 + u < e1;
    c[u] = in ? p.loc_col[e0 + u] : l;
    b[u] = in ? bval[e0 + u] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < SU; ++u) y[u] = *reinterpret_cast<const d4 *>(Y + base + (size_t)c[u] * EIGP + a);
#pragma unroll
  for (int u = 0; u < SU; ++u)
    if (e0 + u < e1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = fma(b[u], y[u][j], acc[j]);
    }
  for (int e = e0 + SU; e < e1; ++e) {
    const double be = bval[e];
    const d4 ye = *reinterpret_cast<const d4 *>(Y + base + (size_t)p.loc_col[e] * EIGP + a);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = fma(be, ye[j], acc[j]);
  }
  *reinterpret_cast<d4 *>(BY + base + (size_t)l * EIGP + a) = d4{acc[0], acc[1], acc[2], acc[3]};
}

// G = Y^T Y and K = Y^T (B Y) into GK[i][2*EIGP*EIGP].  One MFMA 16x16x4
// consumes four rows: lane l supplies Y[row0 + l/16][l%16] as both operands
// (for K, BY as the second), so each wavefront reads 512 contiguous bytes
// per step; wavefronts take interleaved four-row blocks and their
// accumulators are added in a fixed order.  Regions with n_i <= EIGP store
// G = I and K = dense B_i padded with a diagonal above [0, 2].
__global__ void __launch_bounds__(WG) k_eig_gram(Plan p, const double *__restrict__ val,
                                                 const double *__restrict__ sdiag,
                                                 const double *__restrict__ Y,
                                                 const double *__restrict__ BY,
                                                 double *__restrict__ GK,
                                                 const int *__restrict__ conv) {
  const int i = blockIdx.x;
  if (conv[i]) return;
  __shared__ double red[WG / 64][2][EIGP * EIGP];
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  const int t = threadIdx.x;
  double *out = GK + (size_t)i * 2 * EIGP * EIGP;
  if (ni <= EIGP) {
    const int a = t / EIGP, b = t % EIGP;
    out[t] = (a == b) ? 1.0 : 0.0;
    double h = (a == b) ? (a < ni ? 1.0 : 3.0 + a) : 0.0;
    if (a < ni && b < ni && a != b) {
      const double sa = sdiag[r0 + a];
      for (int e = p.loc_rowptr[r0 + a]; e < p.loc_rowptr[r0 + a + 1]; ++e)
        if (p.loc_col[e] == b) h = val[p.loc_src[e]] / sqrt(sa * sdiag[r0 + b]);
    }
    out[EIGP * EIGP + t] = h;
    return;
  }
  const size_t base = (size_t)p.vp_ptr[i] * EIGP;
  const int w = t >> 6, lane = t & 63;
  d4 g = {0.0, 0.0, 0.0, 0.0}, k = {0.0, 0.0, 0.0, 0.0};
  // rows rb .. rb+3 per step; ni > 16 so at least one full step per wave
  int rb = 4 * w;
  for (; rb + 16 < ni; rb += 32) {  // two steps per iteration (loads in flight)
    const int ra = rb + (lane >> 4), rc = ra + 16;
    const double ya = Y[base + (size_t)ra * EIGP + (lane & 15)];
    const double ba = BY[base + (size_t)ra * EIGP + (lane & 15)];
    const double yc = rc < ni ? Y[base + (size_t)rc * EIGP + (lane & 15)] : 0.0;
    const double bc = rc < ni ? BY[base + (size_t)rc * EIGP + (lane & 15)] : 0.0;
    g = mfma16x16x4(ya, ya, g);
    k = mfma16x16x4(ya, ba, k);
    g = mfma16x16x4(yc, yc, g);
    k = mfma16x16x4(yc, bc, k);
  }
  for (; rb < ni; rb += 16) {
    const int ra = rb + (lane >> 4);
    const double ya = ra < ni ? Y[base + (size_t)ra * EIGP + (lane & 15)] : 0.0;
    const double ba = ra < ni ? BY[base + (size_t)ra * EIGP + (lane & 15)] : 0.0;
    g = mfma16x16x4(ya, ya, g);
    k = mfma16x16x4(ya, ba, k);
  }
  // D register q holds entry (lane/16 + 4q, lane%16)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = ((lane >> 4) + 4 * q) * EIGP + (lane & 15);
    red[w][0][e] = g[q];
    red[w][1][e] = k[q];
  }
  __syncthreads();
  {
    double sg = 0.0, sk = 0.0;
    for (int ww = 0; ww < WG / 64; ++ww) {
      sg += red[ww][0][t];
      sk += red[ww][1][t];
    }
    out[t] = sg;
    out[EIGP * EIGP + t] = sk;
  }
}

// Pass 2 (small): L L^T = G, H = L^{-1} K L^{-T} (symmetrised), Jacobi,
// C = L^{-T} V with columns sorted by ascending Ritz value.  One wavefront
// per region.  CC[i] holds C (row-major EIGP x EIGP) then the Ritz values.
__global__ void __launch_bounds__(64) k_eig_ritz(double off_rel2, const double *__restrict__ GK,
                                                 double *__restrict__ CC,
                                                 const int *__restrict__ conv) {
  const int i = blockIdx.x;
  if (conv[i]) return;
  __shared__ double G[EIGP * HP], K[EIGP * HP], Li[EIGP * HP], Hb[EIGP * HP], Vb[EIGP * HP];
  __shared__ int perm[EIGP];
  double *H = Hb, *V = Vb;  // the Jacobi iteration's current buffers (G and K: the others)
  __shared__ double theta[EIGP];
  __shared__ int flag;
  __shared__ double floor_;
  const int t = threadIdx.x;
  const double *in = GK + (size_t)i * 2 * EIGP * EIGP;
  for (int e = t; e < EIGP * EIGP; e += 64) {
    G[(e / EIGP) * HP + e % EIGP] = in[e];
    K[(e / EIGP) * HP + e % EIGP] = in[EIGP * EIGP + e];
  }
  __syncthreads();
  if (t == 0) {
    double tr = 0.0;
    for (int a = 0; a < EIGP; ++a) tr += G[a * HP + a];
    floor_ = 1e-26 * (tr > 0.0 ? tr : 1.0);
  }
  __syncthreads();
  for (int k = 0; k < EIGP; ++k) {  // Cholesky of G (lower, in place)
    if (t == 0) {
      double d = G[k * HP + k];
      if (!(d > floor_)) d = floor_;
      G[k * HP + k] = sqrt(d);
    }
    __syncthreads();
    if (t > k && t < EIGP) G[t * HP + k] /= G[k * HP + k];
    __syncthreads();
    for (int e = t; e < EIGP * EIGP; e += 64) {
      const int r = e / EIGP, c = e % EIGP;
      if (c > k && c <= r) G[r * HP + c] = fma(-G[r * HP + k], G[c * HP + k], G[r * HP + c]);
    }
    __syncthreads();
  }
  if (t < EIGP) {  // Li = L^{-1}: lane j computes column j by forward substitution
    const int j = t;  // (the column in registers; terms m = j .. r-1 in that order)
    double lc[EIGP];
#pragma unroll
    for (int r = 0; r < EIGP; ++r) {
      double s = (r == j) ? 1.0 : 0.0;
#pragma unroll
      for (int m = 0; m < r; ++m)
        if (m >= j) s = fma(-G[r * HP + m], lc[m], s);
      lc[r] = r >= j ? s / G[r * HP + r] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < EIGP; ++r) Li[r * HP + j] = lc[r];
  }
  __syncthreads();
  for (int e = t; e < EIGP * EIGP; e += 64) {  // V <- Li K (temporary)
    const int r = e / EIGP, c = e % EIGP;
    double s = 0.0;
    for (int m = 0; m <= r; ++m) s = fma(Li[r * HP + m], K[m * HP + c], s);
    V[r * HP + c] = s;
  }
  __syncthreads();
  for (int e = t; e < EIGP * EIGP; e += 64) {  // H = (Li K) Li^T
    const int r = e / EIGP, c = e % EIGP;
    double s = 0.0;
    for (int m = 0; m <= c; ++m) s = fma(V[r * HP + m], Li[c * HP + m], s);
    H[r * HP + c] = s;
  }
  __syncthreads();
  for (int e = t; e < EIGP * EIGP; e += 64) {
    const int r = e / EIGP, c = e % EIGP;
    if (c > r) {
      const double m = 0.5 * (H[r * HP + c] + H[c * HP + r]);
      H[r * HP + c] = m;
      H[c * HP + r] = m;
    }
  }
  __syncthreads();
  jacobi16(H, V, G, K, &flag, off_rel2);  // G and K are free by now
  if (t < EIGP) {  // ascending order, ties by index (a stable sort): lane a places value a
    auto key = [&](int a) {
      const double x = H[a * HP + a];
      return x == x ? x : INFINITY;  // a NaN sorts last (the result is then unused)
    };
    const double th = key(t);
    int rank = 0;
#pragma unroll
    for (int b = 0; b < EIGP; ++b) {
      const double x = key(b);
      rank += (x < th || (x == th && b < t)) ? 1 : 0;
    }
    perm[rank] = t;
    theta[rank] = H[t * HP + t];
  }
  __syncthreads();
  double *out = CC + (size_t)i * (EIGP * EIGP + EIGP);
  for (int e = t; e < EIGP * EIGP; e += 64) {  // C = Li^T V (sorted columns)
    const int r = e / EIGP, c = e % EIGP;
    double s = 0.0;
    for (int m = r; m < EIGP; ++m) s = fma(Li[m * HP + r], V[m * HP + perm[c]], s);
    out[e] = s;
  }
  if (t < EIGP) out[EIGP * EIGP + t] = theta[t];
}

// X = Y C and residuals ||B x_j - theta_j x_j|| = ||(BY) C - X Theta||_j for
// the m_i + 1 lowest pairs, convergence flags and eigenvalues.  MFMA over
// 16-row blocks with the K slots permuted (slot q of step s stands for
// k = 4q + s), so a lane reads four contiguous entries of one row of Y and
// of BY and holds C[4q + s][l%16] in registers.  Y and X are distinct
// buffers; padded rows of X are zeroed (they feed the next block solve).
__global__ void __launch_bounds__(WG) k_eig_finish(Plan p, const double *__restrict__ Y,
                                                   const double *__restrict__ BY,
                                                   double *__restrict__ X,
                                                   const double *__restrict__ CC, double tol,
                                                   int *__restrict__ conv,
                                                   double *__restrict__ lam, int ntest_extra) {
  const int i = blockIdx.x;
  if (conv[i]) return;
  __shared__ double C[EIGP * EIGP], theta[EIGP];
  __shared__ double res[WG / 64][EIGP];
  const int t = threadIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0;
  const int npad = p.vp_ptr[i + 1] - p.vp_ptr[i];
  const int m = p.mi[i];
  const double *in = CC + (size_t)i * (EIGP * EIGP + EIGP);
  C[t] = in[t];
  if (t < EIGP) theta[t] = in[EIGP * EIGP + t];
  __syncthreads();
  const size_t base = (size_t)p.vp_ptr[i] * EIGP;
  const bool small = ni <= EIGP;
  const int nchk = (m + 1 < ni ? m + 1 : ni);
  const int ntest = m + ntest_extra;  // pairs whose residuals decide convergence
  const int w = t >> 6, lane = t & 63, q = lane >> 4, col = lane & 15;
  double rs = 0.0;  // this lane's sum of squared residuals of column col
  if (small) {
    for (int e = t; e < npad * EIGP; e += WG) {
      const int l = e / EIGP, j = e % EIGP;
      X[base + e] = (l < ni) ? C[l * EIGP + j] : 0.0;
    }
  } else {
    double cb[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) cb[st] = C[(4 * q + st) * EIGP + col];
    const double th = theta[col];
    for (int rb = 16 * w; rb < npad; rb += 64) {
      const int ra = rb + col;  // A operand row: lane%16
      d4 x = {0.0, 0.0, 0.0, 0.0}, bx = {0.0, 0.0, 0.0, 0.0};
      if (rb < ni) {
        double ya[4], ba[4];
#pragma unroll
        for (int st = 0; st < 4; ++st) {
          ya[st] = ra < ni ? Y[base + (size_t)ra * EIGP + 4 * q + st] : 0.0;
          ba[st] = ra < ni ? BY[base + (size_t)ra * EIGP + 4 * q + st] : 0.0;
        }
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
  if (t == 0) {
    double worst = 0.0;
    if (!small) {
      for (int j = 0; j < min(ntest, nchk); ++j) {
        double s = 0.0;
        for (int ww = 0; ww < WG / 64; ++ww) s += res[ww][j];
        s = sqrt(s);
        if (s > worst || !(s == s)) worst = (s == s) ? s : 1e300;
      }
    }
    conv[i] = (worst <= tol) ? 1 : 0;
    const int ld = p.nev + 1;
    for (int j = 0; j < ld; ++j) lam[(size_t)i * ld + j] = (j < nchk) ? theta[j] : __builtin_nan("");
  }
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
// two for a float64 factor (64 regions of 21 blocks: 91 us with one, 87-96
// with two; 256: 141 / 105; 1024: 335 / 315), one for a float32 factor, whose
// third and fourth workgroup per unit are worth more (256: 105 / 98; 1024:
// 220 / 250), and where the staged entries already fill the registers (512
// regions of 16 blocks in three dimensions: 155 / 170).
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
  const int rows_per_wg = WG / 4;
  hipLaunchKernelGGL(k_eig_spmm, dim3((max_ni + rows_per_wg - 1) / rows_per_wg, p.N), dim3(WG), 0,
                     s, p, bval, Y, BY, conv);
  hipLaunchKernelGGL(k_eig_gram, dim3(p.N), dim3(WG), 0, s, p, val, sdiag, Y, BY, GK, conv);
  // the small eigenproblems are diagonalised to 1e-2 tol relative: their
  // Ritz vectors then carry errors far below the residual bound the sweep
  // tests (on the vectors themselves), so this only saves Jacobi sweeps
  const double rel = fmax(1e-14, 1e-2 * tol);
  hipLaunchKernelGGL(k_eig_ritz, dim3(p.N), dim3(64), 0, s, rel * rel, GK, CC, conv);
  hipLaunchKernelGGL(k_eig_finish, dim3(p.N), dim3(WG), 0, s, p, Y, BY, X, CC, tol, conv, lam,
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
