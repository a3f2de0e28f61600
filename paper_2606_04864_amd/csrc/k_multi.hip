// Several right-hand sides at once: z_k = M^{-1} r_k for up to EIGP columns
// with one pass over the local factors.  With many columns the local solves
// become triangular solves with a block of right-hand sides, whose products
// run on the matrix cores: the block solve that the eigensolver uses
// (env_solve), here with the Dirichlet factor of the apply.
//
// Layout: inside, vectors are rows of W values, W = 8 for up to eight columns
// and EIGP otherwise (columns nr .. W-1 zero), so that whatever reads a row
// through an index (the regions' gathers, the matrix product's neighbours)
// reads one 64- or 128-byte piece of memory; as columns n apart, the gather of
// 16 columns by region took 144 us on the 1024^2 workload against 55 for one
// transposing pass.  The coarse vectors are rows of EIGP values.  XN holds the
// region outputs (local solve plus coarse prolongation), rows of W in the
// region's ascending-global-index layout, which the scatter reads.
#include "k_common.h"
#include "k_solve.h"

namespace amsp {

// f(std::integral_constant<int, W>) for the row width of nr columns
template <typename F>
static void with_width(int nr, F &&f) {
  if (nr <= 8)
    f(std::integral_constant<int, 8>{});
  else
    f(std::integral_constant<int, EIGP>{});
}
int row_width(int nr) { return nr <= 8 ? 8 : EIGP; }

// Rows of W <-> columns ld apart, WG rows per workgroup through LDS (rows a
// padded LDS row apart, so that both sides are contiguous in memory).
template <int W>
__global__ void __launch_bounds__(WG) k_cols_to_rows(int n, size_t ld, int nr,
                                                     const double *__restrict__ A,
                                                     double *__restrict__ R) {
  __shared__ double sh[WG][W + 1];
  const int i0 = blockIdx.x * WG, i = i0 + threadIdx.x;
  const int ic = min(i, n - 1);
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const double x = A[(size_t)min(k, nr - 1) * ld + ic];
    sh[threadIdx.x][k] = k < nr ? x : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < W / 2; ++u) {
    const int e = u * WG + threadIdx.x, r = e / (W / 2), c = 2 * (e % (W / 2));
    if (i0 + r < n)
      *reinterpret_cast<d2 *>(R + (size_t)(i0 + r) * W + c) = d2{sh[r][c], sh[r][c + 1]};
  }
}

// Restriction of every column: c[coff_i + q][k] = sum_l phi_i[l][q] R[dof(l)][k]
// over the region's rows in ascending global order (phi: the copy made by
// launch_basis_to_natural), on the matrix cores: one step takes four rows,
// operand A the basis coefficients (lane's coefficient l & 15), B the rows.
// The wavefronts take interleaved four-row steps, NS at a time with all loads
// issued together, and are added in order.  Columns nr .. are stored as zero.
template <int W, typename TB>
__global__ void __launch_bounds__(WG) k_restrict_rows(Plan p, int nr, const TB *__restrict__ phi,
                                                      const double *__restrict__ R,
                                                      double *__restrict__ c) {
  __shared__ double red[WG / 64][EIGP][EIGP];
  const int i = blockIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0, m = p.mi[i];
  if (m == 0) return;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, a = l & 15, q = l >> 4;
  const TB *ph = phi + (size_t)r0 * p.nev + (size_t)min(a, m - 1) * ni;
  constexpr int NS = 6;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int s0 = 4 * w + q; s0 - q < ni; s0 += 16 * NS) {
    int dof[NS];
    TB raw[NS];
    double x[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const int pos = min(s0 + 16 * u, ni - 1);
      dof[u] = p.asc[r0 + pos];
      raw[u] = ph[pos];
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) x[u] = R[(size_t)dof[u] * W + (a & (W - 1))];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      const bool in = s0 + 16 * u < ni;
      acc = mfma16x16x4(in && a < m ? to_d(raw[u]) : 0.0, in ? x[u] : 0.0, acc);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[w][q + 4 * r][a] = acc[r];
  __syncthreads();
  const int cq = threadIdx.x / EIGP, k = threadIdx.x % EIGP;
  if (cq < m) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < WG / 64; ++u) s += red[u][cq][k];
    c[(size_t)(p.coff[i] + cq) * EIGP + k] = k < nr ? s : 0.0;
  }
}

// The rows of env_solve for the apply: gathered from R by the region's dofs
// (padding rows zero), the forward result kept in Y (rows of W), the output
// with the prolongation Phi_i t_i added (KS matrix-core steps of four
// coefficients) written to XN in the ascending-global-index layout.  For
// W < EIGP the lanes' columns W .. repeat columns 0 .. and are not stored.
template <int W, int KS, typename TB>
struct ApplyIO {
  struct Idx {
    int v[4];
  };
  struct Aux {
    int nat[4];
    TB phi[KS];
  };
  const double *R;      // [n][W]
  double *Y, *XN;       // the region's padded rows
  const int *dofs, *nat;
  const TB *phi;        // [ni][nev], local order
  int ni, nev, m, col, rb, arow, q;
  bool keep, has_t;     // keep: the backward rows are read back (row())
  double t[KS];         // coarse values 4s + q, column col
  template <typename F>
  __device__ __forceinline__ Idx idx(F, int r0) const {
    Idx x;
    if constexpr (F::value) {
#pragma unroll
      for (int r = 0; r < 4; ++r) x.v[r] = dofs[min(r0 + rb + 4 * r, ni - 1)];
    }
    return x;
  }
  template <typename F>
  __device__ __forceinline__ Aux aux(F, int r0) const {
    Aux x;
    if constexpr (!F::value) {
#pragma unroll
      for (int r = 0; r < 4; ++r) x.nat[r] = nat[min(r0 + rb + 4 * r, ni - 1)];
      const TB *ph = phi + (size_t)min(r0 + arow, ni - 1) * nev;
#pragma unroll
      for (int s = 0; s < KS; ++s) x.phi[s] = ph[min(4 * s + q, nev - 1)];
    }
    return x;
  }
  template <typename F>
  __device__ __forceinline__ void load(F, int r0, const Idx &id, d4 &x) const {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = r0 + rb + 4 * r;
      if constexpr (F::value) {
        const double v = R[(size_t)id.v[r] * W + (col & (W - 1))];
        x[r] = row < ni ? v : 0.0;
      } else {  // this lane's own stores (lanes of repeated columns: their pair's)
        x[r] = Y[(size_t)row * W + (col & (W - 1))];
      }
    }
  }
  template <typename F>
  __device__ __forceinline__ void store(F, int r0, const d4 &y, const Aux &a) const {
    if (F::value || keep) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (col < W) Y[(size_t)(r0 + rb + 4 * r) * W + col] = y[r];
    }
    if constexpr (!F::value) {
      d4 z = y;
      if (has_t) {
#pragma unroll
        for (int s = 0; s < KS; ++s) z = mfma16x16x4(4 * s + q < m ? to_d(a.phi[s]) : 0.0, t[s], z);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (col < W && r0 + rb + 4 * r < ni) XN[(size_t)a.nat[r] * W + col] = z[r];
    }
  }
  __device__ __forceinline__ double row(int r) const { return Y[(size_t)r * W + (col & (W - 1))]; }
};

template <int W, int KS, typename T, typename TB, int EVU, int PF, int OCC>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(OCC)))
k_solve_rows(Plan p, const T *__restrict__ diag, const T *__restrict__ erow,
             const T *__restrict__ ecol, const double *__restrict__ R, const TB *__restrict__ phi,
             const double *__restrict__ t, double *Y, double *XN) {
  const int i = blockIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0, npad = p.vp_ptr[i + 1] - p.vp_ptr[i];
  const size_t v0 = p.vp_ptr[i];
  ApplyIO<W, KS, TB> io;
  io.R = R;
  io.Y = Y + v0 * W;
  io.XN = XN + v0 * W;
  io.dofs = p.sd_dofs + r0;
  io.nat = p.nat + r0;
  io.phi = phi + (size_t)r0 * p.nev;
  io.ni = ni;
  io.nev = max(p.nev, 1);
  io.m = t ? p.mi[i] : 0;
  io.has_t = io.m > 0;
  if (!io.has_t) io.phi = phi;  // never null where the basis is empty (see the launcher)
  io.col = l & 15;
  io.q = l >> 4;
  io.rb = 16 * w + io.q;
  io.arow = 16 * w + (l & 15);
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = 4 * s + io.q;
    io.t[s] = k < io.m ? t[(size_t)(p.coff[i] + k) * EIGP + io.col] : 0.0;
  }
  // blocks whose segments reach beyond the ring (a block's longest column
  // segment is its last) or hold more entries than are staged read finished
  // rows from memory: the backward rows are then kept in Y as well
  const int *up = p.uptr + v0 + i;
  int far = 0;
  for (int r = TS * ((int)threadIdx.x + 1) - 1; r < npad; r += TS * WG)
    far |= up[r + 1] - up[r] > SOLVE_RING || up[r + 1] - up[r + 1 - TS] > EVU * WG;
  io.keep = __syncthreads_or(far) != 0;
  env_solve<EVU, PF>(p, i, diag, erow, ecol, io);
}

// XN = Phi_i t_i alone (the coarse part without the local solves); thread per
// row, the region's coarse values in LDS.
template <int W, typename TB>
__global__ void __launch_bounds__(WG) k_prolong_rows(Plan p, const TB *__restrict__ phi,
                                                     const double *__restrict__ t,
                                                     double *__restrict__ XN) {
  __shared__ double tl[MAXNEV][W];
  const int i = blockIdx.x;
  const int r0 = p.sd_ptr[i], ni = p.sd_ptr[i + 1] - r0, m = p.mi[i], nev = p.nev;
  const size_t v0 = p.vp_ptr[i];
  for (int e = threadIdx.x; e < m * W; e += WG)
    tl[e / W][e % W] = t[(size_t)(p.coff[i] + e / W) * EIGP + e % W];
  __syncthreads();
  for (int l = threadIdx.x; l < ni; l += WG) {
    double v[W];
#pragma unroll
    for (int k = 0; k < W; ++k) v[k] = 0.0;
    for (int q = 0; q < m; ++q) {
      const double a = to_d(phi[(size_t)(r0 + l) * nev + q]);
#pragma unroll
      for (int k = 0; k < W; ++k) v[k] = fma(a, tl[q][k], v[k]);
    }
    d2 *dst = reinterpret_cast<d2 *>(XN + (v0 + p.nat[r0 + l]) * W);
#pragma unroll
    for (int k = 0; k < W / 2; ++k) dst[k] = d2{v[2 * k], v[2 * k + 1]};
  }
}

// z_k[j] = sum over the copies of dof j of XN[copy][k], columns n apart:
// W / 2 lanes per row, WG rows per workgroup, through LDS.
template <int W>
__global__ void __launch_bounds__(WG) k_scatter_cols(int n, int nr, const int *__restrict__ inv_ptr,
                                                     const int *__restrict__ ix,
                                                     const double *__restrict__ XN,
                                                     double *__restrict__ z) {
  __shared__ double sh[WG][W + 1];
  const int i0 = blockIdx.x * WG;
#pragma unroll
  for (int u = 0; u < W / 2; ++u) {
    const int e = u * WG + threadIdx.x, r = e / (W / 2), c = 2 * (e % (W / 2));
    const d2 s = sum_copies<W>(min(i0 + r, n - 1), c, inv_ptr, ix, XN);
    sh[r][c] = s[0];
    sh[r][c + 1] = s[1];
  }
  __syncthreads();
  const int i = i0 + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int k = 0; k < W; ++k)
    if (k < nr) z[(size_t)k * n + i] = sh[threadIdx.x][k];
}

// Coarse solve of every column: the product with the tiles of W0 (or W0^T)
// for all columns at once, so W0 is read once, on the matrix cores.  Workgroup
// per lower tile (I, J), wavefront w rows 16w .. of the product; MFMA step
// (g, u), lane quarter q stands for entry 16g + 4q + u of the summed index, so
// a lane reads four neighbouring entries of W0 per group.
// part[(O * T0 + K)][row][k] (rows of W) holds the tile's contribution to
// output tile O (I, or J transposed) from input tile K (J, or I transposed).
template <int W, typename T>
__global__ void __launch_bounds__(WG) k_trmm_tiles(const T *__restrict__ Wt, int T0,
                                                   const double *__restrict__ x,
                                                   double *__restrict__ part, int transpose) {
  const int b = blockIdx.x;
  int I = (int)((sqrt(8.0 * b + 1.0) - 1.0) * 0.5);
  while ((I + 1) * (I + 2) / 2 <= b) ++I;
  while (I * (I + 1) / 2 > b) --I;
  const int J = b - I * (I + 1) / 2;  // J <= I
  const T *t = Wt + ((size_t)I * T0 + J) * TE;
  const int K = transpose ? I : J, O = transpose ? J : I;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, mi = l & 15, mq = l >> 4;
  const T *row = transpose ? t + 4 * mq * TS + 16 * w + mi : t + (16 * w + mi) * TS + 4 * mq;
  const int step = transpose ? TS : 1;
  const double *xr = x + ((size_t)K * TS + 4 * mq) * EIGP + mi;
  T a[16];
  double v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int k = 16 * (e >> 2) + (e & 3);
    a[e] = row[k * step];
    v[e] = xr[k * EIGP];
  }
  d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < 16; ++e) acc = mfma16x16x4((double)a[e], v[e], acc);
  double *dst = part + (((size_t)O * T0 + K) * TS + 16 * w + mq) * W + mi;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (mi < W) dst[4 * r * W] = acc[r];
}

// y[O*64 + r][k] = sum over input tiles K (in order) of part[(O*T0 + K)][r][k];
// columns W .. of y are stored as zero.
template <int W>
__global__ void __launch_bounds__(WG) k_trmm_reduce(int T0, const double *__restrict__ part,
                                                    double *__restrict__ y, int transpose) {
  constexpr int RW = WG / EIGP;  // rows per workgroup
  const int O = blockIdx.x / (TS / RW), r = RW * (blockIdx.x % (TS / RW)) + threadIdx.x / EIGP;
  const int k = threadIdx.x % EIGP;
  const int k0 = transpose ? O : 0, k1 = transpose ? T0 : O + 1;
  double s = 0.0;
  if (k < W) {
#pragma unroll 8
    for (int K = k0; K < k1; ++K) s += part[(((size_t)O * T0 + K) * TS + r) * W + k];
  }
  y[(size_t)(O * TS + r) * EIGP + k] = s;
}

// The mixed forms keep their f32 factor only as the two per-sweep streams;
// the block solve reads packed diagonal tiles and the envelope (row and
// column forms).  One workgroup per tile row g copies them back out: the
// forward block of g is [row-form segments | padding | diagonal tile], the
// backward block [column-form segments | padding | diagonal tile].
__global__ void __launch_bounds__(WG) k_streams_to_env(Plan p, const float *__restrict__ fst,
                                                       const float *__restrict__ bst,
                                                       float *__restrict__ dg,
                                                       float *__restrict__ er,
                                                       float *__restrict__ ec) {
  const int g = blockIdx.x;
  const int i = find_segment(p.trow_ptr, p.N, g);
  const int I = g - p.trow_ptr[i], r0 = I * TS;
  const int *ep = p.eptr + p.vp_ptr[i] + i, *up = p.uptr + p.vp_ptr[i] + i;
  const long long eb = p.ebase[i];
  {
    const float *blk = fst + p.sfr[i] + p.sfb[g];
    const int base = ep[r0], T = ep[r0 + TS] - base, Tp = (T + 3) & ~3;
    for (int k = threadIdx.x; k < T; k += WG) er[eb + base + k] = blk[k];
    for (int e = threadIdx.x; e < DE; e += WG) dg[(size_t)g * DE + e] = blk[Tp + e];
  }
  {
    const float *blk = bst + p.sbr[i] + p.sbb[g];
    const int base = up[r0], T = up[r0 + TS] - base;
    for (int k = threadIdx.x; k < T; k += WG) ec[eb + base + k] = blk[k];
  }
}

// ------------------------------------------------------------- launchers ---
void launch_streams_to_env(hipStream_t s, const Plan &p, int ntilerows, const float *fst,
                           const float *bst, float *dg, float *er, float *ec) {
  if (ntilerows <= 0) return;
  hipLaunchKernelGGL(k_streams_to_env, dim3(ntilerows), dim3(WG), 0, s, p, fst, bst, dg, er, ec);
}

void launch_cols_to_rows(hipStream_t s, int n, size_t ld, int nr, const double *A, double *R) {
  with_width(nr, [&](auto w) {
    hipLaunchKernelGGL((k_cols_to_rows<decltype(w)::value>), dim3((n + WG - 1) / WG), dim3(WG), 0,
                       s, n, ld, nr, A, R);
  });
}

template <typename TB>
void launch_restrict_rows(hipStream_t s, const Plan &p, int nr, const TB *phi, const double *R,
                          double *c) {
  with_width(nr, [&](auto w) {
    hipLaunchKernelGGL((k_restrict_rows<decltype(w)::value, TB>), dim3(p.N), dim3(WG), 0, s, p, nr,
                       phi, R, c);
  });
}

// Staged entries and blocks in flight as for launch_env_solve_block; KS: the
// matrix-core steps of four coefficients that hold nev.  Workgroups per unit
// with a float32 factor: four (128 registers, some spilled) where there are
// regions for more than two (1024 regions, three / four: W = 8 229 / 196 us, W = 16
// 258 / 235; the 2133 regions of 32 problems 446 / 397), three otherwise (64 regions:
// 86 / 95, 256: 94 / 101).
template <typename T, typename TB>
void launch_solve_rows(hipStream_t s, const Plan &p, int nr, const T *diag, const T *erow,
                       const T *ecol, const double *R, const TB *phi, const double *t, double *Y,
                       double *XN) {
  // without a basis the kernel's (unused) coefficient loads read the factor
  if (!phi) phi = reinterpret_cast<const TB *>(diag);
  auto go = [&](auto w, auto ks, auto evu, auto pf, auto occ) {
    hipLaunchKernelGGL((k_solve_rows<decltype(w)::value, decltype(ks)::value, T, TB,
                                     decltype(evu)::value, decltype(pf)::value,
                                     decltype(occ)::value>),
                       dim3(p.N), dim3(WG), 0, s, p, diag, erow, ecol, R, phi, t, Y, XN);
  };
  constexpr std::integral_constant<int, 1> i1{};
  constexpr std::integral_constant<int, 2> i2{};
  constexpr std::integral_constant<int, 3> i3{};
  constexpr std::integral_constant<int, 4> i4{};
  constexpr std::integral_constant<int, 16> i16{};
  auto variant = [&](auto w, auto ks) {
    if (p.env_mean > 700)
      go(w, ks, i16, i1, i2);
    else if constexpr (sizeof(T) == 8)
      go(w, ks, i4, i2, i2);
    else if (p.N > 512)
      go(w, ks, i4, i1, i4);
    else
      go(w, ks, i4, i1, i3);
  };
  with_width(nr, [&](auto w) {
    if (p.nev <= 8)
      variant(w, i2);
    else
      variant(w, i4);
  });
}

template <typename TB>
void launch_prolong_rows(hipStream_t s, const Plan &p, int nr, const TB *phi, const double *t,
                         double *XN) {
  with_width(nr, [&](auto w) {
    hipLaunchKernelGGL((k_prolong_rows<decltype(w)::value, TB>), dim3(p.N), dim3(WG), 0, s, p, phi,
                       t, XN);
  });
}

void launch_scatter_cols(hipStream_t s, int n, int nr, const int *inv_ptr, const int *ix,
                         const double *XN, double *z) {
  with_width(nr, [&](auto w) {
    hipLaunchKernelGGL((k_scatter_cols<decltype(w)::value>), dim3((n + WG - 1) / WG), dim3(WG), 0,
                       s, n, nr, inv_ptr, ix, XN, z);
  });
}

template <typename T>
void launch_trmm(hipStream_t s, const T *Wt, int T0, const double *x, int nr, double *part,
                 double *y, int transpose) {
  const int nb = T0 * (T0 + 1) / 2;
  if (nb == 0) return;
  with_width(nr, [&](auto w) {
    constexpr int W = decltype(w)::value;
    hipLaunchKernelGGL((k_trmm_tiles<W, T>), dim3(nb), dim3(WG), 0, s, Wt, T0, x, part, transpose);
    hipLaunchKernelGGL((k_trmm_reduce<W>), dim3(T0 * (TS * EIGP / WG)), dim3(WG), 0, s, T0, part, y,
                       transpose);
  });
}
template void launch_trmm<double>(hipStream_t, const double *, int, const double *, int, double *,
                                  double *, int);
template void launch_trmm<float>(hipStream_t, const float *, int, const double *, int, double *,
                                 double *, int);

#define AMSP_MULTI_INST(T, TB)                                                                \
  template void launch_restrict_rows<TB>(hipStream_t, const Plan &, int, const TB *,           \
                                         const double *, double *);                           \
  template void launch_prolong_rows<TB>(hipStream_t, const Plan &, int, const TB *,            \
                                        const double *, double *);                            \
  template void launch_solve_rows<T, TB>(hipStream_t, const Plan &, int, const T *, const T *, \
                                         const T *, const double *, const TB *,               \
                                         const double *, double *, double *);
AMSP_MULTI_INST(double, double)
AMSP_MULTI_INST(float, float)
AMSP_MULTI_INST(float, __hip_bfloat16)
#undef AMSP_MULTI_INST

}  // namespace amsp
