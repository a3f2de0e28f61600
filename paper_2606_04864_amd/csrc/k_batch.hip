// CG on several columns and independent problems at once: one recurrence per
// (problem, column), all sharing every matrix product and preconditioner
// application.  Vectors are rows of W values (W = row_width(nr), columns nr ..
// zero; see k_multi.hip), so that one workgroup handles all columns of its
// rows and a neighbour's values are one 64- or 128-byte piece.
//
// Recurrence (s, k), problem s and column k, has index s * W + k.  The rows are
// split into blocks that never cross a problem boundary (rows of block b:
// [brow[b], brow[b+1]), its problem bseg[b]; problem s owns blocks [sblk[s],
// sblk[s+1])); every reduction is a fixed-order sum of whole blocks: results
// are bitwise reproducible, and a problem's scalars do not depend on the
// others.
//
// A step is three passes over the vectors: the direction with its matrix
// product and p.q, the update with r.r, and the scatter of the preconditioner
// with r.z; the scalars in between are one small kernel each.  All three are
// bound by memory: on 32 problems of sides 128 .. 384 with eight columns they
// take 232, 162 and 89 us, which at 5 TB/s is what the update and the scatter
// have to move, and for the direction 1.7 times that.  Column by column (separate product, dots,
// direction, and transpositions to and from the preconditioner's rows) the
// whole step took 1.21 ms, now 1.09; eight columns on 512^2 0.233, now 0.221.
#include "k_common.h"

namespace amsp {

template <typename F>
static void with_width(int nr, F &&f) {
  if (row_width(nr) == 8)
    f(std::integral_constant<int, 8>{});
  else
    f(std::integral_constant<int, EIGP>{});
}

// Lane t of a workgroup handles the columns 2 (t mod W/2), + 1 of the rows
// t / (W/2), + WG / (W/2), ... of its block.
template <int W>
struct Lane {
  static constexpr int L = W / 2, ROWS = WG / L;
  int row, c;
  __device__ __forceinline__ Lane() : row(threadIdx.x / L), c(2 * (threadIdx.x % L)) {}
};

__device__ __forceinline__ d2 ld2(const double *p) { return *reinterpret_cast<const d2 *>(p); }
__device__ __forceinline__ void st2(double *p, d2 v) { *reinterpret_cast<d2 *>(p) = v; }
__device__ __forceinline__ d2 fma2(d2 a, d2 b, d2 c) {
  return d2{fma(a[0], b[0], c[0]), fma(a[1], b[1], c[1])};
}

// part[b * W + k] = sum over the workgroup of the lanes' values, fixed order
template <int W>
__device__ __forceinline__ void block_part(d2 v, double *part) {
  __shared__ double red[WG / 64][W];
  constexpr int L = W / 2;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = L; o < 64; o <<= 1) {
    v[0] += __shfl_xor(v[0], o, 64);
    v[1] += __shfl_xor(v[1], o, 64);
  }
  if (l < L) {
    red[w][2 * l] = v[0];
    red[w][2 * l + 1] = v[1];
  }
  __syncthreads();
  if (threadIdx.x < W) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < WG / 64; ++u) s += red[u][threadIdx.x];
    part[threadIdx.x] = s;
  }
}

// partials of R.R
template <int W>
__global__ void __launch_bounds__(WG) k_rows_norm(const long long *__restrict__ brow,
                                                  const double *__restrict__ R,
                                                  double *__restrict__ part) {
  const Lane<W> ln;
  const int b = blockIdx.x;
  d2 acc = {0.0, 0.0};
  for (long long i = brow[b] + ln.row; i < brow[b + 1]; i += Lane<W>::ROWS) {
    const d2 r = ld2(R + i * W + ln.c);
    acc = fma2(r, r, acc);
  }
  block_part<W>(acc, part + (size_t)b * W);
}

// One row of A times the rows x(j) on the sliced copy of A: J entries' loads
// issued together, longer rows one by one.
template <int J, typename X>
__device__ __forceinline__ d2 sell_row(int i, long long base, int wd, const int *__restrict__ scol,
                                       const double *__restrict__ sval, X &&x) {
  const int lane = i & 63;
  int c[J];
  double v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {  // (past the slice's width: the row itself, dropped)
    const long long e = base + (long long)min(j, wd - 1) * 64 + lane;
    c[j] = scol[e];
    v[j] = sval[e];
  }
  d2 xv[J];
#pragma unroll
  for (int j = 0; j < J; ++j) xv[j] = x(c[j]);
  d2 s = {0.0, 0.0};
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const d2 t = fma2(d2{v[j], v[j]}, xv[j], s);
    s = j < wd ? t : s;
  }
  for (int j = J; j < wd; ++j) {
    const long long e = base + (long long)j * 64 + lane;
    s = fma2(d2{sval[e], sval[e]}, x(scol[e]), s);
  }
  return s;
}

// p = z + beta p_old (first: p = z) for every column, q = A p (the neighbours'
// p formed from z and p_old), partials p.q.  Rows of up to five entries (plane
// grids) issue five entries' loads, longer ones eight.  Neighbouring blocks go
// to the same XCD (workgroups are dealt to the eight in turn), whose L2 then
// serves the rows that both read.
template <int W>
__global__ void __launch_bounds__(WG) k_rows_dir(int nblk,
                                                 const long long *__restrict__ brow,
                                                 const int *__restrict__ bseg,
                                                 const long long *__restrict__ sptr,
                                                 const int *__restrict__ scol,
                                                 const double *__restrict__ sval,
                                                 const double *__restrict__ beta, int first,
                                                 const double *__restrict__ z,
                                                 const double *__restrict__ pold,
                                                 double *__restrict__ pnew, double *__restrict__ q,
                                                 double *__restrict__ part) {
  const int per = (nblk + 7) / 8;
  const int b = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (b >= nblk || ((int)blockIdx.x >> 3) >= per) return;
  const Lane<W> ln;
  const d2 be = first ? d2{0.0, 0.0} : ld2(beta + (size_t)bseg[b] * W + ln.c);
  auto dir = [&](long long i) __attribute__((always_inline)) {
    const d2 zi = ld2(z + i * W + ln.c);
    return first ? zi : fma2(be, ld2(pold + i * W + ln.c), zi);
  };
  d2 acc = {0.0, 0.0};
  for (long long i = brow[b] + ln.row; i < brow[b + 1]; i += Lane<W>::ROWS) {
    const long long base = sptr[i >> 6];
    const int wd = (int)((sptr[(i >> 6) + 1] - base) >> 6);
    const d2 pi = dir(i);
    const d2 s = __all(wd <= 5) ? sell_row<5>((int)i, base, wd, scol, sval, dir)
                                : sell_row<8>((int)i, base, wd, scol, sval, dir);
    st2(pnew + i * W + ln.c, pi);
    st2(q + i * W + ln.c, s);
    acc = fma2(pi, s, acc);
  }
  block_part<W>(acc, part + (size_t)b * W);
}

// x += alpha p (x: columns ld apart), r -= alpha q, partials r.r
template <int W>
__global__ void __launch_bounds__(WG) k_rows_update(int nr, size_t ld,
                                                    const long long *__restrict__ brow,
                                                    const int *__restrict__ bseg,
                                                    const double *__restrict__ alpha,
                                                    const double *__restrict__ P,
                                                    const double *__restrict__ Q,
                                                    double *__restrict__ X, double *__restrict__ R,
                                                    double *__restrict__ part) {
  const Lane<W> ln;
  const int b = blockIdx.x;
  const d2 a = ld2(alpha + (size_t)bseg[b] * W + ln.c);
  double *const x0 = X + (size_t)ln.c * ld, *const x1 = x0 + ld;
  const bool in0 = ln.c < nr, in1 = ln.c + 1 < nr;
  d2 acc = {0.0, 0.0};
  for (long long i = brow[b] + ln.row; i < brow[b + 1]; i += Lane<W>::ROWS) {
    const d2 p = ld2(P + i * W + ln.c), qv = ld2(Q + i * W + ln.c), r = ld2(R + i * W + ln.c);
    if (in0) x0[i] = fma(a[0], p[0], x0[i]);
    if (in1) x1[i] = fma(a[1], p[1], x1[i]);
    const d2 ri = fma2(-a, qv, r);
    st2(R + i * W + ln.c, ri);
    acc = fma2(ri, ri, acc);
  }
  block_part<W>(acc, part + (size_t)b * W);
}

// z = sum of every dof's copies in the regions' outputs XN, partials r.z
template <int W>
__global__ void __launch_bounds__(WG) k_rows_scatter(const long long *__restrict__ brow,
                                                     const int *__restrict__ inv_ptr,
                                                     const int *__restrict__ ix,
                                                     const double *__restrict__ XN,
                                                     const double *__restrict__ R,
                                                     double *__restrict__ Z,
                                                     double *__restrict__ part) {
  const Lane<W> ln;
  const int b = blockIdx.x;
  d2 acc = {0.0, 0.0};
  for (long long i = brow[b] + ln.row; i < brow[b + 1]; i += Lane<W>::ROWS) {
    const d2 r = ld2(R + i * W + ln.c);
    const d2 s = sum_copies<W>((int)i, ln.c, inv_ptr, ix, XN);
    st2(Z + i * W + ln.c, s);
    acc = fma2(r, s, acc);
  }
  block_part<W>(acc, part + (size_t)b * W);
}

// R = F - Q (F: columns ld apart), partials R.R
template <int W>
__global__ void __launch_bounds__(WG) k_rows_residual(int nr, size_t ld,
                                                      const long long *__restrict__ brow,
                                                      const double *__restrict__ F,
                                                      const double *__restrict__ Q,
                                                      double *__restrict__ R,
                                                      double *__restrict__ part) {
  const Lane<W> ln;
  const int b = blockIdx.x;
  d2 acc = {0.0, 0.0};
  for (long long i = brow[b] + ln.row; i < brow[b + 1]; i += Lane<W>::ROWS) {
    d2 f = {0.0, 0.0};
    if (ln.c < nr) f[0] = F[(size_t)ln.c * ld + i];
    if (ln.c + 1 < nr) f[1] = F[(size_t)(ln.c + 1) * ld + i];
    const d2 r = f - ld2(Q + i * W + ln.c);
    st2(R + i * W + ln.c, r);
    acc = fma2(r, r, acc);
  }
  block_part<W>(acc, part + (size_t)b * W);
}

// partials of (|A| |u|)_i^2: the scale of the rounding error of any float64
// residual f - A u (attainable-accuracy floor of the solve)
template <int W>
__global__ void __launch_bounds__(WG) k_rows_floor(const long long *__restrict__ brow,
                                                   const int *__restrict__ rp,
                                                   const int *__restrict__ col,
                                                   const double *__restrict__ val,
                                                   const double *__restrict__ U,
                                                   double *__restrict__ part) {
  const Lane<W> ln;
  const int b = blockIdx.x;
  d2 acc = {0.0, 0.0};
  for (long long i = brow[b] + ln.row; i < brow[b + 1]; i += Lane<W>::ROWS) {
    d2 s = {0.0, 0.0};
    for (int e = rp[i]; e < rp[i + 1]; ++e) {
      const d2 u = ld2(U + (size_t)col[e] * W + ln.c);
      const double a = fabs(val[e]);
      s = fma2(d2{a, a}, d2{fabs(u[0]), fabs(u[1])}, s);
    }
    acc = fma2(s, s, acc);
  }
  block_part<W>(acc, part + (size_t)b * W);
}

// Sum of a problem's block partials for column threadIdx.x (valid for
// threadIdx.x < W): WG / W groups take every (WG / W)-th block, added in order.
template <int W>
__device__ __forceinline__ double seg_sum(const int *__restrict__ sblk, int s,
                                          const double *__restrict__ part, double *sh) {
  constexpr int G = WG / W;
  const int g = threadIdx.x / W, k = threadIdx.x % W;
  double acc = 0.0;
#pragma unroll 4
  for (int b = sblk[s] + g; b < sblk[s + 1]; b += G) acc += part[(size_t)b * W + k];
  __syncthreads();  // earlier readers of sh are done
  sh[g * W + k] = acc;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x < W) {
#pragma unroll
    for (int u = 0; u < G; ++u) t += sh[u * W + threadIdx.x];
  }
  return t;
}

template <int W>
__global__ void __launch_bounds__(WG) k_rows_sum(const int *__restrict__ sblk,
                                                 const double *__restrict__ part,
                                                 double *__restrict__ out) {
  __shared__ double sh[WG];
  const double t = seg_sum<W>(sblk, blockIdx.x, part, sh);
  if (threadIdx.x < W) out[blockIdx.x * W + threadIdx.x] = t;
}

// alpha = (r.z) / (p.Ap) of problem blockIdx.x's active recurrences (0
// otherwise); p.Ap <= 0 or a non-finite ratio stops the recurrence and marks
// it broken.  Clears the count that k_rows_beta adds to.
template <int W>
__global__ void __launch_bounds__(WG) k_rows_alpha(RowCgState st, const int *__restrict__ sblk,
                                                   const double *__restrict__ part,
                                                   double *__restrict__ alpha) {
  __shared__ double sh[WG];
  const double pq = seg_sum<W>(sblk, blockIdx.x, part, sh);
  if (blockIdx.x == 0 && threadIdx.x == 0) *st.nactive = 0;
  if (threadIdx.x >= W) return;
  const int r = blockIdx.x * W + threadIdx.x;
  double c = 0.0;
  if (st.active[r]) {
    const double a = st.rz[r] / pq;
    if (!(pq > 0.0) || !isfinite(a)) {
      st.broken[r] = 1;
      st.active[r] = 0;
    } else {
      c = a;
    }
  }
  alpha[r] = c;
}

// After the update and the preconditioner: an active recurrence with r.r <=
// rtol2 f.f stops (a non-finite r.r stops it as broken); the others take
// beta = (r.z)' / (r.z).  Counts the active ones; the last column of the last
// problem leaves its r.r in hist[it].
template <int W>
__global__ void __launch_bounds__(WG) k_rows_beta(RowCgState st, int nr,
                                                  const int *__restrict__ sblk,
                                                  const double *__restrict__ part_rr,
                                                  const double *__restrict__ part_rz, double rtol2,
                                                  int it, double *__restrict__ beta) {
  __shared__ double sh[WG];
  const double rr = seg_sum<W>(sblk, blockIdx.x, part_rr, sh);
  const double rz = seg_sum<W>(sblk, blockIdx.x, part_rz, sh);
  if (threadIdx.x >= 64) return;
  int act = 0;
  if (threadIdx.x < W) {
    const int r = blockIdx.x * W + threadIdx.x;
    double c = 0.0;
    st.rr[r] = rr;
    if (st.active[r]) {
      st.its[r] += 1;
      if (!isfinite(rr)) {
        st.broken[r] = 1;
        st.active[r] = 0;
      } else if (rr <= rtol2 * st.f2[r]) {
        st.active[r] = 0;
      } else {
        c = rz / st.rz[r];
        st.rz[r] = rz;
      }
    }
    beta[r] = c;
    act = st.active[r];
    if (st.hist && blockIdx.x + 1 == gridDim.x && (int)threadIdx.x == nr - 1 && it < st.hist_cap)
      st.hist[it] = rr;
  }
  const unsigned long long m = __ballot(act != 0);
  if (threadIdx.x == 0 && m) atomicAdd(st.nactive, __popcll(m));
}

// flag[0] = 1 if a stored entry couples two problems (row and column in
// different ones); problem of a row by binary search in sptr (nseg + 1)
__global__ void __launch_bounds__(WG) k_check_blocks(int n, const int *__restrict__ rp,
                                                     const int *__restrict__ col, int nseg,
                                                     const long long *__restrict__ sptr,
                                                     int *__restrict__ flag) {
  const int i = blockIdx.x * WG + threadIdx.x;
  if (i >= n) return;
  int lo = 0, hi = nseg;  // sptr[lo] <= i < sptr[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sptr[mid] <= i) lo = mid; else hi = mid;
  }
  for (int e = rp[i]; e < rp[i + 1]; ++e)
    if (col[e] < sptr[lo] || col[e] >= sptr[lo + 1]) {
      atomicOr(flag, 1);
      return;
    }
}

// ------------------------------------------------------------- launchers ---
#define AMSP_ROWS(kernel, grid, ...)                                                      \
  with_width(nr, [&](auto w) {                                                            \
    hipLaunchKernelGGL((kernel<decltype(w)::value>), dim3(grid), dim3(WG), 0, s, __VA_ARGS__); \
  })

void launch_rows_norm(hipStream_t s, const RowBlocks &b, int nr, const double *R, double *part) {
  AMSP_ROWS(k_rows_norm, b.nblk, b.brow, R, part);
}
void launch_rows_dir(hipStream_t s, const RowBlocks &b, int nr, const long long *sptr,
                     const int *scol, const double *sval, const double *beta, int first,
                     const double *z, const double *pold, double *pnew, double *q, double *part) {
  AMSP_ROWS(k_rows_dir, 8 * ((b.nblk + 7) / 8), b.nblk, b.brow, b.bseg, sptr, scol, sval, beta,
            first, z, pold, pnew, q, part);
}
void launch_rows_update(hipStream_t s, const RowBlocks &b, int nr, size_t ld, const double *alpha,
                        const double *P, const double *Q, double *X, double *R, double *part) {
  AMSP_ROWS(k_rows_update, b.nblk, nr, ld, b.brow, b.bseg, alpha, P, Q, X, R, part);
}
void launch_rows_scatter(hipStream_t s, const RowBlocks &b, int nr, const int *inv_ptr,
                         const int *ix, const double *XN, const double *R, double *Z,
                         double *part) {
  AMSP_ROWS(k_rows_scatter, b.nblk, b.brow, inv_ptr, ix, XN, R, Z, part);
}
void launch_rows_residual(hipStream_t s, const RowBlocks &b, int nr, size_t ld, const double *F,
                          const double *Q, double *R, double *part) {
  AMSP_ROWS(k_rows_residual, b.nblk, nr, ld, b.brow, F, Q, R, part);
}
void launch_rows_floor(hipStream_t s, const RowBlocks &b, int nr, const int *rp, const int *col,
                       const double *val, const double *U, double *part) {
  AMSP_ROWS(k_rows_floor, b.nblk, b.brow, rp, col, val, U, part);
}
void launch_rows_sum(hipStream_t s, const RowBlocks &b, int nr, const double *part, double *out) {
  AMSP_ROWS(k_rows_sum, b.nseg, b.sblk, part, out);
}
void launch_rows_alpha(hipStream_t s, const RowBlocks &b, int nr, const RowCgState &st,
                       const double *part, double *alpha) {
  AMSP_ROWS(k_rows_alpha, b.nseg, st, b.sblk, part, alpha);
}
void launch_rows_beta(hipStream_t s, const RowBlocks &b, int nr, const RowCgState &st,
                      const double *part_rr, const double *part_rz, double rtol2, int it,
                      double *beta) {
  AMSP_ROWS(k_rows_beta, b.nseg, st, nr, b.sblk, part_rr, part_rz, rtol2, it, beta);
}

void launch_check_blocks(hipStream_t s, int n, const int *rp, const int *col, int nseg,
                         const long long *sptr, int *flag) {
  hipLaunchKernelGGL(k_check_blocks, dim3((n + WG - 1) / WG), dim3(WG), 0, s, n, rp, col, nseg,
                     sptr, flag);
}

}  // namespace amsp
