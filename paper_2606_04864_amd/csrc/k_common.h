// Device helpers shared by the HIP kernels (gfx950, wave64).
#pragma once
#include <type_traits>
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include "amsp_internal.h"

namespace amsp {

constexpr int LDT = TS + 1;  // padded LDS row stride (doubles) for 64x64 tiles

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Fixed-order sum over the workgroup; result valid in every thread.
// sh must hold WG/64 doubles; the call contains two barriers.
__device__ __forceinline__ double block_sum(double v, double *sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < WG / 64; ++i) t += sh[i];
  return t;
}

__device__ __forceinline__ float to_f(float x) { return x; }
__device__ __forceinline__ double to_d(double x) { return x; }
__device__ __forceinline__ double to_d(float x) { return (double)x; }
__device__ __forceinline__ double to_d(__hip_bfloat16 x) { return (double)__bfloat162float(x); }
__device__ __forceinline__ float to_f(double x) { return (float)x; }
__device__ __forceinline__ float to_f(__hip_bfloat16 x) { return __bfloat162float(x); }

// Binary search: index i with ptr[i] <= x < ptr[i+1] (ptr nondecreasing, n+1 entries).
__device__ __forceinline__ int find_segment(const int *ptr, int n, int x) {
  int lo = 0, hi = n;  // invariant ptr[lo] <= x < ptr[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (ptr[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ size_t tile_elem(long long tile) { return (size_t)tile * (size_t)TE; }

// Packed diagonal tiles.  The factor pool holds the off-diagonal 64x64 tiles
// (row-major, TE entries each) followed by one lower-triangular diagonal tile
// per tile row.  Row R of a packed tile keeps columns 0..R, zero-padded to a
// multiple of 4 entries, and starts at dpos_row(R), a multiple of 4: rows are
// 16-byte aligned in fp32 and fp64, so they load in 4-entry vectors.
__host__ __device__ constexpr int dpos_row(int R) {
  return 4 * ((R >> 2) + 1) * (2 * (R >> 2) + (R & 3));
}
static_assert(dpos_row(TS) == DE, "packed diagonal tile size");
static_assert((DE * 4) % 16 == 0 && (TE * 4) % 16 == 0, "16-byte aligned tiles");

// first entry of the packed diagonal tile of global tile row g
__device__ __forceinline__ size_t diag_elem(const Plan &p, int g) {
  return (size_t)p.noff * TE + (size_t)g * DE;
}

// Entry (R, C) of a packed diagonal tile (zero above the diagonal).
template <typename T>
__device__ __forceinline__ T packed_at(const T *__restrict__ dtile, int R, int C) {
  return C <= R ? dtile[dpos_row(R) + C] : T(0);
}

// gfx950 gives a workgroup up to 160 KB of LDS; raise the dynamic-LDS limit
// of a kernel once before its first launch with more than 64 KB.
template <typename F>
inline void allow_lds(F *kernel, size_t bytes) {
  if (bytes > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// ---------------------------------------------------------------- MFMA ----
// v_mfma_f64_16x16x4f64: D(16x16) = A(16x4) B(4x16) + C, wave64.
// Lane l supplies A[l%16][l/16] and B[l/16][l%16]; D is returned in four
// registers, D[l/16 + 4r][l%16] in register r (checked on the device by
// amsp_selftest_mfma).
typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma16x16x4(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Copy a 64x64 row-major tile from global memory into padded LDS (coalesced).
template <typename T>
__device__ __forceinline__ void tile_to_lds(const T *__restrict__ g, double *lds) {
  for (int e = threadIdx.x; e < TE; e += WG) lds[(e >> 6) * LDT + (e & 63)] = to_d(g[e]);
}

__device__ __forceinline__ void lds_to_tile(const double *lds, double *__restrict__ g) {
  for (int e = threadIdx.x; e < TE; e += WG) g[e] = lds[(e >> 6) * LDT + (e & 63)];
}

// Packed diagonal tile <-> full tile in padded LDS (upper triangle zero).
__device__ __forceinline__ void packed_to_lds(const double *__restrict__ g, double *lds) {
  for (int e = threadIdx.x; e < TE; e += WG) lds[(e >> 6) * LDT + (e & 63)] = packed_at(g, e >> 6, e & 63);
}

__device__ __forceinline__ void lds_to_packed(const double *lds, double *__restrict__ g) {
  for (int e = threadIdx.x; e < TE; e += WG) {
    const int r = e >> 6, c = e & 63;
    if (c < 4 * ((r >> 2) + 1)) g[dpos_row(r) + c] = c <= r ? lds[r * LDT + c] : 0.0;
  }
}

// Synchronisation of the lanes of one wavefront around LDS traffic: LDS
// operations of a wavefront complete in order; the fences keep the compiler
// from moving loads or stores across the point.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1/sqrt(d) for d > 0 to double precision: hardware estimate y (24 bits or
// more) refined by one third-order step, y (1 + e/2 + 3e^2/8) with e = 1 - d y^2.
__device__ __forceinline__ double rsqrt_d(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-(d * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// Compile-time loop: f(std::integral_constant<int, v>) for v = B, B+S, ... < E.
template <int B, int E, int S = 1, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + S, E, S>(f);
  }
}

// Basis rows with m <= MAXNEV kept coefficients are read as KM = 4, 8 or 16
// values (the smallest that holds nev): with_km(nev, f) calls f with
// std::integral_constant<int, KM>.
template <typename F>
__device__ __forceinline__ void with_km(int nev, F &&f) {
  static_assert(MAXNEV <= 16, "basis rows are read as at most 16 coefficients");
  if (nev <= 4)
    f(std::integral_constant<int, 4>{});
  else if (nev <= 8)
    f(std::integral_constant<int, 8>{});
  else
    f(std::integral_constant<int, 16>{});
}

// Coefficients 0 .. KM-1 of a basis row with m >= 1 kept coefficients, entry
// k at ph[k * stride]; those for k >= m read as zero (basis_coef).  The loads
// are clamped into the m kept entries and issued unconditionally, so that all
// of them are in flight together: a load under "k < m" (a branch on a value
// the compiler cannot see) would be waited for before the next is issued.
template <int KM, typename TB>
__device__ __forceinline__ void basis_row_load(const TB *__restrict__ ph, size_t stride, int m,
                                               TB (&raw)[KM]) {
#pragma unroll
  for (int k = 0; k < KM; ++k) raw[k] = ph[(size_t)min(k, m - 1) * stride];
}
template <int KM, typename TB>
__device__ __forceinline__ double basis_coef(const TB (&raw)[KM], int k, int m) {
  return k < m ? to_d(raw[k]) : 0.0;
}

// Quad permutation of a double across lanes (DPP, no LDS traffic); CTRL is a
// quad_perm control word: 0xB1 swaps neighbours (lane ^ 1), 0x4E swaps pairs
// (lane ^ 2).
template <int CTRL>
__device__ __forceinline__ double dpp_quad(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The same for a float.
template <int CTRL>
__device__ __forceinline__ float dpp_quad_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over the four lanes of a quad, in every lane.
__device__ __forceinline__ double quad_sum(double v) {
  v += dpp_quad<0xB1>(v);
  return v + dpp_quad<0x4E>(v);
}
__device__ __forceinline__ float quad_sum(float v) {
  v += dpp_quad_f<0xB1>(v);
  return v + dpp_quad_f<0x4E>(v);
}

// Cholesky factor of a 64x64 SPD tile and the inverse of the factor, in LDS.
//   a (stride LDT): lower triangle of the tile on entry, L on exit (upper 0)
//   w (stride LDT): inv(L) on exit (upper 0)
// A chain of 64 dependent pivots bounds this; all other work is arranged around
// it, in blocks of 16 rows.  Wavefront 0 factors the diagonal blocks: a lane holds
// a column of the block and of the identity, one elimination turns them into L
// and inv(L), and each step's multipliers reach the 16 lanes through DPP (no LDS
// and no scalar registers on the chain).  The blocks below and left of
// it are products on the matrix cores: behind block b's pivots come its panel
// L_ib = A_ib inv(L_bb)^T and row b of the inverse, W_bj = -inv(L_bb) S_bj, one
// product per wavefront; then wavefront 0 updates and factors the next diagonal
// block, while the other three update the remaining blocks (A_ij -= L_ib
// L_jb^T) and the inverse's sums (S_ij += L_ib W_bj, kept in w).  One tile takes
// 8.2 us, 230 cycles a pivot; 23.3 with all 64 columns in one wavefront's
// registers and the inverse solved row by row behind it.  (Multipliers as
// wave-uniform lane reads: 10.5.)
// Accuracy (condition numbers of general tiles; against 80-bit arithmetic): the
// errors of L, of inv(L) and of a solve and |L L^T - A| are those of the elimination
// column by column up to condition 1e6 and at most twice them at 2e9; |L inv(L) - I|,
// 1e-15 there, grows with the 16-row blocks' condition (3e-15 at 3e6, 5e-14 at 2e9).
// Tiles of Darcy matrices, also at a contrast of 1e6: 4e-16, as before.
// A non-positive or non-finite pivot sets *fail; L and inv(L) then mean nothing (each
// caller's setup ends with an error).  Needs blockDim.x == 256.

// c += X Y^T or X Y of 16x16 blocks in LDS (row stride LD), one wavefront;
// element r of c is row lane / 16 + 4r, column lane % 16.
template <bool YT, int LD = LDT>
__device__ __forceinline__ d4 block_mma(const double *X, const double *Y, d4 c, double sign) {
  const int l = threadIdx.x & 63, i = l & 15, q = l >> 4;
  double x[4], y[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    x[s] = X[i * LD + 4 * q + s];
    y[s] = YT ? Y[i * LD + 4 * q + s] : Y[(4 * q + s) * LD + i];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) c = mfma16x16x4(sign * x[s], y[s], c);
  return c;
}
template <int LD = LDT>
__device__ __forceinline__ d4 block_load(const double *X) {
  const int l = threadIdx.x & 63;
  d4 c;
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = X[((l >> 4) + 4 * r) * LD + (l & 15)];
  return c;
}
template <int LD = LDT>
__device__ __forceinline__ void block_store(double *X, d4 c) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) X[((l >> 4) + 4 * r) * LD + (l & 15)] = c[r];
}

// Lane K of every 16 lanes' value in all 16 of them (DPP, folds into the use).
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x150 + K, 0xF, 0xF, true);
}

// One diagonal block (one wavefront): L over its lower triangle in a, inv(L) in
// w, zeros above both diagonals.  A pivot not above lo (or not finite) is bad and
// its root's inverse replaced by alt; returns whether one was.
template <int LD = LDT>
__device__ __forceinline__ bool block_factor(double *a, double *w, double lo = 0.0,
                                             double alt = 1.0) {
  const int l = threadIdx.x & 63, c = l & 15;
  double v[16], x[16];  // column c of the block and of the identity, in every 16 lanes
  static_for<0, 16>([&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value;
    v[i] = a[max(i, c) * LD + min(i, c)];
    x[i] = i == c ? 1.0 : 0.0;
  });
  wave_sync();
  // lanes 0 .. 15 store row k of L^T, the others (repeatedly) row k of inv(L)
  const bool left = l < 16;
  double *out = left ? a + c * LD : w + c;
  const int step = left ? 1 : LD, kept = left ? c : 16;  // (inv(L) is zero above by itself)
  bool bad = false;
  static_for<0, 16>([&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const double d = row_bcast<k>(v[k]);
    const bool bk = !(d > lo) || !isfinite(d);
    bad = bad || bk;
    double inv = rsqrt_d(d);
    __asm__ volatile("" : "+v"(inv));  // no branch around it
    inv = bk ? alt : inv;
    const double uv = v[k] * inv, ux = x[k] * inv;
    if constexpr (k < 15) {
      const double m = row_bcast<k>(v[k + 1]) * inv;
      x[k + 1] = fma(-m, ux, x[k + 1]);
      v[k + 1] = fma(-m, uv, v[k + 1]);  // the next pivot waits for this one only
      const double tv = -(uv * inv), tx = -(ux * inv);
      static_for<k + 2, 16>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        x[i] = fma(row_bcast<k>(v[i]), tx, x[i]);
        v[i] = fma(row_bcast<k>(v[i]), tv, v[i]);
      });
    }
    *out = kept >= k ? (left ? uv : ux) : 0.0;
    out += step;
  });
  return bad;
}

__device__ __forceinline__ void lds_potrf_trtri(double *a, double *w, int *fail) {
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  auto at = [](double *t, int i, int j) { return t + 16 * i * LDT + 16 * j; };
  for (int b = 0; b < 4; ++b) {
    if (wv == 0) {
      if (b > 0) {
        const double *lb = at(a, b, b - 1);
        block_store(at(a, b, b), block_mma<true>(lb, lb, block_load(at(a, b, b)), -1.0));
        wave_sync();
      }
      if (block_factor(at(a, b, b), at(w, b, b)) && threadIdx.x == 0) *fail = 1;
    } else if (b == 0) {  // the blocks above the diagonal
      for (int e = threadIdx.x - 64; e < 6 * 256; e += 192) {
        const int k = e >> 8, i = k < 3 ? 0 : k < 5 ? 1 : 2, j = k < 3 ? k + 1 : k < 5 ? k - 1 : 3;
        const int o = (16 * i + ((e >> 4) & 15)) * LDT + 16 * j + (e & 15);
        a[o] = 0.0;
        w[o] = 0.0;
      }
    } else {  // what block b - 1 adds to the rows from b on
      const int p = b - 1;
      int k = 0;
      for (int i = b; i < 4; ++i)
        for (int j = 0; j <= i; ++j) {
          if ((i == b && j == b) || k++ % 3 + 1 != wv) continue;
          double *t = j < b ? at(w, i, j) : at(a, i, j);
          if (j < b)
            block_store(t, block_mma<false>(at(a, i, p), at(w, p, j),
                                            j < p ? block_load(t) : d4{0.0, 0.0, 0.0, 0.0}, 1.0));
          else
            block_store(t, block_mma<true>(at(a, i, p), at(a, j, p), block_load(t), -1.0));
        }
    }
    __syncthreads();
    const d4 zero = {0.0, 0.0, 0.0, 0.0};
    if (wv > b)
      block_store(at(a, wv, b), block_mma<true>(at(a, wv, b), at(w, b, b), zero, 1.0));
    else if (wv < b)
      block_store(at(w, b, wv), block_mma<false>(at(w, b, b), at(w, b, wv), zero, -1.0));
    __syncthreads();
  }
}

// ------------------------------------------------ MFMA tile products ------
// One 64x64 output tile per workgroup: wavefront w owns rows 16w..16w+15 as
// four 16x16 MFMA blocks (acc[cb] = columns 16cb..).  K-slot q of MFMA step s
// stands for k = 16q + s, so each lane reads 16 contiguous entries of a row.
// Tiles are row-major 64x64 in global memory.
struct Acc4 {
  d4 v[4];
};

__device__ __forceinline__ void acc_load(Acc4 &c, const double *__restrict__ g) {
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) c.v[cb][r] = g[(16 * wv + (l >> 4) + 4 * r) * TS + 16 * cb + (l & 15)];
}

// acc_load of a packed diagonal tile (zero above the diagonal)
__device__ __forceinline__ void acc_load_packed(Acc4 &c, const double *__restrict__ g) {
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      c.v[cb][r] = packed_at(g, 16 * wv + (l >> 4) + 4 * r, 16 * cb + (l & 15));
}

__device__ __forceinline__ void acc_zero(Acc4 &c) {
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) c.v[cb] = d4{0.0, 0.0, 0.0, 0.0};
}

__device__ __forceinline__ void acc_store(const Acc4 &c, double *__restrict__ g) {
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) g[(16 * wv + (l >> 4) + 4 * r) * TS + 16 * cb + (l & 15)] = c.v[cb][r];
}

__device__ __forceinline__ void acc_to_lds(const Acc4 &c, double *lds) {
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < 4; ++r) lds[(16 * wv + (l >> 4) + 4 * r) * LDT + 16 * cb + (l & 15)] = c.v[cb][r];
}

// c += sign * X Y^T, X and Y with row stride ldx/ldy (global or LDS)
__device__ __forceinline__ void acc_mma_abt(Acc4 &c, const double *X, int ldx, const double *Y,
                                            int ldy, double sign) {
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = l & 15, q = l >> 4;
  double xa[16];
  const double *xr = X + (16 * wv + i) * ldx + 16 * q;
#pragma unroll
  for (int s = 0; s < 16; ++s) xa[s] = sign * xr[s];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    const double *yr = Y + (16 * cb + i) * ldy + 16 * q;
    double yb[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) yb[s] = yr[s];
#pragma unroll
    for (int s = 0; s < 16; ++s) c.v[cb] = mfma16x16x4(xa[s], yb[s], c.v[cb]);
  }
}

// c += sign * X Y
__device__ __forceinline__ void acc_mma_ab(Acc4 &c, const double *X, int ldx, const double *Y,
                                           int ldy, double sign) {
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = l & 15, q = l >> 4;
  double xa[16];
  const double *xr = X + (16 * wv + i) * ldx + 16 * q;
#pragma unroll
  for (int s = 0; s < 16; ++s) xa[s] = sign * xr[s];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
    for (int s = 0; s < 16; ++s) c.v[cb] = mfma16x16x4(xa[s], Y[(16 * q + s) * ldy + 16 * cb + i], c.v[cb]);
  }
}

typedef double d2 __attribute__((ext_vector_type(2)));

// Sum over the copies of row i (fixed map order) of the columns c, c + 1 of XN;
// the first CU copies' index and value loads are issued together.
template <int W>
__device__ __forceinline__ d2 sum_copies(int i, int c, const int *__restrict__ inv_ptr,
                                         const int *__restrict__ ix,
                                         const double *__restrict__ XN) {
  constexpr int CU = 4;
  const int e0 = inv_ptr[i], e1 = inv_ptr[i + 1];
  int src[CU];
  d2 x[CU];
#pragma unroll
  for (int u = 0; u < CU; ++u) src[u] = ix[min(e0 + u, e1 - 1)];
#pragma unroll
  for (int u = 0; u < CU; ++u) x[u] = *reinterpret_cast<const d2 *>(XN + (size_t)src[u] * W + c);
  d2 s = {0.0, 0.0};
#pragma unroll
  for (int u = 0; u < CU; ++u) {
    const d2 a = s + x[u];
    s = e0 + u < e1 ? a : s;
  }
  for (int e = e0 + CU; e < e1; ++e) s += *reinterpret_cast<const d2 *>(XN + (size_t)ix[e] * W + c);
  return s;
}

}  // namespace amsp
