// The block solve shared by the eigensolver's sweeps (k_eigen.hip) and the
// several-column apply (k_multi.hip).
#pragma once
#include "k_common.h"

namespace amsp {

// ------------------------------------------- block solve (EIGP rhs) -------
// Y = (L L^T)^{-1} X for a region's block of up to EIGP columns, one workgroup
// per region, with L in the local apply's layout: packed inverse diagonal
// tiles and the envelope below them (row form forward, column form
// backward).  The caller's IO says where the rows come from and go to.
//
// A sweep is a chain of nt 64-row blocks, and a block's two products are what
// bounds it: the finished rows that its envelope reaches, then inv(L_II) (or
// its transpose) times the 64 x EIGP remainder.  Both run on the matrix
// cores, wavefront w owning rows 16w..16w+15 of both:
//   - the envelope part takes the rows' segments as a 16 x 4 ns operand, ns
//     from the wavefront's longest segment (its first row's forward, its last
//     one's backward: segment lengths are monotone in a block), entries
//     outside a segment being zero;
//   - the diagonal part takes only the 16-column groups of the triangle that
//     the wavefront's rows meet: 4, 8, 12, 16 steps instead of 16 each.
// The two loads are opposite (the wavefront with the longest segments has the
// fewest groups), so that the four SIMDs carry about the same number of
// steps.  MFMA step (g, u), lane quarter q stands for column 16g + 4q + u of
// the triangle, so a lane reads four neighbouring entries per group.
// A block's segments are contiguous: the workgroup stages them in LDS with
// one coalesced load (EVU entries per thread; a block with more reads its
// entries from global memory).  The last RING finished rows stay in LDS (row
// g in slot g mod RING); a wavefront with a longer segment reads the rows
// from global memory.  Every lane loads and stores the same rows and columns
// (rows r0 + 16w + q + 4r of a block, r < 4, column l & 15: the MFMA result
// layout) of the input, the accumulator and the output.
//
// IO, all for this lane's rows of the block at row r0:
//   Idx / Aux            registers loaded 2 PF / PF blocks ahead
//   idx(fwd, r0)         what the loads of the block's rows depend on
//   load(fwd, r0, idx)   the block's right-hand side (forward) or the forward
//                        sweep's result (backward)
//   aux(fwd, r0)         what store needs from memory
//   store(fwd, r0, y, aux)
//   row(r)               column l & 15 of finished row r of the current sweep,
//                        for segments that reach beyond the ring
// Measured (21 blocks of 64 rows per region, float64 / float32 factor): 64
// regions 200 -> 91 / 84 us (1.4 us a block of products, 0.6 of waiting),
// 1024 regions 430 -> 315 / 357 -> 220 us (5 TB/s of factor and rows); in
// three dimensions (1728 regions of 16 blocks) 1320 -> 352 us with a float32
// factor, whose segments of ~100 entries were a serial loop before.
constexpr int SOLVE_RING = 2 * TS;  // finished rows kept in LDS

template <int EVU, int PF, typename T, typename IO>
__device__ __forceinline__ void env_solve(const Plan &p, int i, const T *__restrict__ diag,
                                          const T *__restrict__ erow,
                                          const T *__restrict__ ecol, IO &io) {
  constexpr int LVA = EIGP + 4;  // row strides of the two LDS blocks: rows 4 apart (Acc) and
  constexpr int LVR = EIGP;      // neighbouring rows (ring) fall into different banks
  constexpr int RING = SOLVE_RING;
  constexpr int EVC = EVU * WG;  // envelope entries staged per block
  __shared__ double Rg[RING * LVR];
  __shared__ double Acc[TS * LVA];
  __shared__ T Ev[EVC];
  const int g0 = p.trow_ptr[i], nt = p.trow_ptr[i + 1] - g0;
  const int *ep = p.eptr + p.vp_ptr[i] + i, *up = p.uptr + p.vp_ptr[i] + i;
  const T *erow_i = erow + p.ebase[i], *ecol_i = ecol + p.ebase[i];
  const T *dpool = diag + (size_t)g0 * DE;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int mi = l & 15, mq = l >> 4;  // MFMA operand lane roles
  const int rb = 16 * w + mq;          // D register r: row rb + 4r, column mi
  const int npad = nt * TS;
  // the ring's rows meet zero entries before they are first written
  for (int e = tid; e < RING * LVR; e += WG) Rg[e] = 0.0;
  // Segment bounds of one block: row 16w + mi's first entry within the
  // block's entries [base, base + total) and its length.  The loads are kept
  // as they came (Raw) until the bounds come into use, so that nothing waits
  // for them before; base and total, the same for every lane, then go to
  // scalar registers.
  struct Raw {
    int b0, b1, e0, e1;
  };
  struct Seg {
    int off, len, base, total;
  };
  auto seg_load = [&](const int *ptr, int r0) {
    const int *row = ptr + r0 + 16 * w + mi;
    return Raw{ptr[r0], ptr[r0 + TS], row[0], row[1]};
  };
  auto seg_of = [&](const Raw &r) {
    const int base = __builtin_amdgcn_readfirstlane(r.b0);
    return Seg{r.e0 - base, r.e1 - r.e0, base, __builtin_amdgcn_readfirstlane(r.b1) - base};
  };
  // the block's first EVC entries, this thread's share (clamped into the
  // block and issued unconditionally; a block without entries reads the one
  // before it, or the array's padding entry)
  auto ev_load = [&](const T *src, const Seg &g, T (&ev)[EVU]) {
#pragma unroll
    for (int u = 0; u < EVU; ++u) ev[u] = src[max(g.base + min(tid + WG * u, g.total - 1), 0)];
  };
  // acc -= (segment entries) (finished rows), rows 16w..16w+15.  Row form:
  // a segment ends at column r0 - 1, so the steps count back from r0; column
  // form: it starts at row r0 + TS.
  auto env_part = [&](auto fwd, const T *src, const Seg &g, int r0, d4 &acc) {
    constexpr bool FWD = decltype(fwd)::value;
    const int ltop = __builtin_amdgcn_readlane(g.len, FWD ? 0 : 15);
    const int ns = (ltop + 3) >> 2;
    const int ib = (FWD ? g.len - 4 * ns : 0) + mq;  // this lane's segment index at step 0
    const int vb = (FWD ? r0 - 4 * ns : r0 + TS) + mq;
    if (ns == 0) return;
    if (g.total <= EVC && ltop <= RING) {
      // entries and rows from LDS, four steps' reads issued before the four
      // products before them (the steps past ns read in range and are not used)
      auto fetch = [&](int s0, double(&a)[4], double(&b)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = ib + 4 * (s0 + u);
          const bool ok = k >= 0 && k < g.len;
          const T v = Ev[ok ? g.off + k : 0];
          a[u] = ok ? -(double)v : 0.0;
          // rows outside the wavefront's longest segment count as zero (a zero
          // coefficient would turn their infinities into NaN)
          const int d = 4 * (s0 + u) + mq;
          const double x = Rg[((vb + 4 * (s0 + u)) & (RING - 1)) * LVR + mi];
          b[u] = (FWD ? d >= 4 * ns - ltop : d < ltop) ? x : 0.0;
        }
      };
      auto mul = [&](int s0, const double(&a)[4], const double(&b)[4]) __attribute__((always_inline)) {
        acc = mfma16x16x4(a[0], b[0], acc);
        if (s0 + 1 < ns) acc = mfma16x16x4(a[1], b[1], acc);
        if (s0 + 2 < ns) {
          acc = mfma16x16x4(a[2], b[2], acc);
          acc = mfma16x16x4(a[3], b[3], acc);
        }
      };
      double a0[4], b0[4], a1[4], b1[4];
      fetch(0, a0, b0);
      for (int s0 = 0;; s0 += 8) {
        fetch(s0 + 4, a1, b1);
        mul(s0, a0, b0);
        if (s0 + 4 >= ns) break;
        fetch(s0 + 8, a0, b0);
        mul(s0 + 4, a1, b1);
        if (s0 + 8 >= ns) break;
      }
    } else {  // long segments or many entries: from global memory
      for (int s = 0; s < ns; ++s) {
        const int k = ib + 4 * s;
        const bool ok = k >= 0 && k < g.len;
        const T v = src[g.base + (ok ? g.off + k : 0)];
        const int d = 4 * s + mq;
        double x = io.row(min(max(vb + 4 * s, 0), npad - 1));
        x = (FWD ? d >= 4 * ns - ltop : d < ltop) ? x : 0.0;
        acc = mfma16x16x4(ok ? -(double)v : 0.0, x, acc);
      }
    }
  };
  auto acc_write = [&](const d4 &acc) {
#pragma unroll
    for (int r = 0; r < 4; ++r) Acc[(rb + 4 * r) * LVA + mi] = acc[r];
  };
  auto ring_write = [&](int r0, const d4 &y) {
#pragma unroll
    for (int r = 0; r < 4; ++r) Rg[((r0 + rb + 4 * r) & (RING - 1)) * LVR + mi] = y[r];
  };
  auto ev_write = [&](const T (&ev)[EVU]) {
#pragma unroll
    for (int u = 0; u < EVU; ++u) Ev[tid + WG * u] = ev[u];
  };
  // One sweep.  Slot I % PF of the buffers holds what block I (in sweep
  // order) needs from memory, loaded PF blocks ahead, each part as soon as
  // its registers are free; bounds are loaded 2 PF blocks ahead.
  auto sweep = [&](auto fwd, const int *ptr, const T *env) __attribute__((always_inline)) {
    constexpr bool FWD = decltype(fwd)::value;
    struct Buf {
      T dA[16], ev[EVU];
      d4 x;
      Seg g;
      Raw raw;
      typename IO::Idx idx;
      typename IO::Aux aux;
    } b[PF];
    auto row0 = [&](int I) { return (FWD ? I : nt - 1 - I) * TS; };
    // forward: row 16w + mi, columns 16g + 4q + u for the groups g <= w;
    // backward: column 16w + mi, rows 16g + 4q + u for the groups g >= w
    // (entries outside the triangle lie inside the packed tile and are
    // dropped where they are used)
    auto load_d = [&](int I, T (&dA)[16]) {
      const T *tile = dpool + (size_t)(FWD ? I : nt - 1 - I) * DE;
      const T *row = FWD ? tile + dpos_row(16 * w + mi) + 4 * mq : tile + 16 * w + mi;
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (FWD ? g <= w : g >= w) {
          const int k4 = 4 * g + mq;  // backward: row / 4
#pragma unroll
          for (int u = 0; u < 4; ++u)
            dA[4 * g + u] = FWD ? row[16 * g + u] : row[4 * (k4 + 1) * (2 * k4 + u)];
        }
    };
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      b[j].g = seg_of(seg_load(ptr, row0(min(j, nt - 1))));
      b[j].raw = seg_load(ptr, row0(min(j + PF, nt - 1)));
      ev_load(env, b[j].g, b[j].ev);
      io.load(fwd, row0(min(j, nt - 1)), io.idx(fwd, row0(min(j, nt - 1))), b[j].x);
      b[j].idx = io.idx(fwd, row0(min(j + PF, nt - 1)));
      b[j].aux = io.aux(fwd, row0(min(j, nt - 1)));
      load_d(min(j, nt - 1), b[j].dA);
    }
    for (int I0 = 0; I0 < nt; I0 += PF) {
#pragma unroll
      for (int j = 0; j < PF; ++j) {
        const int I = I0 + j;
        if (I < nt) {
          Buf &c = b[j];
          // the block that takes this slot next (past the last one: the last
          // one again, unused; nothing here is conditional, so that the waits
          // are for the oldest loads only)
          const int In = min(I + PF, nt - 1);
          const Seg g = c.g;
          ev_write(c.ev);
          __syncthreads();  // Ev and the ring complete; the last block's Acc reads done
          d4 acc = c.x;
          c.g = seg_of(c.raw);
          ev_load(env, c.g, c.ev);
          io.load(fwd, row0(In), c.idx, c.x);
          c.raw = seg_load(ptr, row0(min(I + 2 * PF, nt - 1)));
          c.idx = io.idx(fwd, row0(min(I + 2 * PF, nt - 1)));
          env_part(fwd, env, g, row0(I), acc);
          acc_write(acc);
          __syncthreads();  // Acc complete; Ev and the ring free
          d4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            double bd[8];  // two groups' reads, issued (and waited for) together
#pragma unroll
            for (int e = 0; e < 8; ++e)
              bd[e] = Acc[(32 * h + 16 * (e >> 2) + 4 * mq + (e & 3)) * LVA + mi];
#pragma unroll
            for (int e = 0; e < 8; ++e) __asm__ volatile("" : "+v"(bd[e]));
#pragma unroll
            for (int gr = 2 * h; gr < 2 * h + 2; ++gr)
              if (FWD ? gr <= w : gr >= w) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  const bool in = gr != w || (FWD ? 4 * mq + u <= mi : mi <= 4 * mq + u);
                  y = mfma16x16x4(in ? (double)c.dA[4 * gr + u] : 0.0, bd[4 * (gr & 1) + u], y);
                }
              }
          }
          load_d(In, c.dA);
          ring_write(row0(I), y);
          io.store(fwd, row0(I), y, c.aux);
          c.aux = io.aux(fwd, row0(In));
        }
      }
    }
  };
  // forward: Y_I = inv(L_II) (X_I - L[I rows, c < 64I] Y)
  sweep(std::true_type{}, ep, erow_i);
  // backward: X_J = inv(L_JJ)^T (Y_J - L[r >= 64(J+1), J cols]^T X)
  sweep(std::false_type{}, up, ecol_i);
}

}  // namespace amsp
