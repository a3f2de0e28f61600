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
// With several workgroups per unit the instructions between the products count
// (320 vector instructions a block): addresses are one base and constants,
// masks are taken where a step needs one.
// Measured in the eigensolver's sweeps (21 blocks of 64 rows per region, all of them
// at work, float64 / float32 factor): 64 regions 200 -> 75 / 202 -> 78 us, 1024 regions
// 426 -> 297 / 352 -> 213 us (5.2 TB/s of factor and rows); in three dimensions (1728
// regions of 16 blocks) 1442 -> 564 / 1396 -> 391 us, segments of ~100 entries having
// been a serial loop before.
constexpr int SOLVE_RING = 2 * TS;  // finished rows kept in LDS

template <int EVU, int PF, typename T, typename IO>
__device__ __forceinline__ void env_solve(const Plan &p, int i, const T *__restrict__ diag,
                                          const T *__restrict__ erow,
                                          const T *__restrict__ ecol, IO &io) {
  constexpr int LVA = EIGP + 4;  // row strides of the two LDS blocks: rows 4 apart (Acc) and
  constexpr int LVR = EIGP;      // neighbouring rows (ring) fall into different banks
  constexpr int RING = SOLVE_RING;
  constexpr int EVC = EVU * WG;  // envelope entries staged per block
  // one block, so that reads a little before or past a part (dropped by a
  // select) stay inside it
  __shared__ struct {
    double Acc[TS * LVA], Rg[RING * LVR];
    T Ev[EVC + TS];
  } sh;
  double *const Acc = sh.Acc, *const Rg = sh.Rg;
  T *const Ev = sh.Ev;
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
  // acc = (segment entries) (finished rows) for rows 16w..16w+15, ns steps of
  // four.  Row form: a segment ends at row r0 - 1; column form: it starts at
  // row r0 + TS.  The steps end with the longest segment's last entry (row
  // form) or are shifted by pad (column form), so that only the first step
  // holds rows outside that segment; those count as zero (a zero coefficient
  // would turn their infinities into NaN).
  auto env_part = [&](auto fwd, const T *src, const Seg &g, int r0, d4 &acc) {
    constexpr bool FWD = decltype(fwd)::value;
    const int ltop = __builtin_amdgcn_readlane(g.len, FWD ? 0 : 15);
    const int ns = (ltop + 3) >> 2;
    if (ns == 0) return;
    const int pad = 4 * ns - ltop;
    const int kb = (FWD ? g.len - ltop : 0) - pad + mq;  // this lane's segment index at step 0
    const int vb = (FWD ? r0 - ltop : r0 + TS) - pad + mq;
    if (g.total <= EVC && ltop <= TS) {
      // entries and rows from LDS; the rows are the last block's half of the
      // ring, so that every address is one base and a constant
      const T *ea = Ev + g.off + kb;
      const double *rp =
          Rg + (((FWD ? r0 - TS : r0 + TS) & (RING - 1)) + (FWD ? TS - 4 * ns : -pad) + mq) * LVR +
          mi;
      for (int s0 = 0; s0 < ns; s0 += 4) {
        T a[4];
        double b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[u] = ea[4 * (s0 + u)];
          b[u] = rp[4 * (s0 + u) * LVR];
        }
        if (s0 == 0 && mq < pad) b[0] = 0.0;
        auto step = [&](int u) __attribute__((always_inline)) {
          const T v = (unsigned)(kb + 4 * (s0 + u)) < (unsigned)g.len ? a[u] : T(0);
          acc = mfma16x16x4((double)v, b[u], acc);
        };
        step(0);
        if (s0 + 1 < ns) step(1);
        if (s0 + 2 < ns) {
          step(2);
          step(3);
        }
      }
    } else {
      // longer segments: rows from the whole ring or from memory; many
      // entries: those from memory
      const bool staged = g.total <= EVC, in_ring = ltop <= RING;
      for (int s = 0; s < ns; ++s) {
        const int k = kb + 4 * s, row = vb + 4 * s;
        const bool ok = k >= 0 && k < g.len;
        T v;
        if (staged)
          v = Ev[ok ? g.off + k : 0];
        else
          v = src[g.base + (ok ? g.off + k : 0)];
        double x;
        if (in_ring)
          x = Rg[(row & (RING - 1)) * LVR + mi];
        else
          x = io.row(min(max(row, 0), npad - 1));
        acc = mfma16x16x4(ok ? (double)v : 0.0, s == 0 && mq < pad ? 0.0 : x, acc);
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
    // forward: row 16w + mi, columns 16g + 4q + u; backward: column 16w + mi,
    // rows 16g + 4q + u.  Part m = 0: the diagonal group g = w (entries outside
    // the triangle lie inside the packed tile and are dropped where they are
    // used); parts 1 .. 3: the whole groups, g = m - 1 < w forward, g = m > w
    // backward.
    auto group = [&](int m) { return m == 0 ? w : FWD ? m - 1 : m; };
    auto whole = [&](int m) { return FWD ? m - 1 < w : m > w; };
    auto load_d = [&](int I, T (&dA)[16]) {
      const T *tile = dpool + (size_t)(FWD ? I : nt - 1 - I) * DE;
      const T *row = FWD ? tile + dpos_row(16 * w + mi) + 4 * mq : tile + 16 * w + mi;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (m == 0 || whole(m)) {
          const int g = group(m), k4 = 4 * g + mq;  // backward: row / 4
#pragma unroll
          for (int u = 0; u < 4; ++u)
            dA[4 * m + u] = FWD ? row[16 * g + u] : row[4 * (k4 + 1) * (2 * k4 + u)];
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
          const d4 x = c.x;
          c.g = seg_of(c.raw);
          ev_load(env, c.g, c.ev);
          io.load(fwd, row0(In), c.idx, c.x);
          c.raw = seg_load(ptr, row0(min(I + 2 * PF, nt - 1)));
          c.idx = io.idx(fwd, row0(min(I + 2 * PF, nt - 1)));
          d4 acc = {0.0, 0.0, 0.0, 0.0};
          env_part(fwd, env, g, row0(I), acc);
          acc_write(x - acc);
          __syncthreads();  // Acc complete; Ev and the ring free
          d4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            double bd[8];  // two groups' reads, issued (and waited for) together
#pragma unroll
            for (int e = 0; e < 8; ++e)
              bd[e] = Acc[(16 * group(2 * h + (e >> 2)) + 4 * mq + (e & 3)) * LVA + mi];
#pragma unroll
            for (int e = 0; e < 8; ++e) __asm__ volatile("" : "+v"(bd[e]));
#pragma unroll
            for (int m = 2 * h; m < 2 * h + 2; ++m)
              if (m == 0 || whole(m)) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                  T a = c.dA[4 * m + u];
                  if (m == 0) a = (FWD ? 4 * mq + u <= mi : mi <= 4 * mq + u) ? a : T(0);
                  y = mfma16x16x4((double)a, bd[4 * (m & 1) + u], y);
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
