// Compile-time constants and index rules shared by host planning and the HIP kernels.
#pragma once

namespace amsp {

constexpr int TS = 64;       // tile edge: 64x64 tiles, one wavefront-wide row block
constexpr int TE = TS * TS;  // elements per tile
// Entries of a packed diagonal factor tile: row R keeps columns 0..R, padded
// with zeros to a multiple of 4, i.e. sum over R of 4*ceil((R+1)/4).
constexpr int DE = 2176;
constexpr int WG = 256;      // workgroup size of the batched kernels (4 wavefronts)
constexpr int EIGP = 16;     // subspace block width of the local eigensolver
constexpr int EIG_GRAM_ROWS = 128;  // rows of a region per partial Gram matrix
constexpr int MAXNEV = 15;   // nev + 1 must fit in the subspace block
constexpr int MAX_PARTIALS = 1024;  // workgroups (partial sums) of a vector reduction

// ---- One vector's local solves (local_sweep, k_apply.hip): the rules behind its
// LDS reads, also followed by the host's check of them (plan_check.cpp).
// A row's (column's) segment of the envelope is read in passes of 4 batch entries,
// batch per lane, all lanes of a wavefront up to its longest segment.
constexpr int sweep_batch(int evu) { return evu > 4 ? 8 : 4; }
// Row of the vector at the first entry of a segment of len entries (block at row
// r0): row form, the segment ends at row r0 - 1; column form, it starts at r0 + TS.
constexpr int sweep_row(bool fwd, int r0, int len) { return fwd ? r0 - len : r0 + TS; }
// Entries by which a lane moves on after the pass at k0 (one of 4 batch entries): a
// segment that has ended stays where it is, its later passes being dropped whole.  A
// lane then reads less than one pass past its segment, which ends at row r0 - 1 or at
// the region's last row at most, however long the wavefront's longest segment is.
constexpr int sweep_step(int batch, int k0, int len) {
  return k0 + 4 * batch < len ? 4 * batch : 0;
}

}  // namespace amsp
