// Internal declarations shared by the host library and the HIP kernels.
// Not part of the public ABI (see include/amsp.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "amsp_consts.h"

namespace amsp {

// Device view of the planned subdomain structure (all arrays on the device).
struct Plan {
  int N;                    // subdomains
  int nev;                  // requested eigenvectors (row stride of basis arrays)
  const int *sd_ptr;        // [N+1] offsets of each region in the concatenated local vectors
  const int *sd_dofs;       // [sum n_i] global dof of each local index (local order)
  const int *nat;           // [sum n_i] rank of that dof among the region's dofs by global
                            // index: position in the ascending-index layout of the
                            // local corrections and of the basis copy read by the apply
  const int *asc;           // [sum n_i] the region's dofs in ascending order, and the local
  const int *lop;           //   index of each: asc[r0 + nat[r0 + l]] = sd_dofs[r0 + l],
                            //   lop[r0 + nat[r0 + l]] = l
  const int *vp_ptr;        // [N+1] padded offsets (multiples of 64) for tile-aligned vectors
  const int *trow_ptr;      // [N+1] offsets into the per-tile-row arrays
  const int *tfirst;        // [sum nt_i] first tile column of each tile row
  const long long *toff;    // [sum nt_i] pool index of the first off-diagonal tile of each
                            // tile row (tiles J = first(I) .. I-1 follow in order)
  long long noff;           // off-diagonal tiles in the pool; the packed diagonal tiles
                            // follow at entry noff*TE, DE entries per tile row
  const int *eptr;          // [sum npad_i + N] envelope of the factor below the diagonal
  const int *uptr;          //   tiles, per region npad_i + 1 segment starts relative to
  const long long *ebase;   //   ebase[i]: row form (eptr) and column form (uptr)
  int env_mean;             // envelope entries per 64-row block, on average
  const int *sfb, *sbb;     // [sum nt_i] start of each 64-row block in its region's forward
  const long long *sfr;     //   / backward stream; [N+1] region starts of the forward
  const long long *sbr;     //   / backward streams (see launch_local_apply_mixed)
  const int *loc_rowptr;    // [sum n_i + 1] local CSR of A_i (rows in local order)
  const int *loc_col;       //   local column index
  const int *loc_src;       //   index of the value in the global CSR
  const int *mi;            // [N] kept eigenvectors m_i
  const int *coff;          // [N+1] coarse offsets
  const int *mult;          // [n] dof multiplicity
};

// PCG scalar state kept on the device.
struct PcgState {
  double rz, rz_ring[2], pq, rr, alpha, beta, tol2, f2;
  int it, done, breakdown, maxit;
  double *hist;   // rr after each iteration (hist[it]); may be null
  int hist_cap;
};

// ---------------------------------------------------------------- krylov ---
int reduce_blocks(int n);
void launch_spmv(hipStream_t s, int n, const int *rp, const int *col, const double *val,
                 const double *x, double *y, double *partial, const int *done);
// One CG step t in two kernels (direction + update); the scalar reductions
// of the previous kernels are folded in (see k_krylov.hip).
// The direction kernel's matrix product reads the sliced copy of A (64-row
// slices, column-major inside a slice; see launch_csr_to_sell).
void launch_cg_dir(hipStream_t s, int n, const long long *sptr, const int *scol,
                   const double *sval, const double *z, const double *pold, double *pnew, double *q,
                   double *part_pq, PcgState *st, const double *part_rr, const double *part_rz,
                   const double *part_rzo, int t, int first, int flexible);
// y = A x on the sliced copy (amsp_spmv).
void launch_spmv_sell(hipStream_t s, int n, const long long *sptr, const int *scol,
                      const double *sval, const double *x, double *y, const int *done = nullptr);
// Multiplicative cycle steps (all return at once when *done is set):
// x *= a; t = r - q; y += a x with optional partial sums of r.y.
void launch_scale_done(hipStream_t s, int n, double a, double *x, const int *done);
void launch_sub_done(hipStream_t s, int n, const double *r, const double *q, double *t,
                     const int *done);
void launch_axpy_dot(hipStream_t s, int n, double a, const double *x, double *y, const double *r,
                     double *partial, const int *done);
// Sliced copy of A: sptr[s] = first entry of slice s (ceil(n/64) + 1 entries).
void launch_csr_to_sell(hipStream_t s, int n, const int *rp, const int *col, const double *val,
                        const long long *sptr, int *scol, double *sval);
void launch_cg_update(hipStream_t s, int n, double *x, double *r, const double *p, const double *q,
                      PcgState *st, const double *part_pq, int t, double *part_rr,
                      const double *zold, double *part_rzo);
void launch_dot(hipStream_t s, int n, const double *a, const double *b, double *partial,
                const int *done);
// grad[k] = -lambda[row k] * u[col k] for the CSR entries k
void launch_grad_values(hipStream_t s, int n, const int *rp, const int *col, const double *lambda,
                        const double *u, double *grad);
void launch_residual(hipStream_t s, int n, const double *f, const double *Ax, double *r,
                     double *partial);
void launch_copy_scale(hipStream_t s, int n, const double *a, double *b, double alpha);
// GMRES (restarted, flexible right preconditioning) building blocks.  The
// basis columns are V + k * ldv.  One Gram-Schmidt round: out[k] = V_k . w for
// k < k1 (part holds k1 * reduce_blocks(n) partials), w -= V out, with optional
// w.w partials in nrm; v = w / sqrt(*nrm2), *nrm2 summed from part first unless
// that is null; x += Z y.
void launch_gs_round(hipStream_t s, int n, const double *V, size_t ldv, int k1, double *w,
                     double *part, double *out, double *nrm);
void launch_gs_normalize(hipStream_t s, int n, const double *w, double *nrm2, const double *part,
                         double *v);
void launch_basis_combine(hipStream_t s, int n, const double *Z, size_t ldz, int k, const double *y,
                          double *x);

void launch_abs_spmv_sq(hipStream_t s, int n, const int *rp, const int *col, const double *val,
                        const double *x, double *partial);
void launch_fill(hipStream_t s, size_t n, double *a, double v);
void launch_fill_int(hipStream_t s, size_t n, int *a, int v);
void launch_sum_partials(hipStream_t s, const double *partial, int nb, double *out);
void launch_pcg_init(hipStream_t s, PcgState *st, const double *partial_rr, int nb_rr,
                     const double *partial_rz, int nb_rz, double rtol, int maxit);

// ----------------------------------------------------------------- local ---
// s = diag(hat A_i) for every local row; status[i] |= 1 if some s <= 0.
void launch_neumann_diag(hipStream_t s, const Plan &p, const double *val, double *sdiag,
                         int *status);
// Tile-profile storage: mode 0 -> A_i, mode 1 -> S^{-1/2} hat A_i S^{-1/2} + sigma I.
void launch_extract_tiles(hipStream_t s, const Plan &p, int ntilerows, const double *val,
                          const double *sdiag, double *tiles, int mode, double sigma);
// In-place batched profile Cholesky; diagonal tiles then hold inv(L_II).
// status[i] |= bit on a non-positive pivot.
void launch_profile_cholesky(hipStream_t s, const Plan &p, double *tiles, int *status, int bit);
void launch_tiles_to_f32(hipStream_t s, const double *src, float *dst, size_t count);
// Envelope copy (row and column forms, type T) of the off-diagonal part of a
// factored tile pool.
template <typename T>
void launch_env_from_tiles(hipStream_t s, const Plan &p, int ntilerows, const double *tiles,
                           T *erow, T *ecol);
// Largest region (padded rows) of the local apply in the FP64 form and in the mixed
// ones; larger ones are refused at setup.  The mixed line is what the stream kernel's
// LDS holds.  The FP64 line is from a kernel that kept the segment starts beside the
// vector (the present one would hold 14016 rows); it stays, so that what is refused does
// not change.  k_apply.hip checks both lines against its kernels.
constexpr size_t LDS_BYTES = 160 * 1024;  // of a workgroup
constexpr int LOCAL_MAX_NPAD_FP64 = 10112, LOCAL_MAX_NPAD_MIXED = 17280;
// Per-sweep streams of an f32 factor: for every region, its 64-row blocks in
// sweep order (forward: ascending, envelope row form; backward: descending,
// column form), each block's envelope segments zero-padded to a multiple of
// 4 entries and followed by the block's packed inverse diagonal tile.  The
// arrays carry STREAM_TAIL extra entries (read, never used).
constexpr int STREAM_TAIL = 4 * WG;
void launch_stream_from_tiles(hipStream_t s, const Plan &p, int ntilerows, const double *tiles,
                              float *fst, float *bst);
// Coarse restriction c = R0 r: c_i = Phi_i^T r_i for every region (TB basis
// type; the copy made by launch_basis_to_natural).
template <typename TB>
void launch_restrict(hipStream_t s, const Plan &p, const double *r, const TB *phi, double *cvec,
                     const int *done);
// The mixed forms' local apply on the float32 factor's streams (the operation of
// launch_local_apply, whose kernel it takes for up to 640 regions).
template <typename TB>
void launch_local_apply_mixed(hipStream_t s, const Plan &p, int max_npad, const double *r,
                              const float *fst, const float *bst, const TB *phi, const double *t,
                              const double *tpart, int T0, double *xloc, const int *done,
                              hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// Local apply: gather r, envelope forward/backward solve, store into xloc;
// with the coarse solution t (else nullptr) the prolongation Phi_i t_i is
// added to each region's output (phi: the copy made by
// launch_basis_to_natural).  With tpart (else nullptr) the coarse solution
// is instead summed from the per-tile products of W0^T
// (launch_coarse_products with y == nullptr; T0 tiles), as the reduction would
// sum them.  T = double: diag holds the packed inverse diagonal tiles (DE entries
// per tile row), frow / fcol the envelope (with two entries of padding behind
// it); T = float: frow / fcol are the two sweeps' streams, diag is not read.
// ev_start / ev_stop (optional, created with timing): bound to the dispatch
// itself (no extra packets in the stream).
template <typename T, typename TB>
void launch_local_apply(hipStream_t s, const Plan &p, int max_npad, const double *r,
                        const T *diag, const T *frow, const T *fcol, const TB *phi,
                        const double *t, const double *tpart, int T0, double *xloc,
                        const int *done, hipEvent_t ev_start = nullptr,
                        hipEvent_t ev_stop = nullptr);
void launch_selftest_mfma(hipStream_t s, const double *A, const double *B, double *D);
// The regions' dofs in ascending order and their local indices (Plan::asc,
// Plan::lop).
void launch_ascending_dofs(hipStream_t s, const Plan &p, int *asc, int *lop);
// Direct operand indices of the inverse map (see k_inverse_direct).
void launch_inverse_direct(hipStream_t s, int ne, const int *inv_sd, const int *inv_loc,
                           const Plan &p, int *ix);
// z = sum_i R_i^T (x_i + D_i psi_i t_i): with the coarse part, first adds the
// prolongation into the local outputs xloc (overwrites them without the local
// part), then sums every dof's copies; partial r.z per workgroup when r != 0.
template <typename TB>
void launch_scatter_sum_t(hipStream_t s, const Plan &p, int max_ni, int n, const int *inv_ptr,
                          const int *ix, double *xloc, const TB *phi, const double *t, double *z,
                          const double *r, double *partial, int do_local, int do_coarse,
                          const int *done);

// ------------------------------------------------------- several columns ---
// Up to EIGP right-hand sides per pass (k_multi.hip).  Vectors are rows of
// W = row_width(nr) values, coarse vectors rows of EIGP; see k_multi.hip.
int row_width(int nr);
void launch_cols_to_rows(hipStream_t s, int n, size_t ld, int nr, const double *A, double *R);
// c = R0 R (phi: the copy made by launch_basis_to_natural)
template <typename TB>
void launch_restrict_rows(hipStream_t s, const Plan &p, int nr, const TB *phi, const double *R,
                          double *c);
// XN = local solves of the gathered rows + Phi_i t_i (t null: without; phi in
// local order); Y: padded rows of W, scratch
template <typename T, typename TB>
void launch_solve_rows(hipStream_t s, const Plan &p, int nr, const T *diag, const T *erow,
                       const T *ecol, const double *R, const TB *phi, const double *t, double *Y,
                       double *XN);
// XN = Phi_i t_i alone
template <typename TB>
void launch_prolong_rows(hipStream_t s, const Plan &p, int nr, const TB *phi, const double *t,
                         double *XN);
// z (columns n apart) = sum of every dof's copies in XN
void launch_scatter_cols(hipStream_t s, int n, int nr, const int *inv_ptr, const int *ix,
                         const double *XN, double *z);
// y = W0 x (transpose 0) or W0^T x (1), reading W0's tiles once; part holds
// T0 * T0 * 64 * W doubles.
template <typename T>
void launch_trmm(hipStream_t s, const T *Wt, int T0, const double *x, int nr, double *part,
                 double *y, int transpose);
// f32 factor of the mixed forms from its streams back into packed diagonal
// tiles + envelope (the layout of launch_env_solve_block)
void launch_streams_to_env(hipStream_t s, const Plan &p, int ntilerows, const float *fst,
                           const float *bst, float *dg, float *er, float *ec);

// mult[j] (regions containing dof j), inv_ptr (n + 1) and the per-dof lists
// (subdomain, ascending-index position) ordered by subdomain; work holds
// n + ceil(n / 1024) ints; *max_mult receives the largest multiplicity.
void launch_inverse_map(hipStream_t s, const Plan &p, int n, int *mult, int *inv_ptr,
                        int *inv_sd, int *inv_loc, int *work, int *max_mult);
// Local CSR entries (loc_col, loc_src) of every region from the plan's row
// pointers, dofs and ranks, and A's device CSR.  gscratch (2 * sum n_i ints)
// is used only when 2 * max_ni ints exceed LOCAL_CSR_LDS_MAX bytes of LDS.
constexpr size_t LOCAL_CSR_LDS_MAX = 128 * 1024;
size_t local_csr_lds_bytes(int max_ni);
void launch_local_csr(hipStream_t s, const Plan &p, int max_ni, const int *rowptr, const int *col,
                      int *loc_col, int *loc_src, int *gscratch);

// ---------------------------------------------------------------- eigen ---
void launch_eig_init(hipStream_t s, const Plan &p, const double *sdiag, double *X);
// dst[sd_ptr[i] * nev + c * n_i + nat[k]] = src[(sd_ptr[i] + k) * nev + c]: the
// basis in each region's ascending-global-index order, one column after the
// other (read by the single-vector apply's restriction and prolongation).
template <typename TB>
void launch_basis_to_natural(hipStream_t s, const Plan &p, const TB *src, TB *dst);
// Off-diagonal values of the scaled local operators B_i per local CSR entry.
void launch_eig_bval(hipStream_t s, const Plan &p, const double *val, const double *sdiag,
                     double *bval);
// Y = (L L^T)^{-1} X on row-major [rows][EIGP] padded blocks, L given as
// packed inverse diagonal tiles + envelope (as for the local apply).
template <typename T>
void launch_env_solve_block(hipStream_t s, const Plan &p, const T *diag, const T *erow,
                            const T *ecol, const double *X, double *Y, const int *skip);
// Rayleigh-Ritz step on the solve output Y, writing the Ritz vectors into X
// (distinct buffer), residuals, convergence flags and eigenvalues.
// BY: scratch like Y; GK: N*2*EIGP*EIGP doubles; CC: N*(EIGP*EIGP+EIGP).
void launch_eig_rr(hipStream_t s, const Plan &p, int max_ni, const double *val,
                   const double *sdiag, const double *bval, const double *Y, double *BY, double *X,
                   double *GK, double *CC, double tol, int *conv, double *lam,
                   bool test_next);
void launch_build_basis(hipStream_t s, const Plan &p, const double *sdiag, const double *X,
                        double *phi, int pou);
void launch_basis_convert(hipStream_t s, const double *phi, void *dst, size_t count, int bf16);
// phi[e] := phi[e] rounded to float32 (bf16 = 0) or bfloat16 (bf16 = 1), in place
void launch_basis_round(hipStream_t s, double *phi, size_t count, int bf16);

// ---------------------------------------------------------------- coarse ---
struct CoarsePlan {
  int N;
  int nev;
  const int *ext_ptr;       // [N+1] offsets of the extended regions
  const int *ext_rowptr;    // [sum |E_i| + 1] entries coupling each row to region i
  const int *ext_src;       //   global CSR value index
  const int *ext_loc;       //   local index in region i
  int npairs;
  const int *pair_i, *pair_j;
  const int *pair_ptr;      // [npairs+1]
  const int *pair_l;        // local index in region i
  const int *pair_e;        // index in the extended region of j
};
void launch_apply_A_to_basis(hipStream_t s, const Plan &p, const CoarsePlan &c,
                             const double *val, const double *phi, double *W);
void launch_pair_products(hipStream_t s, const Plan &p, const CoarsePlan &c, const double *phi,
                          const double *W, double *A0t, int T0);
void launch_symmetrize_tiles(hipStream_t s, double *A0t, int T0, int nc);
// Singular problems (null space = constants): u = R0 1 (u holds nc doubles),
// alpha = trace(A0) / u.u, A0 += alpha u u^T.
void launch_singular_regularize(hipStream_t s, const Plan &p, const double *phi, double *A0t,
                                int T0, int nc, double *u, double *alpha);
void launch_dense_potrf_diag(hipStream_t s, double *A0t, int T0, int k, double *dinv, int *status);
void launch_dense_trsm_panel(hipStream_t s, double *A0t, int T0, int k, const double *dinv);
// Updates of the blocked Cholesky, split for lookahead: tile column j with the
// columns k .. j - 1, in one launch with its diagonal factor (by the workgroup
// that updates the diagonal tile), and the columns j0 .. with the nk columns
// from k on.
void launch_dense_next_potrf(hipStream_t s, double *A0t, int T0, int k, int j, double *dinv,
                             int *status);
void launch_dense_syrk_rest(hipStream_t s, double *A0t, int T0, int k, int nk, int j0);
void launch_dense_inv_rows(hipStream_t s, const double *Lt, double *Wt, int T0, int k, int nk,
                           const double *dinv);
void launch_dense_inv_update(hipStream_t s, const double *Lt, double *Wt, int T0, int k, int nk);
void launch_tiles_identity(hipStream_t s, double *Wt, int T0);
void launch_dense_tiles_to_f32(hipStream_t s, const double *src, float *dst, int T0);
// y = W^T (W x) over the lower tiles of W.  part: (T0*T0 + T0)*64 doubles of
// scratch holding the per-tile products; t1: T0*64 doubles.  With y == nullptr
// the second product's sums are left to the reader: entry O*64 + r is the sum
// over K = O .. T0-1 of part[(O*T0 + K)*64 + r], split into TRMV_RG consecutive
// pieces of K (piece g: K from O + len*g/TRMV_RG, len = T0 - O), each summed in
// order and the pieces added in order from 0.
constexpr int TRMV_RG = 16;
template <typename T>
void launch_coarse_products(hipStream_t s, const T *Wt, int T0, const double *x, double *part,
                            double *t1, double *y, const int *done);

// ------------------- CG on several columns and problems (k_batch.hip) ---
// Row blocks (never across a problem boundary) and the recurrences' scalars,
// W = row_width(nr) per problem; part: nblk * W doubles.  See k_batch.hip.
struct RowBlocks {
  int nblk, nseg;
  const long long *brow;    // [nblk + 1]
  const int *bseg, *sblk;   // [nblk], [nseg + 1]
};
struct RowCgState {
  double *rz, *f2, *rr;      // nseg * W each
  int *active, *its, *broken;
  int *nactive;              // active recurrences after the step
  double *hist;              // r.r of the last recurrence per step; may be null
  int hist_cap;
};
void launch_rows_norm(hipStream_t s, const RowBlocks &b, int nr, const double *R, double *part);
void launch_rows_dir(hipStream_t s, const RowBlocks &b, int nr, const long long *sptr,
                     const int *scol, const double *sval, const double *beta, int first,
                     const double *z, const double *pold, double *pnew, double *q, double *part);
void launch_rows_update(hipStream_t s, const RowBlocks &b, int nr, size_t ld, const double *alpha,
                        const double *P, const double *Q, double *X, double *R, double *part);
void launch_rows_scatter(hipStream_t s, const RowBlocks &b, int nr, const int *inv_ptr,
                         const int *ix, const double *XN, const double *R, double *Z,
                         double *part);
void launch_rows_residual(hipStream_t s, const RowBlocks &b, int nr, size_t ld, const double *F,
                          const double *Q, double *R, double *part);
void launch_rows_floor(hipStream_t s, const RowBlocks &b, int nr, const int *rp, const int *col,
                       const double *val, const double *U, double *part);
void launch_rows_sum(hipStream_t s, const RowBlocks &b, int nr, const double *part, double *out);
void launch_rows_alpha(hipStream_t s, const RowBlocks &b, int nr, const RowCgState &st,
                       const double *part, double *alpha);
void launch_rows_beta(hipStream_t s, const RowBlocks &b, int nr, const RowCgState &st,
                      const double *part_rr, const double *part_rz, double rtol2, int it,
                      double *beta);
void launch_check_blocks(hipStream_t s, int n, const int *rp, const int *col, int nseg,
                         const long long *sptr, int *flag);

}  // namespace amsp
