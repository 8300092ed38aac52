// Host-side launchers of the device kernels (one per kernel family).  All
// pointers are device pointers; every launch goes on the given stream.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace exg {

// Edge of the output blocks of a dense product, in 32s, for a launch of nb
// blocks of 128 x 128: 4 (128 x 128), 2 or 1.  256 CUs take the blocks in
// rounds; a launch whose last (or only) round is nearly empty is faster on
// smaller blocks, which read more operand bytes per flop.  Cost in units of a
// 128 x 128 block on one CU:
//   128: ceil(nb / 256),  64: 1.15 ceil(4 nb / 256) / 4,  32: 1.6 ceil(16 nb / 256) / 16.
// With 128 x 128 blocks alone and with this rule: panel update and triangular
// solve at n = 1,600 (6 - 12 blocks) 58 and 23 us a launch, 11 and 8 us;
// trailing updates at n = 1,600 (36 blocks) 109 us, 35 us; (l, grad) at
// n = 1,600 3,527 us, 1,823 us; DST l at n = 40,000, 4 tiles wide, 48.5 ms,
// 26.8 ms.
// The weights 1.15 and 1.6 prefer the wider block where the rounds are close.
// They are high: of one launch of 7,440 blocks (n = 16,384, tile 512) 64- and
// 32-wide ones take 0.97 and 1.11 times as long as 128-wide ones, since two or
// more workgroups share a CU and the rounds blur.  All launches of one call on
// 128-, 64- and 32-wide blocks, by the rule, and the best of each launch, us:
//   trailing update     n = 10,000  6,795  5,521  5,748   5,865   5,426
//                       n = 16,384 24,130 22,047 24,396  23,069  21,965
//   inverse's update    n = 10,000  5,975  5,272  6,025   5,828   5,254
//   (tile 768)          n = 20,000 39,268 41,361 46,325  39,268  38,915
//   panel update        n = 16,384  7,663  2,206  1,595   1,973   1,529
//   panel solve         n = 16,384  7,116  2,766  1,517   2,509   1,517
// The last is where the rule is worst: from 33 to 64 blocks it takes 64-wide
// ones (14 us) where 32-wide ones have 10.
inline int block_tiles(int64_t nb) {
  const double c4 = (double)((nb + 255) / 256), c2 = 1.15 * 0.25 * (double)((4 * nb + 255) / 256),
               c1 = 1.6 * 0.0625 * (double)((16 * nb + 255) / 256);
  return c4 <= c2 && c4 <= c1 ? 4 : (c2 <= c1 ? 2 : 1);
}

// The same where the k range differs from block to block (the longest ones
// decide): 128 x 128 only where several rounds even it out.  One launch on 128-,
// 64- and 32-wide blocks, us:
//   fused LAUUM, tile 512   n =   640    15 blocks    194     60     30
//                           n = 1,408    66 blocks    263     86     63
//                           n = 2,560   210 blocks    401    191    194
//                           n = 4,608   666 blocks    874    762    833
//                           n = 6,400 1,275 blocks  2,029  2,028  2,269
//                           n = 8,192 2,080 blocks  3,541  3,701  4,359
//                           n = 14,000 6,105 blocks 15,826 18,286 21,728
// so the upper line lies where 64 and 128 cross; the lower one could lie at 200.
// Fisher products of a call (400 to 900 blocks a launch): xg at n = 6,400 14.2,
// 8.0 and 9.2 ms, at n = 12,000 48.5, 41.2 and 56.8; mxt at n = 6,400 8.8, 5.1 and
// 5.5 ms.
inline int block_tiles_uneven(int64_t nb) { return nb >= 1536 ? 4 : (nb >= 64 ? 2 : 1); }

// Blocks per chunk of the XCD order (xcd_chunk) of a launch of nb blocks of one
// length or longest first, T per tile edge: a whole tile's blocks, one row of
// them, or 1 (dispatch order), whichever first leaves the fullest XCD (64
// workgroups at a time) with no more rounds than the dispatch order does.  At
// n = 40,000 in dispatch order, by rows and by tiles: k_lauum_contract 343, 335
// and 323 ms, k_tri_gemm 307, 306 and 297 ms, k_chol_update 309, 306 and 303 ms.
// Only for 128-wide blocks and eight rounds or more (shorter launches of
// n = 10,000: l 10.05 -> 10.13 ms, (l, grad) 24.2 -> 24.7 ms), and not where
// whole tiles are skipped or differ (the mixed lists and k_update_lp, whose
// chunks would load the XCDs unevenly: k_tri_gemm_band 18 -> 25 ms,
// k_update_lp 88 -> 93 ms).
inline int xcd_chunk_size(int B, int T, int64_t nb) {
  if (B != 4 || nb < 4096) return 1;
  const int64_t plain = ((nb + 7) / 8 + 63) / 64;
  for (int64_t c = (int64_t)T * T; c > 1; c = c > T ? T : 1) {
    const int64_t most = ((nb + c - 1) / c + 7) / 8 * c;  // blocks of the fullest XCD
    if ((most + 63) / 64 <= plain) return (int)c;
  }
  return 1;
}
inline int64_t xcd_chunk_grid(int64_t nb, int chunk) {
  return chunk > 1 ? (nb + 8 * chunk - 1) / (8 * chunk) * (8 * chunk) : nb;
}

// kernel<B> for the block edge 32 B, 256 threads per workgroup
#define EXG_BLOCKS(tiles, kernel, grid, stream, ...)                                                     \
  do {                                                                                                   \
    if ((tiles) == 4)                                                                                    \
      hipLaunchKernelGGL(kernel<4>, dim3((unsigned)(grid)), dim3(256), 0, stream, __VA_ARGS__);          \
    else if ((tiles) == 2)                                                                               \
      hipLaunchKernelGGL(kernel<2>, dim3((unsigned)(grid)), dim3(256), 0, stream, __VA_ARGS__);          \
    else                                                                                                 \
      hipLaunchKernelGGL(kernel<1>, dim3((unsigned)(grid)), dim3(256), 0, stream, __VA_ARGS__);          \
  } while (0)

// k_matern.hip
// doubles of the per-theta table array (quadrature nodes + Chebyshev tables)
int64_t quad_table_doubles();
// info (may be null): reset to "no failed pivot"
void launch_quad_table(const double theta[3], int metric, double nugget, double* qt, double* cst,
                       unsigned long long* info, hipStream_t s);
void launch_gen_tiles(const TileMat& M, int64_t nreal, const double* xs, const double* ys, const double* qt,
                      const double* cst, const uint8_t* tag, bool fill_zero, hipStream_t s);
void launch_gen_dense(double* cov, int64_t ldc, int64_t n, const double* x, const double* y, const double* qt,
                      const double* cst, hipStream_t s);
// r = z - Sigma a in FP64 (Sigma regenerated), sorted order, zero on padding
void launch_sigma_residual(const double* xs, const double* ys, const double* zs, const double* av, int64_t nreal,
                           int64_t npad, const double* qt, const double* cst, double* r, hipStream_t s);

// k_small.hip
void launch_sort_locations(const double* x, const double* y, const double* z, int64_t n, int64_t npad, int64_t P,
                           double* box, uint64_t* keys, int32_t* rank, double* xs, double* ys, double* zs,
                           int32_t* perm, hipStream_t s);
void launch_scatter(const double* v, const int32_t* perm, int64_t n, double* out, hipStream_t s);
void launch_potrf_blk(double* A, int64_t lda, double* dinv, double* ldpart, unsigned long long* info, int64_t col0,
                      hipStream_t s);
// inverses and log-determinant parts of `count` factor blocks in the padding
void launch_pad_blocks(double* dinv, double* ldpart, int64_t count, hipStream_t s);
// forward solve by tiles: y_k = L_kk^-1 rhs_k from the 128-block inverses of
// tile k, then rhs_i -= L_ik y_k below it
void launch_solve_tile(const TileMat& M, int64_t k, const double* dinv_k, int64_t nreal, const double* rhs, double* y,
                       hipStream_t s);
void launch_solve_below(const TileMat& M, int64_t k, int64_t nreal, const double* y, double* rhs, hipStream_t s);
void launch_solve_below_lp(const TileMat& M, const uint8_t* tag, int64_t k, int64_t nreal, const double* y,
                           double* rhs, hipStream_t s);
void launch_trsv_bwd(const TileMat& M, const double* Xd, double* rhs, double* a, hipStream_t s);
// w = L e; part: scratch of TRMV_PARTS vectors of the padded length
constexpr int64_t TRMV_PARTS = 32;
void launch_trmv_lower(const TileMat& M, int64_t nreal, const double* e, double* part, double* w, hipStream_t s);
// out[0..2] = l, log det, quadratic form; out[OUT_INFO], out[OUT_BOX ..] the
// first failed pivot (as an integer) and box[0..4]
enum { OUT_INFO = 6, OUT_BOX = 7, OUT_COUNT = 12 };
void launch_finalize_loglik(const double* yv, int64_t n, const double* ldpart, int64_t nld,
                            const unsigned long long* info, const double* box, double* out, hipStream_t s);
void launch_finalize_grad(const double* part, int64_t nparts, double* out, hipStream_t s);
// eq. (2) with the quadratic form z^T a (a = Sigma^-1 z)
void launch_finalize_loglik_za(const double* zs, const double* av, int64_t n, const double* ldpart, int64_t nld,
                               const unsigned long long* info, const double* box, double* out, hipStream_t s);
// refinement steps on the device: y = a + d; nrm[0] = |r|^2 (trial = 0) or
// nrm[1] = (|r|^2 < nrm[0]) with nrm[0] lowered then (trial = 1); the select
// takes a_try, r_try when nrm[1] is set
void launch_add2(double* y, const double* a, const double* d, int64_t n, hipStream_t s);
void launch_resid_norm(const double* r, int64_t n, double* nrm, int trial, hipStream_t s);
void launch_refine_select(double* a, const double* a_try, double* r, const double* r_try, const double* nrm,
                          int64_t n, hipStream_t s);
void launch_copy(double* dst, const double* src, int64_t n, hipStream_t s);
void launch_copy_diag_lower(double* dst, const double* diag, int64_t ts, int64_t NT, hipStream_t s);
void launch_put_dinv(double* dst, const double* dinv, int64_t ts, int64_t NT, int c, hipStream_t s);

void launch_diag_apply_n(const double* Xk, int64_t ts, const double* b, double* out, hipStream_t s);
void launch_diag_apply_t(const double* Xk, int64_t ts, const double* b, double* out, hipStream_t s);

// k_mixed.hip
void launch_tile_bbox(const double* xs, const double* ys, int64_t ts, int64_t NT, int64_t nreal, double* box,
                      hipStream_t s);
// dmin[off_index(i, j)]: smallest distance between the real points of location
// blocks i > j (sorted, planar); corr: the correlation at that distance
void launch_tile_dmin(const double* xs, const double* ys, int64_t ts, int64_t NT, int64_t nreal, double* dmin,
                      hipStream_t s);
void launch_tile_corr(const double* dmin, int64_t NT, const double* qt, const double* cst, double* corr,
                      hipStream_t s);
void launch_panel_gather(const TileMat& M, int64_t k, const uint8_t* tag, double* pbuf, hipStream_t s);
void launch_panel_scatter(const TileMat& M, int64_t k, const uint8_t* tag, const double* pbuf, float* p32,
                          hipStream_t s);
// BF16 copy of the FP64 panel of step k, each tile transposed (k contiguous)
void launch_panel_bf16t(const TileMat& M, int64_t k, const double* pbuf, uint16_t* pbt, hipStream_t s);
// skip_bf16: BF16 targets are left to launch_update_bf16
void launch_update_lp(const TileMat& M, const uint8_t* tag, const float* p32, const uint16_t* pbt, int64_t k,
                      int64_t nreal, int part, bool skip_bf16, hipStream_t s);
// step k of the mixed update for the BF16 targets (li[e], lj[e]), e0 <= e <
// e0 + count, on 256 x 256 blocks (ts a multiple of 256); pbt: the BF16 panel
// copy of step k (tiles transposed)
void launch_update_bf16(const TileMat& M, const int32_t* li, const int32_t* lj, int64_t e0, int64_t count,
                        const uint16_t* pbt, int64_t k, int64_t nreal, hipStream_t s);
void launch_trsv_bwd_lp(const TileMat& M, const uint8_t* tag, const double* Xd, double* rhs, double* a,
                        hipStream_t s);
// one step of the mixed inverse (FP32 off-diagonal tiles of L^-1, FP32 buffer P)
// The FP64 band tiles of the mixed factor: device lists li / lj (tile (li[e],
// lj[e]), column-major order, pool slot e) and rl (list entries in row-major
// order), with host arrays of the first entry of each tile column (cfirst,
// into li / lj) and of each tile row (rfirst, into rl), NT + 1 each.
struct BandLists {
  const int32_t* li;
  const int32_t* lj;
  const int32_t* rl;
  const int64_t* cfirst;
  const int64_t* rfirst;
};
// step k of the mixed inverse (P: FP32 staging, Q: FP64 staging of the band
// tiles, each (NT - 1) ts^2 elements)
void launch_trtri_right_lp(const TileMat& M, const uint8_t* tag, const double* Xk, float* P, double* Q,
                           const BandLists& bl, int64_t k, int64_t nreal, hipStream_t s);
void launch_trtri_rest_lp(const TileMat& M, const uint8_t* tag, const double* Xk, float* P, double* Q,
                          const BandLists& bl, int64_t k, int64_t nreal, hipStream_t s);
// mixed fused LAUUM + contraction; returns the number of partial triples
int64_t launch_lauum_contract_lp(const TileMat& M, const uint8_t* tag, int64_t nreal, const double* xs,
                                 const double* ys, const double* av, const double* qt, const double* cst,
                                 const int32_t* li, const int32_t* lj, int64_t nband, double* part, hipStream_t s);
void launch_trsv_fwd_lp(const TileMat& M, const uint8_t* tag, const double* Xd, int64_t nreal, double* rhs,
                        double* y, hipStream_t s);

// k_gemm.hip
// trailing update of step k (diag_only: only the diagonal targets); part is
// an UpdatePart: all targets, the first trailing column, or the rest
void launch_chol_update(const TileMat& M, const double* below, int64_t k, int64_t nreal, bool diag_only, int part,
                        hipStream_t s);
// mixed precision: FP64 update of the band tiles (li[e], lj[e]), e0 <= e < e0 + count
void launch_band_update(const TileMat& M, const double* below, int64_t k, int64_t nreal, const int32_t* li,
                        const int32_t* lj, int64_t e0, int64_t count, hipStream_t s);
void launch_panel(double* Dk, double* below, int64_t ts, int64_t NT, int64_t k, int64_t nreal, double* dinv_k,
                  double* ldpart_k, unsigned long long* info, hipStream_t s);
void launch_diag_inverses(double* Xd, const double* diag, const double* dinv, int64_t ts, int64_t NT, hipStream_t s);
// the step's two halves: P_k and column k (any stream), then the rest
void launch_trtri_right(const TileMat& M, const double* Xk, double* P, int64_t k, int64_t nreal, hipStream_t s);
void launch_trtri_rest(const TileMat& M, const double* Xk, double* P, int64_t k, int64_t nreal, hipStream_t s);
// edge (in 32s) of the output blocks of the fused LAUUM and contraction, by the
// number of 128 x 128 blocks with real entries, and the blocks of the lower tiles
inline int lauum_tiles(int64_t nreal) {
  const int64_t R = (nreal + BLK - 1) / BLK;
  return block_tiles_uneven(R * (R + 1) / 2);
}
inline int64_t lauum_blocks(int64_t ts, int64_t NT, int B) {
  const int64_t T = ts / (32 * B);
  return NT * (NT + 1) / 2 * T * T;
}
// part: 3 lauum_blocks(ts, NT, lauum_tiles(nreal)) doubles; returns the number of
// partial triples written
int64_t launch_lauum_contract(const TileMat& M, int64_t nreal, const double* xs, const double* ys, const double* av,
                           const double* qt, const double* cst, double* part, hipStream_t s);

// k_predict.hip
void launch_krige_mean(const double* xs, const double* ys, const double* av, int64_t nreal, const double* xn,
                       const double* yn, int64_t m, const double* qt, const double* cst, double* mean, hipStream_t s);
// variance of new points c0 .. c0 + ncols - 1 (ncols a multiple of 128; C, V: npad x ncols, ld npad)
void launch_krige_mse(const TileMat& M, const double* Xd, const double* xs, const double* ys, int64_t nreal,
                      const double* xn, const double* yn, int64_t m, int64_t c0, int64_t ncols, const double* qt,
                      const double* cst, double* C, double* V, double* mse, hipStream_t s);

// k_fisher.hip (X: the tile matrix holding L^-1; B's: lower tiles packed by
// tile columns, n^2 / 2 doubles each)
int64_t fisher_part_blocks(int64_t ts, int64_t NT);
// doubles of the strip shared by the regenerated derivative rows and the staging
size_t fisher_strip_doubles(int64_t ts, int64_t NT);
void launch_fisher_param(const TileMat& X, int comp, int64_t nreal, const double* xs, const double* ys,
                         const double* qt, const double* cst, double* S, double* Bm, hipStream_t s);
// Bs: B_sigma2 or null (B_sigma2 = I / sigma2); part: 9 fisher_part_blocks
// doubles; out: 9 doubles (device)
void launch_fisher_reduce(const double* Bs, const double* Bb, const double* Bn, int64_t ts, int64_t NT, int64_t nreal,
                          const double* cst, double* part, double* out, hipStream_t s);

}  // namespace exg
