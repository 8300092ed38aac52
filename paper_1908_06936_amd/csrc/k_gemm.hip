// FP64 MFMA kernels of the tile algorithms.  Every kernel maps one 256-thread
// workgroup to 128 x 128 output blocks and calls the shared gemm_blk core.
//
// Cholesky (tile algorithm of Buttari, Langou, Kurzak & Dongarra, Parallel
// Computing 35, 2009, right-looking over tile columns; the paper relies on it
// through its tile library, Section 2.2):
//   panel k: a left-looking sweep over the 128-wide sub-columns c of tile
//   column k: update, factor the 128 x 128 diagonal block (k_potrf_blk),
//   then multiply the blocks below by its inverse (TRSM);
//   trailing update: A_ij -= A_ik A_jk^T for k < j <= i (SYRK on i = j).
//
// Inverse L^-1 (tile TRTRI, in place, step k): A_ik <- -A_ik X_kk (i > k);
// A_ij += A_ik A_kj (i > k > j); A_kj <- X_kk A_kj (j < k); A_kk <- X_kk, with
// X_kk the inverse of the diagonal tile, itself built from the 128-block
// inverses by the same four steps on 128-blocks.
//
// Fused LAUUM and score contraction: W = L^-T L^-1 = Sigma^-1 block by block,
// W_IJ = sum_{K >= I} X_KI^T X_KJ, contracted at once with
//   (a_i a_j / 2 - W_ij / 2) dSigma_m(i, j),  a = Sigma^-1 z,
// so W is never stored.
#include "common.h"
#include "contract.h"
#include "launch.h"

namespace exg {

// -------------------------------------------------------------- Cholesky
// trailing update of step k over the tiles (i, j), k < j <= i < NT
// below: the FP64 tiles (k+1, k), ..., (NT-1, k) of column k, contiguous.
// Mixed precision runs it only on its FP64 targets: the diagonal tiles
// (PAIRS_DIAG) and the FP64 band tiles, given as a list of (i, j) entries
// off, off + 1, ... (PAIRS_LIST; stored in the band pool).
// Block edge 32 B (block_tiles); T = ts / (32 B) blocks per tile edge.
template <int B>
__global__ __launch_bounds__(256, 2) void k_chol_update(TileMat M, const double* __restrict__ below, int T, int64_t k,
                                                        int64_t nreal, int64_t nb, int chunk, int mode, int64_t off,
                                                        const int32_t* __restrict__ li,
                                                        const int32_t* __restrict__ lj) {
  constexpr int E = 32 * B;
  __shared__ double sm[gemm_lds(B, B)];
  const int64_t ts = M.ts;
  const int64_t b = xcd_chunk(nb, chunk);
  if (b < 0) return;
  const int64_t p = b / (T * T);
  const int sub = (int)(b % (T * T));
  const int u = sub / T, v = sub % T;
  int64_t a, c;
  if (mode == PAIRS_LIST) {
    a = li[off + p] - k - 1;
    c = lj[off + p] - k - 1;
  } else {
    pair_map(mode, off, p, &a, &c);
  }
  const int64_t i = k + 1 + a, j = k + 1 + c;
  if (i == j && u < v) return;
  if (i * ts + u * E >= nreal || j * ts + v * E >= nreal) return;  // padding: update is zero
  const double* Ap = below + a * ts * ts + u * E;
  const double* Bp = below + c * ts * ts + v * E;
  double* C = ((i == j || !M.pool) ? tptr(M, i, j) : band64(M, off_index(i, j, M.NT))) + u * E +
              (int64_t)v * E * ts;
  v4d acc[B][B];
  acc_zero(acc);
  gemm_blk<false, false, B, B>(Ap, ts, Bp, ts, (int)ts, acc, sm);
  acc_store(C, ts, acc, -1.0, true);
}

// panel k, sub-column c: rows g0 + ... (128-row blocks, global index)
//   C = A[g, c] -= A[g, 0:c] A[(k,c), 0:c]^T
// The panel of column k is the diagonal tile Dk followed by the contiguous
// FP64 tiles `below`; row block g (global index) lies in tile i = g / T.
__device__ __forceinline__ double* panel_tile(double* Dk, double* below, int64_t i, int64_t k, int64_t ts) {
  return i == k ? Dk : below + (i - k - 1) * ts * ts;
}

// one (32 B) x (32 B) part of a 128 x 128 block per workgroup
template <int B>
__global__ __launch_bounds__(256, 2) void k_panel_update(double* __restrict__ Dk, double* __restrict__ below,
                                                         int64_t ts, int T, int64_t k, int c, int64_t g0) {
  constexpr int E = 32 * B, S = 4 / B;  // S x S parts per block
  __shared__ double sm[gemm_lds(B, B)];
  const int64_t g = g0 + blockIdx.x / (S * S);
  const int q = (int)(blockIdx.x % (S * S)), pu = q / S, pv = q % S;
  const int64_t i = g / T;
  const int u = (int)(g % T);
  double* P = panel_tile(Dk, below, i, k, ts) + u * BLK + pu * E;
  const double* D = Dk + c * BLK + pv * E;
  v4d acc[B][B];
  acc_zero(acc);
  gemm_blk<false, false, B, B>(P, ts, D, ts, c * BLK, acc, sm);
  acc_store(P + (int64_t)(c * BLK + pv * E) * ts, ts, acc, -1.0, true);
}

// panel k, sub-column c: C = A[g, c] Dinv_c^T for the blocks below the diagonal
// block, 32 B rows of a block per workgroup (in place: each workgroup reads
// only the rows that it overwrites)
template <int B>
__global__ __launch_bounds__(256, 2) void k_panel_trsm(double* __restrict__ Dk, double* __restrict__ below, int64_t ts,
                                                       int T, int64_t k, int c, int64_t g0,
                                                       const double* __restrict__ dinv) {
  constexpr int E = 32 * B, S = 4 / B;
  __shared__ double sm[gemm_lds(B, 4)];
  const int64_t g = g0 + blockIdx.x / S;
  const int64_t i = g / T;
  const int u = (int)(g % T);
  double* C = panel_tile(Dk, below, i, k, ts) + u * BLK + (int)(blockIdx.x % S) * E + (int64_t)c * BLK * ts;
  v4d acc[B][4];
  acc_zero(acc);
  gemm_blk<false, true, B, 4>(C, ts, dinv, BLK, BLK, acc, sm);  // Bop(n, q) = X(n, q), X row by row
  acc_store(C, ts, acc, 1.0, false);
}

// ------------------------------------------- inverses of the diagonal tiles
// All NT diagonal tiles at once, on copies Xd[k] (ts x ts) that start as the
// lower part of L_kk; step c of the 128-block algorithm.
// right: X[r, c] <- -X[r, c] Dinv_c for r > c, 32 B rows per workgroup (in place)
template <int B>
__global__ __launch_bounds__(256, 2) void k_dinv_right(double* __restrict__ Xd, const double* __restrict__ dinv,
                                                       int64_t ts, int T, int c) {
  constexpr int E = 32 * B, S = 4 / B;
  __shared__ double sm[gemm_lds(B, 4)];
  const int nr = (T - 1 - c) * S;
  const int64_t k = blockIdx.x / nr;
  const int r = (int)(blockIdx.x % nr);
  double* C = Xd + k * ts * ts + (c + 1) * BLK + r * E + (int64_t)c * BLK * ts;
  const double* D = dinv + (k * T + c) * BLK * BLK;
  v4d acc[B][4];
  acc_zero(acc);
  gemm_blk<false, false, B, 4>(C, ts, D, BLK, BLK, acc, sm);  // Bop(n, q) = X(q, n), X row by row
  acc_store(C, ts, acc, -1.0, false);
}

// gemm: X[r, b] += X[r, c] X[c, b] for r > c > b, on (32 B) x (32 B) blocks
template <int B>
__global__ __launch_bounds__(256, 2) void k_dinv_gemm(double* __restrict__ Xd, int64_t ts, int T, int c) {
  constexpr int E = 32 * B, S = 4 / B;
  __shared__ double sm[gemm_lds(B, B)];
  const int nc = c * S, per = (T - 1 - c) * S * nc;
  const int64_t k = blockIdx.x / per;
  const int q = (int)(blockIdx.x % per);
  const int64_t r = (c + 1) * BLK + (q / nc) * E, bb = (int64_t)(q % nc) * E;
  double* X = Xd + k * ts * ts;
  v4d acc[B][B];
  acc_zero(acc);
  gemm_blk<false, true, B, B>(X + r + (int64_t)c * BLK * ts, ts, X + c * BLK + bb * ts, ts, BLK, acc, sm);
  acc_store(X + r + bb * ts, ts, acc, 1.0, true);
}

// left: X[c, b] <- Dinv_c X[c, b] for b < c, 32 B columns per workgroup (in place)
template <int B>
__global__ __launch_bounds__(256, 2) void k_dinv_left(double* __restrict__ Xd, const double* __restrict__ dinv,
                                                      int64_t ts, int T, int c) {
  constexpr int E = 32 * B, S = 4 / B;
  __shared__ double sm[gemm_lds(4, B)];
  const int64_t k = blockIdx.x / (c * S);
  const int bb = (int)(blockIdx.x % (c * S));
  double* C = Xd + k * ts * ts + c * BLK + (int64_t)bb * E * ts;
  const double* D = dinv + (k * T + c) * BLK * BLK;
  v4d acc[4][B];
  acc_zero(acc);
  // Aop(m, q) = X(m, q), X row by row; Bop(n, q) = C(q, n)
  gemm_blk<true, true, 4, B>(D, BLK, C, ts, BLK, acc, sm);
  acc_store(C, ts, acc, 1.0, false);
}

// --------------------------------------------------------- tile TRTRI step k
// Blocks of edge E = 32 B (block_tiles), T = ts / E per tile edge.
// P_i = -A_ik X_kk for i > k, into the buffer P (tile i - k - 1); one block
// (u, v) per workgroup, k range restricted to the non-zero rows v E.. of the
// lower-triangular X_kk.
template <int B>
__global__ __launch_bounds__(256, 2) void k_tri_right(TileMat M, const double* __restrict__ Xk, double* __restrict__ P,
                                                      int T, int64_t k, int64_t nreal, int64_t nb) {
  const int64_t ts = M.ts;
  constexpr int E = 32 * B;
  __shared__ double sm[gemm_lds(B, B)];
  const int64_t b = blockIdx.x;
  if (b >= nb) return;
  const int64_t i = k + 1 + b / (T * T);
  const int sub = (int)(b % (T * T));
  const int u = sub / T, v = sub % T;
  const int64_t off = (int64_t)v * E * ts;
  const double* Ap = tptr(M, i, k) + u * E + off;
  double* C = P + (i - k - 1) * ts * ts + u * E + off;
  v4d acc[B][B];
  acc_zero(acc);
  // padded rows of L^-1 are zero: store zeros (the buffer is copied back whole)
  if (i * ts + u * E < nreal) gemm_blk<false, true, B, B>(Ap, ts, Xk + v * E + off, ts, (int)(ts - v * E), acc, sm);
  acc_store(C, ts, acc, -1.0, false);
}

// A_ij += P_i A_kj for k < i < NT, 0 <= j < k (P_i = the new A_ik)
template <int B>
__global__ __launch_bounds__(256, 2) void k_tri_gemm(TileMat M, const double* __restrict__ P, int T, int64_t k,
                                                     int64_t nreal, int64_t nb, int chunk) {
  const int64_t ts = M.ts;
  constexpr int E = 32 * B;
  __shared__ double sm[gemm_lds(B, B)];
  const int64_t b = xcd_chunk(nb, chunk);
  if (b < 0) return;
  const int64_t p = b / (T * T);
  const int sub = (int)(b % (T * T));
  const int u = sub / T, v = sub % T;
  const int64_t i = k + 1 + p / k, j = p % k;
  if (i * ts + u * E >= nreal) return;
  const double* Ap = P + (i - k - 1) * ts * ts + u * E;
  const double* Bp = tptr(M, k, j) + (int64_t)v * E * ts;
  double* C = tptr(M, i, j) + u * E + (int64_t)v * E * ts;
  v4d acc[B][B];
  acc_zero(acc);
  gemm_blk<false, true, B, B>(Ap, ts, Bp, ts, (int)ts, acc, sm);
  acc_store(C, ts, acc, 1.0, true);
}

// R_j = X_kk A_kj for j < k, into the buffer P (tile j); k range restricted
// to the non-zero columns ..(u+1) E of row block u of X_kk.
template <int B>
__global__ __launch_bounds__(256, 2) void k_tri_left(TileMat M, const double* __restrict__ Xk, double* __restrict__ P,
                                                     int T, int64_t k, int64_t nb) {
  const int64_t ts = M.ts;
  constexpr int E = 32 * B;
  __shared__ double sm[gemm_lds(B, B)];
  const int64_t b = blockIdx.x;
  if (b >= nb) return;
  const int64_t j = b / (T * T);
  const int sub = (int)(b % (T * T));
  const int u = sub / T, v = sub % T;
  const int64_t off = (int64_t)v * E * ts;
  const double* Bp = tptr(M, k, j) + off;
  double* C = P + j * ts * ts + u * E + off;
  v4d acc[B][B];
  acc_zero(acc);
  gemm_blk<false, true, B, B>(Xk + u * E, ts, Bp, ts, (u + 1) * E, acc, sm);
  acc_store(C, ts, acc, 1.0, false);
}

// tile (i0 + q, jcol) or (irow, j0 + q) <- P tile q, q < count (column or row run)
__global__ void k_copy_back(TileMat M, const double* __restrict__ P, int64_t count, int64_t i0, int64_t j0,
                            int column) {
  const int64_t tt = M.ts * M.ts;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count * tt) return;
  const int64_t q = e / tt, o = e % tt;
  const int64_t i = column ? i0 + q : i0, j = column ? j0 : j0 + q;
  tptr(M, i, j)[o] = P[e];
}

// ------------------------------------------ tile transposition
// Every lower tile of the tile matrix transposed in place, so that the columns
// of X = L^-1 become contiguous rows for the LAUUM below (both of its operands
// are then read along their contiguous index).  One workgroup swaps the 64 x 64
// blocks (a, b) and (b, a), a <= b, of one tile through LDS.
constexpr int TB = 64;
__global__ __launch_bounds__(256) void k_transpose_tiles(TileMat M, int64_t npt, int64_t nb) {
  __shared__ double s1[TB][TB + 1];
  __shared__ double s2[TB][TB + 1];
  const int64_t g = blockIdx.x;
  if (g >= nb) return;
  const int64_t ts = M.ts;
  int64_t I, J, bq, aq;
  tri_decode(g / npt, &I, &J);
  tri_decode(g % npt, &bq, &aq);  // aq <= bq
  double* T = tptr(M, I, J);
  const int64_t ra = aq * TB, rb = bq * TB;
  for (int e = threadIdx.x; e < TB * TB; e += 256) {
    const int r = e & (TB - 1), c = e >> 6;
    s1[c][r] = T[(ra + r) + (rb + c) * ts];
    if (aq != bq) s2[c][r] = T[(rb + r) + (ra + c) * ts];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < TB * TB; e += 256) {
    const int r = e & (TB - 1), c = e >> 6;
    if (aq != bq) {
      T[(ra + r) + (rb + c) * ts] = s2[r][c];
      T[(rb + r) + (ra + c) * ts] = s1[r][c];
    } else {
      T[(ra + r) + (ra + c) * ts] = s1[r][c];
    }
  }
}

// ------------------------------------------ fused LAUUM + score contraction
// Block (I, J, u, v) of W = X^T X with X = L^-1 (lower tiles, in place of L,
// each tile transposed by k_transpose_tiles),
// followed by g_m += sum (w_ij (a_i a_j - W_ij) / 2) dSigma_m(i, j) over its
// entries, w = 2 below the diagonal, 1 on it, 0 above and on padding.
// part[3 b + m] receives the block's sums (zeros for skipped blocks).
template <int B>
__global__ __launch_bounds__(256, 2) void k_lauum_contract(TileMat M, int T, int64_t nreal,
                                                           const double* __restrict__ xs,
                                                           const double* __restrict__ ys, const double* __restrict__ av,
                                                           const double* __restrict__ qt,
                                                           const double* __restrict__ cst, double* __restrict__ part,
                                                           int64_t nb, int chunk) {
  constexpr int E = 32 * B;
  constexpr int LDS = gemm_lds(B, B) > contract_lds(B) ? gemm_lds(B, B) : contract_lds(B);
  __shared__ __attribute__((aligned(16))) double sm[LDS];
  const int64_t ts = M.ts, NT = M.NT;
  const int64_t b = xcd_chunk(nb, chunk);
  if (b < 0) return;
  const int64_t p = b / (T * T);
  const int sub = (int)(b % (T * T));
  const int u = sub / T, v = sub % T;
  int64_t I, J;
  tri_decode(p, &I, &J);
  // DST: dSigma is zero outside the tile band, so are those blocks' terms
  if ((I == J && u < v) || I * ts + u * E >= nreal || J * ts + v * E >= nreal || (M.dst > 0 && I - J >= M.dst)) {
    if (threadIdx.x < 3) part[3 * b + threadIdx.x] = 0.0;
    return;
  }
  v4d acc[B][B];
  acc_zero(acc);
  // One virtual k range over the tiles K = I, ..., NT-1 of tile columns I and
  // J: first rows r0.. of tile row I (X_II is lower triangular, so rows above
  // u E of its column block u are zero), then every row of the tiles below.
  // Transposed tiles: X(K, I)[k, m] sits at k ts + m of tile (K, I).  The
  // off-diagonal tiles of one tile column are stored one after another, so
  // row kk of the stack (K, I), K > I, is at kk ts of the stack's first tile
  // ((kk / ts) ts^2 + (kk % ts) ts = kk ts): no division per stage.
  const int64_t r0 = (int64_t)u * E, c0 = (int64_t)v * E;
  const int64_t L0 = ts - r0;
  const double* XdI = M.diag + I * ts * ts;
  const double* XbI = I + 1 < NT ? (const double*)M.off + off_index(I + 1, I, NT) * ts * ts : XdI;
  // row k0 of either operand's range is at k0 ts of one of two bases
  const double *a1 = XdI + r0 + r0 * ts, *a2 = XbI + r0 - L0 * ts;
  // I > J: the tiles (I, J), (I + 1, J), ... are one stack as well
  const double *b1 = (I == J ? XdI : tptr(M, I, J)) + c0 + r0 * ts, *b2 = I == J ? XbI + c0 - L0 * ts : b1;
  auto ap = [=](int k0) { return (k0 < L0 ? a1 : a2) + (int64_t)k0 * ts; };
  auto bp = [=](int k0) { return (k0 < L0 ? b1 : b2) + (int64_t)k0 * ts; };
  gemm_core<false, false, B, B>(ap, ts, bp, ts, (int)(L0 + (NT - 1 - I) * ts), acc, sm);
  contract_block64(acc, I * ts + r0, J * ts + c0, nreal, xs, ys, av, qt, cst, sm, part + 3 * b);
}

// ------------------------------------------------------------- launchers
static void update_pairs(const TileMat& M, const double* below, int64_t k, int64_t nreal, int mode, int64_t off,
                         int64_t npairs, const int32_t* li, const int32_t* lj, hipStream_t s) {
  const int64_t T4 = M.ts / BLK;
  const int B = block_tiles(npairs * T4 * T4);
  const int T = (int)(M.ts / (32 * B));
  const int64_t nblk = npairs * T * T;
  const int ch = li ? 1 : xcd_chunk_size(B, T, nblk);
  EXG_BLOCKS(B, k_chol_update, xcd_chunk_grid(nblk, ch), s, M, below, T, k, nreal, nblk, ch, mode, off, li, lj);
}

void launch_chol_update(const TileMat& M, const double* below, int64_t k, int64_t nreal, bool diag_only, int part,
                        hipStream_t s) {
  int64_t m = M.NT - k - 1;  // trailing tiles
  if (M.dst > 0 && m > M.dst - 1) m = M.dst - 1;  // DST: L_ik = 0 for i - k >= dst
  if (m <= 0) return;
  int mode;
  int64_t off, npairs;
  if (diag_only) {
    mode = PAIRS_DIAG;
    off = part == UPD_REST ? 1 : 0;
    npairs = part == UPD_ALL ? m : part == UPD_FIRST_COLUMN ? 1 : m - 1;
  } else if (part == UPD_ALL) {
    mode = PAIRS_TRI, off = 0, npairs = m * (m + 1) / 2;
  } else if (part == UPD_FIRST_COLUMN) {
    mode = PAIRS_COL, off = 0, npairs = m;
  } else {
    mode = PAIRS_TRI, off = 1, npairs = (m - 1) * m / 2;
  }
  if (npairs <= 0) return;
  update_pairs(M, below, k, nreal, mode, off, npairs, nullptr, nullptr, s);
}

void launch_band_update(const TileMat& M, const double* below, int64_t k, int64_t nreal, const int32_t* li,
                        const int32_t* lj, int64_t e0, int64_t count, hipStream_t s) {
  if (count <= 0) return;
  update_pairs(M, below, k, nreal, (int)PAIRS_LIST, e0, count, li, lj, s);
}

void launch_panel(double* Dk, double* below, int64_t ts, int64_t NT, int64_t k, int64_t nreal, double* dinv_k,
                  double* ldpart_k, unsigned long long* info, hipStream_t s) {
  const int T = (int)(ts / BLK);
  const int64_t gmax = (nreal + BLK - 1) / BLK;  // blocks holding real rows
  (void)NT;
  for (int c = 0; c < T; ++c) {
    const int64_t gd = k * T + c;  // global index of the diagonal block
    if (gd >= gmax) {  // the rest of the tile is padding, the identity
      launch_pad_blocks(dinv_k + (int64_t)c * BLK * BLK, ldpart_k + c, T - c, s);
      break;
    }
    if (c > 0) {
      const int B = block_tiles(gmax - gd);
      EXG_BLOCKS(B, k_panel_update, (gmax - gd) * (4 / B) * (4 / B), s, Dk, below, ts, T, k, c, gd);
    }
    double* Dblk = Dk + c * BLK + (int64_t)c * BLK * ts;
    launch_potrf_blk(Dblk, ts, dinv_k + (int64_t)c * BLK * BLK, ldpart_k + c, info, gd * BLK, s);
    if (gmax > gd + 1) {
      const int B = block_tiles(gmax - gd - 1);
      EXG_BLOCKS(B, k_panel_trsm, (gmax - gd - 1) * (4 / B), s, Dk, below, ts, T, k, c, gd + 1,
                 dinv_k + (int64_t)c * BLK * BLK);
    }
  }
}

void launch_diag_inverses(double* Xd, const double* diag, const double* dinv, int64_t ts, int64_t NT, hipStream_t s) {
  const int T = (int)(ts / BLK);
  launch_copy_diag_lower(Xd, diag, ts, NT, s);
  for (int c = 0; c < T; ++c) {
    const int64_t nr = T - 1 - c;
    if (nr > 0) {
      const int B = block_tiles(NT * nr), S = 4 / B;
      EXG_BLOCKS(B, k_dinv_right, NT * nr * S, s, Xd, dinv, ts, T, c);
    }
    if (nr > 0 && c > 0) {
      const int B = block_tiles(NT * nr * c), S = 4 / B;
      EXG_BLOCKS(B, k_dinv_gemm, NT * nr * c * S * S, s, Xd, ts, T, c);
    }
    if (c > 0) {
      const int B = block_tiles(NT * c), S = 4 / B;
      EXG_BLOCKS(B, k_dinv_left, NT * c * S, s, Xd, dinv, ts, T, c);
    }
    launch_put_dinv(Xd, dinv, ts, NT, c, s);
  }
}

// Step k of the in-place tile inverse X = L^-1 (after this step rows 0..k of
// X are final), in two halves for two streams.  The first half (P_i = -A_ik
// X_kk into P, then column k <- P) reads only column k of L and X_kk, which no
// earlier step writes, so step k + 1's first half can run beside step k's
// second half (A_ij += P_i A_kj left of column k, row k <- X_kk A_kj, the
// diagonal tile <- X_kk) when the two use different staging buffers.
void launch_trtri_right(const TileMat& M, const double* Xk, double* P, int64_t k, int64_t nreal, hipStream_t s) {
  const int64_t ts = M.ts, NT = M.NT, T4 = ts / BLK;
  const int64_t nbelow = NT - k - 1;
  if (nbelow <= 0) return;
  const int B = block_tiles(nbelow * T4 * T4);
  const int T = (int)(ts / (32 * B));
  const int64_t nr = nbelow * T * T;
  EXG_BLOCKS(B, k_tri_right, nr, s, M, Xk, P, T, k, nreal, nr);
  hipLaunchKernelGGL(k_copy_back, dim3((unsigned)((nbelow * ts * ts + 255) / 256)), dim3(256), 0, s, M, P, nbelow,
                     k + 1, k, 1);
}

void launch_trtri_rest(const TileMat& M, const double* Xk, double* P, int64_t k, int64_t nreal, hipStream_t s) {
  const int64_t ts = M.ts, NT = M.NT, T4 = ts / BLK;
  const int64_t tt = ts * ts;
  const int64_t nbelow = NT - k - 1;
  if (nbelow > 0 && k > 0) {
    const int B = block_tiles(nbelow * k * T4 * T4);
    const int T = (int)(ts / (32 * B));
    const int64_t ng = nbelow * k * T * T;
    const int ch = xcd_chunk_size(B, T, ng);
    EXG_BLOCKS(B, k_tri_gemm, xcd_chunk_grid(ng, ch), s, M, P, T, k, nreal, ng, ch);
  }
  if (k > 0) {
    const int B = block_tiles(k * T4 * T4);
    const int T = (int)(ts / (32 * B));
    const int64_t nl = k * T * T;
    EXG_BLOCKS(B, k_tri_left, nl, s, M, Xk, P, T, k, nl);
    hipLaunchKernelGGL(k_copy_back, dim3((unsigned)((k * tt + 255) / 256)), dim3(256), 0, s, M, P, k, k, (int64_t)0,
                       0);
  }
  launch_copy(M.diag + k * tt, Xk, tt, s);
}

int64_t launch_lauum_contract(const TileMat& M, int64_t nreal, const double* xs, const double* ys, const double* av,
                              const double* qt, const double* cst, double* part, hipStream_t s) {
  const int64_t t64 = M.ts / TB, npt = t64 * (t64 + 1) / 2, ntr = M.NT * (M.NT + 1) / 2 * npt;
  hipLaunchKernelGGL(k_transpose_tiles, dim3((unsigned)ntr), dim3(256), 0, s, M, npt, ntr);
  const int B = lauum_tiles(nreal);
  const int64_t T = M.ts / (32 * B), nb = lauum_blocks(M.ts, M.NT, B);
  const int ch = xcd_chunk_size(B, (int)T, nb);
  EXG_BLOCKS(B, k_lauum_contract, xcd_chunk_grid(nb, ch), s, M, (int)T, nreal, xs, ys, av, qt, cst, part, nb, ch);
  return nb;
}

}  // namespace exg
