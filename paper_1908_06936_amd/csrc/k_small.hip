// Latency-bound pieces of the likelihood path:
//   * location ordering (bounding box, Morton keys, bitonic sort, gather);
//   * Cholesky + inverse of one 128 x 128 diagonal block held in LDS;
//   * the tile-by-tile forward and backward triangular solves;
//   * deterministic reductions for log det Sigma, z^T Sigma^-1 z, l(theta) and
//     the gradient partial sums;
//   * small fills and copies.
#include <float.h>

#include "common.h"
#include "launch.h"
#include "solve.h"

namespace exg {

// ------------------------------------------------------------------ ordering
// box[0..3] = min x, max x, min y, max y; box[4] = number of non-finite
// values among x, y (and z when given)
__global__ __launch_bounds__(1024) void k_bbox(const double* __restrict__ x, const double* __restrict__ y,
                                               const double* __restrict__ z, int64_t n, double* __restrict__ box) {
  __shared__ double red[5][1024];
  double mnx = DBL_MAX, mxx = -DBL_MAX, mny = DBL_MAX, mxy = -DBL_MAX, bad = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 1024) {
    const double a = x[i], b = y[i];
    const double c = z ? z[i] : 0.0;
    if (!(fabs(a) <= DBL_MAX) || !(fabs(b) <= DBL_MAX) || !(fabs(c) <= DBL_MAX)) bad += 1.0;
    mnx = fmin(mnx, a);
    mxx = fmax(mxx, a);
    mny = fmin(mny, b);
    mxy = fmax(mxy, b);
  }
  const int t = threadIdx.x;
  red[0][t] = mnx;
  red[1][t] = mxx;
  red[2][t] = mny;
  red[3][t] = mxy;
  red[4][t] = bad;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (t < s) {
      red[0][t] = fmin(red[0][t], red[0][t + s]);
      red[1][t] = fmax(red[1][t], red[1][t + s]);
      red[2][t] = fmin(red[2][t], red[2][t + s]);
      red[3][t] = fmax(red[3][t], red[3][t + s]);
      red[4][t] += red[4][t + s];
    }
    __syncthreads();
  }
  if (t < 5) box[t] = red[t][0];
}

__device__ __forceinline__ uint32_t spread16(uint32_t v) {
  v &= 0xffffu;
  v = (v | (v << 8)) & 0x00ff00ffu;
  v = (v | (v << 4)) & 0x0f0f0f0fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

// key = Morton code of the 16-bit quantised location (high 32 bits) and the
// caller index (low 32 bits), so keys are distinct and the order is unique.
// rank (may be null): cleared for k_rank.
__global__ void k_morton(const double* __restrict__ x, const double* __restrict__ y, int64_t n, int64_t P,
                         const double* __restrict__ box, uint64_t* __restrict__ keys, int32_t* __restrict__ rank) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  if (rank && i < n) rank[i] = 0;
  if (i >= n) {
    keys[i] = ~(uint64_t)0;
    return;
  }
  const double wx = box[1] - box[0], wy = box[3] - box[2];
  const double sx = wx > 0 ? 65535.999 / wx : 0.0, sy = wy > 0 ? 65535.999 / wy : 0.0;
  const uint32_t qx = (uint32_t)((x[i] - box[0]) * sx), qy = (uint32_t)((y[i] - box[2]) * sy);
  const uint32_t code = spread16(qx) | (spread16(qy) << 1);
  keys[i] = ((uint64_t)code << 32) | (uint64_t)i;
}

// one compare-exchange step of the bitonic network over the whole array
__global__ void k_bitonic_global(uint64_t* __restrict__ keys, int64_t P, int64_t j, int64_t k) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  const int64_t l = i ^ j;
  if (l <= i) return;
  const uint64_t a = keys[i], b = keys[l];
  const bool up = (i & k) == 0;
  if ((a > b) == up) {
    keys[i] = b;
    keys[l] = a;
  }
}

// the steps j = jmax..1 of stage k on chunks of 2048 keys in LDS; with
// kfrom = 2 it runs every stage k <= 2048 (a full sort of each chunk)
__global__ __launch_bounds__(1024) void k_bitonic_local(uint64_t* __restrict__ keys, int64_t kfrom, int64_t kto,
                                                         int64_t jmax) {
  __shared__ uint64_t s[2048];
  const int64_t base = (int64_t)blockIdx.x * 2048;
  const int t = threadIdx.x;
  s[t] = keys[base + t];
  s[t + 1024] = keys[base + t + 1024];
  __syncthreads();
  for (int64_t k = kfrom; k <= kto; k <<= 1) {
    for (int64_t j = (k == kfrom ? jmax : k >> 1); j > 0; j >>= 1) {
      // thread t handles the pair (i, i ^ j) with i having bit j clear
      const int64_t lo = ((t / j) * 2 * j) + (t % j);
      const int64_t hi = lo + j;
      const bool up = ((base + lo) & k) == 0;
      const uint64_t a = s[lo], b = s[hi];
      if ((a > b) == up) {
        s[lo] = b;
        s[hi] = a;
      }
      __syncthreads();
    }
  }
  keys[base + t] = s[t];
  keys[base + t + 1024] = s[t + 1024];
}

// sorted, zero-padded copies of x, y, z and the permutation (sorted -> caller)
__global__ void k_gather(const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
                         int64_t n, int64_t npad, const uint64_t* __restrict__ keys, double* __restrict__ xs,
                         double* __restrict__ ys, double* __restrict__ zs, int32_t* __restrict__ perm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npad) return;
  if (i < n) {
    const int64_t src = (int64_t)(keys[i] & 0xffffffffu);
    perm[i] = (int32_t)src;
    xs[i] = x[src];
    ys[i] = y[src];
    if (zs) zs[i] = z ? z[src] : 0.0;
  } else {
    perm[i] = -1;
    xs[i] = 0.0;
    ys[i] = 0.0;
    if (zs) zs[i] = 0.0;
  }
}

// rank[i] += number of keys among RT of them (block y's) below key i.  The keys
// are distinct, so the ranks are the places in the sorted order.  n^2 key
// comparisons, but one launch: the bitonic network's launches are bound by
// latency (n = 400: 28 us in one workgroup; n = 10,000: ten launches, 64 us).
constexpr int RT = 512;
__global__ __launch_bounds__(256) void k_rank(const uint64_t* __restrict__ keys, int64_t n,
                                              int32_t* __restrict__ rank) {
  __shared__ uint64_t sk[RT];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, j0 = (int64_t)blockIdx.y * RT;
  for (int q = threadIdx.x; q < RT; q += 256) sk[q] = j0 + q < n ? keys[j0 + q] : ~(uint64_t)0;
  __syncthreads();
  if (i >= n) return;
  const uint64_t key = keys[i];
  int c = 0;
#pragma unroll 8
  for (int q = 0; q < RT; ++q) c += sk[q] < key;
  if (c) atomicAdd(rank + i, c);
}

// k_gather from the ranks
__global__ void k_rank_gather(const double* __restrict__ x, const double* __restrict__ y,
                              const double* __restrict__ z, int64_t n, int64_t npad, const int32_t* __restrict__ rank,
                              double* __restrict__ xs, double* __restrict__ ys, double* __restrict__ zs,
                              int32_t* __restrict__ perm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npad) return;
  const int64_t o = i < n ? rank[i] : i;
  perm[o] = i < n ? (int32_t)i : -1;
  xs[o] = i < n ? x[i] : 0.0;
  ys[o] = i < n ? y[i] : 0.0;
  if (zs) zs[o] = i < n && z ? z[i] : 0.0;
}

// out[perm[i]] = v[i] for i < n
__global__ void k_scatter(const double* __restrict__ v, const int32_t* __restrict__ perm, int64_t n,
                          double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[perm[i]] = v[i];
}

// ------------------------------------------------ diagonal 128-block factor
// 1 / sqrt(d) from the hardware reciprocal square root (good to about 2^-24)
// and one third-order step y <- y + y e (1/2 + 3/8 e), e = 1 - d y^2, whose
// error is below e^3 ~ 2^-69: within an ulp or two of the rounded value.
__device__ __forceinline__ double rsqrt_ulp(double d) {
  const double y = __builtin_amdgcn_rsq(d);
  const double e = fma(-d * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// 1 / d likewise: y + y (e + e^2), e = 1 - d y
__device__ __forceinline__ double rcp_ulp(double d) {
  const double y = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, y, 1.0);
  return fma(y, fma(e, e, e), y);
}

// f(integral_constant<int, I>) for I = B, ..., E - 1
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Lane L of each row of 16 lanes, in every lane of the row (DPP row_newbcast,
// the form that double-precision instructions take).  A DPP source must not be
// written by one of the two instructions before; the compiler does not see
// into the block, hence the s_nop.
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
  double r;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v), "n"(L));
  return r;
}

// g[I] += bcast_I(p) gv, u[I] += bcast_I(p) uv for the rows I, ..., I + N - 1
// (N = 1 or 4), the broadcast folded into the multiply-add
template <int I, int N>
__device__ __forceinline__ void row_axpy(double p, double gv, double uv, double* g, double* u) {
#define EXG_AXPY(G, U, L)                                                       \
  "v_fmac_f64_dpp " G ", %[p], %[gv] row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp " U ", %[p], %[uv] row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t"
  if constexpr (N == 4) {
    asm("s_nop 1\n\t" EXG_AXPY("%0", "%1", "%[i0]") EXG_AXPY("%2", "%3", "%[i1]") EXG_AXPY("%4", "%5", "%[i2]")
            EXG_AXPY("%6", "%7", "%[i3]")
        : "+v"(g[I]), "+v"(u[I]), "+v"(g[I + 1]), "+v"(u[I + 1]), "+v"(g[I + 2]), "+v"(u[I + 2]), "+v"(g[I + 3]),
          "+v"(u[I + 3])
        : [p] "v"(p), [gv] "v"(gv), [uv] "v"(uv), [i0] "n"(I), [i1] "n"(I + 1), [i2] "n"(I + 2), [i3] "n"(I + 3));
  } else {
    static_assert(N == 1, "one row or four");
    asm("s_nop 1\n\t" EXG_AXPY("%0", "%1", "%[i0]")
        : "+v"(g[I]), "+v"(u[I])
        : [p] "v"(p), [gv] "v"(gv), [uv] "v"(uv), [i0] "n"(I));
  }
#undef EXG_AXPY
}

// the same for the rows B, ..., E - 1
template <int B, int E>
__device__ __forceinline__ void rows_axpy(double p, double gv, double uv, double* g, double* u) {
  if constexpr (E - B >= 4) {
    row_axpy<B, 4>(p, gv, uv, g, u);
    rows_axpy<B + 4, E>(p, gv, uv, g, u);
  } else if constexpr (B < E) {
    row_axpy<B, 1>(p, gv, uv, g, u);
    rows_axpy<B + 1, E>(p, gv, uv, g, u);
  }
}

// barrier of a workgroup that exchanges data through LDS only: global stores
// in flight are not waited for
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Cholesky of one 128 x 128 block and the inverse of its factor, by 16-wide
// steps k = 0..7 of row elimination on [A | I].  With A = L L^T, d_j = L_jj^2
// and X = L^-1, row j of the eliminated panel holds sqrt(d_j) L_cj in the
// columns c > j and sqrt(d_j) X_jc in the columns c <= j: the rows stay
// unscaled, so the serial chain of pivots needs no square root.
//   The 36 lower 16 x 16 blocks live in LDS.  Slot (r, c) holds A(r, c)^T until
//   step c consumes it and then T(r, c), the running right-hand side that
//   becomes X(r, c); the eliminated row panel k is kept in P.  Both halves of
//   the elimination share one update on MFMA, with P_c = 16 columns c of P:
//     A(r, c)^T -= P_c^T D^-1 P_r  (c > k),   T(r, c) -= P_r^T D^-1 P_c  (c <= k).
//   Waves 0 and 1 eliminate a row panel as one instruction stream with lanes
//   as columns: every lane carries one of the 128 panel columns and, in each
//   row of 16 lanes, a copy of the diagonal block's columns, so pivots and
//   multipliers are broadcast within 16 lanes by DPP moves, without LDS.
//   While they eliminate panel k, waves 2, 3, 6 and 7 (the SIMDs without an
//   eliminating wave) finish step k - 1's update and waves 4 and 5 write panel
//   k - 1, scaled, to global memory; between eliminations the eight waves bring
//   the eight blocks of the next panel up to date.
// What bounds it is the chain of 128 pivots (about 200 cycles each: a chain of
// 98 and the multiply-adds of the rows below) and, in steps 1 to 4, the updates
// beside it, which only two SIMDs can take: an FP64 MFMA holds up the FP64
// multiply-adds of its SIMD (4.6 -> 20.7 cycles).  Their blocks come from a table
// (one scalar load per step), fetched one ahead.  The LDS (95 KB) and 128
// registers per lane leave room for one trailing-update workgroup on the same
// CU.  It takes 27 us alone and 49 / 93 us on average in the factorisations of
// n = 10,000 / 22,500 (the wait for a CU included); with the blocks' indices
// formed on the way and a branch per row in the elimination's loads 32 us alone
// (two blocks at a time: 31), with one barrier per column (255 in all) 99 us.
// Writes L (zeros above the diagonal) over the block, X row by row to dinv
// (X(r, c) at 128 r + c, the order in which the panels leave LDS), the block's
// sum of 2 ln L_jj to *ldpart and the first failing global column
// (1-based) to *info with an atomic minimum.  The strict upper part of the
// input does not enter the result.
constexpr int PB = 16;           // step width
constexpr int PNB = BLK / PB;    // steps
constexpr int PLD = BLK + PB;  // row panel: 128 columns, then its 16 x 16 diagonal block; 16 columns of two rows
                               // a stride apart fall into different halves of the banks
constexpr int PSLOT = PB * PB;
constexpr int PSLOTS = PNB * (PNB + 1) / 2;
constexpr int POTRF_LDS = ((PSLOTS + 1) * PSLOT + PB * PLD + 6 * PB + BLK) * 8;  // bytes
static_assert(POTRF_LDS + GEMM_LDS * 8 <= 160 * 1024, "one trailing-update workgroup beside it");

// One block update as a scalar: slot, the column blocks of P of the scaled and
// the plain operand, and whether the slot starts from zero.
constexpr uint32_t potrf_job(int r, int c, int k) {
  return (uint32_t)((r * (r + 1) / 2 + c) | (c > k ? c : r) << 6 | (c > k ? r : c) << 9 | (c == k) << 12);
}
// The rest of step k - 1: rows r > k, columns c <= r except k, dealt in turn to
// the four waves that update beside the elimination of panel k; at most seven
// blocks for one wave, 16 bits each, then their number.
struct PotrfJobs {
  uint64_t j[PNB][4][2];
};
constexpr PotrfJobs potrf_jobs() {
  PotrfJobs t{};
  for (int k = 1; k < PNB; ++k) {
    int e = 0;
    for (int r = k + 1; r < PNB; ++r)
      for (int c = 0; c <= r; ++c)
        if (c != k) {
          const int v = e % 4, i = e / 4;
          t.j[k][v][i / 4] |= (uint64_t)potrf_job(r, c, k - 1) << (16 * (i % 4));
          t.j[k][v][1] += (uint64_t)1 << 48;
          ++e;
        }
  }
  return t;
}
__constant__ const PotrfJobs POTRF_JOBS = potrf_jobs();

// The LDS is dynamic so that the compiler keeps to 128 registers per lane: two
// waves per SIMD then fit beside a trailing-update workgroup's two.
__global__ __launch_bounds__(512, 4) void k_potrf_blk(
    double* __restrict__ A, int64_t lda, double* __restrict__ dinv, double* __restrict__ ldpart,
    unsigned long long* __restrict__ info, int64_t col0) {
  extern __shared__ double potrf_lds[];
  double* slots = potrf_lds;
  double* ident = slots + PSLOTS * PSLOT;  // the 16 x 16 identity
  double* P = ident + PSLOT;
  double* nrd = P + PB * PLD;  // -1 / d_j of the panels k (even, odd; a copy per eliminating wave)
  double* rsc = nrd + 4 * PB;  // 1 / L_jj (a copy per writing wave)
  double* piv = rsc + 2 * PB;  // d_j
  const int t = threadIdx.x;
  int lane = t & 63, l16 = lane & 15, q16 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  auto slot = [&](int r, int c) { return slots + (r * (r + 1) / 2 + c) * PSLOT; };
  {
    v4d v[5];
    int r = 0, c = 0;
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      const int b = min(8 * s + w, PSLOTS - 1);  // spare turns repeat the last block
      while ((r + 1) * (r + 2) / 2 <= b) ++r;
      c = b - r * (r + 1) / 2;
      const double* Ab = A + PB * r + (int64_t)(PB * c) * lda;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[s][q] = Ab[l16 + (4 * q + q16) * lda];
    }
    if (t < PSLOT) ident[t] = t / PB == t % PB ? 1.0 : 0.0;
#pragma unroll
    for (int s = 0; s < 5; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) slots[min(8 * s + w, PSLOTS - 1) * PSLOT + 64 * q + lane] = v[s][q];
  }
  // the lane's -1 / d_j of panel k
  auto upd_scale = [&](int k, v4d& nv) {
    const double* nd = nrd + 2 * PB * (k & 1) + q16;
#pragma unroll
    for (int q = 0; q < 4; ++q) nv[q] = nd[4 * q];
  };
  // the update of one block (potrf_job); T(r, k) starts in step k, from zero
  struct Upd {
    v4d acc, x, y;
  };
  auto upd_load = [&](uint32_t job, Upd& u) {
    const double* S = slots + (job & 63) * PSLOT + lane;
    const double* pl = P + q16 * PLD + l16;
    const double *px = pl + (job >> 6 & 7) * PB, *py = pl + (job >> 9 & 7) * PB;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u.x[q] = px[4 * q * PLD];
      u.y[q] = py[4 * q * PLD];
      u.acc[q] = S[64 * q];
    }
  };
  auto upd_apply = [&](uint32_t job, const v4d& nv, Upd& u) {
    double* S = slots + (job & 63) * PSLOT + lane;
    asm volatile("" : "+v"(u.acc));  // loaded in any case: a branch per element costs more
    if (job >> 12 & 1) u.acc = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) u.acc = mfma64(u.x[q] * nv[q], u.y[q], u.acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) S[64 * q] = u.acc[q];
  };
#pragma unroll 1
  for (int k = 0;; ++k) {
    // addresses are formed anew in each step, not kept in registers across them
    asm volatile("" : "+v"(lane), "+v"(l16), "+v"(q16));
    lds_barrier();  // panel k's blocks are up to date with step k - 1
    if (w < 2) {
      if (k == PNB) break;
      const int col = 64 * w + lane, cb = col >> 4;
      const double* src = (cb > k ? slot(cb, k) : cb == k ? ident : slot(k, cb)) + l16;
      const double* dsrc = slot(k, k) + l16;
      double* nd = nrd + 2 * PB * (k & 1) + PB * w;
      double u[PB], g[PB];  // the lane's panel column, its copy of a diagonal column
#pragma unroll
      for (int j = 0; j < PB; ++j) {
        g[j] = dsrc[j * PB];
        u[j] = src[j * PB];
      }
      static_for<0, PB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const double d = row_bcast<j>(g[j]);
        const double r = -rcp_ulp(d), gv = g[j] * r, uv = u[j] * r;  // -row j / d_j
        nd[j] = r;
        if constexpr (j + 1 < PB) {
          row_axpy<j + 1, 1>(g[j], gv, uv, g, u);  // the next pivot's row first
          rows_axpy<j + 2, PB>(g[j], gv, uv, g, u);
        }
      });
      lds_barrier();  // nobody reads panel k - 1 any more
#pragma unroll
      for (int j = 0; j < PB; ++j) P[j * PLD + col] = u[j];
      if (lane < PB) {  // half of the diagonal block's rows each
        double* Pd = P + BLK + lane;
        if (w == 0) {
#pragma unroll
          for (int j = 0; j < PB / 2; ++j) Pd[j * PLD] = g[j];
        } else {
#pragma unroll
          for (int j = PB / 2; j < PB; ++j) Pd[j * PLD] = g[j];
        }
      }
    } else if (w == 4 || w == 5) {
      if (k > 0) {  // panel k - 1 to global memory
        const int col = 64 * (w - 4) + lane, cb = col >> 4;
        const double pv = P[l16 * PLD + BLK + l16], sd = sqrt(pv);  // pivot l16
        double* rs = rsc + PB * (w - 4);
        rs[l16] = rsqrt_ulp(pv);
        const int d = col - PB * (k - 1);  // > j below the diagonal
        double* Ak = A + PB * (k - 1) * lda + col;
        double* X = dinv + PB * (k - 1) * BLK + col;
        // L takes its diagonal block's columns from the panel's tail
        const double *Pc = P + (cb == k - 1 ? BLK + l16 : col), *Px = P + col;
#pragma unroll
        for (int j = 0; j < PB; ++j) {
          const double rj = rs[j];
          double v = Pc[j * PLD] * rj, x = Px[j * PLD] * rj;
          asm volatile("" : "+v"(v), "+v"(x));  // selected, not branched over
          Ak[(uint32_t)j * (uint32_t)lda] = d > j ? v : 0.0;
          X[j * BLK] = cb < k ? x : 0.0;
        }
        if (cb == k - 1) {
          Ak[(uint32_t)l16 * (uint32_t)lda] = sd;
          piv[col] = pv;
          if (!(pv > 0.0) || !(pv <= DBL_MAX)) atomicMin(info, (unsigned long long)(col0 + col + 1));
        }
      }
      if (k == PNB) break;
      lds_barrier();
    } else {
      if (k == PNB) break;
      // the wave's share of the rest of step k - 1; each block's operands are read
      // while the products of the one before run
      const int v = (w & 1) + 2 * (w >> 2);
      uint64_t j0 = POTRF_JOBS.j[k][v][0], j1 = POTRF_JOBS.j[k][v][1];
      int left = (int)(j1 >> 48);
      if (left > 0) {
        auto next = [&]() {
          const uint32_t job = (uint32_t)j0 & 0xffff;
          j0 = j0 >> 16 | j1 << 48;
          j1 >>= 16;
          return job;
        };
        v4d nv;
        Upd a, b;
        upd_scale(k - 1, nv);
        uint32_t ja = next(), jb;
        upd_load(ja, a);
#pragma unroll 1
        for (;;) {
          jb = left > 1 ? next() : ja;  // the last one's reads are not used
          upd_load(jb, b);
          upd_apply(ja, nv, a);
          if (--left == 0) break;
          ja = left > 1 ? next() : jb;
          upd_load(ja, a);
          upd_apply(jb, nv, b);
          if (--left == 0) break;
        }
      }
      lds_barrier();
    }
    // the blocks of panel k + 1, one per wave
    const int r = w <= k + 1 ? k + 1 : w, c = w <= k + 1 ? w : k + 1;
    const uint32_t job = potrf_job(r, c, k);
    lds_barrier();  // panel k eliminated
    if (k < PNB - 1) {
      v4d nv;
      Upd a;
      upd_load(job, a);
      upd_scale(k, nv);
      upd_apply(job, nv, a);
    }
  }
  // 2 sum ln L_jj = sum ln d_j, in a fixed order
  lds_barrier();
  if (w == 0) {
    const double s = wave_sum(log(piv[lane]) + log(piv[64 + lane]));
    if (t == 0) *ldpart = s;
  }
}

// factor blocks that lie in the padding (the identity): their inverses (row
// by row) and log-determinant parts, block blockIdx.x of dinv / ldpart
__global__ __launch_bounds__(256) void k_pad_blk(double* __restrict__ dinv, double* __restrict__ ldpart) {
  double* X = dinv + (int64_t)blockIdx.x * BLK * BLK;
  for (int e = threadIdx.x; e < BLK * BLK; e += 256) X[e] = e / BLK == e % BLK ? 1.0 : 0.0;
  if (threadIdx.x == 0) ldpart[blockIdx.x] = 0.0;
}

// ------------------------------------------------------- triangular solves
// Forward substitution on one diagonal tile, y = L_kk^-1 rhs, by the 128-blocks
// and their inverses (nblk blocks with real rows; y = 0 on the others): one
// workgroup, bound by what one CU reads (128 KB a block, most of it written on
// other XCDs): 21 us for four blocks, 36 for six (23 and 37 with the zero half of
// the inverses read too).  58 registers, so that it fits on a CU beside a
// trailing-update workgroup; fetching the next block ahead took 96, 32 us alone,
// and waited 2 ms a tile for a free CU at n = 40,000.
__global__ __launch_bounds__(1024) void k_tile_fwd(const double* __restrict__ L, int64_t ts,
                                                   const double* __restrict__ dinv, const double* __restrict__ rhs,
                                                   double* __restrict__ y, int nblk) {
  extern __shared__ double fy[];  // ts (y), 128 (right-hand side of a block), 1024
  double* sb = fy + ts;
  double* red = sb + BLK;
  const int t = threadIdx.x, r = t & 127, h = t >> 7;
  for (int q = t; q < ts; q += 1024) fy[q] = 0.0;
  __syncthreads();
  for (int c = 0; c < nblk; ++c) {
    const double* Lr = L + c * BLK + r;
    double s = 0.0;
    int q = h;
    for (; q < c * BLK; q += 128) {  // 16 loads in flight per thread
      double v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = Lr[(int64_t)(q + 8 * e) * ts];
#pragma unroll
      for (int e = 0; e < 16; ++e) s += v[e] * fy[q + 8 * e];
    }
    red[t] = s;
    __syncthreads();
    if (t < BLK) {
      double a = 0.0;
#pragma unroll
      for (int g = 0; g < 8; ++g) a += red[g * BLK + t];
      sb[t] = rhs[c * BLK + t] - a;
    }
    __syncthreads();
    // y_c = X s, X row by row: eight lanes per row
    {
      const int row = t >> 3, l = t & 7, rb = __builtin_amdgcn_readfirstlane(t >> 6);  // X is lower triangular
      const double* X = dinv + ((int64_t)c * BLK + row) * BLK;
      double a = 0.0;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (e <= rb) a += X[8 * e + l] * sb[8 * e + l];
      a += __shfl_xor(a, 4, 8);
      a += __shfl_xor(a, 2, 8);
      a += __shfl_xor(a, 1, 8);
      if (l == 0) fy[c * BLK + row] = a;
    }
    __syncthreads();
  }
  for (int q = t; q < ts; q += 1024) y[q] = fy[q];
}

// rhs_i -= L_ik y_k for the 128-row blocks g0 <= g < gmax below tile k.
__global__ __launch_bounds__(SOLVE_THREADS) void k_gemv_fwd(TileMat M, int64_t k, int64_t g0,
                                                           const double* __restrict__ yk, double* __restrict__ rhs) {
  const int64_t ts = M.ts;
  extern __shared__ double sy[];  // ts + SOLVE_THREADS
  double* red = sy + ts;
  const int T = (int)(ts / BLK);
  const int64_t g = g0 + blockIdx.x;
  const int64_t i = g / T;
  const int u = (int)(g % T);
  const int t = threadIdx.x;
  for (int q = t; q < ts; q += SOLVE_THREADS) sy[q] = yk[q];
  __syncthreads();
  const double* L = tptr(M, i, k) + u * BLK;
  const double s = slab_rowdot([=](int r, int c) { return L[r + (int64_t)c * ts]; }, sy, (int)ts, red);
  if (t < BLK) rhs[i * ts + u * BLK + t] -= s;
}

// out = X b on one diagonal tile, X lower triangular (explicit inverse);
// one 128-row block per workgroup
__global__ __launch_bounds__(SOLVE_THREADS) void k_diag_apply_n(const double* __restrict__ X, int64_t ts,
                                                               const double* __restrict__ b,
                                                               double* __restrict__ out) {
  __shared__ double sb[4096];  // ts <= 4096
  __shared__ double red[SOLVE_THREADS];
  const int rb = blockIdx.x, t = threadIdx.x;
  const int cmax = (rb + 1) * BLK;  // X(row, c) = 0 for c >= cmax
  for (int q = t; q < cmax; q += SOLVE_THREADS) sb[q] = b[q];
  __syncthreads();
  const double* Xr = X + rb * BLK;
  const double s = slab_rowdot([=](int r, int c) { return Xr[r + (int64_t)c * ts]; }, sb, cmax, red);
  if (t < BLK) out[rb * BLK + t] = s;
}

// out = X^T b on one diagonal tile, X lower triangular; one 128-column block
// per workgroup, eight columns per wave (lanes run down the columns)
__global__ __launch_bounds__(SOLVE_THREADS) void k_diag_apply_t(const double* __restrict__ X, int64_t ts,
                                                               const double* __restrict__ b,
                                                               double* __restrict__ out) {
  const int64_t col0 = (int64_t)blockIdx.x * BLK + 8 * (threadIdx.x >> 6);
  double s[8];
  wave_coldot8([=](int64_t r, int64_t c) { return X[r + c * ts]; }, b, col0, true, ts, s);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) out[col0 + e] = s[e];
  }
}

// rhs_j -= L_kj^T a_k over the 128-column blocks of the tiles j < k (one
// block per workgroup)
__global__ __launch_bounds__(SOLVE_THREADS) void k_gemv_bwd(TileMat M, int64_t k, const double* __restrict__ ak,
                                                           double* __restrict__ rhs) {
  const int64_t ts = M.ts;
  const int T = (int)(ts / BLK);
  const int64_t cb = blockIdx.x;
  const int64_t j = cb / T;
  const int64_t col0 = (cb % T) * BLK + 8 * (threadIdx.x >> 6);
  const double* L = tptr(M, k, j);
  double s[8];
  wave_coldot8([=](int64_t r, int64_t c) { return L[r + c * ts]; }, ak, col0, false, ts, s);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) rhs[j * ts + col0 + e] -= s[e];
  }
}

// w = L e on the lower tiles (diagonal tiles read up to their diagonal only).
// Workgroup (g, h): 128-row block g against the tiles j = h, h + H, ... of its
// tile row; its sums go to part[h npad + row], added in order of h by
// k_trmv_sum.  Bound by reading L once (n = 22,500: 2.0 GB, 0.39 ms; one
// workgroup of 256 threads per row block and two loads in flight per thread
// took 4.55 ms).
__global__ __launch_bounds__(SOLVE_THREADS) void k_trmv_lower(TileMat M, const double* __restrict__ e,
                                                             double* __restrict__ part, int64_t npad) {
  const int64_t ts = M.ts;
  extern __shared__ double se[];  // ts + SOLVE_THREADS
  double* red = se + ts;
  const int T = (int)(ts / BLK);
  const int64_t g = blockIdx.x, i = g / T;
  const int u = (int)(g % T), t = threadIdx.x;
  double s = 0.0;
  for (int64_t j = blockIdx.y; j <= i; j += gridDim.y) {
    for (int q = t; q < ts; q += SOLVE_THREADS) se[q] = e[j * ts + q];
    __syncthreads();
    const double* L = tptr(M, i, j) + u * BLK;
    if (j < i) {
      s += slab_rowdot([=](int r, int c) { return L[r + (int64_t)c * ts]; }, se, (int)ts, red);
    } else {
      const int r = t & 127, row = u * BLK + r;
      double a = 0.0;
#pragma unroll 4
      for (int c = t >> 7; c <= row; c += 8) a += L[r + (int64_t)c * ts] * se[c];
      red[t] = a;
      __syncthreads();
      if (t < BLK) {
#pragma unroll
        for (int h = 0; h < 8; ++h) s += red[h * BLK + t];
      }
    }
    __syncthreads();
  }
  if (t < BLK) part[blockIdx.y * npad + g * BLK + t] = s;
}

__global__ __launch_bounds__(256) void k_trmv_sum(const double* __restrict__ part, int64_t npad, int H, int64_t nrows,
                                                  double* __restrict__ w) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= nrows) return;
  double s = 0.0;
  for (int h = 0; h < H; ++h) s += part[h * npad + r];
  w[r] = s;
}

// ------------------------------------------------------------- reductions
// the first failed pivot and the bounding box / input check behind the results,
// so that one copy brings everything to the host
__device__ __forceinline__ void append_status(double* out, const unsigned long long* info, const double* box) {
  out[OUT_INFO] = __longlong_as_double((long long)*info);
  for (int q = 0; q < 5; ++q) out[OUT_BOX + q] = box[q];
}

// out[0] = l, out[1] = log det, out[2] = y^T y  (eq. 2 with the true n)
__global__ __launch_bounds__(256) void k_finalize_loglik(const double* __restrict__ yv, int64_t n,
                                                         const double* __restrict__ ldpart, int64_t nld,
                                                         const unsigned long long* __restrict__ info,
                                                         const double* __restrict__ box, double* __restrict__ out) {
  __shared__ double red[2 * 256];
  double v[2] = {0.0, 0.0};
  for (int64_t i = threadIdx.x; i < n; i += 256) v[0] += yv[i] * yv[i];
  for (int64_t i = threadIdx.x; i < nld; i += 256) v[1] += ldpart[i];
  block_sum<2>(v, red);
  if (threadIdx.x == 0) {
    const double q = v[0], ld = v[1];
    out[0] = -0.5 * ((double)n * 1.8378770664093454836 + ld + q);
    out[1] = ld;
    out[2] = q;
    append_status(out, info, box);
  }
}

// eq. (2) from log det Sigma (sum of ldpart) and the quadratic form
// z^T Sigma^-1 z = z^T a with a = Sigma^-1 z (refined solve)
__global__ __launch_bounds__(256) void k_finalize_loglik_za(const double* __restrict__ zs, const double* __restrict__ av,
                                                            int64_t n, const double* __restrict__ ldpart, int64_t nld,
                                                            const unsigned long long* __restrict__ info,
                                                            const double* __restrict__ box,
                                                            double* __restrict__ out) {
  __shared__ double red[2 * 256];
  double v[2] = {0.0, 0.0};
  for (int64_t i = threadIdx.x; i < n; i += 256) v[0] += zs[i] * av[i];
  for (int64_t i = threadIdx.x; i < nld; i += 256) v[1] += ldpart[i];
  block_sum<2>(v, red);
  if (threadIdx.x == 0) {
    const double q = v[0], ld = v[1];
    out[0] = -0.5 * ((double)n * 1.8378770664093454836 + ld + q);
    out[1] = ld;
    out[2] = q;
    append_status(out, info, box);
  }
}

// y = a + d
__global__ void k_add2_f64(double* __restrict__ y, const double* __restrict__ a, const double* __restrict__ d,
                           int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a[i] + d[i];
}

// Refinement bookkeeping on the device (no host round trip): nrm[0] holds
// the squared norm of the accepted residual.  init: nrm[0] = |r|^2.  trial:
// flag = |r_try|^2 < nrm[0], and then nrm[0] = |r_try|^2.
__global__ __launch_bounds__(1024) void k_resid_norm(const double* __restrict__ r, int64_t n, double* __restrict__ nrm,
                                                     int trial) {
  __shared__ double red[1024];
  double v[1] = {0.0};
  for (int64_t i = threadIdx.x; i < n; i += 1024) v[0] += r[i] * r[i];
  block_sum<1>(v, red);
  if (threadIdx.x == 0) {
    if (!trial) {
      nrm[0] = v[0];
    } else {
      const bool better = v[0] < nrm[0];
      nrm[1] = better ? 1.0 : 0.0;
      if (better) nrm[0] = v[0];
    }
  }
}

// accept the trial step when the flag is set: a <- a_try, r <- r_try
__global__ void k_refine_select(double* __restrict__ a, const double* __restrict__ a_try, double* __restrict__ r,
                                const double* __restrict__ r_try, const double* __restrict__ nrm, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && nrm[1] != 0.0) {
    a[i] = a_try[i];
    r[i] = r_try[i];
  }
}

// out[0..2] = sum over parts of part[3 p + k]
__global__ __launch_bounds__(256) void k_finalize_grad(const double* __restrict__ part, int64_t nparts,
                                                       double* __restrict__ out) {
  __shared__ double red[3 * 256];
  double v[3] = {0.0, 0.0, 0.0};
  for (int64_t p = threadIdx.x; p < nparts; p += 256) {
    v[0] += part[3 * p];
    v[1] += part[3 * p + 1];
    v[2] += part[3 * p + 2];
  }
  block_sum<3>(v, red);
  if (threadIdx.x == 0) {
    out[0] = v[0];
    out[1] = v[1];
    out[2] = v[2];
  }
}

// ------------------------------------------------------------ fills/copies
__global__ void k_copy_f64(double* __restrict__ dst, const double* __restrict__ src, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// dst[k] = lower part of diagonal tile k (zeros above the diagonal), k < NT
__global__ void k_copy_diag_lower(double* __restrict__ dst, const double* __restrict__ diag, int64_t ts, int64_t NT) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tt = ts * ts;
  if (e >= NT * tt) return;
  const int64_t k = e / tt, q = e % tt;
  const int64_t r = q % ts, c = q / ts;
  dst[e] = (r >= c) ? diag[k * tt + q] : 0.0;
}

// dst[k] block (c, c) = dinv[k][c] (stored row by row) for every diagonal tile k
__global__ void k_put_dinv(double* __restrict__ dst, const double* __restrict__ dinv, int64_t ts, int64_t NT, int c) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= NT * BLK * BLK) return;
  const int T = (int)(ts / BLK);
  const int64_t k = e / (BLK * BLK), q = e % (BLK * BLK);
  const int cc = (int)(q % BLK), r = (int)(q / BLK);
  dst[k * ts * ts + (int64_t)c * BLK + r + ((int64_t)c * BLK + cc) * ts] = dinv[(k * T + c) * BLK * BLK + q];
}

// ------------------------------------------------------------- launchers
static inline unsigned nb(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

void launch_sort_locations(const double* x, const double* y, const double* z, int64_t n, int64_t npad, int64_t P,
                           double* box, uint64_t* keys, int32_t* rank, double* xs, double* ys, double* zs,
                           int32_t* perm, hipStream_t s) {
  hipLaunchKernelGGL(k_bbox, dim3(1), dim3(1024), 0, s, x, y, z, n, box);
  // ranks by counting up to 16,384 points (20 us there; the bitonic network 75 us)
  if (n <= 16384) {
    hipLaunchKernelGGL(k_morton, dim3(nb(n, 256)), dim3(256), 0, s, x, y, n, n, box, keys, rank);
    hipLaunchKernelGGL(k_rank, dim3(nb(n, 256), nb(n, RT)), dim3(256), 0, s, keys, n, rank);
    hipLaunchKernelGGL(k_rank_gather, dim3(nb(npad, 256)), dim3(256), 0, s, x, y, z, n, npad, rank, xs, ys, zs, perm);
    return;
  }
  hipLaunchKernelGGL(k_morton, dim3(nb(P, 256)), dim3(256), 0, s, x, y, n, P, box, keys, (int32_t*)nullptr);
  // P is a power of two >= 2048
  hipLaunchKernelGGL(k_bitonic_local, dim3((unsigned)(P / 2048)), dim3(1024), 0, s, keys, (int64_t)2, (int64_t)2048,
                     (int64_t)1);
  for (int64_t k = 4096; k <= P; k <<= 1) {
    int64_t j = k >> 1;
    for (; j >= 2048; j >>= 1)
      hipLaunchKernelGGL(k_bitonic_global, dim3(nb(P, 256)), dim3(256), 0, s, keys, P, j, k);
    hipLaunchKernelGGL(k_bitonic_local, dim3((unsigned)(P / 2048)), dim3(1024), 0, s, keys, k, k, j);
  }
  hipLaunchKernelGGL(k_gather, dim3(nb(npad, 256)), dim3(256), 0, s, x, y, z, n, npad, keys, xs, ys, zs, perm);
}

void launch_scatter(const double* v, const int32_t* perm, int64_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_scatter, dim3(nb(n, 256)), dim3(256), 0, s, v, perm, n, out);
}

void launch_potrf_blk(double* A, int64_t lda, double* dinv, double* ldpart, unsigned long long* info, int64_t col0,
                      hipStream_t s) {
  hipLaunchKernelGGL(k_potrf_blk, dim3(1), dim3(512), POTRF_LDS, s, A, lda, dinv, ldpart, info, col0);
}

void launch_pad_blocks(double* dinv, double* ldpart, int64_t count, hipStream_t s) {
  if (count > 0) hipLaunchKernelGGL(k_pad_blk, dim3((unsigned)count), dim3(256), 0, s, dinv, ldpart);
}

void launch_solve_tile(const TileMat& M, int64_t k, const double* dinv_k, int64_t nreal, const double* rhs, double* y,
                       hipStream_t s) {
  const int64_t ts = M.ts, T = ts / BLK, gmax = (nreal + BLK - 1) / BLK;
  const int nblk = (int)(gmax - k * T < T ? gmax - k * T : T);
  hipLaunchKernelGGL(k_tile_fwd, dim3(1), dim3(1024), (size_t)(ts + BLK + 1024) * sizeof(double), s,
                     (const double*)(M.diag + k * ts * ts), ts, dinv_k, rhs + k * ts, y + k * ts, nblk);
}

void launch_solve_below(const TileMat& M, int64_t k, int64_t nreal, const double* y, double* rhs, hipStream_t s) {
  const int64_t ts = M.ts, T = ts / BLK;
  int64_t gmax = (nreal + BLK - 1) / BLK;  // row blocks holding real rows
  if (M.dst > 0 && gmax > (k + M.dst) * T) gmax = (k + M.dst) * T;  // zero below the band
  const int64_t g0 = (k + 1) * T;
  if (gmax > g0)
    hipLaunchKernelGGL(k_gemv_fwd, dim3((unsigned)(gmax - g0)), dim3(SOLVE_THREADS),
                       (size_t)(ts + SOLVE_THREADS) * sizeof(double), s, M, k, g0, y + k * ts, rhs);
}

void launch_diag_apply_n(const double* Xk, int64_t ts, const double* b, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_apply_n, dim3((unsigned)(ts / BLK)), dim3(SOLVE_THREADS), 0, s, Xk, ts, b, out);
}

void launch_diag_apply_t(const double* Xk, int64_t ts, const double* b, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_apply_t, dim3((unsigned)(ts / BLK)), dim3(SOLVE_THREADS), 0, s, Xk, ts, b, out);
}

void launch_trsv_bwd(const TileMat& M, const double* Xd, double* rhs, double* a, hipStream_t s) {
  const int64_t ts = M.ts, NT = M.NT;
  const int T = (int)(ts / BLK);
  for (int64_t k = NT - 1; k >= 0; --k) {
    launch_diag_apply_t(Xd + k * ts * ts, ts, rhs + k * ts, a + k * ts, s);
    if (k > 0)
      hipLaunchKernelGGL(k_gemv_bwd, dim3((unsigned)(k * T)), dim3(SOLVE_THREADS), 0, s, M, k, a + k * ts, rhs);
  }
}

void launch_trmv_lower(const TileMat& M, int64_t nreal, const double* e, double* part, double* w, hipStream_t s) {
  const int64_t gmax = (nreal + BLK - 1) / BLK, npad = M.NT * M.ts;
  // about 1,024 workgroups, where there are tiles for them
  int64_t H = (1024 + gmax - 1) / gmax;
  H = H < M.NT ? H : M.NT;
  H = H < TRMV_PARTS ? H : TRMV_PARTS;
  hipLaunchKernelGGL(k_trmv_lower, dim3((unsigned)gmax, (unsigned)H), dim3(SOLVE_THREADS),
                     (M.ts + SOLVE_THREADS) * sizeof(double), s, M, e, part, npad);
  hipLaunchKernelGGL(k_trmv_sum, dim3((unsigned)((gmax * BLK + 255) / 256)), dim3(256), 0, s, (const double*)part,
                     npad, (int)H, gmax * BLK, w);
}

void launch_finalize_loglik(const double* yv, int64_t n, const double* ldpart, int64_t nld,
                            const unsigned long long* info, const double* box, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize_loglik, dim3(1), dim3(256), 0, s, yv, n, ldpart, nld, info, box, out);
}

void launch_finalize_loglik_za(const double* zs, const double* av, int64_t n, const double* ldpart, int64_t nld,
                               const unsigned long long* info, const double* box, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize_loglik_za, dim3(1), dim3(256), 0, s, zs, av, n, ldpart, nld, info, box, out);
}

void launch_add2(double* y, const double* a, const double* d, int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_add2_f64, dim3(nb(n, 256)), dim3(256), 0, s, y, a, d, n);
}

void launch_resid_norm(const double* r, int64_t n, double* nrm, int trial, hipStream_t s) {
  hipLaunchKernelGGL(k_resid_norm, dim3(1), dim3(1024), 0, s, r, n, nrm, trial);
}

void launch_refine_select(double* a, const double* a_try, double* r, const double* r_try, const double* nrm,
                          int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_refine_select, dim3(nb(n, 256)), dim3(256), 0, s, a, a_try, r, r_try, nrm, n);
}

void launch_finalize_grad(const double* part, int64_t nparts, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize_grad, dim3(1), dim3(256), 0, s, part, nparts, out);
}

void launch_copy(double* dst, const double* src, int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_copy_f64, dim3(nb(n, 256)), dim3(256), 0, s, dst, src, n);
}

void launch_copy_diag_lower(double* dst, const double* diag, int64_t ts, int64_t NT, hipStream_t s) {
  hipLaunchKernelGGL(k_copy_diag_lower, dim3(nb(NT * ts * ts, 256)), dim3(256), 0, s, dst, diag, ts, NT);
}

void launch_put_dinv(double* dst, const double* dinv, int64_t ts, int64_t NT, int c, hipStream_t s) {
  hipLaunchKernelGGL(k_put_dinv, dim3(nb(NT * BLK * BLK, 256)), dim3(256), 0, s, dst, dinv, ts, NT, c);
}


}  // namespace exg
