// Covariance generation (paper eq. 3) on the device: per-theta quadrature
// tables, the packed lower-tile matrix used by the factorisation, and a dense
// n x n matrix in the caller's order (used to check generation entry by entry).
#include "common.h"
#include "launch.h"
#include "matern_dev.h"

namespace exg {

// psi(z), z > 0: shift with psi(z) = psi(z + 1) - 1/z until z >= 12, then
// psi(z) ~ ln z - 1/(2z) - sum_k B_2k / (2k z^2k)  (DLMF 5.5.2, 5.11.2).
__device__ double dev_digamma(double z) {
  double acc = 0.0;
  while (z < 12.0) {
    acc -= 1.0 / z;
    z += 1.0;
  }
  const double iz2 = 1.0 / (z * z);
  const double s =
      iz2 * (1.0 / 12 - iz2 * (1.0 / 120 - iz2 * (1.0 / 252 - iz2 * (1.0 / 240 - iz2 * (1.0 / 132 - iz2 * (691.0 / 32760))))));
  return acc + log(z) - 0.5 / z - s;
}

// One thread per (bucket m, node k): node t = k h_m, weights of the three
// integrands including the trapezoidal end weight h/2 at t = 0.
// info (may be null): the first failed pivot, reset for the factorisation.
__global__ void k_quad_table(double s2, double beta, double nu, double metric, double nugget,
                             double* __restrict__ qt, double* __restrict__ cst, unsigned long long* info) {
  const int m = blockIdx.x, k = threadIdx.x;
  const double h = 0.1 * exp2(-0.5 * m);
  const double t = k * h;
  const double sh = sinh(0.5 * t);
  const double w = (k == 0) ? 0.5 * h : h;
  double* q = qt + ((int64_t)m * QNK + k) * QW;
  q[0] = 2.0 * sh * sh;  // cosh t - 1 without cancellation
  q[1] = t;
  q[2] = w * cosh(nu * t);
  q[3] = w * cosh((nu - 1.0) * t);
  q[4] = w * t * sinh(nu * t);
  if (m == 0 && k == 0) {
    const double c = exp((1.0 - nu) * 0.69314718055994530942 - lgamma(nu));
    cst[C_S2] = s2;
    cst[C_BETA] = beta;
    cst[C_NU] = nu;
    cst[C_C] = c;
    cst[C_PSI] = dev_digamma(nu);
    cst[C_S2C] = s2 * c;
    cst[C_METRIC] = metric;
    cst[C_NUG] = nugget;
    cst[C_RBETA] = 1.0 / beta;
    int se, be;
    frexp(s2, &se);
    frexp(beta, &be);
    cst[C_S2E] = __longlong_as_double(se);
    cst[C_D1E] = __longlong_as_double(se - be);
    if (info) *info = ~0ull;
  }
}

// CH_POW.t[n][k]: the coefficient of t^k in the Chebyshev polynomial T_n
struct ChebPowers {
  int t[CH_N][CH_N];
};
constexpr ChebPowers cheb_powers() {
  ChebPowers p{};
  p.t[0][0] = p.t[1][1] = 1;
  for (int n = 2; n < CH_N; ++n)
    for (int k = 0; k <= n; ++k) p.t[n][k] = (k > 0 ? 2 * p.t[n - 1][k - 1] : 0) - p.t[n - 2][k];
  return p;
}
__constant__ const ChebPowers CH_POW = cheb_powers();

// Tables of u0, u1, u2 on segment blockIdx.x of ln x (see matern_dev.h): the
// functions at the 13 Chebyshev points by the quadrature; stored per function
// are factors with its value at the segment centre (the middle point, t = 0) and
// the coefficients of ln(u / u_centre) in powers of t, from the Chebyshev
// coefficients c_k = (2/N) sum_j d_j cos(pi k (j + 1/2) / N).  Runs after
// k_quad_table.  Bound by latency: 16 lanes share the exponentials of the up to
// 400 nodes of one point, one thread per function then adds them in node order
// (so the table does not depend on the split), and the logarithms and cosines
// are formed once, one per thread.  With a thread per point and per
// coefficient: 68 us.
__global__ __launch_bounds__(256) void k_cheb_table(double* __restrict__ qt, const double* __restrict__ cst) {
  constexpr int LP = 16;  // lanes per point
  __shared__ double fv[3][CH_N], lg[3][CH_N], ch[3][CH_N], cs[CH_N][CH_N], ex[CH_N][QNK + 1], xs[CH_N];
  __shared__ int nk[CH_N];
  const int seg = blockIdx.x, t = threadIdx.x;
  const double pi = 3.14159265358979323846;
  const double nu = cst[C_NU], cnu = cst[C_C];
  int e;
  const double sc = frexp(cst[C_S2], &e) * cnu, bm = frexp(cst[C_BETA], &e);  // the mantissas'
  if (t < CH_N * CH_N) cs[t / CH_N][t % CH_N] = cos(pi * (t / CH_N) * (t % CH_N + 0.5) / CH_N);
  if (t < CH_N * LP) {
    const int j = t / LP, l = t % LP;
    const double tj = cos(pi * (j + 0.5) / CH_N);
    const double x = exp(CH_SLO + (seg + 0.5 * (tj + 1.0)) * CH_DS);
    const double* q = qt + (quad_bucket(x) * QNK + l) * QW;
    int k = l;
    for (; k < QNK; k += LP, q += LP * QW) {
      const double c = q[0];
      if (k > 0 && x * c - nu * q[1] > QCUT + 5.0) break;
      ex[j][k] = exp(-x * c);
    }
    for (int o = LP / 2; o > 0; o >>= 1) k = min(k, __shfl_xor(k, o, LP));
    if (l == 0) xs[j] = x, nk[j] = min(k, QNK);
  }
  __syncthreads();
  if (t < 3 * CH_N) {
    const int f = t / CH_N, j = t % CH_N, n = nk[j];
    const double x = xs[j], xn = pow(x, nu);
    const double* q = qt + quad_bucket(x) * QNK * QW + 2 + f;
    double a = 0.0;
    int k = 0;
    for (; k + 8 <= n; k += 8) {
      double v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = q[(k + e) * QW];
#pragma unroll
      for (int e = 0; e < 8; ++e) a += ex[j][k + e] * v[e];
    }
    for (; k < n; ++k) a += ex[j][k] * q[k * QW];
    fv[f][j] = f == 1 ? xn * x * a : xn * a;
  }
  __syncthreads();
  if (t < 3 * CH_N) lg[t / CH_N][t % CH_N] = log(fv[t / CH_N][t % CH_N] / fv[t / CH_N][CH_MID]);
  __syncthreads();
  if (t < 3 * CH_N) {
    const int f = t / CH_N, k = t % CH_N;
    double c = 0.0;
    for (int q = 0; q < CH_N; ++q) c += lg[f][q] * cs[k][q];
    ch[f][k] = c * (2.0 / CH_N);
  }
  __syncthreads();
  if (t < 3 * 16) {
    const int f = t >> 4, k = t & 15;
    const double A = sc * fv[f][CH_MID];
    double c = 0.0;
    if (k < CH_A) {  // coefficient of t^(k + 1), the small terms first
      for (int q = CH_N - 1; q > k; --q) c = fma((double)CH_POW.t[q][k + 1], ch[f][q], c);
    } else if (k == CH_A) {
      c = f == 1 ? A / bm : A;
    } else if (k == CH_A + 1) {
      c = cnu * fv[f][CH_MID];
    }
    if (k < CH_STRIDE) qt[QT_CHEB_OFF + f * CH_TAB + seg * CH_STRIDE + k] = c;
  }
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Lower tiles of the padded covariance.  One 256-thread block per 128 x 128
// block (u, v) of tile (I, J); blocks above the diagonal of a diagonal tile
// are not needed by any later step and are skipped.  Mixed precision (tag !=
// NULL): diagonal tiles FP64, off-diagonal tiles FP32 (tag 0) or BF16 (tag 1),
// each rounded to nearest even from the FP64 value, or FP64 in the band pool
// (tag 2).  A block's columns are shared by `parts` workgroups: 1 where the
// blocks fill the chip, 8 where they would not.  Bound by the entries'
// instructions and table reads (matern_dev.h): n = 40,000 in 6.0 ms, 1.3e11
// entries/s and 1.1 TB/s written.  Tiles outside the DST band are zero and are
// written only if fill_zero.
__global__ __launch_bounds__(256) void k_gen_tiles(TileMat M, int T, int64_t nreal, const double* __restrict__ xs,
                                                   const double* __restrict__ ys, const double* __restrict__ qt,
                                                   const double* __restrict__ cst, const uint8_t* __restrict__ tag,
                                                   int64_t tile_first, int parts, int fill_zero) {
  const int64_t ts = M.ts;
  const int64_t b = blockIdx.x / parts;
  const int part = blockIdx.x % parts, ncol = BLK / parts;
  const int64_t p = tile_first + b / (T * T);
  const int sub = (int)(b % (T * T));
  const int u = sub / T, v = sub % T;
  int64_t I, J;
  tri_decode(p, &I, &J);
  if (I == J && u < v) return;
  const bool zero_tile = M.dst > 0 && I - J >= M.dst;  // outside the DST band
  if (zero_tile && !fill_zero) return;
  __shared__ __attribute__((aligned(16))) double tab[CH_TAB];
  stage_tables<1>(qt, tab);
  __syncthreads();
  const int r = threadIdx.x & 127, c0 = part * ncol + (threadIdx.x >> 7);
  const int64_t gi = I * ts + u * BLK + r;
  const bool ipad = gi >= nreal;
  const double xi = ipad ? 0.0 : xs[gi], yi = ipad ? 0.0 : ys[gi];
  const int64_t o = (u * BLK + r) + (int64_t)(v * BLK) * ts;  // element offset in the tile
  // 0: FP64, 1: FP32, 2: BF16
  const int64_t idx = I == J ? 0 : off_index(I, J, M.NT);
  const int tg = (!tag || I == J) ? -1 : tag[idx];
  const int kind = (tg < 0 || tg == TAG_F64) ? 0 : (tg == TAG_BF16 ? 2 : 1);
  double* out64 = nullptr;
  float* out32 = nullptr;
  uint16_t* out16 = nullptr;
  if (kind == 0) {
    out64 = (tg == TAG_F64 ? band64(M, idx) : tptr(M, I, J)) + o;
  } else if (kind == 1) {
    out32 = (float*)M.off + off_index(I, J, M.NT) * ts * ts + o;
  } else {
    out16 = (uint16_t*)((float*)M.off + off_index(I, J, M.NT) * ts * ts) + o;
  }
  for (int c = c0; c < (part + 1) * ncol; c += 2) {
    const int64_t gj = J * ts + v * BLK + c;
    double val;
    if (zero_tile) {
      val = 0.0;
    } else if (ipad || gj >= nreal) {
      val = (gi == gj) ? 1.0 : 0.0;
    } else {
      val = matern_value(loc_dist(xi, yi, xs[gj], ys[gj], cst), cst, qt, tab);
      if (gi == gj) val += cst[C_NUG];  // the observation's own noise
    }
    const int64_t e = (int64_t)c * ts;
    if (kind == 0) out64[e] = val;
    else if (kind == 1) out32[e] = (float)val;
    else out16[e] = f32_to_bf16_rne((float)val);
  }
}

// cov[i + j ldc] = Sigma(s_i, s_j) in the caller's order.
__global__ __launch_bounds__(256) void k_gen_dense(double* __restrict__ cov, int64_t ldc, int64_t n,
                                                   const double* __restrict__ x, const double* __restrict__ y,
                                                   const double* __restrict__ qt, const double* __restrict__ cst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double xi = x[i], yi = y[i];
  for (int64_t j = blockIdx.y; j < n; j += gridDim.y) {
    cov[i + j * ldc] = matern_value(loc_dist(xi, yi, x[j], y[j], cst), cst, qt, qt + QT_CHEB_OFF) + (i == j ? cst[C_NUG] : 0.0);
  }
}

int64_t quad_table_doubles() { return QT_TOTAL; }

// qt: QT_TOTAL doubles (quadrature nodes, then the Chebyshev tables)
void launch_quad_table(const double theta[3], int metric, double nugget, double* qt, double* cst,
                       unsigned long long* info, hipStream_t s) {
  hipLaunchKernelGGL(k_quad_table, dim3(QNB), dim3(QNK), 0, s, theta[0], theta[1], theta[2], (double)metric, nugget,
                     qt, cst, info);
  hipLaunchKernelGGL(k_cheb_table, dim3(CH_NSEG), dim3(256), 0, s, qt, (const double*)cst);
}

void launch_gen_tiles(const TileMat& M, int64_t nreal, const double* xs, const double* ys, const double* qt,
                      const double* cst, const uint8_t* tag, bool fill_zero, hipStream_t s) {
  const int64_t ts = M.ts, NT = M.NT;
  const int T = (int)(ts / BLK);
  const int64_t ntile = NT * (NT + 1) / 2;
  // 1 and 8 workgroups per block of the R (R + 1) / 2 with real rows: n = 400 56 and
  // 11 us, n = 4,096 (528 blocks) 84 and 66, n = 6,400 (1,275) 141 and 131, n = 8,100
  // (2,080) 195 and 199, n = 10,000 287 and 302, n = 20,000 991 and 1,163
  const int64_t R = (nreal + BLK - 1) / BLK;
  const int parts = R * (R + 1) / 2 < 2048 ? 8 : 1;
  // keep each launch's grid below 2^31 blocks
  const int64_t per = ((int64_t)1 << 30) / (T * T * parts);
  for (int64_t f = 0; f < ntile; f += per) {
    const int64_t cnt = (ntile - f < per) ? ntile - f : per;
    hipLaunchKernelGGL(k_gen_tiles, dim3((unsigned)(cnt * T * T * parts)), dim3(256), 0, s, M, T, nreal, xs, ys, qt,
                       cst, tag, f, parts, (int)fill_zero);
  }
}

// r_i = z_i - sum_j Sigma_ij a_j over the real points (Sigma regenerated in
// FP64, the nugget on the diagonal), r_i = 0 on padded rows; one 256-thread
// workgroup per row, fixed-order reduction.  The residual of a solve done
// through a lower-precision factor.  Bound by the entries, as k_gen_tiles:
// n = 40,000 in 7.0 ms, 2.3e11 entries/s (12.1 ms with the table in global memory
// and the library's functions).
__global__ __launch_bounds__(256) void k_sigma_residual(const double* __restrict__ xs, const double* __restrict__ ys,
                                                        const double* __restrict__ zs, const double* __restrict__ av,
                                                        int64_t nreal, int64_t npad, const double* __restrict__ qt,
                                                        const double* __restrict__ cst, double* __restrict__ r) {
  __shared__ double red[256];
  __shared__ __attribute__((aligned(16))) double tab[CH_TAB];
  const int64_t i = blockIdx.x;
  if (i >= npad) return;
  if (i >= nreal) {
    if (threadIdx.x == 0) r[i] = 0.0;
    return;
  }
  stage_tables<1>(qt, tab);
  __syncthreads();
  const double px = xs[i], py = ys[i];
  double s = 0.0;
  for (int64_t j = threadIdx.x; j < nreal; j += 256)
    s += matern_value(loc_dist(px, py, xs[j], ys[j], cst), cst, qt, tab) * av[j];
  double v[1] = {s};
  block_sum<1>(v, red);
  if (threadIdx.x == 0) r[i] = zs[i] - (v[0] + cst[C_NUG] * av[i]);
}

void launch_sigma_residual(const double* xs, const double* ys, const double* zs, const double* av, int64_t nreal,
                           int64_t npad, const double* qt, const double* cst, double* r, hipStream_t s) {
  hipLaunchKernelGGL(k_sigma_residual, dim3((unsigned)npad), dim3(256), 0, s, xs, ys, zs, av, nreal, npad, qt, cst, r);
}

void launch_gen_dense(double* cov, int64_t ldc, int64_t n, const double* x, const double* y, const double* qt,
                      const double* cst, hipStream_t s) {
  const unsigned gx = (unsigned)((n + 255) / 256);
  const unsigned gy = (unsigned)(n < 8192 ? n : 8192);
  hipLaunchKernelGGL(k_gen_dense, dim3(gx, gy), dim3(256), 0, s, cov, ldc, n, x, y, qt, cst);
}

}  // namespace exg
