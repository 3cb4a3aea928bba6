// Type-1 non-uniform FFT on gfx950: exponential-of-semicircle spreading onto an
// oversampled grid, FP64 FFT, deconvolution.
//
// What is computed (Sec. 2.3 of the paper, "Covariance vector" / "Covariance
// matrix"): for C real weight channels w_c and points x_j on the torus,
//     c_c[q] = sum_j w_cj exp(-i q.x_j),   |q_a| <= K.
// Method (Barnett, Magland, af Klinteberg, SIAM J. Sci. Comput. 41(5), 2019):
// with grid spacing h = 2 pi / nf and grid point l <-> x = -pi + l h, spread
//     g_c[l] = sum_j w_cj phi(l - u_j),  u_j = (x_j + pi) / h,
// phi(t) = psi(2 t / w), psi(z) = exp(beta (sqrt(1 - z^2) - 1)) on |z| <= 1, then
//     c_c[q] ~= (-1)^q DFT(g_c)[q mod nf] / prod_a Phihat(q_a h),
// Phihat(omega) = int phi(t) exp(-i omega t) dt (Poisson summation; the
// aliased terms are the error, bounded here by the plan's error estimate).
//
// Design for MI355X:
// * 1-D grids (<= 1024 points per channel) live whole in LDS: each workgroup
//   streams a contiguous chunk of points (coalesced), accumulates partials
//   with LDS atomics and flushes them once into an FP64 global grid.
// * 2-D grids (up to 512 x 512) do not fit in 160 KB of LDS, so points are
//   counting-sorted by bin (a T x T tile of the grid): per-workgroup LDS
//   histograms, a scan, and a scatter into bin-contiguous records
//   (two 32-bit fixed-point grid coordinates + FP32 weights).  One workgroup
//   per (bin, slice of the bin's points) then spreads into an LDS subgrid of
//   (T + 2 ceil(w/2))^2 cells x C channels and flushes it with FP64 atomics.
// * LDS partials are FP64: on gfx950 ds_add_f64 sustains ~7 lane-ops/clk/CU
//   while ds_add_f32 sustains ~0.33 (measured), so the wider type is also the
//   fast one, and the per-bin partials carry no FP32 rounding.
// * Grid coordinates are computed in FP64 and carried as fixed point (error
//   <= 2^-(33 - log2 nf) grid units), so the phase error stays below 1e-7
//   even at the highest frequency.
// * The FFT and deconvolution run in FP64 (the grids are tiny).
#include "fk_internal.h"
#include "fk_device.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace fk {

// ------------------------------------------------------------------ plan (host)

static double es_psi(double z, double beta) {
  double r = 1.0 - z * z;
  return r < 0 ? 0.0 : std::exp(beta * (std::sqrt(r) - 1.0));
}

// Gauss-Legendre nodes/weights on [-1, 1] (Newton on the Legendre recurrence).
static void gauss_legendre(int n, std::vector<double>& x, std::vector<double>& w) {
  x.resize(n);
  w.resize(n);
  for (int i = 0; i < n; ++i) {
    double z = std::cos(kPi * (i + 0.75) / (n + 0.5));
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= n; ++k) {
        double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      double dp = n * (z * p1 - p0) / (z * z - 1.0);
      double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    double p0 = 1.0, p1 = z;
    for (int k = 2; k <= n; ++k) {
      double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    double dp = n * (z * p1 - p0) / (z * z - 1.0);
    x[i] = z;
    w[i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

// Phihat(omega) = (w/2) int_{-1}^{1} psi(z) cos(omega w z / 2) dz.
static double es_phihat(double omega, int w, double beta, const std::vector<double>& gx,
                        const std::vector<double>& gw) {
  double s = 0.0;
  for (size_t i = 0; i < gx.size(); ++i) s += gw[i] * es_psi(gx[i], beta) * std::cos(omega * w * gx[i] * 0.5);
  return 0.5 * w * s;
}

// Worst case over sub-grid shifts of |sum_l phi(l - u) e^{-i omega (l-u)} - Phihat(omega)| / Phihat(omega)
// for omega = q h, 0 <= q <= K.
static double es_error(int nf, int K, int w, double beta, const std::vector<double>& gx,
                       const std::vector<double>& gw) {
  const double h = 2.0 * kPi / nf;
  std::vector<double> ph(K + 1);
  for (int q = 0; q <= K; ++q) ph[q] = es_phihat(q * h, w, beta, gx, gw);
  double worst = 0.0;
  const int nu = 24;
  for (int iu = 0; iu <= nu; ++iu) {
    double u = double(iu) / nu;
    for (int q = 0; q <= K; q += std::max(1, K / 48)) {
      double re = 0.0, im = 0.0;
      for (int l = -w; l <= w + 1; ++l) {
        double t = l - u;
        double z = 2.0 * t / w;
        if (std::fabs(z) > 1.0) continue;
        double v = es_psi(z, beta);
        re += v * std::cos(q * h * t);
        im -= v * std::sin(q * h * t);
      }
      double e = std::hypot(re - ph[q], im) / std::fabs(ph[q]);
      worst = std::max(worst, e);
    }
  }
  return worst;
}

EsPlan make_es_plan(int K, double eps, int nf_fixed) {
  // Fine grid: nf_fixed when given, else the smallest power of two with oversampling
  // nf / (2K+1) >= 2.
  EsPlan p;
  p.K = K;
  int nf = 16;
  while (nf < 2 * (2 * K + 1)) nf <<= 1;
  if (nf_fixed > 0) nf = nf_fixed;
  p.nf = nf;
  std::vector<double> gx, gw;
  gauss_legendre(160, gx, gw);
  const double sigma = double(nf) / (2 * K + 1);
  int best_w = kMaxW;
  double best_beta = 2.3 * kMaxW, best_err = 1.0;
  for (int w = 4; w <= kMaxW; ++w) {
    // shape parameter: scan around the published heuristic beta ~ pi w (1 - 1/(2 sigma)) * 0.97
    double b0 = 0.97 * kPi * w * (1.0 - 0.5 / sigma);
    double bb = b0, be = 1.0;
    for (int i = -6; i <= 6; ++i) {
      double beta = b0 * (1.0 + 0.02 * i);
      double e = es_error(nf, K, w, beta, gx, gw);
      if (e < be) { be = e; bb = beta; }
    }
    if (be <= eps || w == kMaxW) {
      best_w = w;
      best_beta = bb;
      best_err = be;
      break;
    }
  }
  p.w = best_w;
  p.beta = best_beta;
  p.err = best_err;
  p.phihat.resize(K + 1);
  const double h = 2.0 * kPi / nf;
  for (int q = 0; q <= K; ++q) p.phihat[q] = es_phihat(q * h, p.w, p.beta, gx, gw);
  return p;
}

fk_status get_es_plan(fk_ctx* ctx, int K, EsPlan* plan, const double** d_phihat, int nf_fixed) {
  double eps = ctx->opt.eps > 0 ? ctx->opt.eps : 2e-7;
  uint64_t bits;
  std::memcpy(&bits, &eps, 8);
  auto key = std::make_pair(K + (nf_fixed << 16), bits);
  auto it = ctx->es_cache.find(key);
  if (it == ctx->es_cache.end()) {
    EsPlan p = make_es_plan(K, eps, nf_fixed);
    double* d = nullptr;
    FK_HIP(hipMalloc(&d, sizeof(double) * (K + 1)));
    FK_HIP(hipMemcpy(d, p.phihat.data(), sizeof(double) * (K + 1), hipMemcpyHostToDevice));
    it = ctx->es_cache.emplace(key, std::make_pair(p, d)).first;
  }
  *plan = it->second.first;
  *d_phihat = it->second.second;
  return FK_OK;
}

fk_status get_es_plan_host(fk_ctx* ctx, int K, EsPlan* plan, int nf_fixed) {
  double eps = ctx->opt.eps > 0 ? ctx->opt.eps : 2e-7;
  uint64_t bits;
  std::memcpy(&bits, &eps, 8);
  auto key = std::make_pair(K + (nf_fixed << 16), bits);
  auto dev = ctx->es_cache.find(key);
  if (dev != ctx->es_cache.end()) {
    *plan = dev->second.first;
    return FK_OK;
  }
  auto it = ctx->es_host_cache.find(key);
  if (it == ctx->es_host_cache.end()) it = ctx->es_host_cache.emplace(key, make_es_plan(K, eps, nf_fixed)).first;
  *plan = it->second;
  return FK_OK;
}

// ------------------------------------------------------------------ device helpers

// beta is pre-multiplied by log2(e): the exponent lies in [-beta log2 e, 0], so the hardware exp2
// needs no range handling, and the hardware square root no denormal scaling.
struct EsDev {
  float beta_log2e;
  float two_over_w;
};

__device__ __forceinline__ float es_eval(float s, EsDev es) {
  // s: distance in grid units; |s| <= w/2 inside the support.
  const float z = s * es.two_over_w;
  const float r = fmaxf(fmaf(-z, z, 1.0f), 0.0f);
  return __builtin_amdgcn_exp2f(fmaf(es.beta_log2e, __builtin_amdgcn_sqrtf(r), -es.beta_log2e));
}

// Window start i0 = ceil(u - w/2) and first offset s0 = i0 - u (grid units) from
// a fixed-point coordinate with fb fraction bits.
__device__ __forceinline__ void window_start(uint32_t U, int fb, int w, int* i0, float* s0) {
  int64_t V = (int64_t)U - ((int64_t)w << (fb - 1));
  int64_t one = (int64_t)1 << fb;
  int64_t c = (V >= 0) ? ((V + one - 1) >> fb) : -((-V) >> fb);
  *i0 = (int)c;
  *s0 = (float)((double)((c << fb) - (int64_t)U) * (1.0 / (double)one));
}

// ------------------------------------------------------------------ 1-D spread (whole grid in LDS)
// grid: gridDim.x workgroups over contiguous chunks of points.  LDS: C nf doubles, 1 << lc copies of each side by
// side.  Channel 0 carries weight 1 when ones != 0; channels ones..C-1 read Y rows.
// Bound by LDS atomics: 64 lanes add into random cells, and lanes whose cells share banks (or are the same) wait
// for each other.  A lane adds into the copy of its number, so that only lanes 1 << lc apart can meet: 2e7 points,
// two channels of 512 cells, 285 us with one copy -> 155 with 16.
template <int W>
__global__ __launch_bounds__(1024) void k_spread_1d(const void* __restrict__ X, fk_dtype dt, int64_t n,
                                                    const void* __restrict__ Y, int nw, int ones,
                                                    int nf, int fb, double scale, EsDev es,
                                                    double* __restrict__ grid, int* flags,
                                                    int64_t chunk, int lc) {
  extern __shared__ double lds[];
  const int C = nw + ones;
  for (int i = threadIdx.x; i < (C * nf) << lc; i += blockDim.x) lds[i] = 0.0;
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = min(n, beg + chunk);
  const uint32_t nf_fix = (uint32_t)nf << fb;
  double* copy = lds + (threadIdx.x & ((1 << lc) - 1));
  for (int64_t j = beg + threadIdx.x; j < end; j += blockDim.x) {
    uint32_t U;
    if (!to_fixed(load_coord(X, dt, j), scale, nf_fix, &U, flags)) continue;
    int i0;
    float s0;
    window_start(U, fb, W, &i0, &s0);
    float k[W];
#pragma unroll
    for (int a = 0; a < W; ++a) k[a] = es_eval(s0 + (float)a, es);
    int base = i0 < 0 ? i0 + nf : i0;
    if (ones) {
#pragma unroll
      for (int a = 0; a < W; ++a) {
        int l = base + a;
        l = l >= nf ? l - nf : l;
        atomicAdd(&copy[l << lc], (double)k[a]);
      }
    }
    for (int c = 0; c < nw; ++c) {
      float wc = load_weight(Y, dt, (int64_t)c * n + j);
      if (!(wc == wc) || isinf(wc)) { atomicOr(&flags[kFlagNaN], 1); continue; }
      double* g = copy + (((c + ones) * nf) << lc);
#pragma unroll
      for (int a = 0; a < W; ++a) {
        int l = base + a;
        l = l >= nf ? l - nf : l;
        atomicAdd(&g[l << lc], (double)(wc * k[a]));
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < C * nf; i += blockDim.x) {
    double v = 0.0;
    for (int q = 0; q < 1 << lc; ++q) v += lds[(i << lc) + ((q + threadIdx.x) & ((1 << lc) - 1))];
    if (v != 0.0) atomicAdd(&grid[i], v);
  }
}

// ------------------------------------------------------------------ 3-D spread (FP64 global atomics)
// One thread per point: the w^3 window of every channel (channel 0 with weight 1) is added into
// the FP64 grid [C][nf][nf][nf] by hardware FP64 atomics.  Kernel values in FP32, as in 1-D.
template <int W>
__global__ __launch_bounds__(256) void k_spread_3d(const void* __restrict__ X, fk_dtype dt, int64_t n,
                                                   int64_t xstride, const void* __restrict__ Y, int nw, int nf,
                                                   int fb, double scale, EsDev es, double* __restrict__ grid,
                                                   int* flags) {
  const uint32_t nf_fix = (uint32_t)nf << fb;
  const int64_t cube = (int64_t)nf * nf * nf;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
    uint32_t U[3];
    bool ok = true;
    for (int a = 0; a < 3; ++a) ok = to_fixed(load_coord(X, dt, a * xstride + j), scale, nf_fix, &U[a], flags) && ok;
    if (!ok) continue;
    float k[3][W];
    int base[3];
    for (int a = 0; a < 3; ++a) {
      int i0;
      float s0;
      window_start(U[a], fb, W, &i0, &s0);
#pragma unroll
      for (int t = 0; t < W; ++t) k[a][t] = es_eval(s0 + (float)t, es);
      base[a] = i0 < 0 ? i0 + nf : i0;
    }
    for (int c = 0; c <= nw; ++c) {
      float wc = 1.0f;
      if (c > 0) {
        wc = load_weight(Y, dt, (int64_t)(c - 1) * n + j);
        if (!(wc == wc) || isinf(wc)) {
          atomicOr(&flags[kFlagNaN], 1);
          continue;
        }
      }
      double* g = grid + (int64_t)c * cube;
      for (int a1 = 0; a1 < W; ++a1) {
        int l1 = base[0] + a1;
        l1 = l1 >= nf ? l1 - nf : l1;
        const float v1 = wc * k[0][a1];
        for (int a2 = 0; a2 < W; ++a2) {
          int l2 = base[1] + a2;
          l2 = l2 >= nf ? l2 - nf : l2;
          const float v12 = v1 * k[1][a2];
          double* row = g + ((int64_t)l1 * nf + l2) * nf;
#pragma unroll
          for (int a3 = 0; a3 < W; ++a3) {
            int l3 = base[2] + a3;
            l3 = l3 >= nf ? l3 - nf : l3;
            atomicAdd(&row[l3], (double)(v12 * k[2][a3]));
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------ 2-D binned spread
// Bins are T x T tiles of the nf x nf grid: nbx = nf / T bins per axis.

__global__ __launch_bounds__(256) void k_bin_count(const void* __restrict__ X, fk_dtype dt, int64_t n,
                                                   int64_t xstride, int nf, int fb, double scale,
                                                   int tshift, int nbx, uint32_t* __restrict__ cnt,
                                                   int nblk, int64_t chunk, int* flags) {
  extern __shared__ uint32_t hist[];
  const int nb = nbx * nbx;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) hist[i] = 0;
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = min(n, beg + chunk);
  const uint32_t nf_fix = (uint32_t)nf << fb;
  for (int64_t j = beg + threadIdx.x; j < end; j += blockDim.x) {
    uint32_t U1, U2;
    bool ok = to_fixed(load_coord(X, dt, j), scale, nf_fix, &U1, flags);
    ok = to_fixed(load_coord(X, dt, xstride + j), scale, nf_fix, &U2, flags) && ok;
    if (!ok) continue;
    int b = ((U1 >> fb) >> tshift) * nbx + ((U2 >> fb) >> tshift);
    atomicAdd(&hist[b], 1u);
  }
  __syncthreads();
  // count table is [workgroup][bin]: one contiguous row per workgroup
  uint32_t* row = cnt + (int64_t)blockIdx.x * nb;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) row[i] = hist[i];
  (void)nblk;
}

// Exclusive scan over workgroups of cnt[.][bin] in place, one thread per bin
// (consecutive threads read consecutive bins of a row); bin totals out.
__global__ __launch_bounds__(256) void k_scan_cols(uint32_t* __restrict__ cnt, int nb, int nblk,
                                                   uint32_t* __restrict__ totals) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  uint32_t run = 0;
  for (int k = 0; k < nblk; ++k) {
    uint32_t* p = cnt + (int64_t)k * nb + b;
    uint32_t c = *p;
    *p = run;
    run += c;
  }
  totals[b] = run;
}

// Exclusive scan of the bin totals (nb <= 65536) by one workgroup; start[nb] = total.
__global__ __launch_bounds__(1024) void k_scan_totals(const uint32_t* __restrict__ totals, int nb,
                                                      uint64_t* __restrict__ start) {
  __shared__ uint64_t part[1024];
  const int per = (nb + 1023) / 1024;
  const int b0 = threadIdx.x * per;
  uint64_t s = 0;
  for (int i = 0; i < per; ++i)
    if (b0 + i < nb) s += totals[b0 + i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    uint64_t v = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  uint64_t run = part[threadIdx.x] - s;
  for (int i = 0; i < per; ++i)
    if (b0 + i < nb) {
      start[b0 + i] = run;
      run += totals[b0 + i];
    }
  if (threadIdx.x == 1023) start[nb] = part[1023];
}

// Scatter points into bin-contiguous records [U1, U2, w_0 .. w_{nw-1}] (32-bit words).
// Each workgroup keeps the next write position of every bin in LDS (64-bit,
// seeded from the scans) and claims a slot with one LDS atomic per point.
__global__ __launch_bounds__(1024) void k_bin_scatter(const void* __restrict__ X, fk_dtype dt, int64_t n,
                                                      int64_t xstride, const void* __restrict__ Y,
                                                      int nw, int nf, int fb, double scale, int tshift,
                                                      int nbx, const uint32_t* __restrict__ cnt,
                                                      const uint64_t* __restrict__ start, int64_t chunk,
                                                      uint32_t* __restrict__ rec, int* flags) {
  extern __shared__ unsigned long long nextpos[];
  const int nb = nbx * nbx;
  const uint32_t* row = cnt + (int64_t)blockIdx.x * nb;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) nextpos[i] = start[i] + row[i];
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = min(n, beg + chunk);
  const uint32_t nf_fix = (uint32_t)nf << fb;
  const int R = 2 + nw;
  for (int64_t j = beg + threadIdx.x; j < end; j += blockDim.x) {
    uint32_t U1, U2;
    bool ok = to_fixed(load_coord(X, dt, j), scale, nf_fix, &U1, flags);
    ok = to_fixed(load_coord(X, dt, xstride + j), scale, nf_fix, &U2, flags) && ok;
    if (!ok) continue;
    int b = ((U1 >> fb) >> tshift) * nbx + ((U2 >> fb) >> tshift);
    uint64_t pos = atomicAdd(&nextpos[b], 1ull);
    uint32_t* o = rec + pos * R;
    o[0] = U1;
    o[1] = U2;
    for (int c = 0; c < nw; ++c) {
      float wc = load_weight(Y, dt, (int64_t)c * n + j);
      if (!(wc == wc) || isinf(wc)) {
        atomicOr(&flags[kFlagNaN], 1);
        wc = 0.f;
      }
      o[2 + c] = __float_as_uint(wc);
    }
  }
}

// The same with lanes over the channels, for 17 channels and more: a lane per point computes the window and the
// kernel values of 64 points, then the wave adds one point at a time (two with up to 32 channels, half a wave each),
// lane c the channel c, so that an addition goes to adjacent addresses.  The products and sums are those of the
// kernel below (with a lane per point, 64 windows met in the LDS banks): 2e6 points, 32 targets, w = 7, 2691 -> 2144 us;
// whole transforms of 2.7e6 points, m = 32: 17 targets 3640 -> 2555, 20 targets, m = 60, 4864 -> 3410.  Bound by the rate of
// FP64 additions in LDS, about 2.5 per clock and CU.
template <int W>
__global__ __launch_bounds__(1024) void k_spread_2d_lanes(const uint32_t* __restrict__ rec, int nw,
                                                          const uint64_t* __restrict__ start, int nbx, int T, int nf,
                                                          int fb, EsDev es, int slices, double* __restrict__ grid) {
  extern __shared__ double sub[];
  constexpr int H = (W + 1) / 2;     // halo each side
  const int S = T + 2 * H, C = nw + 1, R = 2 + nw;
  const int b = blockIdx.x / slices, sl = blockIdx.x - b * slices;
  const uint64_t p0 = start[b], len = start[b + 1] - p0;
  const uint64_t q0 = p0 + len * sl / slices, q1 = p0 + len * (sl + 1) / slices;
  if (q0 == q1) return;
  for (int i = threadIdx.x; i < S * S * C; i += blockDim.x) sub[i] = 0.0;
  __syncthreads();
  const int bx = b / nbx, by = b - bx * nbx;
  const int o1 = bx * T - H, o2 = by * T - H;   // subgrid origin (may be negative: periodic)
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  const bool two = C <= 32;
  const int half = two ? lane >> 5 : 0, c = two ? lane & 31 : lane, step = two ? 2 : 1;
  for (uint64_t base = q0 + 64u * w; base < q1; base += 64u * nwave) {
    const int np = (int)min((uint64_t)64, q1 - base);
    const uint32_t* r = rec + (base + min(lane, np - 1)) * R;
    int i1, i2;
    float s1, s2;
    window_start(r[0], fb, W, &i1, &s1);
    window_start(r[1], fb, W, &i2, &s2);
    float k1[W], k2[W];
#pragma unroll
    for (int a = 0; a < W; ++a) {
      k1[a] = es_eval(s1 + (float)a, es);
      k2[a] = es_eval(s2 + (float)a, es);
    }
    const int cell0 = (i1 - o1) * S + (i2 - o2);   // each axis in [0, S - W]
    auto weight = [&](int p) { return c == 0 ? 1.f : __uint_as_float(rec[(base + min(p, np - 1)) * R + 2 + min(c, nw) - 1]); };
    float wn = weight(half);
    for (int p = 0; p < np; p += step) {
      const int src = min(p + half, np - 1);
      const bool on = c < C && p + half < np;
      const float wv = wn;
      wn = weight(p + step + half);
      double* row = sub + __shfl(cell0, src, 64) * C + c;
      float y[W];
#pragma unroll
      for (int a = 0; a < W; ++a) y[a] = __shfl(k2[a], src, 64);
#pragma unroll
      for (int a = 0; a < W; ++a) {
        const float x = __shfl(k1[a], src, 64);
        if (on) {
#pragma unroll
          for (int e = 0; e < W; ++e) atomicAdd(&row[(a * S + e) * C], (double)(wv * (x * y[e])));
        }
      }
    }
  }
  __syncthreads();
  // flush: periodic wrap into the FP64 global grid [C][nf][nf]
  for (int i = threadIdx.x; i < S * S * C; i += blockDim.x) {
    const double v = sub[i];
    if (v == 0.0) continue;
    const int ch = i % C, cell = i / C, a = cell / S, bb = cell - a * S;
    int g1 = o1 + a, g2 = o2 + bb;
    g1 = g1 < 0 ? g1 + nf : (g1 >= nf ? g1 - nf : g1);
    g2 = g2 < 0 ? g2 + nf : (g2 >= nf ? g2 - nf : g2);
    atomicAdd(&grid[((int64_t)ch * nf + g1) * nf + g2], v);
  }
}

// One workgroup per (bin, slice).  LDS subgrid S x S cells x C channels,
// cell-major ([cell][channel]) so the channels of one cell are adjacent.
template <int W>
__global__ __launch_bounds__(256) void k_spread_2d_binned(const uint32_t* __restrict__ rec, int nw,
                                                          int ones, const uint64_t* __restrict__ start,
                                                          int nbx, int T, int nf, int fb, EsDev es,
                                                          int slices, double* __restrict__ grid) {
  extern __shared__ double sub[];
  constexpr int H = (W + 1) / 2;     // halo each side
  const int S = T + 2 * H;
  const int C = nw + ones;
  const int b = blockIdx.x / slices;
  const int sl = blockIdx.x - b * slices;
  const uint64_t p0 = start[b], p1 = start[b + 1];
  const uint64_t len = p1 - p0;
  const uint64_t q0 = p0 + len * sl / slices;
  const uint64_t q1 = p0 + len * (sl + 1) / slices;
  if (q0 == q1) return;
  for (int i = threadIdx.x; i < S * S * C; i += blockDim.x) sub[i] = 0.0;
  __syncthreads();
  const int bx = b / nbx, by = b - bx * nbx;
  const int o1 = bx * T - H, o2 = by * T - H;   // subgrid origin (may be negative: periodic)
  const int R = 2 + nw;
  for (uint64_t j = q0 + threadIdx.x; j < q1; j += blockDim.x) {
    const uint32_t* r = rec + j * R;
    int i1, i2;
    float s1, s2;
    window_start(r[0], fb, W, &i1, &s1);
    window_start(r[1], fb, W, &i2, &s2);
    float k1[W], k2[W];
#pragma unroll
    for (int a = 0; a < W; ++a) {
      k1[a] = es_eval(s1 + (float)a, es);
      k2[a] = es_eval(s2 + (float)a, es);
    }
    const int l1 = i1 - o1, l2 = i2 - o2;      // in [0, S - W]
    if (ones) {
#pragma unroll
      for (int a = 0; a < W; ++a) {
        double* row = sub + ((l1 + a) * S + l2) * C;
#pragma unroll
        for (int c2 = 0; c2 < W; ++c2) atomicAdd(&row[c2 * C], (double)(k1[a] * k2[c2]));
      }
    }
    for (int cg = 0; cg < nw; cg += 4) {
      float wv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) wv[u] = (cg + u < nw) ? __uint_as_float(r[2 + cg + u]) : 0.f;
      const int cn = min(4, nw - cg);
#pragma unroll
      for (int a = 0; a < W; ++a) {
        double* row = sub + ((l1 + a) * S + l2) * C + ones + cg;
#pragma unroll
        for (int c2 = 0; c2 < W; ++c2) {
          float kk = k1[a] * k2[c2];
          double* cell = row + c2 * C;
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (u < cn) atomicAdd(&cell[u], (double)(wv[u] * kk));
        }
      }
    }
  }
  __syncthreads();
  // flush: periodic wrap into the FP64 global grid [C][nf][nf]
  for (int i = threadIdx.x; i < S * S * C; i += blockDim.x) {
    double v = sub[i];
    if (v == 0.0) continue;
    int c = i % C;
    int cell = i / C;
    int a = cell / S, bb = cell - a * S;
    int g1 = o1 + a, g2 = o2 + bb;
    g1 = g1 < 0 ? g1 + nf : (g1 >= nf ? g1 - nf : g1);
    g2 = g2 < 0 ? g2 + nf : (g2 >= nf ? g2 - nf : g2);
    atomicAdd(&grid[((int64_t)c * nf + g1) * nf + g2], v);
  }
}

// ------------------------------------------------------------------ FFT (FP64, radix 4, in LDS)
// A workgroup transforms lb lines of length nf (a power of two, 16 .. 1024) and writes the pruned,
// deconvolved frequencies q = -K..K of each:
//   out[line][q + K] = scale * (-1)^q / phihat[|q|] * sum_l in[l] e^{-2 pi i q l / nf}.
// The lines are brought into LDS together (neighbouring columns in runs of lb complex entries), a wave
// transforms one line at a time without a workgroup barrier (decimation in frequency, two radix-2
// levels per LDS round trip, bit-reversed result), and the frequencies leave in runs again.
// REAL: 2 lb contiguous real lines, two per complex transform (Z = A + iB gives A[q] = (Z[q] + conj
// Z[-q]) / 2 and B[q] = (Z[q] - conj Z[-q]) / 2i); line r at in + r nf, its output at out + r (2K + 1).
// Else line (lo, li): entry i at in[lo in_outer + li + i inner] (complex), li < inner; output q at
// out[lo out_outer + li + (q + K) inner].
// Bound by memory for large batches: one workgroup per line with its twiddles computed in every radix-2
// stage took 771 us for the three passes of a 256^3 grid of two channels (0.62 GB), these 317, and 120 against
// 71 us for 17 channels of 512^2.
constexpr int FFT_T = 256;          // threads: four waves
constexpr int FFT_PTS = 4096;       // points per workgroup at most

__device__ __forceinline__ int fft_pad(int i) { return i + (i >> 3); }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// In-place transform of one padded line by one wave; tw[k] = e^{-2 pi i k / nf}, k < nf / 2.
__device__ __forceinline__ void wave_fft(double2* B, const double2* tw, int nf, int lane) {
  int len = nf, step = 1;
  for (; len >= 4; len >>= 2, step <<= 2) {
    const int q = len >> 2, lq = __ffs(q) - 1;
    for (int t = lane; t < nf / 4; t += 64) {
      const int pos = t & (q - 1), i0 = ((t >> lq) << (lq + 2)) + pos;
      double2* p0 = B + fft_pad(i0);
      double2* p1 = B + fft_pad(i0 + q);
      double2* p2 = B + fft_pad(i0 + 2 * q);
      double2* p3 = B + fft_pad(i0 + 3 * q);
      const double2 a0 = *p0, a1 = *p1, a2 = *p2, a3 = *p3;
      const double2 w1 = tw[pos * step], w2 = tw[pos * step * 2];
      // b2 = (a0 - a2) w1, b3 = (a1 - a3) w1 (-i)
      const double2 b0 = make_double2(a0.x + a2.x, a0.y + a2.y), b1 = make_double2(a1.x + a3.x, a1.y + a3.y);
      const double2 d2 = zmul(make_double2(a0.x - a2.x, a0.y - a2.y), w1);
      const double2 d3 = zmul(make_double2(a1.y - a3.y, a3.x - a1.x), w1);
      *p0 = make_double2(b0.x + b1.x, b0.y + b1.y);
      *p1 = zmul(make_double2(b0.x - b1.x, b0.y - b1.y), w2);
      *p2 = make_double2(d2.x + d3.x, d2.y + d3.y);
      *p3 = zmul(make_double2(d2.x - d3.x, d2.y - d3.y), w2);
    }
    wave_sync();
  }
  if (len == 2) {
    for (int t = lane; t < nf / 2; t += 64) {
      double2* p0 = B + fft_pad(2 * t);
      double2* p1 = B + fft_pad(2 * t + 1);
      const double2 u = *p0, v = *p1;
      *p0 = make_double2(u.x + v.x, u.y + v.y);
      *p1 = make_double2(u.x - v.x, u.y - v.y);
    }
    wave_sync();
  }
}

template <bool REAL>
__global__ __launch_bounds__(FFT_T) void k_fft_lines(const double* __restrict__ in, int64_t nlines, int64_t in_outer,
                                                     int inner, int nf, int logn, int lb,
                                                     const double* __restrict__ phihat, int K, double scale,
                                                     double* __restrict__ out, int64_t out_outer) {
  extern __shared__ __align__(16) double2 fbuf[];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int ls = fft_pad(nf), L = 2 * K + 1;
  double2* tw = fbuf + (size_t)lb * ls;
  double* fac = reinterpret_cast<double*>(tw + nf / 2);   // scale (-1)^q / phihat[q], q = 0..K
  for (int k = tid; k < nf / 2; k += FFT_T) {
    double sn, cs;
    sincospi(-2.0 * k / nf, &sn, &cs);
    tw[k] = make_double2(cs, sn);
  }
  for (int q = tid; q <= K; q += FFT_T) {
    const double f = scale / phihat[q];
    fac[q] = (q & 1) ? -f : f;
  }
  int64_t line0, lo = 0;
  int cnt;   // lines of this workgroup (REAL: real lines)
  if constexpr (REAL) {
    line0 = (int64_t)blockIdx.x * 2 * lb;
    cnt = (int)min((int64_t)2 * lb, nlines - line0);
    const double* src = in + line0 * nf;
    double* dst = reinterpret_cast<double*>(fbuf);
    for (int e = tid; e < 2 * lb * nf; e += FFT_T) {
      const int r = e >> logn, i = e & (nf - 1);
      dst[2 * ((r >> 1) * ls + fft_pad(i)) + (r & 1)] = r < cnt ? src[e] : 0.0;
    }
  } else {
    const int per = (inner + lb - 1) / lb;
    lo = blockIdx.x / per;
    line0 = (int64_t)(blockIdx.x - lo * per) * lb;
    cnt = (int)min((int64_t)lb, inner - line0);
    const double2* src = reinterpret_cast<const double2*>(in) + lo * in_outer + line0;
    for (int e = tid; e < lb * nf; e += FFT_T) {
      const int i = e / lb, j = e - i * lb;
      if (j < cnt) fbuf[j * ls + fft_pad(i)] = src[(int64_t)i * inner + j];
    }
  }
  __syncthreads();
  const int nz = REAL ? (cnt + 1) / 2 : cnt;
  for (int j = w; j < nz; j += FFT_T / 64) wave_fft(fbuf + j * ls, tw, nf, lane);
  __syncthreads();
  auto at = [&](const double2* B, int l) { return B[fft_pad((int)(__brev((unsigned)l) >> (32 - logn)))]; };
  if constexpr (REAL) {
    double2* dst = reinterpret_cast<double2*>(out) + line0 * L;
    for (int e = tid; e < cnt * L; e += FFT_T) {
      const int r = e / L, q = e - r * L - K;
      const double2* B = fbuf + (r >> 1) * ls;
      const double2 z1 = at(B, q & (nf - 1)), z2 = at(B, -q & (nf - 1));
      const double f = 0.5 * fac[abs(q)];
      dst[e] = (r & 1) ? make_double2((z1.y + z2.y) * f, (z2.x - z1.x) * f)
                       : make_double2((z1.x + z2.x) * f, (z1.y - z2.y) * f);
    }
  } else {
    double2* dst = reinterpret_cast<double2*>(out) + lo * out_outer + line0;
    for (int e = tid; e < lb * L; e += FFT_T) {
      const int qi = e / lb, j = e - qi * lb, q = qi - K;
      if (j >= cnt) continue;
      const double2 z = at(fbuf + j * ls, q & (nf - 1));
      const double f = fac[abs(q)];
      dst[(int64_t)qi * inner + j] = make_double2(z.x * f, z.y * f);
    }
  }
}

// Lines per workgroup: FFT_PTS points, fewer while that would leave CUs without a workgroup.
static int fft_lb(int64_t lines, int nf) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(FFT_PTS / nf, lines / 512));
}

// Real lines along the contiguous axis: `lines` lines of nf doubles -> [lines][2K + 1] complex.
static void fft_real(hipStream_t st, const double* in, int64_t lines, int nf, int logn, const double* phihat, int K,
                     double scale, double* out) {
  const int64_t pairs = (lines + 1) / 2;
  const int lb = fft_lb(pairs, nf);
  const size_t lds = sizeof(double2) * ((size_t)lb * (nf + nf / 8) + nf / 2) + sizeof(double) * (K + 1);
  hipLaunchKernelGGL(k_fft_lines<true>, dim3((unsigned)((pairs + lb - 1) / lb)), dim3(FFT_T), lds, st, in, lines,
                     (int64_t)0, 1, nf, logn, lb, phihat, K, scale, out, (int64_t)0);
}

// Complex lines along the middle axis of [outer][nf][inner] -> [outer][2K + 1][inner].
static void fft_mid(hipStream_t st, const double* in, int64_t outer, int inner, int nf, int logn, const double* phihat,
                    int K, double scale, double* out) {
  int lb = fft_lb(outer * inner, nf);
  lb = std::min(lb, inner);
  const size_t lds = sizeof(double2) * ((size_t)lb * (nf + nf / 8) + nf / 2) + sizeof(double) * (K + 1);
  const int64_t blocks = outer * ((inner + lb - 1) / lb);
  hipLaunchKernelGGL(k_fft_lines<false>, dim3((unsigned)blocks), dim3(FFT_T), lds, st, in, outer * inner,
                     (int64_t)nf * inner, inner, nf, logn, lb, phihat, K, scale, out, (int64_t)(2 * K + 1) * inner);
}

// ------------------------------------------------------------------ host driver

static int ilog2(int v) {
  int r = 0;
  while ((1 << r) < v) ++r;
  return r;
}

struct BinGeom {
  int T, tshift, nbx, nb, nblk;
  int64_t chunk;
};

// Spread used by the 2-D type-1 stage.  kRows: 8..16 weighted channels as the rows
// of matrix-core products (spread_mfma.hip); kOuter: 0..7 weighted channels as
// per-channel outer products (spread_op.hip); both after the two-pass bin sort.
// kAtomic: one counting pass and FP64 LDS atomics (other channel counts or widths).
enum class Spread2 { kAtomic, kRows, kOuter };

static Spread2 spread2_kind(int nw, int nf, int W, int64_t n) {
  if (nw >= 8 && nw <= 16 && spread_mfma_ok(nw, W) && sort2_ok(nf / spread_mfma_bin(nf, n))) return Spread2::kRows;
  if (spread_op_ok(nw, W) && nf % spread_op_bin() == 0 && sort2_ok(nf / spread_op_bin())) return Spread2::kOuter;
  return Spread2::kAtomic;
}

// Bin edge of the channel-row spread: the shape's choice when the sort can take it, else the
// density rule.
static int rows_bin(int nf, int64_t n, int mb) {
  if ((mb == 2 || mb == 4) && sort2_ok(nf / mb)) return mb;
  return spread_mfma_bin(nf, n);
}

static BinGeom bin_geom(int nf, int C, int64_t n, Spread2 kind, int mb = 0) {
  BinGeom g;
  g.T = kind == Spread2::kRows ? rows_bin(nf, n, mb)
        : kind == Spread2::kOuter ? spread_op_bin() : ((C > 8) ? 16 : 32);
  if (g.T > nf) g.T = nf;
  g.tshift = ilog2(g.T);
  g.nbx = nf / g.T;
  g.nb = g.nbx * g.nbx;
  const int64_t cap = std::max<int64_t>(1, (int64_t)(1 << 23) / g.nb);   // count table <= 8M entries
  g.nblk = (int)std::min<int64_t>(std::min<int64_t>(2048, cap), std::max<int64_t>(1, (n + 8191) / 8192));
  g.chunk = (n + g.nblk - 1) / g.nblk;
  return g;
}

// 3-D: the points are sorted into bins of 8^3 window-start cells before the spread wherever their
// positions fit 32 bits.  Spread alone (every point adding its window into the grid by itself) against sort
// and binned spread: 460 / 282 us with one point for every four bins, 1053 / 513 with one per bin (nf = 256,
// two channels), and 625 / 88 us at nf = 128, w = 9.
static bool spread3_sorted(int nf, int64_t n, int nw) { return sort3_ok(nf, n, nw); }

// Workspace of type1(): the largest layout any kernel width can select (the width
// follows from K and the context's tolerance, not known here).
size_t type1_workspace(int d, int64_t n, int nw, int K, double eps) {
  (void)eps;
  int nf = 16;
  while (nf < 2 * (2 * K + 1)) nf <<= 1;
  const int C = nw + 1;
  const int L = 2 * K + 1;
  auto layout = [&](Spread2 kind) {
    Carve cv(nullptr, 0);
    if (d == 1) {
      cv.take<double>((size_t)C * nf);
      return cv.off;
    }
    if (d == 3) {
      cv.take<double>((size_t)C * nf * nf * nf);      // FP64 grid
      cv.take<double>((size_t)C * nf * nf * L * 2);   // after the axis-2 transform
      cv.take<double>((size_t)C * nf * L * L * 2);    // after the axis-1 transform
      if (spread3_sorted(nf, n, nw)) {
        const size_t nb = (size_t)(nf / 8) * (nf / 8) * (nf / 8);
        cv.take<uint64_t>(nb + 1);                    // bin starts
        cv.take<uint32_t>((size_t)n * (3 + nw));      // records
        Sort2Bufs sb;
        sort3_carve(cv, n, nf, nw, &sb);
      }
      return cv.off;
    }
    BinGeom g = bin_geom(nf, C, n, kind);
    if (kind == Spread2::kRows) {                   // bin starts for the finest bins any shape takes
      const BinGeom g2 = bin_geom(nf, C, n, kind, 2);
      if (g2.nb > g.nb) g = g2;
    }
    cv.take<double>((size_t)C * nf * nf);          // FP64 grid
    if (kind != Spread2::kAtomic) {
      cv.take<uint32_t>((size_t)g.nbx);             // the sort's totals (one-pass sort: see type1)
    } else {
      cv.take<uint32_t>((size_t)g.nb * g.nblk);
      cv.take<uint32_t>((size_t)g.nb);
    }
    cv.take<double>((size_t)C * nf * L * 2);        // row-FFT output
    cv.take<uint64_t>((size_t)g.nb + 1);
    if (kind != Spread2::kAtomic) {
      const int wv = sort2_words(nw);
      cv.take<uint32_t>((size_t)n * 2);
      cv.take<uint32_t>((size_t)n * (kind == Spread2::kRows ? 1 : wv));
      Sort2Bufs sb;
      sort2_carve(cv, n, g.nbx, wv, &sb);
    } else {
      cv.take<uint32_t>((size_t)n * (2 + nw));
    }
    return cv.off;
  };
  size_t sz = layout(Spread2::kAtomic);
  for (int w = 4; w <= 8; ++w) sz = std::max(sz, layout(spread2_kind(nw, nf, w, n)));
  return sz + 256;
}

// Copies of the 1-D grid in LDS: as many as 144 KB hold, with one workgroup of 1024 threads per CU, from 2^19 points on
// (2e7 points: 72 KB and two workgroups 237 us for the whole transform, 36 KB and four 263, 144 KB 222).  Below,
// many small workgroups have fewer cells to clear and to add up.
constexpr int64_t kCopies1dPoints = 1 << 19;
constexpr size_t kCopies1dBytes = 144 * 1024;
constexpr int k1dBlocks = 256;

template <int W>
static void launch_spread_1d(fk_ctx* ctx, const void* X, fk_dtype dt, int64_t n, const void* Y, int nw, int ones, int nf,
                             int fb, double scale, EsDev es, double* grid) {
  const size_t cells = (size_t)(nw + ones) * nf;
  // workgroups of 4096 points; few points in smaller ones, down to 512, over up to 256 CUs (a thread's points follow
  // one another: 10000 points 16.7 -> 5.3 us)
  int blocks = (int)std::min<int64_t>(1024, std::max<int64_t>((n + 4095) / 4096, std::min<int64_t>(256, (n + 511) / 512)));
  int threads = 256, lc = 0;
  if (n >= kCopies1dPoints) {
    while (lc < 5 && (sizeof(double) * cells << (lc + 1)) <= kCopies1dBytes) ++lc;
    if (lc > 0) {
      blocks = k1dBlocks;
      threads = 1024;
    }
  }
  hipLaunchKernelGGL(k_spread_1d<W>, dim3(blocks), dim3(threads), sizeof(double) * cells << lc, ctx->stream, X, dt, n, Y,
                     nw, ones, nf, fb, scale, es, grid, ctx->flags, (n + blocks - 1) / blocks, lc);
}

template <int W>
static void launch_spread_3d(fk_ctx* ctx, const void* X, fk_dtype dt, int64_t n, int64_t xstride, const void* Y,
                             int nw, int nf, int fb, double scale, EsDev es, double* grid) {
  const int blocks = (int)std::min<int64_t>(65536, std::max<int64_t>(1, (n + 255) / 256));
  hipLaunchKernelGGL(k_spread_3d<W>, dim3(blocks), dim3(256), 0, ctx->stream, X, dt, n, xstride, Y, nw, nf, fb,
                     scale, es, grid, ctx->flags);
}

template <int W>
static void launch_spread_2d(fk_ctx* ctx, int blocks, size_t lds, const uint32_t* rec, int nw,
                             const uint64_t* start, int nbx, int T, int nf, int fb, EsDev es, int slices,
                             double* grid) {
  if (nw >= 16 && nw < 64) {
    hipLaunchKernelGGL(k_spread_2d_lanes<W>, dim3(blocks), dim3(1024), lds, ctx->stream, rec, nw, start, nbx, T, nf, fb, es,
                       slices, grid);
    return;
  }
  hipLaunchKernelGGL(k_spread_2d_binned<W>, dim3(blocks), dim3(256), lds, ctx->stream, rec, nw, 1, start,
                     nbx, T, nf, fb, es, slices, grid);
}

#define FK_W_SWITCH(w, CALL)                         \
  switch (w) {                                       \
    case 4: { constexpr int WW = 4; CALL; } break;   \
    case 5: { constexpr int WW = 5; CALL; } break;   \
    case 6: { constexpr int WW = 6; CALL; } break;   \
    case 7: { constexpr int WW = 7; CALL; } break;   \
    case 8: { constexpr int WW = 8; CALL; } break;   \
    case 9: { constexpr int WW = 9; CALL; } break;   \
    case 10: { constexpr int WW = 10; CALL; } break; \
    case 11: { constexpr int WW = 11; CALL; } break; \
    case 12: { constexpr int WW = 12; CALL; } break; \
    case 13: { constexpr int WW = 13; CALL; } break; \
    case 14: { constexpr int WW = 14; CALL; } break; \
    case 15: { constexpr int WW = 15; CALL; } break; \
    case 16: { constexpr int WW = 16; CALL; } break; \
    default: return FK_EINVAL;                       \
  }

// Launch shape of the sorted 2-D type-1 stage: the table's entry for this shape, or (when the
// problem is large enough for shapes to matter and the mode allows) coordinate descent over the
// candidates, each run on the call's own data and timed between ev[0] and ev[2].
template <class Run>
static fk_status tune_t1(fk_ctx* ctx, int d, int nf, int W, int nw, int64_t n, bool rows, Run& run, T1Shape* out) {
  T1Shape sh;
  const int mode = tune_mode(ctx);
  if (mode == kTuneOff) {
    *out = sh;
    return FK_OK;
  }
  char key[160];
  std::snprintf(key, sizeof(key), "%s t1 d=%d nf=%d w=%d nw=%d n=2^%d", tune_arch(ctx->device).c_str(), d, nf, W, nw,
                ilog2((int)std::min<int64_t>(n >> 10, 1 << 30)) + 10);
  std::map<std::string, double> v;
  if (mode != kTuneForce && tune_lookup(key, &v)) {
    if (v.count("mb")) sh.mb = (int)v["mb"];
    if (v.count("spread_pts") && v["spread_pts"] >= 256) sh.spread_pts = (int)v["spread_pts"];
    if (v.count("sort_blk") && v["sort_blk"] >= 1 && v["sort_blk"] <= kSortBlkMax) sh.sort_blk = (int)v["sort_blk"];
    if (v.count("sort_slice") && v["sort_slice"] >= kSortSliceMin) sh.sort_slice = (int)v["sort_slice"];
    *out = sh;
    return FK_OK;
  }
  if (n < ((int64_t)1 << 22)) {   // small problems: launch and latency bound, the defaults
    *out = sh;
    return FK_OK;
  }
  // a candidate's time is the better of two runs: the candidates of a knob differ by about as much
  // as one run varies (1-2 % of the stage), and the first run of the stage also pays first touches
  auto time_of = [&](const T1Shape& s, float* ms) -> fk_status {
    *ms = 0.f;
    for (int rep = 0; rep < 2; ++rep) {
      fk_status st = run(s);
      if (st != FK_OK) return st;
      FK_HIP(hipEventSynchronize(ctx->ev[2]));
      float t = 0.f;
      FK_HIP(hipEventElapsedTime(&t, ctx->ev[0], ctx->ev[2]));
      *ms = rep == 0 ? t : std::min(*ms, t);
    }
    return FK_OK;
  };
  float best;
  fk_status st = time_of(sh, &best);
  if (st != FK_OK) return st;
  auto knob = [&](int T1Shape::*field, std::initializer_list<int> cands) -> fk_status {
    for (int c : cands) {
      if (sh.*field == c) continue;
      T1Shape t = sh;
      t.*field = c;
      float ms;
      fk_status s = time_of(t, &ms);
      if (s != FK_OK) return s;
      if (ms < best) {
        best = ms;
        sh = t;
      }
    }
    return FK_OK;
  };
  if (rows) {
    sh.mb = spread_mfma_bin(nf, n);
    st = knob(&T1Shape::mb, {2, 4});
    if (st != FK_OK) return st;
  }
  if ((st = knob(&T1Shape::spread_pts, {4096, 8192, 16384, 32768})) != FK_OK) return st;
  if ((st = knob(&T1Shape::sort_blk, {256, 512, 1024})) != FK_OK) return st;
  if ((st = knob(&T1Shape::sort_slice, {32768, 65536, 131072})) != FK_OK) return st;
  std::map<std::string, double> rec{{"spread_pts", sh.spread_pts}, {"sort_blk", sh.sort_blk},
                                    {"sort_slice", sh.sort_slice}};
  if (rows) rec["mb"] = sh.mb;
  tune_store(key, rec, best);
  *out = sh;
  return FK_OK;
}

// out: complex128 [C][(2K+1)^d], C = nw + 1, channel 0 = weight 1.
// out_c[q] = sign_scale * sum_j w_cj exp(-i q.x_j).
fk_status type1(fk_ctx* ctx, int d, int64_t n, fk_dtype dt, const void* X, int64_t xstride, int nw,
                const void* Y, int K, double sign_scale, double* out, Carve& cv, fk_fit_info* info) {
  EsPlan plan;
  const double* phihat;
  fk_status st = get_es_plan(ctx, K, &plan, &phihat);
  if (st != FK_OK) return st;
  const int nf = plan.nf, W = plan.w, logn = ilog2(nf);
  const int fb = 32 - ilog2(nf) - 1;        // fixed-point fraction bits (u < nf <= 2^(31-fb))
  const double scale = (double)nf / (2.0 * kPi) * (double)(1u << fb);
  EsDev es{(float)(plan.beta * 1.44269504088896340736), 2.0f / (float)W};
  const int C = nw + 1;
  const int L = 2 * K + 1;
  if (info) {
    info->w = W;
    info->nf = nf;
    info->beta = plan.beta;
  }
  hipEvent_t* ev = ctx->ev;
  if (d == 1) {
    double* grid = cv.take<double>((size_t)C * nf);
    if (!cv.ok()) return FK_ENOMEM;
    FK_HIP(hipEventRecord(ev[0], ctx->stream));
    FK_HIP(hipMemsetAsync(grid, 0, sizeof(double) * C * nf, ctx->stream));
    // channels per launch: as many whole FP64 grids as 160 KB of LDS holds (the ones channel
    // goes with the first launch); the grid is [C][nf], so a launch writes channels ones + c0 ..
    const int per = (int)((160 * 1024) / (sizeof(double) * nf));
    if (per < 2) return FK_EINVAL;
    const size_t esz = dt == FK_F64 ? sizeof(double) : sizeof(float);
    FK_HIP(hipEventRecord(ev[1], ctx->stream));
    for (int c0 = 0, first = 1; first || c0 < nw; first = 0) {
      const int cnt = std::min(per - first, nw - c0);
      const void* Yc = Y ? static_cast<const void*>(static_cast<const char*>(Y) + esz * (size_t)c0 * n) : nullptr;
      double* gc = grid + (size_t)(first ? 0 : 1 + c0) * nf;
      FK_W_SWITCH(W, launch_spread_1d<WW>(ctx, X, dt, n, Yc, cnt, first, nf, fb, scale, es, gc));
      c0 += cnt;
    }
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[2], ctx->stream));
    fft_real(ctx->stream, grid, C, nf, logn, phihat, K, sign_scale, out);
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[3], ctx->stream));
    if (info) info->bin = 0;
    return FK_OK;
  }
  if (d == 3) {
    // spread, then transforms along axis 2 (C nf^2 lines), axis 1 (C nf L lines) and axis 0
    // (C L^2 lines), each pruned to |q| <= K and deconvolved along its own axis
    const int64_t nf3 = (int64_t)nf * nf * nf;
    double* grid = cv.take<double>((size_t)C * nf3);
    double* ta = cv.take<double>((size_t)C * nf * nf * L * 2);
    double* tb = cv.take<double>((size_t)C * nf * L * L * 2);
    const bool sorted = spread3_sorted(nf, n, nw);
    uint64_t* start3 = nullptr;
    uint32_t* rec3 = nullptr;
    Sort2Bufs sb;
    if (sorted) {
      start3 = cv.take<uint64_t>((size_t)(nf / 8) * (nf / 8) * (nf / 8) + 1);
      rec3 = cv.take<uint32_t>((size_t)n * (3 + nw));
      sort3_carve(cv, n, nf, nw, &sb);
    }
    if (!cv.ok()) return FK_ENOMEM;
    if (info) info->bin = sorted ? 8 : 0;
    FK_HIP(hipEventRecord(ev[0], ctx->stream));
    FK_HIP(hipMemsetAsync(grid, 0, sizeof(double) * C * nf3, ctx->stream));
    if (sorted) {
      st = sort3(ctx->stream, X, dt, n, xstride, Y, nw, nf, fb, W, scale, sb, rec3, start3, ctx->flags);
      if (st != FK_OK) return st;
    }
    FK_HIP(hipEventRecord(ev[1], ctx->stream));
    if (sorted) {
      st = launch_spread3(ctx->stream, W, rec3, nw, start3, nf, fb, plan.beta, n, grid);
      if (st != FK_OK) return st;
    } else {
      FK_W_SWITCH(W, launch_spread_3d<WW>(ctx, X, dt, n, xstride, Y, nw, nf, fb, scale, es, grid));
    }
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[2], ctx->stream));
    fft_real(ctx->stream, grid, (int64_t)C * nf * nf, nf, logn, phihat, K, 1.0, ta);
    fft_mid(ctx->stream, ta, (int64_t)C * nf, L, nf, logn, phihat, K, 1.0, tb);
    fft_mid(ctx->stream, tb, C, L * L, nf, logn, phihat, K, sign_scale, out);
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[3], ctx->stream));
    return FK_OK;
  }
  if (d != 2) return FK_EINVAL;
  const Spread2 kind = spread2_kind(nw, nf, W, n);
  const bool split = kind != Spread2::kAtomic;   // two-pass sort, then an MFMA spread
  const int wv = sort2_words(nw);
  BinGeom gmax = bin_geom(nf, C, n, kind);
  if (kind == Spread2::kRows) {
    const BinGeom g2 = bin_geom(nf, C, n, kind, 2);
    if (g2.nb > gmax.nb) gmax = g2;
  }
  // the sort's totals follow the grid, so that one fill clears both; those of a one-pass sort, nb words (nf^2 / 64),
  // run on into rowfft, which is written after the sort
  double* grid = cv.take<double>((size_t)C * nf * nf);
  uint32_t* cnt = split ? nullptr : cv.take<uint32_t>((size_t)gmax.nb * gmax.nblk);
  uint32_t* totals = cv.take<uint32_t>(split ? (size_t)gmax.nbx : (size_t)gmax.nb);
  double* rowfft = cv.take<double>((size_t)C * nf * L * 2);
  uint64_t* start = cv.take<uint64_t>((size_t)gmax.nb + 1);
  uint32_t* rec = cv.take<uint32_t>((size_t)n * (split ? 2 : 2 + nw));
  // second sorted array: weight words (outer-product spread) or, for the channel-row
  // spread, each point's position in the row-grouped weight blocks sb.wts1
  uint32_t* wts = split ? cv.take<uint32_t>((size_t)n * (kind == Spread2::kRows ? 1 : wv)) : nullptr;
  Sort2Bufs sb;
  if (split) sort2_carve(cv, n, gmax.nbx, wv, &sb);
  if (!cv.ok()) return FK_ENOMEM;
  // The binning and the spread for one launch shape, between events ev[0] .. ev[2].
  auto run = [&](const T1Shape& sh) -> fk_status {
    const BinGeom g = bin_geom(nf, C, n, kind, sh.mb);
    if (info) info->bin = g.T;
    FK_HIP(hipEventRecord(ev[0], ctx->stream));
    size_t clear = sizeof(double) * C * nf * nf;
    if (split) clear = (size_t)(reinterpret_cast<char*>(totals + sort2_totals(n, g.nbx, nw)) - reinterpret_cast<char*>(grid));
    FK_HIP(hipMemsetAsync(grid, 0, clear, ctx->stream));
    if (split) {
      // records for the MFMA spreads: two-pass sort, coordinates and weight words
      fk_status s2 = sort2(ctx->stream, X, dt, n, xstride, Y, nw, nf, fb, W, scale, g.tshift, g.nbx, sh, sb, totals,
                           rec, wts, start, ctx->flags);
      if (s2 != FK_OK) return s2;
    } else {
      hipLaunchKernelGGL(k_bin_count, dim3(g.nblk), dim3(256), sizeof(uint32_t) * g.nb, ctx->stream, X, dt, n,
                         xstride, nf, fb, scale, g.tshift, g.nbx, cnt, g.nblk, g.chunk, ctx->flags);
      FK_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_scan_cols, dim3((g.nb + 255) / 256), dim3(256), 0, ctx->stream, cnt, g.nb, g.nblk,
                         totals);
      hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(1024), 0, ctx->stream, totals, g.nb, start);
      hipLaunchKernelGGL(k_bin_scatter, dim3(g.nblk), dim3(1024), sizeof(unsigned long long) * g.nb, ctx->stream, X,
                         dt, n, xstride, Y, nw, nf, fb, scale, g.tshift, g.nbx, cnt, start, g.chunk, rec,
                         ctx->flags);
    }
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[1], ctx->stream));
    int64_t per_bin = (n + g.nb - 1) / g.nb;
    if (kind == Spread2::kRows) {
      fk_status s2 = launch_spread_mfma(ctx->stream, W, g.T, rec, wts, sb.wts1, nw, start, g.nbx, g.nb, nf, fb,
                                        plan.beta, n, sh.spread_pts, grid);
      if (s2 != FK_OK) return s2;
      if (info) info->bin = -g.T;   // negative: MFMA spread over T x T bins
    } else if (kind == Spread2::kOuter) {
      fk_status s2 = launch_spread_op(ctx->stream, W, rec, wts, nw, start, g.nbx, g.nb, nf, fb, plan.beta, n,
                                      sh.spread_pts, grid);
      if (s2 != FK_OK) return s2;
      if (info) info->bin = -g.T;
    } else {
      const int H = (W + 1) / 2;
      const int S = g.T + 2 * H;
      size_t lds = sizeof(double) * S * S * C;
      if (lds > 160 * 1024) return FK_EINVAL;
      int slices = (int)std::max<int64_t>(1, std::min<int64_t>(4096, (per_bin + 8191) / 8192));
      int blocks = g.nb * slices;
      FK_W_SWITCH(W, launch_spread_2d<WW>(ctx, blocks, lds, rec, nw, start, g.nbx, g.T, nf, fb, es, slices, grid));
    }
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[2], ctx->stream));
    return FK_OK;
  };
  T1Shape shape;
  if (split) {
    fk_status s2 = tune_t1(ctx, d, nf, W, nw, n, kind == Spread2::kRows, run, &shape);
    if (s2 != FK_OK) return s2;
  }
  st = run(shape);
  if (st != FK_OK) return st;
  // rows along dim 2 (contiguous) -> rowfft[c][i1][q2], then columns along i1
  fft_real(ctx->stream, grid, (int64_t)C * nf, nf, logn, phihat, K, 1.0, rowfft);
  fft_mid(ctx->stream, rowfft, C, L, nf, logn, phihat, K, sign_scale, out);
  FK_HIP(hipGetLastError());
  FK_HIP(hipEventRecord(ev[3], ctx->stream));
  return FK_OK;
}

}  // namespace fk
