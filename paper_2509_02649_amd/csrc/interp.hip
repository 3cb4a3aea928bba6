// Type-2 non-uniform FFT (prediction) and the on-device synthetic-input generator.
//
// Prediction evaluates the estimator f_theta(x) = sum_k theta_k exp(+i k.x)
// (Sec. 2.1) at new points: the coefficients are divided by the kernel's
// Fourier transform, placed on an oversampled grid, inverse-FFT'd in FP64, and
// each point gathers its w^d grid neighbours weighted by the same
// exponential-of-semicircle kernel as the type-1 spread.  Only the real part is
// kept (a real estimator has Hermitian-symmetric theta).
//   Re f(x) ~= sum_l Re(g_l) phi(l - u),  g_l = sum_q (-1)^q theta_q / Phihat(q h) e^{2 pi i q l / nf}.
#include "fk_internal.h"
#include "cg_fft.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

namespace fk {

// Inverse DFT of a line with pruned input frequencies q = -K..K:
//   out[l] = sum_q in[q + K] * f(q) * e^{+2 pi i q l / nf},  f(q) = (-1)^q / phihat[|q|].
// Line (lo, li), li < inner: input elements (complex) at in + lo in_outer + li in_inner + (q + K) istride, output
// (complex; REAL: the real part in FP32) at out + lo out_outer + li out_inner + l ostride, all in elements.
// Bound by LDS and memory: NT = nf / 4 lanes (at most 64) per line, radix 4, 256 / NT lines per workgroup, one
// twiddle table for all.  (A workgroup per line with radix-2 levels and a sine and cosine per butterfly took 40.8 us
// per pass for two 128^3 grids, and a FP64 grid and its conversion came after it; this takes 11 us, and
// 30 for the last, to FP32.)
template <int NT, bool REAL>
__global__ __launch_bounds__(256) void k_ifft_lines(const double2* __restrict__ in, int64_t istride, int64_t in_outer,
                                                    int64_t in_inner, int inner, int64_t nlines, int K,
                                                    const double* __restrict__ phihat, int nf, int logn,
                                                    void* __restrict__ out, int64_t ostride, int64_t out_outer,
                                                    int64_t out_inner) {
  extern __shared__ __align__(16) double2 ibuf[];
  constexpr int LINES = 256 / NT;
  const int tid = threadIdx.x, L = 2 * K + 1, ls = nf + 1;
  double2* tw = ibuf + LINES * ls;
  double* fac = reinterpret_cast<double*>(tw + nf / 2);
  const int64_t line0 = (int64_t)blockIdx.x * LINES;
  const int cnt = (int)min((int64_t)LINES, nlines - line0);
  for (int k = tid; k < nf / 2; k += 256) {
    double sn, cs;
    sincospi(-2.0 * k / nf, &sn, &cs);
    tw[k] = make_double2(cs, sn);
  }
  for (int q = tid; q <= K; q += 256) fac[q] = (q & 1) ? -1.0 / phihat[q] : 1.0 / phihat[q];
  for (int e = tid; e < LINES * ls; e += 256) ibuf[e] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int e = tid; e < LINES * L; e += 256) {   // along the line where it is contiguous, else across the lines
    const int j = istride == 1 ? e / L : e % LINES, qi = istride == 1 ? e - j * L : e / LINES, q = qi - K;
    if (j >= cnt) continue;
    const int64_t line = line0 + j, lo = line / inner, li = line - lo * inner;
    const double2 v = in[lo * in_outer + li * in_inner + qi * istride];
    const double f = fac[q < 0 ? -q : q];
    ibuf[j * ls + (__brev((unsigned)(q & (nf - 1))) >> (32 - logn))] = make_double2(v.x * f, v.y * f);
  }
  __syncthreads();
  dit_inverse<NT>(ibuf + tid / NT * ls, tw, nf, tid % NT);
  for (int e = tid; e < LINES * nf; e += 256) {
    const int j = ostride == 1 ? e / nf : e % LINES, l = ostride == 1 ? e - j * nf : e / LINES;
    if (j >= cnt) continue;
    const int64_t line = line0 + j, lo = line / inner, li = line - lo * inner;
    const int64_t o = lo * out_outer + li * out_inner + l * ostride;
    const double2 v = ibuf[j * ls + l];
    if constexpr (REAL) static_cast<float*>(out)[o] = (float)v.x;
    else static_cast<double2*>(out)[o] = v;
  }
}

template <bool REAL>
static void ifft_lines(hipStream_t st, const double* in, int64_t istride, int64_t in_outer, int64_t in_inner, int inner,
                       int64_t nlines, int K, const double* phihat, int nf, int logn, void* out, int64_t ostride,
                       int64_t out_outer, int64_t out_inner) {
  auto launch = [&](auto kernel, int nt) {
    const int lines = 256 / nt;
    const size_t lds = sizeof(double2) * ((size_t)lines * (nf + 1) + nf / 2) + sizeof(double) * (K + 1);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((nlines + lines - 1) / lines)), dim3(256), lds, st,
                       reinterpret_cast<const double2*>(in), istride, in_outer, in_inner, inner, nlines, K, phihat, nf,
                       logn, out, ostride, out_outer, out_inner);
  };
  if (nf <= 16) launch(k_ifft_lines<4, REAL>, 4);
  else if (nf == 32) launch(k_ifft_lines<8, REAL>, 8);
  else if (nf == 64) launch(k_ifft_lines<16, REAL>, 16);
  else if (nf == 128) launch(k_ifft_lines<32, REAL>, 32);
  else launch(k_ifft_lines<64, REAL>, 64);
}

// ES kernel psi(s) = exp(beta (sqrt(1 - (2s/w)^2) - 1)) with beta pre-multiplied by log2 e, so that
// the hardware exp2 takes the exponent directly (it lies in [-beta log2 e, 0]: no range handling) and
// the hardware square root needs no denormal scaling (1 - z^2 below 2^-126 gives psi ~ e^-beta).
struct EsDev2 {
  float beta_log2e;
  float two_over_w;
};

__device__ __forceinline__ float es_eval2(float s, EsDev2 es) {
  const float z = s * es.two_over_w;
  const float r = fmaxf(fmaf(-z, z, 1.0f), 0.0f);
  return __builtin_amdgcn_exp2f(fmaf(es.beta_log2e, __builtin_amdgcn_sqrtf(r), -es.beta_log2e));
}

// Grid coordinate in FP64 -> window start i0 = ceil(u - w/2) and offset s0 = i0 - u.
__device__ __forceinline__ bool window_of(double x, int nf, int w, int* i0, float* s0) {
  const double two_pi = 6.283185307179586476925;
  if (!(x == x) || x < -two_pi || x >= two_pi) return false;
  if (x < -3.14159265358979323846) x += two_pi;
  if (x >= 3.14159265358979323846) x -= two_pi;
  double u = (x + 3.14159265358979323846) * ((double)nf / two_pi);
  double c = ceil(u - 0.5 * w);
  *i0 = (int)c;
  *s0 = (float)(c - u);
  return true;
}

// window_of with the grid scale nf / 2 pi given (no division per point).
__device__ __forceinline__ bool window_at(double x, double scale, int w, int* i0, float* s0) {
  const double two_pi = 6.283185307179586476925;
  if (!(x == x) || x < -two_pi || x >= two_pi) return false;
  if (x < -3.14159265358979323846) x += two_pi;
  if (x >= 3.14159265358979323846) x -= two_pi;
  double u = (x + 3.14159265358979323846) * scale;
  double c = ceil(u - 0.5 * w);
  *i0 = (int)c;
  *s0 = (float)(c - u);
  return true;
}

// d = 2 and 3, W <= 8, from grids in memory: a wave per point, lane b W + c at cell (b, c) of the window's last two
// axes (d = 3: the first axis in a loop).  A load then touches W rows of the window instead of 64 unrelated cells,
// which is what a lane per point waits for.  A wave takes ppw points in turn: a lane per point computes the window
// and the kernel values first.  300 000 points x 2 sets, d = 3, 128^3 cells: 1107 us with a lane per point, 392 so.
template <int W, int D>
__global__ __launch_bounds__(256) void k_interp_wave(const float* __restrict__ grid, int nf, int T,
                                                     const void* __restrict__ Xq, fk_dtype dt, int64_t nq, int ppw,
                                                     EsDev2 es, float* __restrict__ out, int* flags) {
  static_assert(W * W <= 64 && (D == 2 || D == 3), "a window's plane in one wave");
  constexpr int RW = 2 * W + 1;
  __shared__ float tab[4][64 * RW];   // kernel values of the last two axes, per point
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t j0 = ((int64_t)blockIdx.x * 4 + w) * ppw, j = j0 + lane;
  if (j0 >= nq) return;
  const bool mine = lane < ppw && j < nq;
  auto ld = [&](int64_t idx) -> double {
    return dt == FK_F64 ? static_cast<const double*>(Xq)[idx] : (double)static_cast<const float*>(Xq)[idx];
  };
  int i[3] = {0, 0, 0};
  float s[3] = {0.f, 0.f, 0.f};
  bool ok = mine;
#pragma unroll
  for (int a = 0; a < D; ++a) ok = mine && window_of(ld(a * nq + (mine ? j : j0)), nf, W, &i[a + 3 - D], &s[a + 3 - D]) && ok;
  if (mine && !ok) atomicOr(&flags[kFlagRange], 1);
  float k1[W];
#pragma unroll
  for (int a = 0; a < W; ++a) {
    k1[a] = D == 3 ? es_eval2(s[0] + (float)a, es) : 1.f;
    tab[w][lane * RW + a] = ok ? es_eval2(s[1] + (float)a, es) : 0.f;
    tab[w][lane * RW + W + a] = es_eval2(s[2] + (float)a, es);
  }
  if (!ok) i[0] = i[1] = i[2] = 0;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const bool cell = lane < W * W;
  const int b = cell ? lane / W : 0, c = cell ? lane - b * W : 0;
  const int64_t plane = (int64_t)nf * nf, cells = D == 3 ? plane * nf : plane;
  const int np = (int)min((int64_t)ppw, nq - j0);
  for (int t = 0; t < T; ++t) {
    const float* g = grid + t * cells;
    float res = 0.f;
#pragma unroll 4
    for (int p = 0; p < np; ++p) {
      const int p1 = __builtin_amdgcn_readlane(i[0], p), p2 = __builtin_amdgcn_readlane(i[1], p),
                p3 = __builtin_amdgcn_readlane(i[2], p);
      int l2 = p2 + b, l3 = p3 + c;
      l2 = l2 < 0 ? l2 + nf : (l2 >= nf ? l2 - nf : l2);
      l3 = l3 < 0 ? l3 + nf : (l3 >= nf ? l3 - nf : l3);
      const float* q = g + l2 * nf + l3;
      const float wt = cell ? tab[w][p * RW + b] * tab[w][p * RW + W + c] : 0.f;
      float acc = 0.f;
      if constexpr (D == 3) {
#pragma unroll
        for (int a = 0; a < W; ++a) {
          int l1 = p1 + a;
          l1 = l1 < 0 ? l1 + nf : (l1 >= nf ? l1 - nf : l1);
          acc = fmaf(q[l1 * plane], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(k1[a]), p)), acc);
        }
      } else {
        acc = *q;
      }
      acc *= wt;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
      res = lane == p ? acc : res;
    }
    if (mine) out[(int64_t)t * nq + j] = ok ? res : __int_as_float(0x7fc00000);
  }
}

template <int W>
__global__ __launch_bounds__(256) void k_interp(const float* __restrict__ grid, int d, int nf, int T,
                                                const void* __restrict__ Xq, fk_dtype dt, int64_t nq, EsDev2 es,
                                                float* __restrict__ out, int* flags) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nq) return;
  auto ld = [&](int64_t idx) -> double {
    return dt == FK_F64 ? static_cast<const double*>(Xq)[idx] : (double)static_cast<const float*>(Xq)[idx];
  };
  int i1, i2 = 0, i3 = 0;
  float s1, s2 = 0.f, s3 = 0.f;
  bool ok = window_of(ld(j), nf, W, &i1, &s1);
  if (d >= 2) ok = window_of(ld(nq + j), nf, W, &i2, &s2) && ok;
  if (d == 3) ok = window_of(ld(2 * nq + j), nf, W, &i3, &s3) && ok;
  if (!ok) {
    atomicOr(&flags[kFlagRange], 1);
    for (int t = 0; t < T; ++t) out[(int64_t)t * nq + j] = __int_as_float(0x7fc00000);
    return;
  }
  float k1[W], k2[W], k3[W];
#pragma unroll
  for (int a = 0; a < W; ++a) {
    k1[a] = es_eval2(s1 + (float)a, es);
    k2[a] = d >= 2 ? es_eval2(s2 + (float)a, es) : 1.f;
    k3[a] = d == 3 ? es_eval2(s3 + (float)a, es) : 1.f;
  }
  for (int t = 0; t < T; ++t) {
    float acc = 0.f;
    if (d == 1) {
      const float* g = grid + (int64_t)t * nf;
#pragma unroll
      for (int a = 0; a < W; ++a) {
        int l = i1 + a;
        l = l < 0 ? l + nf : (l >= nf ? l - nf : l);
        acc += g[l] * k1[a];
      }
    } else if (d == 3) {
      const float* g = grid + (int64_t)t * nf * nf * nf;
      for (int a = 0; a < W; ++a) {
        int l1 = i1 + a;
        l1 = l1 < 0 ? l1 + nf : (l1 >= nf ? l1 - nf : l1);
        float ra = 0.f;
        for (int b = 0; b < W; ++b) {
          int l2 = i2 + b;
          l2 = l2 < 0 ? l2 + nf : (l2 >= nf ? l2 - nf : l2);
          const float* row = g + ((int64_t)l1 * nf + l2) * nf;
          float rb = 0.f;
#pragma unroll
          for (int c = 0; c < W; ++c) {
            int l3 = i3 + c;
            l3 = l3 < 0 ? l3 + nf : (l3 >= nf ? l3 - nf : l3);
            rb += row[l3] * k3[c];
          }
          ra += rb * k2[b];
        }
        acc += ra * k1[a];
      }
    } else {
      const float* g = grid + (int64_t)t * nf * nf;
#pragma unroll
      for (int a = 0; a < W; ++a) {
        int l1 = i1 + a;
        l1 = l1 < 0 ? l1 + nf : (l1 >= nf ? l1 - nf : l1);
        const float* row = g + (int64_t)l1 * nf;
        float ra = 0.f;
#pragma unroll
        for (int b = 0; b < W; ++b) {
          int l2 = i2 + b;
          l2 = l2 < 0 ? l2 + nf : (l2 >= nf ? l2 - nf : l2);
          ra += row[l2] * k2[b];
        }
        acc += ra * k1[a];
      }
    }
    out[(int64_t)t * nq + j] = acc;
  }
}

// ------------------------------------------------------------------ 2-D prediction from an LDS grid
// For d = 2 the oversampled grid of one coefficient set is small enough for LDS when its length is
// any even number near 2.2 (2m + 1) (not a power of two): the inverse transforms are then plain
// FP64 DFTs (a few hundred lines of at most 186 outputs), and every interpolation read is an LDS
// read instead of an L2 request.

constexpr int kNf2Max = 186;   // (nf + kMaxW)^2 FP32 values fit 160 KB of LDS

// Grid length of the LDS path for d = 2 (0 when the grid would not fit LDS).
static int predict_nf2(int m) {
  const int L = 2 * m + 1;
  const int nf = ((int)std::ceil(2.2 * L) + 7) & ~7;
  return nf <= kNf2Max ? nf : 0;
}

static size_t pad_stride(int nf, int W) { return ((size_t)(nf + W) * (nf + W) + 63) & ~size_t(63); }

// Inverse DFT along axis 0 of theta (one line per (set, q2)), pruned input frequencies q1 = -K..K,
// deconvolved:  tmp[t][l1][q2] = sum_q1 theta[t][q1][q2] (-1)^q1 / phihat[|q1|] e^{+2 pi i q1 l1 / nf}.
__global__ __launch_bounds__(256) void k_idft_cols(const double* __restrict__ theta, int K, int nf,
                                                   const double* __restrict__ phihat, double* __restrict__ tmp) {
  __shared__ double twr[kNf2Max], twi[kNf2Max];
  __shared__ double ar[129], ai[129];
  const int L = 2 * K + 1;
  const int line = blockIdx.x;   // t * L + q2
  const int t = line / L, q2 = line - t * L;
  for (int i = threadIdx.x; i < nf; i += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * i / nf, &sn, &cs);
    twr[i] = cs;
    twi[i] = sn;
  }
  const double* src = theta + 2 * ((size_t)t * L * L + q2);
  for (int q = threadIdx.x; q < L; q += blockDim.x) {
    const int aq = q - K < 0 ? K - q : q - K;
    double f = 1.0 / phihat[aq];
    if (aq & 1) f = -f;
    ar[q] = src[2 * (size_t)q * L] * f;
    ai[q] = src[2 * (size_t)q * L + 1] * f;
  }
  __syncthreads();
  double* dst = tmp + 2 * ((size_t)t * nf * L + q2);
  for (int l = threadIdx.x; l < nf; l += blockDim.x) {
    int r = (int)(((int64_t)(nf - K) * l) % nf);   // (-K) l mod nf
    double sr = 0.0, si = 0.0;
    for (int q = 0; q < L; ++q) {
      sr += ar[q] * twr[r] - ai[q] * twi[r];
      si += ar[q] * twi[r] + ai[q] * twr[r];
      r += l;
      if (r >= nf) r -= nf;
    }
    dst[2 * (size_t)l * L] = sr;
    dst[2 * (size_t)l * L + 1] = si;
  }
}

// Inverse DFT along axis 1 (one line per (set, l1)), deconvolved, real part in FP32, written into
// the periodically padded grid g[t][p1][p2] (P = nf + W rows and columns, padded index p holding the
// grid point (p - W/2) mod nf), so that every window of W cells is contiguous without wrapping.
__global__ __launch_bounds__(256) void k_idft_rows_pad(const double* __restrict__ tmp, int K, int nf, int W,
                                                       const double* __restrict__ phihat, size_t pstride,
                                                       float* __restrict__ g) {
  __shared__ double twr[kNf2Max], twi[kNf2Max];
  __shared__ double ar[129], ai[129];
  const int L = 2 * K + 1, P = nf + W, H = W / 2;
  const int line = blockIdx.x;   // t * nf + l1
  const int t = line / nf, l1 = line - t * nf;
  for (int i = threadIdx.x; i < nf; i += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * i / nf, &sn, &cs);
    twr[i] = cs;
    twi[i] = sn;
  }
  const double* src = tmp + 2 * ((size_t)t * nf * L + (size_t)l1 * L);
  for (int q = threadIdx.x; q < L; q += blockDim.x) {
    const int aq = q - K < 0 ? K - q : q - K;
    double f = 1.0 / phihat[aq];
    if (aq & 1) f = -f;
    ar[q] = src[2 * q] * f;
    ai[q] = src[2 * q + 1] * f;
  }
  __syncthreads();
  float* gt = g + (size_t)t * pstride;
  for (int p2 = threadIdx.x; p2 < P; p2 += blockDim.x) {
    int l = p2 - H;
    l = l < 0 ? l + nf : (l >= nf ? l - nf : l);
    int r = (int)(((int64_t)(nf - K) * l) % nf);
    double sr = 0.0;
    for (int q = 0; q < L; ++q) {
      sr += ar[q] * twr[r] - ai[q] * twi[r];
      r += l;
      if (r >= nf) r -= nf;
    }
    const float v = (float)sr;
    // padded rows of grid row l1: l1 + H, and its periodic copies inside [0, P)
    for (int p1 = l1 + H - nf; p1 < P; p1 += nf)
      if (p1 >= 0) gt[(size_t)p1 * P + p2] = v;
  }
}

// f_t(x_j) for the points of one chunk (1024 NPT points, NPT per thread) and the sets t0 .. t0 + ts - 1,
// each set's padded grid in LDS in turn.
//
// Bound by LDS: w^2 reads per point and set at unrelated addresses.  All reads of a point have its base
// address plus an offset that is the same for every lane, so lanes whose base addresses lie in different
// banks never conflict.  The chunk is therefore ordered by the bank of the base address (a counting sort
// over the 64 banks in LDS): lane l takes points of bank l, and the few points over a bank's share fill
// the slots that other banks leave empty.  The kernel values are computed once per point, and kept in
// registers for all sets.  Results are staged in LDS in the order of the input and written as runs.
// 3e6 points x 16 sets at m = 32, w = 8: 675 us with unordered points, one set per workgroup and the
// kernel values per set; 390 us now (LDS busy 250 of them).  Loading the next set's grid into registers
// meanwhile costs a point per thread: 421 us.
constexpr int kLds = 160 * 1024;
constexpr int kBanks = 64;
template <int W>
constexpr int interp_npt() { return W <= 8 ? 4 : (W <= 12 ? 2 : 1); }
constexpr int IT = 1024;   // threads (four waves per SIMD, 128 registers each)

template <int W, int NPT>
__global__ __launch_bounds__(IT) void k_interp2_lds(const float* __restrict__ gpad, size_t pstride, int nf, int T,
                                                      int ts, const void* __restrict__ Xq, fk_dtype dt, int64_t nq,
                                                      double scale, EsDev2 es, int staged, float* __restrict__ out,
                                                      int* flags) {
  extern __shared__ __align__(16) float gl[];   // records of the ordered points, then grid and staging
  constexpr int H = W / 2, PTS = IT * NPT, CAP = PTS / kBanks;
  const int P = nf + W, tid = threadIdx.x;
  const int ngrp = (T + ts - 1) / ts;
  const int t0 = (blockIdx.x % ngrp) * ts, t1 = min(T, t0 + ts);
  const int64_t j0 = (int64_t)(blockIdx.x / ngrp) * PTS;
  const int count = (int)min((int64_t)PTS, nq - j0);
  // record of a point: offsets s1, s2, base address (all ones: outside [-2 pi, 2 pi)), index in the chunk
  struct __align__(16) Rec {
    float s1, s2;
    uint32_t addr, j;
  };
  Rec* rec = reinterpret_cast<Rec*>(gl);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(rec + PTS);   // points, points over and slots free, per bank
  uint32_t* over = cnt + kBanks;
  uint32_t* hole = over + kBanks;
  if (tid < kBanks) cnt[tid] = 0;
  __syncthreads();
  auto ld = [&](int64_t idx) -> double {
    return dt == FK_F64 ? static_cast<const double*>(Xq)[idx] : (double)static_cast<const float*>(Xq)[idx];
  };
  constexpr uint32_t kOut = 0xffffffffu, kNone = 0xfffffffeu;   // out of range; an empty slot
  Rec r[NPT];
  uint32_t rank[NPT];
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    const int j = u * IT + tid;
    r[u].addr = kNone;
    r[u].j = j;
    if (j < count) {
      int i1, i2;
      const bool ok1 = window_at(ld(j0 + j), scale, W, &i1, &r[u].s1);
      const bool ok2 = window_at(ld(nq + j0 + j), scale, W, &i2, &r[u].s2);
      r[u].addr = ok1 && ok2 ? (uint32_t)((i1 + H) * P + (i2 + H)) : kOut;
      if (!(ok1 && ok2)) atomicOr(&flags[kFlagRange], 1);
      rank[u] = atomicAdd(&cnt[r[u].addr % kBanks], 1u);
    }
  }
#pragma unroll
  for (int u = 0; u < NPT; ++u) rec[u * IT + tid].addr = kNone;
  __syncthreads();
  if (tid < kBanks) {   // exclusive sums of the points over, and of the slots free, per bank
    const int c = (int)cnt[tid];
    uint32_t a = (uint32_t)max(0, c - CAP), b = (uint32_t)max(0, CAP - c);
    const uint32_t a0 = a, b0 = b;
#pragma unroll
    for (int o = 1; o < kBanks; o <<= 1) {
      const uint32_t x = __shfl_up(a, o, 64), y = __shfl_up(b, o, 64);
      if (tid >= o) {
        a += x;
        b += y;
      }
    }
    over[tid] = a - a0;
    hole[tid] = b - b0;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    if (r[u].addr == kNone) continue;
    const uint32_t bank = r[u].addr % kBanks;
    uint32_t slot;
    if (rank[u] < (uint32_t)CAP) {
      slot = rank[u] * kBanks + bank;
    } else {
      const uint32_t o = over[bank] + (rank[u] - CAP);   // the o-th free slot: last bank with hole[] <= o
      int lo = 0;
#pragma unroll
      for (int st = kBanks / 2; st > 0; st >>= 1)
        if (hole[lo + st] <= o) lo += st;
      slot = (cnt[lo] + (o - hole[lo])) * kBanks + lo;
    }
    rec[slot] = r[u];
  }
  __syncthreads();
  float k1[NPT][W], k2[NPT][W];
  uint32_t base[NPT], jj[NPT];
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    const Rec q = rec[u * IT + tid];
    const bool real = q.addr < kNone;
    base[u] = real ? q.addr : (uint32_t)(tid % kBanks);   // any address inside the grid, of the lane's bank
    jj[u] = q.addr == kNone ? kNone : (q.addr == kOut ? (q.j | 0x80000000u) : q.j);
#pragma unroll
    for (int a = 0; a < W; ++a) {
      k1[u][a] = es_eval2((real ? q.s1 : 0.f) + (float)a, es);
      k2[u][a] = es_eval2((real ? q.s2 : 0.f) + (float)a, es);
    }
  }
  __syncthreads();   // the records are read: the grids take their memory
  float* so = gl + pstride;
  const int n4 = (int)(pstride / 4);
  for (int t = t0; t < t1; ++t) {
    const float4* src = reinterpret_cast<const float4*>(gpad + (size_t)t * pstride);
    for (int i = tid; i < n4; i += IT) reinterpret_cast<float4*>(gl)[i] = src[i];
    __syncthreads();
    float* ot = out + (int64_t)t * nq + j0;
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      // (a branch around each point: without it the compiler issues the reads of all points at once and
      // runs out of registers)
      if (jj[u] == kNone) continue;
      const float* gp = gl + base[u];
      float acc = 0.f;
#pragma unroll
      for (int a = 0; a < W; ++a) {
        const float* row = gp + a * P;
        float ra = 0.f;
#pragma unroll
        for (int c = 0; c < W; ++c) ra += row[c] * k2[u][c];
        acc += ra * k1[u][a];
      }
      if (jj[u] & 0x80000000u) acc = __int_as_float(0x7fc00000);
      const uint32_t j = jj[u] & 0x7fffffffu;
      if (staged) so[j] = acc;
      else ot[j] = acc;
    }
    __syncthreads();
    if (staged)
      for (int j = tid; j < count; j += IT) ot[j] = so[j];
  }
}

// ------------------------------------------------------------------ few points: direct sums
// f_t(x_j) = Re sum_k theta_k e^{i k.x_j} in FP64, for calls so small that the grids of the type-2
// transform cost more than the sums.  A workgroup takes DP points of one set: lane (p, s) of a wave the
// last-axis modes s, s + 8, ... of point p, whose phases stay in registers (a rotation by e^{8 i x}
// from one to the next), the waves the rows (the modes of the other axes) in turn.  Bound by latency at
// the sizes that take it: 1000 points at m = 32 in 8.2 us, against 18.5 us for the three kernels of the
// transform.
constexpr int DP = 8;              // points per workgroup
constexpr int DW = 8;              // waves per workgroup

// sin and cos of a, |a| < 1e4: Cody-Waite reduction by pi/2 in two parts and the Taylor series on
// [-pi/4, pi/4] (to a^17 and a^16, below 1e-16).
__device__ __forceinline__ void sincos_small(double a, double* sn, double* cs) {
  const double k = rint(a * 0.63661977236758134308);
  double r = fma(-k, 1.57079632679489655800, a);
  r = fma(-k, 6.12323399573676603587e-17, r);
  const double z = r * r;
  double p = 1.0 / 355687428096000.0, q = 1.0 / 20922789888000.0;
  p = fma(p, z, -1.0 / 1307674368000.0);
  q = fma(q, z, -1.0 / 87178291200.0);
  p = fma(p, z, 1.0 / 6227020800.0);
  q = fma(q, z, 1.0 / 479001600.0);
  p = fma(p, z, -1.0 / 39916800.0);
  q = fma(q, z, -1.0 / 3628800.0);
  p = fma(p, z, 1.0 / 362880.0);
  q = fma(q, z, 1.0 / 40320.0);
  p = fma(p, z, -1.0 / 5040.0);
  q = fma(q, z, -1.0 / 720.0);
  p = fma(p, z, 1.0 / 120.0);
  q = fma(q, z, 1.0 / 24.0);
  p = fma(p, z, -1.0 / 6.0);
  q = fma(q, z, -0.5);
  const double s = fma(p * z, r, r), c = fma(q, z, 1.0);
  const int n = (int)k;
  const double u = (n & 1) ? c : s, v = (n & 1) ? s : c;
  *sn = (n & 2) ? -u : u;
  *cs = ((n + 1) & 2) ? -v : v;
}

__device__ __forceinline__ void rot(double& re, double& im, double cr, double ci) {
  const double t = re * cr - im * ci;
  im = fma(re, ci, im * cr);
  re = t;
}

// DK: last-axis modes per lane (8 DK >= 2m + 1).
template <int D, int DK>
__global__ __launch_bounds__(64 * DW) void k_direct(const double2* __restrict__ theta, int m, int64_t nq, fk_dtype dt,
                                                    const void* __restrict__ Xq, float* __restrict__ out, int* flags) {
  __shared__ double part[DW][DP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = lane & 7, s = lane >> 3;
  const int L = 2 * m + 1;
  const int64_t j = (int64_t)blockIdx.x * DP + p, jc = min(j, nq - 1);
  const int t = blockIdx.y;
  double x[D];
  bool ok = true;
  const double two_pi = 6.283185307179586476925;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    x[a] = dt == FK_F64 ? static_cast<const double*>(Xq)[a * nq + jc]
                        : (double)static_cast<const float*>(Xq)[a * nq + jc];
    ok = ok && x[a] >= -two_pi && x[a] < two_pi;
    x[a] = ok ? x[a] : 0.0;
  }
  // last axis: e^{i k x} for k = -m + s + 8 q
  double er[DK], ei[DK], br, bi;
  sincos_small(8.0 * x[D - 1], &bi, &br);
  sincos_small((double)(s - m) * x[D - 1], &ei[0], &er[0]);
#pragma unroll
  for (int q = 1; q < DK; ++q) {
    er[q] = er[q - 1];
    ei[q] = ei[q - 1];
    rot(er[q], ei[q], br, bi);
  }
  const int rows = D == 1 ? 1 : (D == 2 ? L : L * L);
  double acc = 0.0;
  const double2* th = theta + (size_t)t * rows * L;
  double cs = 1.0, sn = 0.0, dr = 1.0, di = 0.0;   // D = 2: phase of row r, and from row r to row r + DW
  if constexpr (D == 2) {
    sincos_small((double)(w - m) * x[0], &sn, &cs);
    sincos_small((double)DW * x[0], &di, &dr);
  }
  for (int r = w; r < rows; r += DW) {
    double sr = 0.0, si = 0.0;
    const double2* row = th + (size_t)r * L;
    double2 v[DK];
#pragma unroll
    for (int q = 0; q < DK; ++q) v[q] = row[min(s + 8 * q, L - 1)];
#pragma unroll
    for (int q = 0; q < DK; ++q) {
      if (8 * q + 8 > L && s + 8 * q >= L) v[q] = make_double2(0.0, 0.0);
      sr = fma(v[q].x, er[q], fma(-v[q].y, ei[q], sr));
      si = fma(v[q].x, ei[q], fma(v[q].y, er[q], si));
    }
    if constexpr (D == 1) {
      acc += sr;
    } else {
      if constexpr (D == 3) sincos_small((double)(r / L - m) * x[0] + (double)(r % L - m) * x[1], &sn, &cs);
      acc = fma(sr, cs, fma(-si, sn, acc));
      if constexpr (D == 2) rot(cs, sn, dr, di);
    }
  }
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
  if (s == 0) part[w][p] = acc;
  __syncthreads();
  if (threadIdx.x < DP && j < nq) {
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < DW; ++i) v += part[i][p];
    if (!ok) atomicOr(&flags[kFlagRange], 1);
    out[(int64_t)t * nq + j] = ok ? (float)v : __int_as_float(0x7fc00000);
  }
}

static int ilog2i(int v) {
  int r = 0;
  while ((1 << r) < v) ++r;
  return r;
}

static size_t grid_cells(int d, int nf) {
  size_t g = 1;
  for (int a = 0; a < d; ++a) g *= (size_t)nf;
  return g;
}

static size_t predict_ws(int d, int m, int T) {
  int nf = 16;
  while (nf < 2 * (2 * m + 1)) nf <<= 1;
  const int L = 2 * m + 1;
  Carve cv(nullptr, 0);
  if (d == 2 && predict_nf2(m)) {
    const int nf2 = predict_nf2(m);
    cv.take<double>((size_t)T * nf2 * L * 2);
    cv.take<float>((size_t)T * pad_stride(nf2, kMaxW));
    return cv.off + 512;
  }
  if (d == 2) cv.take<double>((size_t)T * nf * L * 2);
  if (d == 3) {
    cv.take<double>((size_t)T * nf * L * L * 2);
    cv.take<double>((size_t)T * nf * nf * L * 2);
  }
  cv.take<double>((size_t)T * grid_cells(d, nf));
  cv.take<float>((size_t)T * grid_cells(d, nf));
  return cv.off + 512;
}

// d = 3 is limited to m <= 31 (grid 128^3) and 64 coefficient sets per call.
static bool predict_shape_ok(int d, int m, int T) {
  if (d < 1 || d > 3 || m < 1 || m > 64 || T < 1 || T > 4096) return false;
  return d < 3 || (m <= 31 && T <= 64);
}

}  // namespace fk

using namespace fk;

extern "C" fk_status fk_predict_workspace_size(fk_ctx* ctx, int d, int m, int ntheta, size_t* bytes) {
  if (!bytes || !predict_shape_ok(d, m, ntheta)) return FK_EINVAL;
  *bytes = predict_ws(d, m, ntheta);
  return FK_OK;
}

#define FK_W_SWITCH2(w, CALL)                        \
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

namespace fk {

template <int W, int NPT>
static fk_status launch_interp2_n(hipStream_t st, const float* gp, size_t pst, int nf, int T, const void* Xq,
                                  fk_dtype dt, int64_t nq, EsDev2 es, float* out, int* flags) {
  const int64_t chunks = (nq + IT * NPT - 1) / (IT * NPT);
  // sets per workgroup: all of them once the chunks fill the CUs twice, fewer below
  const int ts = (int)std::max<int64_t>(1, std::min<int64_t>(T, T * chunks / 512));
  const int64_t blocks = chunks * ((T + ts - 1) / ts);
  if (blocks > 0x7fffffff) return FK_EINVAL;
  const size_t grid = sizeof(float) * pst, stage = sizeof(float) * IT * NPT;
  const size_t rec = 16 * IT * NPT + 3 * sizeof(uint32_t) * kBanks;
  const int staged = grid + stage <= (size_t)kLds;
  const size_t lds = std::max(rec, grid + (staged ? stage : 0));
  hipLaunchKernelGGL((k_interp2_lds<W, NPT>), dim3((unsigned)blocks), dim3(IT), lds, st, gp, pst, nf, T, ts, Xq, dt,
                     nq, (double)nf / (2.0 * 3.14159265358979323846), es, staged, out, flags);
  return hipGetLastError() == hipSuccess ? FK_OK : FK_EHIP;
}

// Points per thread: as many as the registers allow, fewer where that would leave CUs without a chunk or
// the results without room behind the grid.
template <int W>
static fk_status launch_interp2(hipStream_t st, const float* gp, size_t pst, int nf, int T, const void* Xq,
                                fk_dtype dt, int64_t nq, EsDev2 es, float* out, int* flags) {
  constexpr int NPT = interp_npt<W>();
  auto fits = [&](int npt) {
    return sizeof(float) * (pst + IT * npt) <= (size_t)kLds && nq * T >= (int64_t)256 * IT * npt;
  };
  if constexpr (NPT >= 4)
    if (fits(4)) return launch_interp2_n<W, 4>(st, gp, pst, nf, T, Xq, dt, nq, es, out, flags);
  if constexpr (NPT >= 2)
    if (fits(2)) return launch_interp2_n<W, 2>(st, gp, pst, nf, T, Xq, dt, nq, es, out, flags);
  return launch_interp2_n<W, 1>(st, gp, pst, nf, T, Xq, dt, nq, es, out, flags);
}

template <int DK>
static void launch_direct(fk_ctx* ctx, int d, dim3 grid, const double2* th, int m, int64_t nq, fk_dtype dt,
                          const void* Xq, float* out) {
  if (d == 1)
    hipLaunchKernelGGL((k_direct<1, DK>), grid, dim3(64 * DW), 0, ctx->stream, th, m, nq, dt, Xq, out, ctx->flags);
  else if (d == 2)
    hipLaunchKernelGGL((k_direct<2, DK>), grid, dim3(64 * DW), 0, ctx->stream, th, m, nq, dt, Xq, out, ctx->flags);
  else
    hipLaunchKernelGGL((k_direct<3, DK>), grid, dim3(64 * DW), 0, ctx->stream, th, m, nq, dt, Xq, out, ctx->flags);
}

// Direct sums instead of the transform, where they are estimated to take less: per point and set 0.25 ns
// and 0.45 (d = 3: 0.65, a sine and cosine per row) ps per mode, lanes past the last mode counted
// (measured: 0.65, 2.1 and 8.0 ns at d = 2, m = 8, 32 and 60; 4.7 and 28 ns at d = 3, m = 6 and 16; 0.23
// at d = 1, m = 50), and a workgroup's chain of 58 ns per row, against what the transform costs before its first
// point: launches more, and grids that grow with m (about 5 us at d = 1; 9, 13 and 25 us at d = 2, m = 8, 32 and
// 60, of which three quarters are taken; 20 us at d = 3).  Whole calls, direct / transform: d = 3, m = 6, 2000
// points 36 / 46 us, m = 8, 2000 points 44 / 49, 4000 points 60 / 49, m = 12 and 16, 50 points 62 / 46 and 91 / 62.  Up to 16 points (two workgroups) take the direct
// sums at any m, for their FP64 results.
static bool direct_ok(int d, int m, int T, int64_t nq) {
  const int L = 2 * m + 1;
  const double rows = std::pow((double)L, d - 1), lanes = 8.0 * (L <= 40 ? 5 : (L <= 72 ? 9 : 17));
  const double per_point = 0.25e-3 + rows * lanes * (d == 3 ? 0.65e-6 : 0.45e-6);   // microseconds
  const double fixed = d == 1 ? 4.0 : (d == 2 ? 6.0 + 0.2 * m : 20.0);
  return (double)nq * T * per_point <= fixed && (d < 3 || nq <= 16 || 0.058 * rows <= fixed);
}

// The type-2 stage on a caller-given workspace and deconvolution table (device, plan.K + 1 doubles).
static fk_status predict_impl(fk_ctx* ctx, const EsPlan& plan, const double* phihat, int d, int m, int T,
                              const double* theta, int64_t nq, fk_dtype dt, const void* Xq, float* out, void* ws,
                              size_t ws_bytes) {
  fk_status st = reset_flags(ctx);
  if (st != FK_OK) return st;
  const int nf = plan.nf, logn = ilog2i(nf), L = 2 * m + 1;
  if (direct_ok(d, m, T, nq)) {
    const double2* th = reinterpret_cast<const double2*>(theta);
    const dim3 grid((unsigned)((nq + DP - 1) / DP), T);
    if (L <= 40) launch_direct<5>(ctx, d, grid, th, m, nq, dt, Xq, out);
    else if (L <= 72) launch_direct<9>(ctx, d, grid, th, m, nq, dt, Xq, out);
    else launch_direct<17>(ctx, d, grid, th, m, nq, dt, Xq, out);
    FK_HIP(hipGetLastError());
    return read_flags(ctx);
  }
  Carve cv(ws, ws_bytes);
  if (d == 2 && predict_nf2(m) == nf) {
    // two pruned FP64 DFTs into padded FP32 grids, then one LDS-resident grid per workgroup
    const int W = plan.w;
    const size_t pst = pad_stride(nf, W);
    double* t2 = cv.take<double>((size_t)T * nf * L * 2);
    float* gp = cv.take<float>((size_t)T * pst);
    if (!cv.ok()) return FK_ENOMEM;
    hipLaunchKernelGGL(k_idft_cols, dim3(T * L), dim3(256), 0, ctx->stream, theta, m, nf, phihat, t2);
    hipLaunchKernelGGL(k_idft_rows_pad, dim3(T * nf), dim3(256), 0, ctx->stream, t2, m, nf, W, phihat, pst, gp);
    EsDev2 es{(float)(plan.beta * 1.44269504088896340736), 2.0f / (float)W};
    st = FK_EINVAL;
    FK_W_SWITCH2(W, st = launch_interp2<WW>(ctx->stream, gp, pst, nf, T, Xq, dt, nq, es, out, ctx->flags));
    if (st != FK_OK) return st;
    FK_HIP(hipGetLastError());
    return read_flags(ctx);
  }
  double* tmp = d == 2 ? cv.take<double>((size_t)T * nf * L * 2) : nullptr;
  double* ta = d == 3 ? cv.take<double>((size_t)T * nf * L * L * 2) : nullptr;
  double* tb = d == 3 ? cv.take<double>((size_t)T * nf * nf * L * 2) : nullptr;
  (void)cv.take<double>((size_t)T * grid_cells(d, nf));   // (the sizes that the workspace queries give are kept)
  float* g32 = cv.take<float>((size_t)T * grid_cells(d, nf));
  if (!cv.ok()) return FK_ENOMEM;
  const int64_t L1 = L, nf1 = nf;
  if (d == 1) {
    // one line per target: theta[t][q + m] -> g32[t][l]
    ifft_lines<true>(ctx->stream, theta, 1, L1, 0, 1, T, m, phihat, nf, logn, g32, 1, nf1, 0);
  } else if (d == 3) {
    // axis 0: for each (t, q2, q3) the line over q1 (stride L^2) -> ta[t][l1][q2][q3]
    ifft_lines<false>(ctx->stream, theta, L1 * L1, L1 * L1 * L1, 1, L * L, T * L1 * L1, m, phihat, nf, logn, ta, L1 * L1,
                      nf1 * L1 * L1, 1);
    // axis 1: for each (t, l1, q3) the line over q2 (stride L) -> tb[t][l1][l2][q3]
    ifft_lines<false>(ctx->stream, ta, L1, L1 * L1, 1, L, T * nf1 * L1, m, phihat, nf, logn, tb, L1, nf1 * L1, 1);
    // axis 2: for each (t, l1, l2) the contiguous line over q3 -> g32[t][l1][l2][l3]
    ifft_lines<true>(ctx->stream, tb, 1, L1, 0, 1, T * nf1 * nf1, m, phihat, nf, logn, g32, 1, nf1, 0);
  } else {
    // for each (t, q2): line over q1 (stride L) -> tmp[t][l1][q2]
    ifft_lines<false>(ctx->stream, theta, L1, L1 * L1, 1, L, T * L1, m, phihat, nf, logn, tmp, L1, nf1 * L1, 1);
    // for each (t, l1): line over q2 (contiguous) -> g32[t][l1][l2]
    ifft_lines<true>(ctx->stream, tmp, 1, L1, 0, 1, T * nf1, m, phihat, nf, logn, g32, 1, nf1, 0);
  }
  EsDev2 es{(float)(plan.beta * 1.44269504088896340736), 2.0f / (float)plan.w};
  if (d >= 2 && plan.w <= 8) {
    // points per wave: 64, fewer where the waves would not fill the chip
    const int ppw = (int)std::max<int64_t>(4, std::min<int64_t>(64, nq / 4096));
    const unsigned wb = (unsigned)((nq + 4 * ppw - 1) / (4 * ppw));
    switch (plan.w) {
#define FK_WAVE(WW)                                                                                                 \
  case WW:                                                                                                          \
    if (d == 2)                                                                                                     \
      hipLaunchKernelGGL((k_interp_wave<WW, 2>), dim3(wb), dim3(256), 0, ctx->stream, g32, nf, T, Xq, dt, nq, ppw, es, \
                         out, ctx->flags);                                                                          \
    else                                                                                                            \
      hipLaunchKernelGGL((k_interp_wave<WW, 3>), dim3(wb), dim3(256), 0, ctx->stream, g32, nf, T, Xq, dt, nq, ppw, es, \
                         out, ctx->flags);                                                                          \
    break;
      FK_WAVE(4) FK_WAVE(5) FK_WAVE(6) FK_WAVE(7) FK_WAVE(8)
#undef FK_WAVE
      default: return FK_EINVAL;
    }
    FK_HIP(hipGetLastError());
    return read_flags(ctx);
  }
  const int blocks = (int)((nq + 255) / 256);
  FK_W_SWITCH2(plan.w, hipLaunchKernelGGL(k_interp<WW>, dim3(blocks), dim3(256), 0, ctx->stream, g32, d, nf, T, Xq,
                                          dt, nq, es, out, ctx->flags));
  FK_HIP(hipGetLastError());
  return read_flags(ctx);
}

static bool predict_args_ok(fk_ctx* ctx, int d, int m, int T, const double* theta, int64_t nq, fk_dtype dt,
                            const void* Xq, const float* out) {
  return ctx && theta && Xq && out && predict_shape_ok(d, m, T) && nq >= 1 && (dt == FK_F32 || dt == FK_F64);
}

// ------------------------------------------------------------------ allocation-free prediction
// A file-scope device array holds the intermediates of fk_predict_noalloc: the deconvolution table
// at its start, then the workspace that fk_predict would take from the caller.  Each device has its
// own copy; host code uses only the address hipGetSymbolAddress returns for the device (the array's
// name on the host is a stand-in, not a device address).
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr size_t kScratchTable = 1024;   // phihat, at most 65 doubles
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch[kMaxDevices] = {};

// Resolves this device's copy of the array; called with the device current (from fk_create, and
// again by the entry point if that failed).  Returns FK_EHIP if the address cannot be taken.
fk_status scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return FK_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[device]) return FK_OK;
  void* ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return FK_EHIP;
  g_scratch[device] = ptr;
  return FK_OK;
}

struct Table65 {
  double v[65];
};

__global__ void k_put_table(Table65 t, int count, double* __restrict__ dst) {
  const int i = threadIdx.x;
  if (i < count) dst[i] = t.v[i];
}

}  // namespace fk

extern "C" fk_status fk_predict(fk_ctx* ctx, int d, int m, int T, const double* theta, int64_t nq, fk_dtype dt,
                                const void* Xq, float* out, void* ws, size_t ws_bytes) {
  if (!predict_args_ok(ctx, d, m, T, theta, nq, dt, Xq, out)) return FK_EINVAL;
  if (!ws || ws_bytes < predict_ws(d, m, T)) return FK_ENOMEM;
  FK_HIP(hipSetDevice(ctx->device));
  kept_invalidate(ws, ws_bytes);
  EsPlan plan;
  const double* phihat;
  fk_status st = get_es_plan(ctx, m, &plan, &phihat, d == 2 ? predict_nf2(m) : 0);
  if (st != FK_OK) return st;
  return predict_impl(ctx, plan, phihat, d, m, T, theta, nq, dt, Xq, out, ws, ws_bytes);
}

extern "C" size_t fk_predict_noalloc_max_bytes(void) { return kScratchBytes - kScratchTable; }

extern "C" fk_status fk_predict_noalloc(fk_ctx* ctx, int d, int m, int T, const double* theta, int64_t nq,
                                        fk_dtype dt, const void* Xq, float* out) {
  if (!predict_args_ok(ctx, d, m, T, theta, nq, dt, Xq, out)) return FK_EINVAL;
  if (predict_ws(d, m, T) > kScratchBytes - kScratchTable) return FK_ENOMEM;
  FK_HIP(hipSetDevice(ctx->device));
  fk_status st = scratch_init(ctx->device);
  if (st != FK_OK) return st;
  unsigned char* base = static_cast<unsigned char*>(g_scratch[ctx->device]);
  EsPlan plan;
  st = get_es_plan_host(ctx, m, &plan, d == 2 ? predict_nf2(m) : 0);
  if (st != FK_OK) return st;
  if (plan.phihat.size() != (size_t)m + 1 || m + 1 > 65) return FK_EINVAL;
  // the deconvolution table goes in by value (a kernel argument), so no host buffer must outlive the call
  Table65 tab{};
  for (int i = 0; i <= m; ++i) tab.v[i] = plan.phihat[i];
  double* phihat = reinterpret_cast<double*>(base);
  hipLaunchKernelGGL(k_put_table, dim3(1), dim3(128), 0, ctx->stream, tab, m + 1, phihat);
  FK_HIP(hipGetLastError());
  return predict_impl(ctx, plan, phihat, d, m, T, theta, nq, dt, Xq, out, base + kScratchTable,
                      kScratchBytes - kScratchTable);
}

// ------------------------------------------------------------------ Philox4x32-10 generator
// Salmon et al., SC'11: ten rounds of (hi, lo) = M * c with the Weyl key schedule.

__device__ __forceinline__ void philox10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  for (int r = 0; r < 10; ++r) {
    uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
    uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
    uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

struct Box16 {
  double lo[16], hi[16];
};

__global__ void k_gen_uniform(uint64_t seed, int d, int64_t n, int64_t start, Box16 box, float* __restrict__ X) {
  const double* lo = box.lo;
  const double* hi = box.hi;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint64_t j = (uint64_t)(i + start);
  for (int g = 0; g < (d + 3) / 4; ++g) {
    uint32_t c[4] = {(uint32_t)j, (uint32_t)(j >> 32), (uint32_t)(g == 0 ? 0 : 16 + g), 0u};
    philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    for (int r = 0; r < 4; ++r) {
      int a = 4 * g + r;
      if (a >= d) break;
      double u = (double)(c[r] >> 8) * 5.9604644775390625e-08;  // 2^-24
      double span = __dadd_rn(hi[a], -lo[a]);
      X[(int64_t)a * n + i] = (float)__dadd_rn(lo[a], __dmul_rn(span, u));
    }
  }
}

__global__ void k_gen_targets(uint64_t seed, int ntgt, int64_t n, int64_t start, const float* __restrict__ X,
                              double sigma, float* __restrict__ Y) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint64_t j = (uint64_t)(i + start);
  const double x1 = X[i], x2 = X[n + i];
  const double c2 = cos(x2);
  for (int t = 1; t <= ntgt; ++t) {
    uint32_t c[4] = {(uint32_t)j, (uint32_t)(j >> 32), (uint32_t)t, 0u};
    philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    double u1 = ((double)c[0] + 1.0) * 2.3283064365386963e-10;  // (0, 1]
    double u2 = (double)c[1] * 2.3283064365386963e-10;          // [0, 1)
    double z = sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
    double v = sin((double)t * x1) * c2 + sigma * z;
    Y[(int64_t)(t - 1) * n + i] = (float)v;
  }
}

extern "C" fk_status fk_generate_uniform(fk_ctx* ctx, uint64_t seed, int d, int64_t n, int64_t start,
                                         const double* lo, const double* hi, float* X) {
  if (!ctx || !lo || !hi || !X || d < 1 || d > 16 || n < 1 || start < 0) return FK_EINVAL;
  FK_HIP(hipSetDevice(ctx->device));
  Box16 box;
  for (int a = 0; a < 16; ++a) {
    box.lo[a] = a < d ? lo[a] : 0.0;
    box.hi[a] = a < d ? hi[a] : 0.0;
  }
  hipLaunchKernelGGL(k_gen_uniform, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, seed, d, n, start,
                     box, X);
  FK_HIP(hipGetLastError());
  FK_HIP(hipStreamSynchronize(ctx->stream));
  return FK_OK;
}

extern "C" fk_status fk_generate_targets(fk_ctx* ctx, uint64_t seed, int ntgt, int64_t n, int64_t start,
                                         const float* X, double sigma, float* Y) {
  if (!ctx || !X || !Y || ntgt < 1 || ntgt > 1024 || n < 1 || start < 0) return FK_EINVAL;
  FK_HIP(hipSetDevice(ctx->device));
  hipLaunchKernelGGL(k_gen_targets, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, seed, ntgt, n,
                     start, X, sigma, Y);
  FK_HIP(hipGetLastError());
  FK_HIP(hipStreamSynchronize(ctx->stream));
  return FK_OK;
}
