// Complex FP64 arithmetic and the LDS line transforms of the Toeplitz products: NT threads (lane = 0 .. NT - 1 of
// the line) transform one line of L points; every thread of the workgroup calls them together.
#ifndef FK_CG_FFT_H
#define FK_CG_FFT_H
#include "fk_internal.h"

namespace fk {
namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// Decimation in frequency, natural order in, bit-reversed order out, e^{-2 pi i / L}; tw[k] =
// e^{-2 pi i k / L}, k < L / 2.  Two radix-2 levels per LDS round trip (lengths len and len / 2
// over the four points pos, pos + len/4, pos + len/2, pos + 3 len/4 of a block), then a last
// radix-2 level when log2 L is odd.
template <int NT>
__device__ __forceinline__ void dif_forward(double2* B, const double2* tw, int L, int lane) {
  int len = L, step = 1;
  for (; len >= 4; len >>= 2, step <<= 2) {
    const int q = len >> 2;
    for (int t = lane; t < L / 4; t += NT) {
      const int grp = t / q, pos = t - grp * q;
      const int i0 = grp * len + pos, i1 = i0 + q, i2 = i1 + q, i3 = i2 + q;
      const double2 a0 = B[i0], a1 = B[i1], a2 = B[i2], a3 = B[i3];
      const double2 b0 = cadd(a0, a2), b2 = cmul(csub(a0, a2), tw[pos * step]);
      const double2 b1 = cadd(a1, a3), b3 = cmul(csub(a1, a3), tw[(pos + q) * step]);
      const double2 w = tw[pos * step * 2];
      B[i0] = cadd(b0, b1);
      B[i1] = cmul(csub(b0, b1), w);
      B[i2] = cadd(b2, b3);
      B[i3] = cmul(csub(b2, b3), w);
    }
    __syncthreads();
  }
  if (len == 2) {
    for (int t = lane; t < L / 2; t += NT) {
      const double2 u = B[2 * t], v = B[2 * t + 1];
      B[2 * t] = cadd(u, v);
      B[2 * t + 1] = csub(u, v);
    }
    __syncthreads();
  }
}

// Decimation in time, bit-reversed order in, natural order out, e^{+2 pi i / L} (unnormalised
// inverse): a first radix-2 level when log2 L is odd, then two levels per LDS round trip
// (lengths len and 2 len over the points pos, pos + len/2, pos + len, pos + 3 len/2).
template <int NT>
__device__ __forceinline__ void dit_inverse(double2* B, const double2* tw, int L, int lane) {
  int len = 2, step = L / 2;
  int lg = 0;
  while ((1 << lg) < L) ++lg;
  if (lg & 1) {
    for (int t = lane; t < L / 2; t += NT) {
      const double2 u = B[2 * t], v = B[2 * t + 1];
      B[2 * t] = cadd(u, v);
      B[2 * t + 1] = csub(u, v);
    }
    __syncthreads();
    len = 4;
    step = L / 4;
  }
  for (; len <= L / 2; len <<= 2, step >>= 2) {
    const int h = len >> 1;
    for (int t = lane; t < L / 4; t += NT) {
      const int grp = t / h, pos = t - grp * h;
      const int i0 = grp * 2 * len + pos, i1 = i0 + h, i2 = i0 + len, i3 = i2 + h;
      const double2 w = cconj(tw[pos * step]);
      const double2 c1 = cmul(B[i1], w), c3 = cmul(B[i3], w);
      const double2 a0 = B[i0], a2 = B[i2];
      const double2 b0 = cadd(a0, c1), b1 = csub(a0, c1), b2 = cadd(a2, c3), b3 = csub(a2, c3);
      const double2 v2 = cmul(b2, cconj(tw[pos * (step >> 1)]));
      const double2 v3 = cmul(b3, cconj(tw[(pos + h) * (step >> 1)]));
      B[i0] = cadd(b0, v2);
      B[i2] = csub(b0, v2);
      B[i1] = cadd(b1, v3);
      B[i3] = csub(b1, v3);
    }
    __syncthreads();
  }
}

}  // namespace
}  // namespace fk
#endif
