// Conjugate gradients with one workgroup per system: the whole iteration (product by FFT, dot products, vector
// updates) runs in one kernel, with the intermediate of the product in LDS.  For d = 1, and for d = 2 with
// 8 <= m <= 32; the other sizes run the passes of cg.hip.
//
// d = 2.  The product needs Lf^2 points of which an axis-0 transform fills Lf x (2m + 1): 135 KB of the 160 KB
// of LDS for Lf = 128 and m = 32, 35 KB for Lf = 64 and m <= 16.  Lf = 4m is one short of 4m + 1: of the
// generator's lags -2m .. 2m only the two ends share a cyclic position, and each acts on one pair of
// positions, c[2m] on (2m, 0) and c[-2m] on (0, 2m).  They are left out of the spectrum and added by hand: along
// axis 1 as two products per line, along axis 0 as two more lines (the convolutions of the first and last row
// of x with the generator's end rows).  So m = 32 runs with Lf = 128, not 256.
//
// A line's Lf = 8 P points lie in 8 lanes, point l + 8 r in lane l, register r < P, before and after a
// transform: P-point DFT in registers, twiddle, exchange over the 8 lanes through the line's own LDS storage,
// 8-point DFTs.  Lines of one transform belong to one wave, so exchanges need no barrier.  The direction and the
// product are handed over in LDS too, where the vector updates read them in memory order.
//
// Bound by LDS and FP64 issue in turn (44 and 40 % of the cycles; waves of a phase run it together): at m = 32
// one product is 388 transforms of 128 points.  256 systems of 4225 unknowns, up to 36 iterations: 5143 -> 1233 us
// (before: three passes of Lf = 256 per product, 113 x 36 us, and the vector updates, 36 x 26 us, all through
// device memory).  One system of 2401 unknowns with the collocation term, 48 iterations: 2784 -> 2287 us here (before:
// 420 launches of 2 to 15 us), and 1358 us in four launches per iteration (below).
// Ten waves at Lf = 128: 65 columns need nine, and the registers allow 640 threads without much spilling (1024:
// 1399 against 1320 us).  Keeping the vectors in the columns' registers spilled (3040 us); in row order per
// column, the updates were longer than the product.
#include "fk_internal.h"
#include "cg_fft.h"

#include <algorithm>

namespace fk {
namespace {

constexpr double kC8 = 0.70710678118654752440;    // cos(pi / 4)
constexpr double kC16 = 0.92387953251128675613;   // cos(pi / 8)
constexpr double kS16 = 0.38268343236508977173;   // sin(pi / 8)

// The LDS accesses of a wave are done in order; this keeps the compiler from moving them.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v (c + i s) forward, v (c - i s) inverse, for a forward twiddle c + i s
template <bool INV>
__device__ __forceinline__ double2 twmul(double2 v, double c, double s) {
  return INV ? make_double2(v.x * c + v.y * s, v.y * c - v.x * s) : make_double2(v.x * c - v.y * s, v.x * s + v.y * c);
}
template <bool INV>
__device__ __forceinline__ double2 mul_mi(double2 v) {   // -i v, inverse +i v
  return INV ? make_double2(-v.y, v.x) : make_double2(v.y, -v.x);
}

// The same value, opaque to the compiler: addresses and tests made from it are not kept over the whole iteration
// (kept, they took 190 registers and the transforms spilled).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// (a, b, c, d) -> their 4-point DFT; NZ of them may differ from zero.
template <bool INV, int NZ>
__device__ __forceinline__ void dft4n(double2& a, double2& b, double2& c, double2& d) {
  if constexpr (NZ == 2) {
    const double2 jb = mul_mi<INV>(b), a0 = a;
    a = cadd(a0, b);
    c = csub(a0, b);
    b = cadd(a0, jb);
    d = csub(a0, jb);
  } else {
    const double2 s0 = cadd(a, c), d0 = csub(a, c);
    const double2 s1 = NZ == 3 ? b : cadd(b, d), d1 = NZ == 3 ? b : csub(b, d);
    const double2 jd1 = mul_mi<INV>(d1);
    a = cadd(s0, s1);
    c = csub(s0, s1);
    b = cadd(d0, jd1);
    d = csub(d0, jd1);
  }
}

// 8-point DFT in place; HALF: v[5 .. 7] are zero.
template <bool INV, bool HALF>
__device__ __forceinline__ void dft8(double2* v) {
  dft4n<INV, HALF ? 3 : 4>(v[0], v[2], v[4], v[6]);
  dft4n<INV, HALF ? 2 : 4>(v[1], v[3], v[5], v[7]);
  const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
  const double2 o0 = v[1], o1 = twmul<INV>(v[3], kC8, -kC8), o2 = mul_mi<INV>(v[5]), o3 = twmul<INV>(v[7], -kC8, -kC8);
  v[0] = cadd(e0, o0);
  v[1] = cadd(e1, o1);
  v[2] = cadd(e2, o2);
  v[3] = cadd(e3, o3);
  v[4] = csub(e0, o0);
  v[5] = csub(e1, o1);
  v[6] = csub(e2, o2);
  v[7] = csub(e3, o3);
}

// 16-point DFT in place; HALF: v[9 .. 15] are zero.
template <bool INV, bool HALF>
__device__ __forceinline__ void dft16n(double2* v) {
  dft4n<INV, HALF ? 3 : 4>(v[0], v[4], v[8], v[12]);
#pragma unroll
  for (int a = 1; a < 4; ++a) dft4n<INV, HALF ? 2 : 4>(v[a], v[a + 4], v[a + 8], v[a + 12]);
  v[5] = twmul<INV>(v[5], kC16, -kS16);     // W16^1
  v[6] = twmul<INV>(v[6], kC8, -kC8);       // 2
  v[7] = twmul<INV>(v[7], kS16, -kC16);     // 3
  v[9] = twmul<INV>(v[9], kC8, -kC8);       // 2
  v[10] = mul_mi<INV>(v[10]);               // 4
  v[11] = twmul<INV>(v[11], -kC8, -kC8);    // 6
  v[13] = twmul<INV>(v[13], kS16, -kC16);   // 3
  v[14] = twmul<INV>(v[14], -kC8, -kC8);    // 6
  v[15] = twmul<INV>(v[15], -kC16, kS16);   // 9
  // v[na + 4 kb]: the DFT over na gives frequency kb + 4 ka
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) dft4n<INV, 4>(v[4 * kb], v[4 * kb + 1], v[4 * kb + 2], v[4 * kb + 3]);
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
#pragma unroll
    for (int ka = kb + 1; ka < 4; ++ka) {   // transpose 4 x 4: frequency k at v[k]
      const double2 t = v[4 * kb + ka];
      v[4 * kb + ka] = v[4 * ka + kb];
      v[4 * ka + kb] = t;
    }
}

// Exchange over the 8 lanes of a line: lane l's register k1 goes to lane k1 % 8, register 8 (k1 / 8) + l.  Slot
// of (k1, l): 8 k1 + (l ^ (k1 & 7)); the XOR keeps both sides free of bank conflicts.
struct RowExchange {      // through P x 8 doubles, real parts first
  double* x;
  template <int P>
  __device__ __forceinline__ void run(double2* v, int l) const {
    wave_order();
#pragma unroll
    for (int k = 0; k < P; ++k) x[8 * k + (l ^ (k & 7))] = v[k].x;
    wave_order();
#pragma unroll
    for (int j = 0; j < P / 8; ++j)
#pragma unroll
      for (int a = 0; a < 8; ++a) v[8 * j + a].x = x[8 * (l + 8 * j) + (a ^ l)];
    wave_order();
#pragma unroll
    for (int k = 0; k < P; ++k) x[8 * k + (l ^ (k & 7))] = v[k].y;
    wave_order();
#pragma unroll
    for (int j = 0; j < P / 8; ++j)
#pragma unroll
      for (int a = 0; a < 8; ++a) v[8 * j + a].y = x[8 * (l + 8 * j) + (a ^ l)];
    wave_order();
  }
};
// Element i of row f is at row_at<RS>(f) + i.  Rows 16 banks apart keep the exchanges of four lines apart that an
// 8-byte access of half a wave makes; the two elements by which every other four rows are shifted keep the eight
// rows apart that a 16-byte access down a column makes.
template <int RS>
__device__ __forceinline__ int row_at(int f) { return f * RS + ((f >> 1) & 2); }

template <int RS>
struct ColExchange {      // through the column's own L entries
  double2* x;
  template <int P>
  __device__ __forceinline__ void run(double2* v, int l) const {
    wave_order();
#pragma unroll
    for (int k = 0; k < P; ++k) x[8 * k * RS + row_at<RS>(l ^ (k & 7))] = v[k];
    wave_order();
#pragma unroll
    for (int j = 0; j < P / 8; ++j)
#pragma unroll
      for (int a = 0; a < 8; ++a) v[8 * j + a] = x[8 * (l + 8 * j) * RS + row_at<RS>(a ^ l)];
    wave_order();
  }
};

// Transform of one line; tw[8 k + l] = e^{-2 pi i k l / (8 P)}.  HALF: the registers past P / 2 hold zeros; mid()
// runs between its two stages.
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <int P, bool INV, bool HALF, class Ex, class Mid = Nothing>
__device__ __forceinline__ void line_dft(double2* v, const double2* tw, int l, const Ex& ex, const Mid& mid = Mid{}) {
  if constexpr (P == 16) dft16n<INV, HALF>(v);
  else dft8<INV, HALF>(v);
#pragma unroll
  for (int k = 1; k < P; ++k) {
    const double2 w = tw[8 * k + l];
    v[k] = twmul<INV>(v[k], w.x, w.y);
  }
  ex.template run<P>(v, l);
  mid();
#pragma unroll
  for (int j = 0; j < P / 8; ++j) dft8<INV, false>(v + 8 * j);
  if constexpr (P == 16) {   // v[8 j + k2] holds frequency l + 8 (j + 2 k2): register j + 2 k2
    double2 u[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) u[k] = v[k];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < 8; ++k) v[j + 2 * k] = u[8 * j + k];
  }
}

template <int P>
__device__ __forceinline__ void fill_twiddles(double2* tw, int nt) {
  for (int i = threadIdx.x; i < 8 * P; i += nt) {
    double s, c;
    sincospi(-2.0 * ((i >> 3) * (i & 7)) / (8 * P), &s, &c);
    tw[i] = make_double2(c, s);
  }
}

// ------------------------------------------------------------------ spectrum (d = 2)

// Of a generator, for Lf = L: S[f0][f1] / L^2 with the ends of both axes left out when they alias (4m = L), then
// the two rows of axis-0 lags +2m and -2m, S[L + e][f1] / L; edge[row][2]: the axis-1 lags +2m and -2m of each
// row, as it is added to the line's output (/ L for the frequencies of axis 0).
template <int P>
struct Spec2 {
  static constexpr int L = 8 * P;
  static constexpr size_t elems = (size_t)(L + 2) * (L + 2);
  double2* S;
  __host__ __device__ double2* edge() const { return S + (size_t)(L + 2) * L; }
};

// AXIS 1: rows of the generator; AXIS 0: columns, in place (a line is read whole before it is written).
template <int P, int AXIS>
__global__ __launch_bounds__(256) void k_spec2(const double2* __restrict__ M, int m, Spec2<P> sp) {
  constexpr int L = 8 * P;
  __shared__ __align__(16) double2 tw[L];
  __shared__ double xch[32 * L];
  fill_twiddles<P>(tw, 256);
  __syncthreads();
  const int l = threadIdx.x & 7, line = blockIdx.x * 32 + (threadIdx.x >> 3);
  const int K = 4 * m + 1;
  const bool alias = 4 * m == L;
  const int lim = alias ? 2 * m - 1 : 2 * m;
  const bool live = line < L + 2;
  double2* edge = sp.edge();
  double2 v[P];
  bool row = false;
  int r0 = 0;
  if (AXIS == 1) {
    row = live && (line >= L ? alias : line <= lim || line >= L - lim);
    r0 = line >= L ? (line == L ? 2 * m : -2 * m) : (line <= lim ? line : line - L);
  }
  const double2* g = M + (2 * m - r0) * (int64_t)K;
#pragma unroll
  for (int r = 0; r < P; ++r) {
    const int t = l + 8 * r;
    v[r] = make_double2(0.0, 0.0);
    if (AXIS == 1) {
      if (row && (t <= lim || t >= L - lim)) v[r] = g[2 * m - (t <= lim ? t : t - L)];
    } else if (live) {
      v[r] = line < L ? sp.S[(size_t)t * L + line] : edge[2 * t + line - L];
    }
  }
  line_dft<P, false, false>(v, tw, l, RowExchange{xch + (threadIdx.x >> 3) * L});
  if (!live) return;
  if (AXIS == 1) {
    const double sc = line >= L ? 1.0 / L : 1.0;
#pragma unroll
    for (int r = 0; r < P; ++r) sp.S[(size_t)line * L + l + 8 * r] = make_double2(v[r].x * sc, v[r].y * sc);
    if (l == 0) {
      edge[2 * line] = row ? g[0] : make_double2(0.0, 0.0);
      edge[2 * line + 1] = row ? g[4 * m] : make_double2(0.0, 0.0);
    }
  } else {
    const double sc = line < L ? 1.0 / ((double)L * L) : 1.0 / L;
#pragma unroll
    for (int r = 0; r < P; ++r) {
      const int t = l + 8 * r;
      const double2 o = make_double2(v[r].x * sc, v[r].y * sc);
      if (line < L) sp.S[(size_t)t * L + line] = o;
      else edge[2 * t + line - L] = o;
    }
  }
}

// ------------------------------------------------------------------ products

// One line of axis 1 in place: transform, spectrum row `row`, inverse; x: 8 L bytes of LDS of the line.
template <int P>
__device__ __forceinline__ void conv_regs(double2* v, const double2* tw, double2* x, const Spec2<P>& s, int row, int l,
                                          bool alias) {
  const double2 x0 = v[0], x1 = v[P / 2];   // lane 0, 4m = L: positions 0 and 2m
  const double2* S = s.S + (size_t)row * Spec2<P>::L;
  double2 sv[P];
  const RowExchange ex{reinterpret_cast<double*>(x)};
  line_dft<P, false, true>(v, tw, l, ex, [&] {   // the spectrum's latency behind the second stage
#pragma unroll
    for (int r = 0; r < P; ++r) sv[r] = S[l + 8 * r];
    __builtin_amdgcn_sched_barrier(0);
  });
#pragma unroll
  for (int r = 0; r < P; ++r) v[r] = cmul(v[r], sv[r]);
  line_dft<P, true, false>(v, tw, l, ex);
  if (alias && l == 0) {
    const double2 ep = s.edge()[2 * row], em = s.edge()[2 * row + 1];
    v[P / 2] = cadd(v[P / 2], cmul(ep, x0));
    v[0] = cadd(v[0], cmul(em, x1));
  }
}

// vec[k] <- (Sigma vec)[k], k < N, in LDS; every thread of the workgroup calls apply(), after a barrier, and the
// result is there for all when it returns.
template <int P_>
struct Product2 {
  static constexpr int P = P_, kLines = P, L = 8 * P, NT = P == 16 ? 640 : 512, RS = L / 2 + 4;
  static constexpr int E = ((L / 2 + 1) * (L / 2 + 1) + NT - 1) / NT;   // elements per thread of a vector
  static constexpr size_t lds_elems = (size_t)L * RS + L + 4 * RS;
  Spec2<P> sp[2];
  int m;
  double2 *vec, *tw, *vx, *vy;   // [L][RS] (vectors in its front), twiddles, the first and last row of x, what they
                                 // add to the last and first
  int lane, line;                // of the thread: lane of its line, line

  __device__ __forceinline__ void refresh() {
    lane = fresh(threadIdx.x & 7);
    line = fresh(threadIdx.x >> 3);
  }
  __device__ __forceinline__ void init(double2* lds) {
    vec = lds;
    tw = vec + L * RS;
    vx = tw + L;
    vy = vx + 2 * RS;
    fill_twiddles<P>(tw, NT);
    __syncthreads();
  }
  __device__ __forceinline__ int n0() const { return 2 * m + 1; }

  // one line of axis 1: in[t] -> out[t], t < 2m + 1, through x (8 L bytes); in and out may be x
  __device__ __forceinline__ void conv_line(double2* v, const double2* in, double2* out, double2* x,
                                            const Spec2<P>& s, int row, int l, bool alias) const {
#pragma unroll
    for (int r = 0; r < P; ++r)
      v[r] = r <= P / 2 && l + 8 * r < n0() ? in[l + 8 * r] : make_double2(0.0, 0.0);
    conv_regs<P>(v, tw, x, s, row, l, alias);
#pragma unroll
    for (int r = 0; r <= P / 2; ++r)
      if (l + 8 * r < n0()) out[l + 8 * r] = v[r];
  }

  __device__ __forceinline__ void apply(int which) {
    double2* A = vec;
    const bool alias = 4 * m == L;
    const Spec2<P> s = sp[which];
    refresh();
    int l = lane;
    double2 v[P];
    if (line < n0()) {
#pragma unroll
      for (int r = 0; r < P; ++r)
        v[r] = r <= P / 2 && l + 8 * r < n0() ? vec[(l + 8 * r) * n0() + line] : make_double2(0.0, 0.0);
      if (alias && l == 0) {
        vx[line] = v[0];
        vx[RS + line] = v[P / 2];
      }
    }
    __syncthreads();
    if (line < n0()) {   // axis 0 forward
      line_dft<P, false, true>(v, tw, l, ColExchange<RS>{A + line});
#pragma unroll
      for (int r = 0; r < P; ++r) A[8 * r * RS + row_at<RS>(l) + line] = v[r];
    }
    __syncthreads();
    // axis 1: tasks of 8 lines, one per wave, with 10 waves and 16 tasks a second one for the waves 0-3, 6 and 7
    // (waves go to the four SIMDs in turn: four tasks each)
    const int wv = threadIdx.x >> 6;
    refresh();
    l = lane;
#pragma nounroll
    for (int t = wv; t < L / 8; t = t >= 10 ? L : (wv < 4 ? 10 + wv : (wv < 6 ? L : 8 + wv))) {
      const int row = 8 * t + (line & 7);
      conv_line(v, A + row_at<RS>(row), A + row_at<RS>(row), A + row_at<RS>(row), s, row, l, alias);
    }
    __syncthreads();
    refresh();
    l = lane;
    // axis 0 inverse; the two end rows in a wave that has no column
    const int vl = line - ((n0() + 7) & ~7);
    if (line < n0()) {
#pragma unroll
      for (int r = 0; r < P; ++r) v[r] = A[8 * r * RS + row_at<RS>(l) + line];
      line_dft<P, true, false>(v, tw, l, ColExchange<RS>{A + line});
    } else if (alias && (vl == 0 || vl == 1)) {
      conv_line(v, vx + vl * RS, vy + vl * RS, vy + vl * RS, s, L + vl, l, alias);
    }
    __syncthreads();
    if (line < n0()) {
      if (alias && l == 0) {
        v[P / 2] = cadd(v[P / 2], vy[line]);
        v[0] = cadd(v[0], vy[RS + line]);
      }
#pragma unroll
      for (int r = 0; r <= P / 2; ++r)
        if (l + 8 * r < n0()) vec[(l + 8 * r) * n0() + line] = v[r];
    }
    __syncthreads();
  }
};

// d = 1: the line in LDS, all 256 threads on it; the spectrum is that of the passes (bit-reversed order).
struct Product1 {
  static constexpr int NT = 256, E = 2, kLines = 0;
  const double2* spec[2];
  const double2* tw_g;
  int m, L;
  double2 *vec, *tw;

  __device__ __forceinline__ void init(double2* lds) {
    vec = lds;
    tw = vec + L;
    for (int k = threadIdx.x; k < L / 2; k += NT) tw[k] = tw_g[k];
    __syncthreads();
  }
  __device__ __forceinline__ void apply(int which) {
    for (int t = 2 * m + 1 + threadIdx.x; t < L; t += NT) vec[t] = make_double2(0.0, 0.0);
    __syncthreads();
    dif_forward<NT>(vec, tw, L, threadIdx.x);
    const double sc = 1.0 / L;
    for (int t = threadIdx.x; t < L; t += NT) {
      const double2 s = spec[which][t];
      vec[t] = cmul(vec[t], make_double2(s.x * sc, s.y * sc));
    }
    __syncthreads();
    dit_inverse<NT>(vec, tw, L, threadIdx.x);
  }
};

// ------------------------------------------------------------------ the iteration

struct CgArgs {
  const double2 *M, *Mr, *b, *D;   // Mr, D: with the collocation term only
  int64_t centre;                  // index of lag 0 in M
  int ntgt, N;
  const double *lams, *pw;
  double mu, tol2;
  int first, last, run;            // this launch: starts, ends the solve; its iterations
  double2 *theta, *r, *p, *q;
  double *rho, *bb, *m0, *relres;  // m0: the diagonals of Sigma and Sigma_r, for the host to check
  int *iters, *active, *flags;
};

// sums of a and b over the workgroup, the same bits in every thread; red is free again after the next barrier
template <int NT>
__device__ __forceinline__ void block_sum2(double& a, double& b, double* red) {
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o, 64);
    b += __shfl_down(b, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = a;
    red[2 * (threadIdx.x >> 6) + 1] = b;
  }
  __syncthreads();
  a = b = 0.0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    a += red[2 * k];
    b += red[2 * k + 1];
  }
}

// One system: q = (Sigma + lambda P [+ mu D^* Sigma_r D]) p, alpha = rho / <p, q>, theta += alpha p, r -= alpha q,
// stop if ||r||^2 <= tol2 ||b||^2, else z = r / dg, beta = <r, z> / rho, p = z + beta p; at most `run`
// iterations, and the true residual where the system leaves.  A non-positive <p, q> (the matrix is not positive
// definite in FP64) stops the system and raises the flag.  Thread i has the elements i + e NT of every vector:
// theta, r and p in device memory (no other thread reads them), q and z in LDS.
template <class Prod, bool COL>
__global__ __launch_bounds__(Prod::NT) void k_cg_fused(Prod prod, CgArgs a) {
  extern __shared__ __align__(16) double2 lds_cg[];
  __shared__ double red[2][2 * (Prod::NT / 64)];
  constexpr int E = Prod::E, NT = Prod::NT;
  const int s = blockIdx.x, N = a.N;
  const double m0 = a.M[a.centre].x, m0r = COL ? a.Mr[a.centre].x : 1.0;
  if (s == 0 && threadIdx.x == 0) {
    a.m0[0] = m0;
    a.m0[1] = m0r;
  }
  if (!(m0 > 0.0) || isinf(m0) || !(m0r > 0.0) || isinf(m0r)) return;   // the host refuses the call
  if (!a.first && !a.active[s]) return;
  prod.init(lds_cg);
  const double lam = a.lams[s / a.ntgt];
  const double2* bt = a.b + (int64_t)(s % a.ntgt) * N;
  double2* th = a.theta + (int64_t)s * N;
  double2* rs = a.r + (int64_t)s * N;
  double2* ps = a.p + (int64_t)s * N;
  double2* qs = a.q + (int64_t)s * N;
  double2* vec = prod.vec;
  // elements of a stage: loads without branches (past the end: the last entry), so that they are in flight together
  auto at = [&](int e, int i) { return min(i + e * NT, N - 1); };
  auto load = [&](auto* x, const auto* src, int i) {
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = src[at(e, i)];
  };
  auto inv_diag = [&](double lp, double2 d) {
    double dg = m0 + lp;
    if constexpr (COL) dg += a.mu * m0r * (d.x * d.x + d.y * d.y);
    return 1.0 / dg;
  };
  double rho, bb;
  int it = 0, act = 1;
  if (a.first) {
    double rz = 0.0, b2 = 0.0;
    for (int k = threadIdx.x; k < N; k += NT) {
      const double2 x = bt[k];
      const double inv = inv_diag(lam * a.pw[k], COL ? a.D[k] : x), n2 = x.x * x.x + x.y * x.y;
      const double2 z = make_double2(x.x * inv, x.y * inv);
      th[k] = make_double2(0.0, 0.0);
      rs[k] = x;
      ps[k] = z;
      vec[k] = z;
      b2 += n2;
      rz += n2 * inv;
    }
    block_sum2<NT>(rz, b2, red[1]);
    rho = rz;
    bb = b2;
    if (!(b2 > 0.0) || isinf(b2)) {
      if (threadIdx.x == 0) {
        if (!(b2 == b2) || isinf(b2)) atomicOr(&a.flags[kFlagNaN], 1);   // a NaN or Inf right-hand side
        a.relres[s] = b2 == 0.0 ? 0.0 : nan("");
        a.iters[s] = 0;
        a.active[s] = 0;
      }
      return;
    }
  } else {
    rho = a.rho[s];
    bb = a.bb[s];
    it = a.iters[s];
    for (int k = threadIdx.x; k < N; k += NT) vec[k] = ps[k];
    __syncthreads();
  }
  bool resid = false;
  int todo = a.run;
  for (;;) {
    if (!resid && todo == 0) {
      if (!a.last) break;
      resid = true;
    }
    const double2* xs = resid ? th : ps;
    if (resid) {
      for (int k = threadIdx.x; k < N; k += NT) vec[k] = xs[k];
      __syncthreads();
    }
    prod.apply(0);
    if constexpr (COL) {
      const int i = fresh(threadIdx.x);
      double2 d[E], x[E];
      load(d, a.D, i);
      load(x, xs, i);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int k = i + e * NT;
        if (k < N) {
          qs[k] = vec[k];
          vec[k] = cmul(d[e], x[e]);
        }
      }
      __syncthreads();
      prod.apply(1);
      const int j = fresh(threadIdx.x);
      load(d, a.D, j);
      load(x, qs, j);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int k = j + e * NT;
        if (k < N) {
          const double2 y = vec[k];
          vec[k] = make_double2(x[e].x + a.mu * (d[e].x * y.x + d[e].y * y.y),
                                x[e].y + a.mu * (d[e].x * y.y - d[e].y * y.x));
        }
      }
    }
    double s1 = 0.0, s2 = 0.0;
    if (resid) {
      for (int k = threadIdx.x; k < N; k += NT) {
        const double lp = lam * a.pw[k];
        const double2 x = bt[k], t = th[k], q = vec[k];
        const double rx = x.x - q.x - lp * t.x, ry = x.y - q.y - lp * t.y;
        s1 += rx * rx + ry * ry;
      }
      block_sum2<NT>(s1, s2, red[0]);
      if (threadIdx.x == 0) a.relres[s] = sqrt(s1 / bb);
      break;
    }
    // p, theta, r and the weights are read once, before the first reduction
    const int i = fresh(threadIdx.x);
    double2 x[E], t[E], w[E];
    double dg[E];
    load(x, ps, i);
    load(dg, a.pw, i);
    load(t, th, i);
    load(w, rs, i);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int k = i + e * NT;
      dg[e] *= lam;
      if (k < N) {
        double2 q = vec[k];
        q.x += dg[e] * x[e].x;
        q.y += dg[e] * x[e].y;
        vec[k] = q;
        s1 += x[e].x * q.x + x[e].y * q.y;
      }
    }
    block_sum2<NT>(s1, s2, red[0]);
    if (!(s1 > 0.0)) {
      if (threadIdx.x == 0) atomicOr(&a.flags[s1 == s1 ? kFlagNotPD : kFlagNaN], 1);   // NaN: one in M or b
      act = 0;
      resid = true;
      continue;
    }
    const double alpha = rho / s1;
    double rr = 0.0, rz = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int k = i + e * NT;
      if (k < N) {
        const double2 q = vec[k];
        const double inv = inv_diag(dg[e], COL ? a.D[k] : q);
        const double2 y = make_double2(w[e].x - alpha * q.x, w[e].y - alpha * q.y);
        const double n2 = y.x * y.x + y.y * y.y;
        th[k] = make_double2(t[e].x + alpha * x[e].x, t[e].y + alpha * x[e].y);
        rs[k] = y;
        rr += n2;
        rz += n2 * inv;
        vec[k] = make_double2(y.x * inv, y.y * inv);
      }
    }
    block_sum2<NT>(rr, rz, red[1]);
    ++it;
    --todo;
    if (rr <= a.tol2 * bb) {
      act = 0;
      resid = true;
      continue;
    }
    const double beta = rz / rho;
    rho = rz;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int k = i + e * NT;
      if (k < N) {
        const double2 z = vec[k], p = make_double2(z.x + beta * x[e].x, z.y + beta * x[e].y);
        ps[k] = p;
        vec[k] = p;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.rho[s] = rho;
    a.bb[s] = bb;
    a.iters[s] = it;
    a.active[s] = act;
  }
}

// ------------------------------------------------------------------ few systems: an iteration in four launches

// With the collocation term (two products per iteration) and Lf = 128, one workgroup per system takes 48 us (m = 24)
// to 59 us (m = 32) per iteration.  For few systems a wave takes 8 lines of one system and one product instead,
// and an iteration is four launches, between which the intermediate and the partial sums go through memory:
// columns forward (with the new direction), rows, columns inverse (with the dot product), vector updates.  Every
// workgroup that needs a sum adds the same partial sums in the same order.  Bound by latency: the four kernels
// take 5.9, 5.3, 5.9 and 3.4 us, and a launch costs the host 6 us.
// One system, m = 24, 48 iterations: 2287 us in one workgroup -> 1358 us.
struct CgSplit {
  CgArgs a;
  int m, n0, N, it, resid;         // it: this iteration; resid: the product of theta, for the true residual
  double2 *T[2], *p2[2], *vy;      // [nsys][L][n0] per product, directions by parity, [nsys][2][2][n0]
  double *part1, *part2, *rho2;    // [nsys][kParts], 2 x [nsys][kParts], rho by parity [2][nsys]
  double* dinv;                    // [nsys][N], 1 / diagonal
  double2* tw;                     // the twiddles
  int nsys, nc, nd;                // workgroups of the column and of the update launches
};
constexpr int kParts = 64, SP = 16, SL = 8 * SP;

__device__ __forceinline__ void load_twiddles(double2* tw, const double2* g, int nt) {
  for (int i = threadIdx.x; i < SL; i += nt) tw[i] = g[i];
}

// sum over the wave, the same bits in every lane
__device__ __forceinline__ double wave_sum(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ double parts_sum(const double* p, int n) {
  const int lane = threadIdx.x & 63;
  return wave_sum(lane < n ? p[lane] : 0.0);
}
__global__ __launch_bounds__(1024) void k_split_init(CgSplit c) {
  __shared__ double red[2 * 16];
  const CgArgs& a = c.a;
  const int s = blockIdx.x, N = c.N;
  const double m0 = a.M[a.centre].x, m0r = a.Mr[a.centre].x;
  if (s == 0 && threadIdx.x == 0) {
    a.m0[0] = m0;
    a.m0[1] = m0r;
  }
  if (s == 0) fill_twiddles<SP>(c.tw, 1024);
  const bool ok = m0 > 0.0 && !isinf(m0) && m0r > 0.0 && !isinf(m0r);
  const double lam = a.lams[s / a.ntgt];
  double rz = 0.0, b2 = 0.0;
  for (int k = threadIdx.x; ok && k < N; k += 1024) {
    const double2 x = a.b[(int64_t)(s % a.ntgt) * N + k];
    double dg = m0 + lam * a.pw[k];
    dg += a.mu * m0r * (a.D[k].x * a.D[k].x + a.D[k].y * a.D[k].y);
    const double inv = 1.0 / dg, n2 = x.x * x.x + x.y * x.y;
    const int64_t e = (int64_t)s * N + k;
    c.dinv[e] = inv;
    a.theta[e] = make_double2(0.0, 0.0);
    a.r[e] = x;
    c.p2[0][e] = make_double2(x.x * inv, x.y * inv);
    b2 += n2;
    rz += n2 * inv;
  }
  block_sum2<1024>(rz, b2, red);
  if (threadIdx.x == 0) {
    c.rho2[s] = rz;
    a.bb[s] = b2;
    a.iters[s] = 0;
    a.active[s] = ok && b2 > 0.0 && !isinf(b2);
    if (ok && (!(b2 == b2) || isinf(b2))) atomicOr(&a.flags[kFlagNaN], 1);   // a NaN or Inf right-hand side
  }
}

// Columns of one product, 8 per wave: stop test of the last iteration, p = r / dg + beta p, axis 0 forward.
__global__ __launch_bounds__(64) void k_split_fwd(CgSplit c) {
  constexpr int P = SP, L = SL, RS = 12;
  __shared__ __align__(16) double2 tw[L], xch[L * RS];
  const CgArgs& a = c.a;
  const int s = blockIdx.y, h = blockIdx.x % 2, blk = blockIdx.x / 2;
  const int l = threadIdx.x & 7, line = threadIdx.x >> 3, i = blk * 8 + line, N = c.N;
  const bool first = blockIdx.x == 0 && threadIdx.x == 0, live = i < c.n0;
  const int64_t o = (int64_t)s * N;
  const double2* src = (c.resid ? a.theta : c.it > 0 ? c.p2[(c.it - 1) & 1] : c.p2[0]) + o;
  // everything is read before the sums are waited for (what a lane does not need: entry 0)
  const bool step = !c.resid && c.it > 0;
  load_twiddles(tw, c.tw, 64);
  double2 v[P], y[P / 2 + 1], d[P / 2 + 1];
  double inv[P / 2 + 1];
#pragma unroll
  for (int r = 0; r <= P / 2; ++r) {
    const int k = live && l + 8 * r < c.n0 ? (l + 8 * r) * c.n0 + i : 0;
    v[r] = src[k];
    y[r] = a.r[o + k];
    inv[r] = c.dinv[o + k];
    d[r] = a.D[k];
  }
  double beta = 0.0;
  if (!c.resid) {
    const int on = a.active[s];
    if (c.it > 0) {
      const double rr = parts_sum(c.part2 + 2 * s * kParts, c.nd), rz = parts_sum(c.part2 + (2 * s + 1) * kParts, c.nd);
      const double rho = c.rho2[((c.it - 1) & 1) * c.nsys + s], bb = a.bb[s];
      if (!on) return;
      if (first) a.iters[s] = c.it;
      if (rr <= a.tol2 * bb) {   // seen alike, or as active = 0, by every workgroup of the system
        if (first) a.active[s] = 0;
        return;
      }
      beta = rz / rho;
      if (first) c.rho2[(c.it & 1) * c.nsys + s] = rz;
    }
    if (!on) return;
  }
  __syncthreads();
  if (!live) return;
  double2* dst = c.p2[c.it & 1] + o;
#pragma unroll
  for (int r = 0; r < P; ++r) {
    if (r > P / 2 || l + 8 * r >= c.n0) {
      v[r] = make_double2(0.0, 0.0);
      continue;
    }
    if (step) {
      v[r] = make_double2(y[r].x * inv[r] + beta * v[r].x, y[r].y * inv[r] + beta * v[r].y);
      if (h == 0) dst[(l + 8 * r) * c.n0 + i] = v[r];
    }
    if (h) v[r] = cmul(d[r], v[r]);
  }
  line_dft<P, false, true>(v, tw, l, ColExchange<RS>{xch + line});
  double2* T = c.T[h] + (int64_t)s * L * c.n0 + i;
#pragma unroll
  for (int r = 0; r < P; ++r) T[(l + 8 * r) * c.n0] = v[r];
}

// Rows of one product, 8 per wave, in place; the two end rows (4m = L) from the direction.
__global__ __launch_bounds__(64) void k_split_rows(CgSplit c, Spec2<SP> s0, Spec2<SP> s1) {
  constexpr int P = SP, L = SL;
  __shared__ __align__(16) double2 tw[L], xch[8 * (L / 2 + 4)];
  const CgArgs& a = c.a;
  const int s = blockIdx.y, h = blockIdx.x % 2, blk = blockIdx.x / 2;
  const int l = threadIdx.x & 7, line = threadIdx.x >> 3, row = blk * 8 + line, n0 = c.n0;
  load_twiddles(tw, c.tw, 64);
  if (!c.resid && !a.active[s]) return;
  __syncthreads();
  const bool alias = 4 * c.m == L;
  if (row >= (alias ? L + 2 : L)) return;
  double2* T = c.T[h] + ((int64_t)s * L + row) * n0;
  const int k0 = row == L ? 0 : 2 * c.m * n0;   // end rows: the first row of x for lag +2m, the last for -2m
  const double2* p = (c.resid ? a.theta : c.p2[c.it & 1]) + (int64_t)s * c.N + k0;
  double2 v[P];
#pragma unroll
  for (int r = 0; r < P; ++r) {
    const int t = l + 8 * r;
    v[r] = make_double2(0.0, 0.0);
    if (r <= P / 2 && t < n0) v[r] = row < L ? T[t] : h ? cmul(a.D[k0 + t], p[t]) : p[t];
  }
  conv_regs<P>(v, tw, xch + line * (L / 2 + 4), h ? s1 : s0, row, l, alias);
  double2* out = row < L ? T : c.vy + ((int64_t)(s * 2 + h) * 2 + row - L) * n0;
#pragma unroll
  for (int r = 0; r <= P / 2; ++r)
    if (l + 8 * r < n0) out[l + 8 * r] = v[r];
}

// Columns, 8 per workgroup and a wave per product: axis 0 inverse, q = all terms (into the first N entries of
// T[0], whose columns the wave has read), and the partial <p, q> or ||b - q||^2.
__global__ __launch_bounds__(128) void k_split_inv(CgSplit c) {
  constexpr int P = SP, L = SL, RS = 12;
  __shared__ __align__(16) double2 tw[L], xch[2][L * RS];
  const CgArgs& a = c.a;
  const int s = blockIdx.y, h = threadIdx.x >> 6, l = threadIdx.x & 7, line = (threadIdx.x >> 3) & 7;
  const int i = blockIdx.x * 8 + line, n0 = c.n0, N = c.N;
  const bool live = i < n0, alias = 4 * c.m == L;
  const int64_t o = (int64_t)s * N;
  const double2* T = c.T[h] + (int64_t)s * L * n0 + (live ? i : 0);
  const double2* p = (c.resid ? a.theta : c.p2[c.it & 1]) + o;
  load_twiddles(tw, c.tw, 128);
  // read before the transform (what a lane does not need: entry 0)
  double2 v[P], x[P / 2 + 1], d[P / 2 + 1];
  double lp[P / 2 + 1];
#pragma unroll
  for (int r = 0; r < P; ++r) v[r] = T[(l + 8 * r) * n0];
#pragma unroll
  for (int r = 0; r <= P / 2; ++r) {
    const int k = live && l + 8 * r < n0 ? (l + 8 * r) * n0 + i : 0;
    x[r] = p[k];
    lp[r] = a.pw[k];
    d[r] = a.D[k];
  }
  if (!c.resid && !a.active[s]) return;
  __syncthreads();
  if (live) {
    line_dft<P, true, false>(v, tw, l, ColExchange<RS>{xch[h] + line});
    if (alias && l == 0) {
      const double2* vy = c.vy + (int64_t)(s * 2 + h) * 2 * n0 + i;
      v[P / 2] = cadd(v[P / 2], vy[0]);
      v[0] = cadd(v[0], vy[n0]);
    }
  }
  if (live && h == 1) {
#pragma unroll
    for (int r = 0; r <= P / 2; ++r) xch[1][(l + 8 * r) * 8 + line] = v[r];
  }
  __syncthreads();
  if (h == 1) return;
  double sum = 0.0;
  const double lam = a.lams[s / a.ntgt];
  double2* q = c.T[0] + (int64_t)s * L * n0;
#pragma unroll
  for (int r = 0; r <= P / 2; ++r)
    if (live && l + 8 * r < n0) {
      const int k = (l + 8 * r) * n0 + i;
      double2 y = make_double2(v[r].x + lam * lp[r] * x[r].x, v[r].y + lam * lp[r] * x[r].y);
      const double2 w = xch[1][(l + 8 * r) * 8 + line];
      y.x += a.mu * (d[r].x * w.x + d[r].y * w.y);
      y.y += a.mu * (d[r].x * w.y - d[r].y * w.x);
      if (c.resid) {
        const double2 b = a.b[(int64_t)(s % a.ntgt) * N + k];
        sum += (b.x - y.x) * (b.x - y.x) + (b.y - y.y) * (b.y - y.y);
      } else {
        q[k] = y;
        sum += x[r].x * y.x + x[r].y * y.y;
      }
    }
  sum = wave_sum(sum);
  if (threadIdx.x == 0) c.part1[s * kParts + blockIdx.x] = sum;
}

// theta += alpha p, r -= alpha q and the partial ||r||^2 and <r, r / dg>.
__global__ __launch_bounds__(256) void k_split_update(CgSplit c) {
  __shared__ double red[2 * 4];
  const CgArgs& a = c.a;
  const int s = blockIdx.y, k = blockIdx.x * 256 + threadIdx.x, N = c.N;
  const int kc = min(k, N - 1);
  const int64_t e = (int64_t)s * N + kc;
  const double2 p = c.p2[c.it & 1][e], q = c.T[0][(int64_t)s * SL * c.n0 + kc];
  double2 t = a.theta[e], r = a.r[e];
  const double inv = c.dinv[e], rho = c.rho2[(c.it & 1) * c.nsys + s];
  const double pq = parts_sum(c.part1 + s * kParts, c.nc);
  if (!a.active[s]) return;
  if (!(pq > 0.0)) {   // seen alike, or as active = 0, by every workgroup of the system
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.active[s] = 0;
      atomicOr(&a.flags[pq == pq ? kFlagNotPD : kFlagNaN], 1);
    }
    return;
  }
  const double alpha = rho / pq;
  double rr = 0.0, rz = 0.0;
  if (k < N) {
    t.x += alpha * p.x;
    t.y += alpha * p.y;
    r.x -= alpha * q.x;
    r.y -= alpha * q.y;
    a.theta[e] = t;
    a.r[e] = r;
    rr = r.x * r.x + r.y * r.y;
    rz = rr * inv;
  }
  block_sum2<256>(rr, rz, red);
  if (threadIdx.x == 0) {
    c.part2[2 * s * kParts + blockIdx.x] = rr;
    c.part2[(2 * s + 1) * kParts + blockIdx.x] = rz;
  }
}

// After the last launch: the stop test of the last iteration, and the true residual.
__global__ __launch_bounds__(64) void k_split_end(CgSplit c) {
  const CgArgs& a = c.a;
  const int s = blockIdx.x;
  const double rr = parts_sum(c.part2 + 2 * s * kParts, c.nd), e = parts_sum(c.part1 + s * kParts, c.nc);
  if (threadIdx.x) return;
  if (a.active[s] && c.it > 0) {
    a.iters[s] = c.it;
    if (rr <= a.tol2 * a.bb[s]) a.active[s] = 0;
  }
  a.relres[s] = a.bb[s] > 0.0 ? sqrt(e / a.bb[s]) : 0.0;
}

fk_status run_split(fk_ctx* ctx, CgSplit c, const Spec2<SP>* sp, int maxit, double* back, size_t back_bytes,
                    int* iters_out, double* relres_out) {
  constexpr int kCheck = 8;   // iterations between reads of the active systems
  hipStream_t st = ctx->stream;
  const int nsys = c.nsys;
  char* h = static_cast<char*>(stage_take(ctx, back_bytes));
  if (!h) return FK_EHIP;
  const double* hm0 = reinterpret_cast<const double*>(h);
  const int* hit = reinterpret_cast<const int*>(hm0 + 2 + nsys);
  const int* hact = hit + nsys;
  const dim3 cols((unsigned)(2 * c.nc), (unsigned)nsys), rows((unsigned)(2 * (4 * c.m == SL ? SP + 1 : SP)), (unsigned)nsys);
  auto product = [&] {
    hipLaunchKernelGGL(k_split_fwd, cols, dim3(64), 0, st, c);
    hipLaunchKernelGGL(k_split_rows, rows, dim3(64), 0, st, c, sp[0], sp[1]);
    hipLaunchKernelGGL(k_split_inv, dim3(c.nc, nsys), dim3(128), 0, st, c);
  };
  hipLaunchKernelGGL(k_split_init, dim3(nsys), dim3(1024), 0, st, c);
  int nact = 1, done = 0;
  while (nact > 0 && done < maxit) {
    for (const int to = std::min(maxit, done + kCheck); done < to; ++done) {
      c.it = done;
      product();
      hipLaunchKernelGGL(k_split_update, dim3(c.nd, nsys), dim3(256), 0, st, c);
    }
    FK_HIP(hipMemcpyAsync(h, back, back_bytes, hipMemcpyDeviceToHost, st));
    FK_HIP(hipStreamSynchronize(st));
    for (int i = 0; i < 2; ++i)
      if (!(hm0[i] > 0.0) || std::isinf(hm0[i])) return FK_EINVAL;
    nact = 0;
    for (int i = 0; i < nsys; ++i) nact += hact[i];
  }
  c.it = done;
  c.resid = 1;
  product();
  hipLaunchKernelGGL(k_split_end, dim3(nsys), dim3(64), 0, st, c);
  FK_HIP(hipMemcpyAsync(h, back, back_bytes, hipMemcpyDeviceToHost, st));
  const fk_status fs = read_flags(ctx);
  if (fs == FK_EHIP) return fs;
  nact = 0;
  int mx = 0;
  for (int i = 0; i < nsys; ++i) {
    nact += hact[i];
    mx = std::max(mx, hit[i]);
  }
  if (relres_out) std::copy(hm0 + 2, hm0 + 2 + nsys, relres_out);
  if (iters_out) *iters_out = mx;
  return fs == FK_OK && nact > 0 ? FK_ENOCONV : fs;
}

template <class Prod>
fk_status run_cg(fk_ctx* ctx, const Prod& prod, CgArgs a, size_t lds, int nsys, int maxit, bool colloc, double* back,
                 size_t back_bytes, int* iters_out, double* relres_out) {
  hipStream_t st = ctx->stream;
  char* h = static_cast<char*>(stage_take(ctx, back_bytes));
  if (!h) return FK_EHIP;
  const double* hm0 = reinterpret_cast<const double*>(h);
  const double* hrel = hm0 + 2;
  const int* hit = reinterpret_cast<const int*>(hrel + nsys);
  const int* hact = hit + nsys;
  // iterations of a launch: enough for most solves, a few ms for one round of workgroups, and fewer with many
  const int chunk = std::max(16, std::min(256, 65536 / nsys));
  int done = 0, mx = 0;
  bool open = true;
  fk_status fs = FK_OK;
  while (open) {
    a.first = done == 0;
    a.run = std::min(chunk, maxit - done);
    done += a.run;
    a.last = done == maxit;
    if (colloc) hipLaunchKernelGGL((k_cg_fused<Prod, true>), dim3(nsys), dim3(Prod::NT), lds, st, prod, a);
    else hipLaunchKernelGGL((k_cg_fused<Prod, false>), dim3(nsys), dim3(Prod::NT), lds, st, prod, a);
    if (hipGetLastError() != hipSuccess) return FK_EHIP;
    FK_HIP(hipMemcpyAsync(h, back, back_bytes, hipMemcpyDeviceToHost, st));
    fs = read_flags(ctx);
    if (fs == FK_EHIP) return fs;
    // the diagonal of Sigma is M[0], real and positive for a positive definite Sigma
    for (int i = 0; i < 2; ++i)
      if (!(hm0[i] > 0.0) || std::isinf(hm0[i])) return FK_EINVAL;
    int nact = 0;
    for (int i = 0; i < nsys; ++i) {
      nact += hact[i];
      mx = std::max(mx, hit[i]);
    }
    open = nact > 0 && done < maxit;
    if (!open) {
      if (relres_out) std::copy(hrel, hrel + nsys, relres_out);
      if (iters_out) *iters_out = mx;
      if (fs == FK_OK && nact > 0) fs = FK_ENOCONV;
    }
  }
  return fs;
}

struct CgInput {
  int m, ntgt, N;
  const double *M, *b, *Mr, *Dsym;
  const std::vector<double>&lams, &pw;
  double mu, tol;
  int maxit;
  double* theta;
  int* iters_out;
  double* relres_out;
};

// The workspace is that of the passes, which has room for their two intermediates where this needs a few KB.
// Four launches per iteration with the collocation term and Lf = 128 up to this many systems (per solve, m = 24 and
// 32: 1450 and 1632 against 2293 and 3069 us with 4 systems, 2041 and 2547 against 2318 and 3088 with 64).  At
// Lf = 64 (15 us per iteration in one workgroup), and without the term (26 to 32 us), the four launches, 25 us and
// more, gain little or lose.
constexpr int kSplitSystems = 64;

template <class Prod>
fk_status solve_fused(fk_ctx* ctx, const CgInput& in, const Prod& prod, size_t lds, Carve& cv) {
  const int nlam = (int)in.lams.size(), nsys = nlam * in.ntgt;
  const bool colloc = in.Mr != nullptr;
  CgArgs a{};
  a.M = reinterpret_cast<const double2*>(in.M);
  a.Mr = reinterpret_cast<const double2*>(in.Mr);
  a.b = reinterpret_cast<const double2*>(in.b);
  a.D = reinterpret_cast<const double2*>(in.Dsym);
  a.centre = 2 * in.m;
  if (in.N > 2 * in.m + 1) a.centre += (int64_t)(2 * in.m) * (4 * in.m + 1);
  a.ntgt = in.ntgt;
  a.N = in.N;
  a.mu = in.mu;
  a.tol2 = in.tol * in.tol;
  a.theta = reinterpret_cast<double2*>(in.theta);
  a.r = cv.take<double2>((size_t)nsys * in.N);
  a.p = cv.take<double2>((size_t)nsys * in.N);
  a.q = colloc ? cv.take<double2>((size_t)nsys * in.N) : nullptr;
  double* up = cv.take<double>((size_t)nlam + in.N);
  a.lams = up;
  a.pw = up + nlam;
  a.rho = cv.take<double>((size_t)nsys);
  a.bb = cv.take<double>((size_t)nsys);
  const size_t back_bytes = sizeof(double) * (2 + (size_t)nsys) + sizeof(int) * 2 * (size_t)nsys;
  double* back = cv.take<double>(2 + 2 * (size_t)nsys);
  a.m0 = back;
  a.relres = back + 2;
  a.iters = reinterpret_cast<int*>(back + 2 + nsys);
  a.active = a.iters + nsys;
  a.flags = ctx->flags;
  if (!cv.ok()) return FK_ENOMEM;
  std::vector<double> h(in.lams);
  h.insert(h.end(), in.pw.begin(), in.pw.begin() + in.N);
  const fk_status s = stage_upload(ctx, up, h.data(), sizeof(double) * h.size());
  if (s != FK_OK) return s;
  if constexpr (Prod::kLines == SP) {
    if (colloc && nsys <= kSplitSystems) {
      const size_t n0 = 2 * (size_t)in.m + 1, t = (size_t)nsys * SL * n0;
      CgSplit c{};
      c.a = a;
      c.m = in.m;
      c.n0 = (int)n0;
      c.N = in.N;
      c.nsys = nsys;
      c.nc = (int)(n0 + 7) / 8;
      c.nd = (in.N + 255) / 256;   // at most 17 (kParts)
      c.p2[0] = a.p;
      c.p2[1] = a.q;
      c.T[0] = cv.take<double2>(t);
      c.T[1] = cv.take<double2>(t);
      c.vy = cv.take<double2>((size_t)nsys * 4 * n0);
      c.part1 = cv.take<double>((size_t)nsys * kParts);
      c.part2 = cv.take<double>((size_t)nsys * 2 * kParts);
      c.rho2 = cv.take<double>((size_t)nsys * 2);
      c.dinv = cv.take<double>((size_t)nsys * in.N);
      c.tw = cv.take<double2>(SL);
      if (!cv.ok()) return FK_ENOMEM;
      return run_split(ctx, c, prod.sp, in.maxit, back, back_bytes, in.iters_out, in.relres_out);
    }
  }
  return run_cg(ctx, prod, a, lds, nsys, in.maxit, colloc, back, back_bytes, in.iters_out, in.relres_out);
}

template <int P>
fk_status solve_fused2(fk_ctx* ctx, const CgInput& in, Carve& cv) {
  Product2<P> prod{};
  prod.m = in.m;
  constexpr unsigned blocks = (8 * P + 2 + 31) / 32;
  for (int i = 0; i <= (in.Mr != nullptr); ++i) {
    prod.sp[i].S = cv.take<double2>(Spec2<P>::elems);
    if (!cv.ok()) return FK_ENOMEM;
    const double2* g = reinterpret_cast<const double2*>(i ? in.Mr : in.M);
    hipLaunchKernelGGL((k_spec2<P, 1>), dim3(blocks), dim3(256), 0, ctx->stream, g, in.m, prod.sp[i]);
    hipLaunchKernelGGL((k_spec2<P, 0>), dim3(blocks), dim3(256), 0, ctx->stream, g, in.m, prod.sp[i]);
  }
  return solve_fused(ctx, in, prod, sizeof(double2) * Product2<P>::lds_elems, cv);
}

}  // namespace

bool cg_fused_ok(int d, int m) { return d == 1 || (d == 2 && m >= 8 && m <= 32); }

fk_status cg_fused_impl(fk_ctx* ctx, int d, int m, const double* M, int ntgt, const double* b,
                        const std::vector<double>& lams, const std::vector<double>& pw, double mu, const double* Mr,
                        const double* Dsym, double tol, int maxit, double* theta_out, int* iters_out,
                        double* relres_out, Carve& cv) {
  const int n0 = 2 * m + 1;
  const CgInput in{m, ntgt, d == 1 ? n0 : n0 * n0, M, b, Mr, Dsym, lams, pw, mu, tol, maxit, theta_out, iters_out,
                   relres_out};
  if (d == 2) return m <= 16 ? solve_fused2<8>(ctx, in, cv) : solve_fused2<16>(ctx, in, cv);
  Product1 prod{};
  prod.m = m;
  const fk_status s = toeplitz_spectra_1d(ctx, m, M, Mr, prod.spec, &prod.tw_g, &prod.L, cv);
  if (s != FK_OK) return s;
  return solve_fused(ctx, in, prod, sizeof(double2) * (size_t)(prod.L + prod.L / 2), cv);
}

}  // namespace fk
