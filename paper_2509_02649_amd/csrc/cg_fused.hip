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
// device memory).  One system of 2401 unknowns with the collocation term, 48 iterations: 2784 -> 2287 us (before:
// 420 launches of 2 to 15 us).
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

// vec[k] <- (Sigma vec)[k], k < N, in LDS; every thread of the workgroup calls apply(), after a barrier, and the
// result is there for all when it returns.
template <int P_>
struct Product2 {
  static constexpr int P = P_, L = 8 * P, NT = P == 16 ? 640 : 512, RS = L / 2 + 4;
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
    const double2 x0 = v[0], x1 = v[P / 2];   // lane 0, 4m = L: positions 0 and 2m
    const double2* S = s.S + (size_t)row * L;
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
  static constexpr int NT = 256, E = 2;
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
