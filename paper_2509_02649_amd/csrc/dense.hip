// Dense stage: assembly of the normal equations in real cosine/sine form, a
// batched blocked Cholesky of FP32 matrices on MFMA (finished panels kept as FP16
// pairs, products on the FP16 matrix cores), FP32 triangular solves, and FP64
// iterative refinement (eq. kenrel_reg; the paper's additive model solves the
// same kind of system directly, Sec. 5 "Complexity").
//
// Real form.  For real data the complex system A theta = b with
// A[-k,-l] = conj A[k,l] and b[-k] = conj b[k] has a Hermitian-symmetric
// solution, and theta = U c with the unitary change of basis
//   c_0 <-> exp(0),  c_{k,cos} <-> sqrt2 cos(k.x),  c_{k,sin} <-> sqrt2 sin(k.x)
// (k in a half space) turns it into the real symmetric system
// (U^* A U) c = U^* b of the same size N and condition number, which costs
// a quarter of the complex factorization.  Real index r of a block of L modes:
// r = 0 constant, r = 2h-1 cosine and r = 2h sine of mode h = 1..(L-1)/2 (the
// modes are counted from the centre of the block in row-major order).
//
// Layout in HBM: every real matrix is Np x Np row-major, Np = N rounded up to a
// multiple of 64, padded with the identity (factor) or zeros (FP64 Gram), so the
// blocked kernels never see a ragged edge.  One FP64 Gram H64 (with any dense,
// lambda-independent penalty folded in) serves all lambdas; each lambda has its
// own FP32 matrix, overwritten by its Cholesky factor below the diagonal blocks (as FP16
// pairs in the same 32-bit slots), and the inverses of its 64 x 64 diagonal blocks.
#include "fk_internal.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

namespace fk {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int NB = 64;     // block size of the factorization
constexpr int LDT = NB + 4; // LDS row stride (floats) of a 64 x 64 tile

// ------------------------------------------------------------------ factor panels as FP16 pairs
// A finished panel of the factor keeps each entry as two FP16 halves in its 32-bit slot:
// a = hi + 2^-11 lo with hi = fp16(a) and lo = fp16(2^11 (a - hi)), both rounded to nearest (the
// splitting of Ootomo and Yokota, 2022, for FP32-accurate products on FP16 matrix units).  The
// left-looking updates multiply such panels as hi*hi + 2^-11 (hi*lo + lo*hi) with FP32 accumulation,
// the lo*lo term (2^-22 relative) dropped: about 22 significant bits per operand at the FP16 matrix
// rate (one v_mfma_f32_16x16x32_f16, 16 cycles, per 16 x 16 x 32 term against eight FP32 16x16x4
// steps, 256 cycles).  The equilibrated factor's entries are at most 1 in magnitude, far inside the
// FP16 range, and the scaled lo keeps entries below the FP16 normal range to 2^-35 absolute.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
constexpr float kSplitScale = 2048.f;

__device__ __forceinline__ uint32_t split_pack(float a) {
  const _Float16 hi = (_Float16)a;
  const _Float16 lo = (_Float16)((a - (float)hi) * kSplitScale);
  return (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}

__device__ __forceinline__ float split_unpack(uint32_t w) {
  const float hi = (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu));
  const float lo = (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
  return fmaf(lo, 1.f / kSplitScale, hi);
}

// A 64 x 64 split tile in LDS: the hi and the lo halves as two row-major FP16 tiles of 128-byte
// rows, unpadded (three tiles per workgroup, three workgroups per CU).  The 16-byte chunk j of row r
// is stored at chunk j ^ sw(r), sw(r) = (r mod 8) ^ (r / 8 mod 2): the 16 rows that one matrix-core
// operand read touches (16 lanes, 16 bytes each) then fall on distinct banks.
struct SplitTile {
  _Float16 hi[NB * NB];
  _Float16 lo[NB * NB];
};
__device__ __forceinline__ int split_off(int r, int c) {   // c: first of 4 (staging) or 8 (reads) columns
  return r * NB + ((((c >> 3) ^ (r & 7) ^ ((r >> 3) & 1))) << 3) + (c & 7);
}

// Four packed entries of one tile row (LDS offset off = split_off(row, first column)) into the hi
// and lo tiles.
__device__ __forceinline__ void split_stage(SplitTile& T, int off, uint4 v) {
  uint2 h, o;
  h.x = (v.x & 0xffffu) | (v.y << 16);
  h.y = (v.z & 0xffffu) | (v.w << 16);
  o.x = (v.x >> 16) | (v.y & 0xffff0000u);
  o.y = (v.z >> 16) | (v.w & 0xffff0000u);
  *reinterpret_cast<uint2*>(&T.hi[off]) = h;
  *reinterpret_cast<uint2*>(&T.lo[off]) = o;
}

// ------------------------------------------------------------------ real-form index maps

struct RealMap {
  int L;      // complex modes per block
  int nblk;   // number of blocks (1, or d for the additive model)
};

// complex index of the mode of real index r, its negation, and the entry type
// (0 const, 1 cos, 2 sin)
__device__ __forceinline__ void real_to_complex(int r, int L, int* type, int* kidx, int* nkidx) {
  int a = r / L, rho = r - a * L;
  int c0 = a * L + (L - 1) / 2;
  if (rho == 0) {
    *type = 0;
    *kidx = c0;
    *nkidx = c0;
  } else {
    int h = (rho + 1) >> 1;
    *type = (rho & 1) ? 1 : 2;
    *kidx = c0 + h;
    *nkidx = c0 - h;
  }
}

struct cplx {
  double re, im;
};
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return {a.re - b.re, a.im - b.im}; }

// Real-form entry from four complex entries (see header comment).
template <class Q>
__device__ double real_entry(const Q& q, int r, int s, int L) {
  int tr, k, nk, ts, l, nl;
  real_to_complex(r, L, &tr, &k, &nk);
  real_to_complex(s, L, &ts, &l, &nl);
  const double rs2 = 0.70710678118654752440;
  if (tr == 0 && ts == 0) return q(k, l).re;
  if (tr == 0) {
    cplx a = q(k, l), b = q(k, nl);
    // (0, cos): (Q(0,l) + Q(0,-l))/sqrt2 ; (0, sin): Re[i (Q(0,-l) - Q(0,l))]/sqrt2
    return ts == 1 ? (a.re + b.re) * rs2 : -(b.im - a.im) * rs2;
  }
  if (ts == 0) {
    cplx a = q(k, l), b = q(nk, l);
    // (cos, 0): (Q(k,0) + Q(-k,0))/sqrt2 ; (sin, 0): Re[-i (Q(-k,0) - Q(k,0))]/sqrt2
    return tr == 1 ? (a.re + b.re) * rs2 : (b.im - a.im) * rs2;
  }
  cplx kl = q(k, l), knl = q(k, nl), nkl = q(nk, l), nknl = q(nk, nl);
  if (tr == 1 && ts == 1) return 0.5 * (kl.re + knl.re + nkl.re + nknl.re);
  if (tr == 2 && ts == 2) return 0.5 * (nknl.re - nkl.re - knl.re + kl.re);
  if (tr == 1) {  // (cos k, sin l) = Re[(i/2)(Q(k,-l) - Q(k,l) + Q(-k,-l) - Q(-k,l))]
    cplx z = csub(cadd(knl, nknl), cadd(kl, nkl));
    return -0.5 * z.im;
  }
  // (sin k, cos l) = Re[(-i/2)(Q(-k,l) + Q(-k,-l) - Q(k,l) - Q(k,-l))]
  cplx z = csub(cadd(nkl, nknl), cadd(kl, knl));
  return 0.5 * z.im;
}

// Complex entry providers ------------------------------------------------

// Toeplitz Gram Sigma[k, l] = M[l - k] from the generator over {-2m..2m}^d.
struct ToeplitzQ {
  const double* M;
  int m, d;
  // Linear offset of mode i in the generator grid (sum over axes of k_a G^a): the entry (i, j) is at
  // off(j) - off(i) + centre, so four entries of one real-form element need four decodes, not eight.
  __device__ int off(int i) const {
    const int L = 2 * m + 1, G = 4 * m + 1;
    int o = 0, mul = 1;
    for (int a = d - 1; a >= 0; --a) {
      const int qd = i / L;
      o += (i - qd * L - m) * mul;
      i = qd;
      mul *= G;
    }
    return o;
  }
  __device__ int centre() const {
    const int G = 4 * m + 1;
    int c = 0, mul = 1;
    for (int a = 0; a < d; ++a) {
      c += 2 * m * mul;
      mul *= G;
    }
    return c;
  }
};

// The four complex entries that real_entry reads for one real-form element (modes k, -k of the
// row and l, -l of the column), through mode offsets: entry (i, j) at M[off(j) - off(i) + centre].
struct ToeplitzPairQ {
  const double* M;
  int c, k, l, ok, onk, ol, onl;
  __device__ cplx operator()(int i, int j) const {
    const int idx = (j == l ? ol : onl) - (i == k ? ok : onk) + c;
    return {M[2 * idx], M[2 * idx + 1]};
  }
};

// Physics-informed penalty of a box (Sec. 4, tractable domains): mu conj(D_k) C[k, l] D_l with the
// operator symbol D (device, N complex) and C[k, l] = (2 pi)^-d prod_a int_{lo_a}^{hi_a}
// exp(i (l_a - k_a) u) du, so that theta^* C theta = (2 pi)^-d int_box |f_theta|^2 for
// f_theta = sum_k theta_k exp(i k.x).  d = 1 or 2.
struct PdeQ {
  const double* dsym;
  int m, d;
  double mu, lo0, hi0, lo1, hi1;
  __device__ static cplx box(int q, double lo, double hi) {
    if (q == 0) return {hi - lo, 0.0};
    double s1, c1, s0, c0;
    sincos(q * hi, &s1, &c1);
    sincos(q * lo, &s0, &c0);
    // (e^{iqhi} - e^{iqlo}) / (iq) = ((s1 - s0) - i (c1 - c0)) / q
    return {(s1 - s0) / q, -(c1 - c0) / q};
  }
  // entry (i, j) with the box integrals of axis a at boxt[a G + (l_a - k_a) + 2m], G = 4m + 1
  __device__ cplx entry(int i, int j, const cplx* boxt, int G) const {
    const int L = 2 * m + 1;
    cplx C;
    if (d == 1) {
      C = boxt[(j - m) - (i - m) + 2 * m];
      const double s = 1.0 / (2.0 * kPi);
      C = {C.re * s, C.im * s};
    } else {
      const int k0 = i / L - m, k1 = i % L - m, l0 = j / L - m, l1 = j % L - m;
      const cplx c0 = boxt[l0 - k0 + 2 * m], c1 = boxt[G + l1 - k1 + 2 * m];
      const double s = 1.0 / (4.0 * kPi * kPi);
      C = {(c0.re * c1.re - c0.im * c1.im) * s, (c0.re * c1.im + c0.im * c1.re) * s};
    }
    const cplx Dk = {dsym[2 * i], dsym[2 * i + 1]}, Dl = {dsym[2 * j], dsym[2 * j + 1]};
    // conj(Dk) * C * Dl
    const cplx t = {Dk.re * C.re + Dk.im * C.im, Dk.re * C.im - Dk.im * C.re};
    return {mu * (t.re * Dl.re - t.im * Dl.im), mu * (t.re * Dl.im + t.im * Dl.re)};
  }
};

// Dense complex matrix [Nc][Nc] (additive block Gram).
struct DenseQ {
  const double* B;
  int Nc;
  __device__ cplx operator()(int i, int j) const {
    size_t o = 2 * ((size_t)i * Nc + j);
    return {B[o], B[o + 1]};
  }
};

// H64[r][s] = real form of Q (r, s < N); zero padding up to Np.  Any block structure (L modes per block).
template <class Q>
__global__ __launch_bounds__(256) void k_assemble_real(Q q, int N, int L, int Np, double* __restrict__ H) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)Np * Np) return;
  int r = (int)(idx / Np), s = (int)(idx - (int64_t)r * Np);
  H[idx] = r < N && s < N ? real_entry(q, r, s, L) : 0.0;
}

// The same for one block of N modes (N odd) with a Toeplitz part: rows 2g - 1 and 2g are the cosine and the
// sine of one pair of modes +-k, so the 2 x 2 entries of a pair of rows and a pair of columns come from the
// same four complex entries.  A thread computes such a block (rows and columns past N: zeros): a quarter of the
// index arithmetic, of the generator reads and, with the physics-informed part, of the box integrals (which
// come from a table per axis here, boxt[q + 2m], filled by the workgroup: they depend on k - l only).
// Toeplitz, N = 4225: 146 us -> 42 (143 MB written); with the heat penalty, N = 1681: 177 -> 22 us.
template <bool PDE>
__global__ __launch_bounds__(256) void k_assemble_pairs(ToeplitzQ tq, PdeQ pq, int N, int Np, double* __restrict__ H) {
  extern __shared__ cplx boxt[];
  const int G = 4 * tq.m + 1;
  if constexpr (PDE) {
    for (int i = threadIdx.x; i < G * pq.d; i += 256) {
      const int ax = i / G, q = i - ax * G - 2 * tq.m;
      boxt[i] = PdeQ::box(q, ax == 0 ? pq.lo0 : pq.lo1, ax == 0 ? pq.hi0 : pq.hi1);
    }
    __syncthreads();
  }
  const int gc = blockIdx.x * 256 + threadIdx.x, gr = blockIdx.y;   // groups 0 .. Np / 2
  if (gc > Np / 2) return;
  const int h = (N - 1) / 2, c0 = h;   // group g <= h: modes c0 + g and c0 - g
  const bool in = gr <= h && gc <= h;
  const int k = c0 + gr, nk = c0 - gr, l = c0 + gc, nl = c0 - gc;
  cplx kl{0, 0}, knl{0, 0}, nkl{0, 0}, nknl{0, 0};
  if (in) {
    const ToeplitzPairQ t{tq.M, tq.centre(), k, l, tq.off(k), tq.off(nk), tq.off(l), tq.off(nl)};
    auto at = [&](int i, int j) -> cplx {
      cplx v = t(i, j);
      if constexpr (PDE) v = cadd(v, pq.entry(i, j, boxt, G));
      return v;
    };
    kl = at(k, l);
    knl = gc ? at(k, nl) : kl;
    nkl = gr ? at(nk, l) : kl;
    nknl = gr ? (gc ? at(nk, nl) : nkl) : knl;
  }
  const double rs2 = 0.70710678118654752440;
  auto put = [&](int r, int c, double v) {
    if (r >= 0 && r < Np && c >= 0 && c < Np) H[(size_t)r * Np + c] = in ? v : 0.0;
  };
  const int r1 = 2 * gr - 1, s1 = 2 * gc - 1;   // cosine rows and columns; sine: + 1; the constant: 0 = 2 * 0
  if (gr == 0 && gc == 0) {
    put(0, 0, kl.re);
  } else if (gr == 0) {
    put(0, s1, (kl.re + knl.re) * rs2);
    put(0, s1 + 1, -(knl.im - kl.im) * rs2);
  } else if (gc == 0) {
    put(r1, 0, (kl.re + nkl.re) * rs2);
    put(r1 + 1, 0, (nkl.im - kl.im) * rs2);
  } else {
    put(r1, s1, 0.5 * (kl.re + knl.re + nkl.re + nknl.re));
    put(r1, s1 + 1, -0.5 * csub(cadd(knl, nknl), cadd(kl, nkl)).im);
    put(r1 + 1, s1, 0.5 * csub(cadd(nkl, nknl), cadd(kl, knl)).im);
    put(r1 + 1, s1 + 1, 0.5 * (nknl.re - nkl.re - knl.re + kl.re));
  }
}

static void launch_assemble_pairs(hipStream_t st, const ToeplitzQ& tq, const PdeQ* pq, int N, int Np, double* H) {
  const dim3 grid((Np / 2 + 256) / 256, Np / 2 + 1);
  if (pq)
    hipLaunchKernelGGL(k_assemble_pairs<true>, grid, dim3(256), sizeof(cplx) * (4 * tq.m + 1) * pq->d, st, tq, *pq, N,
                       Np, H);
  else
    hipLaunchKernelGGL(k_assemble_pairs<false>, grid, dim3(256), 0, st, tq, PdeQ{}, N, Np, H);
}

// Symmetric diagonal equilibration of each lambda's matrix: scl[l][r] =
// 1/sqrt(H64[r][r] + lambda_l preal[r]) (1 on the padding).  The FP32 factor is
// taken of S A S, which keeps the PDE-penalty systems (diagonal spread over many
// decades) inside FP32's reach; refinement applies S on both sides.
__global__ void k_make_scale(const double* __restrict__ H, const double* __restrict__ preal,
                             const double* __restrict__ lams, int N, int Np, double* __restrict__ scl) {
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  const int l = blockIdx.y;
  if (r >= Np) return;
  double v = 1.0;
  if (r < N) {
    double dgl = H[(size_t)r * Np + r] + lams[l] * preal[r];
    v = dgl > 0.0 ? 1.0 / sqrt(dgl) : 1.0;
  }
  scl[(size_t)l * Np + r] = v;
}

// A32[l] = S_l (H64 + lambda_l diag(p_real)) S_l in FP32, identity padding; blocks
// above the block diagonal are not written (no kernel reads them).  One workgroup per 64 x 64
// tile of the lower block triangle (blockIdx.x enumerates them row by row); a thread takes four
// consecutive columns of four rows of H64, read once, and writes them for every lambda.
__global__ __launch_bounds__(256) void k_make_a32(const double* __restrict__ H, const double* __restrict__ preal,
                                                  const double* __restrict__ lams, const double* __restrict__ scl,
                                                  int N, int Np, int nlam, float* __restrict__ A) {
  // tile index x -> (rb, cb), cb <= rb, x = rb (rb + 1) / 2 + cb
  const int x = blockIdx.x;
  int rb = (int)((sqrt(8.0 * x + 1.0) - 1.0) * 0.5);
  while ((rb + 1) * (rb + 2) / 2 <= x) ++rb;
  while (rb * (rb + 1) / 2 > x) --rb;
  const int cb = x - rb * (rb + 1) / 2;
  const int cc = (threadIdx.x & 15) * 4, r0 = threadIdx.x >> 4;
  const int s = cb * NB + cc;
  double h[4][4], pr[4];
  int rows[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = rb * NB + r0 + 16 * u;
    rows[u] = r;
    pr[u] = (r < N) ? preal[r] : 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[u][e] = (r < N && s + e < N) ? H[(size_t)r * Np + s + e] : 0.0;
  }
  for (int l = 0; l < nlam; ++l) {
    const double* sl = scl + (size_t)l * Np;
    const double lam = lams[l];
    double ss[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) ss[e] = sl[s + e];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = rows[u];
      const double sr = sl[r];
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = s + e;
        const bool in = r < N && c < N;
        const double pd = (in && r == c) ? pr[u] : 0.0;
        o[e] = in ? (float)(sr * (h[u][e] + lam * pd) * ss[e]) : (r == c ? 1.0f : 0.0f);
      }
      *reinterpret_cast<float4*>(A + (size_t)l * Np * Np + (size_t)r * Np + s) = make_float4(o[0], o[1], o[2], o[3]);
    }
  }
}

// Workgroups of k_make_a32: the 64 x 64 tiles of the lower block triangle.
static unsigned a32_tiles(int Np) {
  const unsigned nb = (unsigned)(Np / NB);
  return nb * (nb + 1) / 2;
}

// grid.y = 0 (with p): real-form weights preal[r] = p[complex mode of r], zero padded; grid.y = t + 1: real
// right-hand sides Bre[t][r] (Np rows, zero padded) from complex b[t][k].  The real form reads
// the mode k of each pair (k, -k) only (b_-k = conj b_k for real data); a NaN or Inf in either entry
// of the pair is carried into the row, so that the residual norms report it.
__global__ void k_real_inputs(const double* __restrict__ p, const double* __restrict__ b, int N, int L, int Np,
                              double* __restrict__ preal, double* __restrict__ Bre) {
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= Np) return;
  int ty = 0, k = 0, nk = 0;
  if (r < N) real_to_complex(r, L, &ty, &k, &nk);
  if (blockIdx.y == 0) {
    if (p) preal[r] = r < N ? p[k] : 0.0;
    return;
  }
  const int t = blockIdx.y - 1;
  double v = 0.0;
  if (r < N) {
    const double* bt = b + 2 * (size_t)t * N;
    const double s2 = 1.41421356237309504880;
    v = ty == 0 ? bt[2 * k] : (ty == 1 ? s2 * bt[2 * k] : -s2 * bt[2 * k + 1]);
    const double pair = bt[2 * k] + bt[2 * k + 1] + bt[2 * nk] + bt[2 * nk + 1];
    if (!isfinite(pair)) v = pair - pair;   // NaN
  }
  Bre[(size_t)t * Np + r] = v;
}

// theta[l][t][k] (complex) from real solutions X[l][t][r].
__global__ void k_theta_from_real(const double* __restrict__ X, int N, int L, int Np, int ntgt,
                                  double* __restrict__ theta) {
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  int lt = blockIdx.y;  // l * ntgt + t
  if (r >= N) return;
  const double* x = X + (size_t)lt * Np;
  double* th = theta + 2 * (size_t)lt * N;
  int ty, k, nk;
  real_to_complex(r, L, &ty, &k, &nk);
  const double rs2 = 0.70710678118654752440;
  if (ty == 0) {
    th[2 * k] = x[r];
    th[2 * k + 1] = 0.0;
  } else if (ty == 1) {
    double c = x[r], s = x[r + 1];
    th[2 * k] = c * rs2;
    th[2 * k + 1] = -s * rs2;
    th[2 * nk] = c * rs2;
    th[2 * nk + 1] = s * rs2;
  }
}

// ------------------------------------------------------------------ MFMA 64x64x64 tile
// acc += As * Bs^T, As and Bs are 64 x 64 FP32 tiles in LDS with row stride LDT
// (As[row][k], Bs[col][k]).  Wave w owns rows 32*(w>>1).. and cols 32*(w&1)..,
// as 2 x 2 blocks of v_mfma_f32_16x16x4f32.  For that instruction lane l holds
// A[l%16][l/16] and B[l/16][l%16]; the 16 x 16 result row 4*(l/16)+v, column
// l%16 sits in element v of the lane's accumulator.
__device__ __forceinline__ void mfma_tile64(const float* As, const float* Bs, floatx4 acc[2][2]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll 4
  for (int k = 0; k < NB; k += 4) {
    float a0 = As[(r0 + li) * LDT + k + lk];
    float a1 = As[(r0 + 16 + li) * LDT + k + lk];
    float b0 = Bs[(c0 + li) * LDT + k + lk];
    float b1 = Bs[(c0 + 16 + li) * LDT + k + lk];
    acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
  }
}

// Load a 64 x 64 FP32 tile (row-major, leading dimension ld) into LDS (rows of LDT
// floats, 16-byte aligned).
// A 64 x 64 FP32 tile (row stride ld) in four float4 registers per lane of a 256-thread
// workgroup, and its store into an LDS tile of row stride LDT (named registers: an array would be
// kept in scratch memory by the compiler where it lives across other work).
#define FK_F32_LOAD4(src, ld, a0, a1, a2, a3)                                                \
  do {                                                                                       \
    _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_) {                                       \
      const int i_ = threadIdx.x + 256 * u_, r_ = i_ / (NB / 4), c_ = (i_ - r_ * (NB / 4)) * 4; \
      const float4 v_ = *reinterpret_cast<const float4*>((src) + r_ * (ld) + c_);          \
      if (u_ == 0) a0 = v_;                                                                  \
      if (u_ == 1) a1 = v_;                                                                  \
      if (u_ == 2) a2 = v_;                                                                  \
      if (u_ == 3) a3 = v_;                                                                  \
    }                                                                                        \
  } while (0)
#define FK_F32_STORE4(T, a0, a1, a2, a3)                                                     \
  do {                                                                                       \
    _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_) {                                       \
      const int i_ = threadIdx.x + 256 * u_, r_ = i_ / (NB / 4), c_ = (i_ - r_ * (NB / 4)) * 4; \
      *reinterpret_cast<float4*>((T) + r_ * LDT + c_) = u_ == 0 ? a0 : u_ == 1 ? a1 : u_ == 2 ? a2 : a3; \
    }                                                                                        \
  } while (0)

// Two tiles into LDS, all eight loads of a lane issued before any store (one memory latency).
__device__ __forceinline__ void load_tiles2(float* T0, const float* src0, int64_t ld0, float* T1, const float* src1,
                                            int64_t ld1) {
  float4 v0, v1, v2, v3, w0, w1, w2, w3;
  FK_F32_LOAD4(src0, ld0, v0, v1, v2, v3);
  FK_F32_LOAD4(src1, ld1, w0, w1, w2, w3);
  FK_F32_STORE4(T0, v0, v1, v2, v3);
  FK_F32_STORE4(T1, w0, w1, w2, w3);
}

// dst tile (+)= sign * acc
__device__ __forceinline__ void store_acc(float* dst, int64_t ld, const floatx4 acc[2][2], bool add, float sign) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        int r = r0 + rb * 16 + 4 * (lane >> 4) + v;
        int c = c0 + cb * 16 + (lane & 15);
        float x = sign * acc[rb][cb][v];
        if (add) dst[r * ld + c] += x;
        else dst[r * ld + c] = x;
      }
}

// acc[t] += As Bt^T over the 64 k of split tiles (t = 0: B0, t = 1: B1), for the 2 x 2 blocks of
// 16 x 16 a wave owns (rows 32 (w >> 1).., columns 32 (w & 1)..): hi*hi into acc, hi*lo + lo*hi into
// accx.  For v_mfma_f32_16x16x32_f16 lane l supplies row l % 16 of A and column l % 16 of B at the
// 8 k of its lane group l / 16 (the same 8 for both operands); its result layout is the one of
// the FP32 instruction above.
template <int NBT>
__device__ __forceinline__ void mfma_split64(const SplitTile& As, const SplitTile& B0, const SplitTile& B1,
                                             floatx4 (&acc)[NBT][2][2], floatx4 (&accx)[NBT][2][2]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
  const int li = lane & 15, kq = 8 * (lane >> 4);
#pragma unroll
  for (int k = 0; k < NB; k += 32) {
    half8 ah[2], al[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int o = split_off(r0 + 16 * u + li, k + kq);
      ah[u] = *reinterpret_cast<const half8*>(&As.hi[o]);
      al[u] = *reinterpret_cast<const half8*>(&As.lo[o]);
    }
#pragma unroll
    for (int t = 0; t < NBT; ++t) {
      const SplitTile& Bt = t == 0 ? B0 : B1;
      half8 bh[2], bl[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int o = split_off(c0 + 16 * u + li, k + kq);
        bh[u] = *reinterpret_cast<const half8*>(&Bt.hi[o]);
        bl[u] = *reinterpret_cast<const half8*>(&Bt.lo[o]);
      }
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          acc[t][rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[rb], bh[cb], acc[t][rb][cb], 0, 0, 0);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          accx[t][rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[rb], bl[cb], accx[t][rb][cb], 0, 0, 0);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          accx[t][rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[rb], bh[cb], accx[t][rb][cb], 0, 0, 0);
    }
  }
}

// dst tile -= acc + 2^-11 accx
__device__ __forceinline__ void store_split_update(float* dst, int64_t ld, const floatx4 (&acc)[2][2],
                                                   const floatx4 (&accx)[2][2]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + rb * 16 + 4 * (lane >> 4) + v;
        const int c = c0 + cb * 16 + (lane & 15);
        dst[r * ld + c] -= fmaf(accx[rb][cb][v], 1.f / kSplitScale, acc[rb][cb][v]);
      }
}

// dst tile = acc as packed FP16 pairs (a finished panel tile of the factor)
__device__ __forceinline__ void store_acc_split(float* dst, int64_t ld, const floatx4 acc[2][2]) {
  uint32_t* d = reinterpret_cast<uint32_t*>(dst);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + rb * 16 + 4 * (lane >> 4) + v;
        const int c = c0 + cb * 16 + (lane & 15);
        d[r * ld + c] = split_pack(acc[rb][cb][v]);
      }
}

// ------------------------------------------------------------------ Cholesky kernels

// XCD-aware placement of a (rows x nlam) grid launched as one dimension.  The hardware deals the
// workgroups round-robin over the 8 XCDs (XCD = id mod 8); this bijection gives XCD x the
// consecutive run of pairs (lambda, row) in the order (lambda mod 8, lambda / 8, row), so that the
// workgroups of one lambda share one L2, which then holds the column tiles they all read.  Any
// dealing order gives the same result; only the locality depends on it.
__device__ __forceinline__ void xcd_place(int rows, int nlam, int* lam, int* row) {
  const int G = rows * nlam, id = blockIdx.x;
  const int x = id & 7, slot = id >> 3;
  int off = 0;   // workgroups dealt to the XCDs before x
  for (int y = 0; y < x; ++y) off += (G - y + 7) >> 3;
  const int q = off + slot;
  int c = 0, base = 0;   // lambda class c = lambda mod 8 holds ceil((nlam - c) / 8) lambdas
  while (c < 7) {
    const int n = ((nlam - c + 7) >> 3) * rows;
    if (q < base + n) break;
    base += n;
    ++c;
  }
  const int r = q - base;
  *lam = c + 8 * (r / rows);
  *row = r % rows;
}

// 1/x for a positive normal x: hardware reciprocal and two Newton steps
// (r <- r + r (1 - x r)), a few ulp in FP64.
__device__ inline double recip64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// The same update for the two block columns kb and kb + 1 at once, over the panels
// k < kb:  A[i][kb] -= sum L[i][k] L[kb][k]^T  and (i > kb) A[i][kb+1] -= sum
// L[i][k] L[kb+1][k]^T.  The row panel L[i][.], the bulk of the traffic, is read once
// for both columns.  The finished panels are FP16 pairs (split tiles in LDS, products on the
// FP16 matrix cores); one LDS buffer per operand, the next k's tiles loaded into registers
// while the current ones are multiplied.
// Without PART: the panels kfirst <= k < kend, and G pairs of columns from kb on in one launch.  The workgroups of a row's
// G pairs run side by side on one XCD, so that its panel, the bulk of the traffic, comes from memory once for all
// (64 lambdas, N = 4225: 8.7 -> 7.9 ms of updates with G = 2).
template <bool PART>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_left_update2(float* __restrict__ A,
                                                                                             int Np, int kb, int kfirst,
                                                                                             int kend, int G, int nlam,
                                                                                             int nsplit,
                                                                                             float* __restrict__ part) {
  __shared__ __align__(16) SplitTile As;
  __shared__ __align__(16) SplitTile B0;
  __shared__ __align__(16) SplitTile B1;
  const int rows = Np / NB - kb;
  int l, i, k0 = kfirst, k1 = kend, sidx = 0;
  if constexpr (PART) {
    // workgroup (sidx, l, i): panels k0 <= k < k1 of the split sidx of the sum
    const int b = blockIdx.x;
    i = b % rows;
    l = (b / rows) % nlam;
    sidx = b / (rows * nlam);
    k0 = (int)((int64_t)kb * sidx / nsplit);
    k1 = (int)((int64_t)kb * (sidx + 1) / nsplit);
  } else {
    xcd_place(rows * G, nlam, &l, &i);
    const int p = i % G;
    i = i / G - 2 * p;
    if (i < 0) return;   // above the pair's diagonal blocks
    kb += 2 * p;
  }
  i += kb;
  float* Al = A + (size_t)l * Np * Np;
  const uint32_t* Ai = reinterpret_cast<const uint32_t*>(Al + (size_t)i * NB * Np);
  const uint32_t* A0 = reinterpret_cast<const uint32_t*>(Al + (size_t)kb * NB * Np);
  const uint32_t* A1 = reinterpret_cast<const uint32_t*>(Al + (size_t)(kb + 1) * NB * Np);
  int off_g[4], off_s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int idx = threadIdx.x + q * 256, r = idx / (NB / 4), c = (idx % (NB / 4)) * 4;
    off_g[q] = r * Np + c;
    off_s[q] = split_off(r, c);
  }
  uint4 ra[4], rb[4], rc[4];
  auto gload = [&](int k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ra[q] = *reinterpret_cast<const uint4*>(Ai + k * NB + off_g[q]);
      rb[q] = *reinterpret_cast<const uint4*>(A0 + k * NB + off_g[q]);
      rc[q] = *reinterpret_cast<const uint4*>(A1 + k * NB + off_g[q]);
    }
  };
  floatx4 acc[2][2][2] = {}, accx[2][2][2] = {};
  if (k0 < k1) gload(k0);
  for (int k = k0; k < k1; ++k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      split_stage(As, off_s[q], ra[q]);
      split_stage(B0, off_s[q], rb[q]);
      split_stage(B1, off_s[q], rc[q]);
    }
    __syncthreads();
    if (k + 1 < k1) gload(k + 1);
    mfma_split64<2>(As, B0, B1, acc, accx);
    __syncthreads();
  }
  if constexpr (PART) {
    // this split's part of the 64 x 128 update, row-major, columns kb then kb + 1
    float* dst = part + ((size_t)(sidx * nlam + l) * rows + (i - kb)) * (NB * 2 * NB);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int rb2 = 0; rb2 < 2; ++rb2)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int r = r0 + rb2 * 16 + 4 * (lane >> 4) + v;
            const int c = c0 + cb * 16 + (lane & 15);
            dst[r * (2 * NB) + t * NB + c] = fmaf(accx[t][rb2][cb][v], 1.f / kSplitScale, acc[t][rb2][cb][v]);
          }
  } else {
    store_split_update(Al + (size_t)i * NB * Np + kb * NB, Np, acc[0], accx[0]);
    if (i > kb) store_split_update(Al + (size_t)i * NB * Np + (kb + 1) * NB, Np, acc[1], accx[1]);
  }
}

// The split update's parts added in a fixed order (the result does not depend on timing) and
// subtracted from block columns kb, kb + 1 (the tile above the diagonal left alone).  Workgroup
// (tile, eighth): 256 threads x 4 consecutive entries; all parts of an entry are loaded before the
// first addition, so a workgroup waits for memory once.
constexpr int kMaxSplit = 16;
__global__ __launch_bounds__(256) void k_left_update2_sum(float* __restrict__ A, int Np, int kb, int nlam,
                                                          int nsplit, const float* __restrict__ part) {
  const int rows = Np / NB - kb;
  const int tile_id = blockIdx.x >> 3, eighth = blockIdx.x & 7;
  const int ii = tile_id % rows, l = tile_id / rows, i = kb + ii;
  const size_t tile = (size_t)NB * 2 * NB, stride = (size_t)nlam * rows * tile;
  const int e = (eighth * 256 + threadIdx.x) * 4, r = e / (2 * NB), c = e - r * (2 * NB);
  if (c >= NB && i == kb) return;   // above the diagonal (all four entries: c is a multiple of 4)
  const float* src = part + ((size_t)l * rows + ii) * tile + e;
  float4 v[kMaxSplit];
#pragma unroll
  for (int sp = 0; sp < kMaxSplit; ++sp)
    if (sp < nsplit) v[sp] = *reinterpret_cast<const float4*>(src + sp * stride);
  float4 sum = v[0];
#pragma unroll
  for (int sp = 1; sp < kMaxSplit; ++sp)
    if (sp < nsplit) {
      sum.x += v[sp].x;
      sum.y += v[sp].y;
      sum.z += v[sp].z;
      sum.w += v[sp].w;
    }
  float4* dst = reinterpret_cast<float4*>(A + (size_t)l * Np * Np + (size_t)i * NB * Np + kb * NB + (size_t)r * Np + c);
  float4 d = *dst;
  d.x -= sum.x;
  d.y -= sum.y;
  d.z -= sum.z;
  d.w -= sum.w;
  *dst = d;
}

// The diagonal block kb of every lambda (one workgroup per lambda) factored in FP64, for launch
// shapes that ask for it (diag64): inv(L_kk) to Linv[l][kb]; L_kk itself is read by nothing.
// Within the 64 x 64 block the sweep is right-looking:
// Thread (r, q) = (tid / 8, tid % 8) keeps entries r, q + 8u (u = 0..7) of the block, and
// of T below, in registers.  Unscaled: at step j column j has received every
// update, its owners publish it to P[.][j] (never written again), one barrier, and each row
// below applies a[r][k] -= f P[k][j] with f = P[r][j] / P[j][j].  The same row operations turn the identity into T = diag(sqrt P) inv(L):
// T[i][c] = delta_ic - sum_{k<i} (P[i][k] / P[k][k]) T[k][c], so row j of T is final at step j,
// is published with column j (two-slot LDS buffer), and rows r > j take t[r][.] -= f T[j][.]
// in the same step: one sweep of 64 barriers for the factor and its inverse.
constexpr int kPotrfThreads = 512;
__global__ __launch_bounds__(kPotrfThreads) void k_potrf_diag64(const float* __restrict__ A, int Np, int kb,
                                                    float* __restrict__ Linv, int* flags) {
  __shared__ double P[NB][NB + 1];
  __shared__ double trow[2][NB];
  __shared__ double piv[NB], rsq[NB];
  __shared__ int bad;
  constexpr int TPR = kPotrfThreads / NB, EPT = NB / TPR;   // threads per row, entries per thread
  const int l = blockIdx.x;
  const float* Ab = A + (size_t)l * Np * Np + (size_t)kb * NB * Np + kb * NB;
  const int r = threadIdx.x / TPR, q = threadIdx.x % TPR;
  double a[EPT], t[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int k = TPR * u + q;
    a[u] = (k <= r) ? (double)Ab[(size_t)r * Np + k] : double(0);
    t[u] = (k == r) ? double(1) : double(0);
  }
  if (threadIdx.x == 0) bad = 0;
  // unrolled, so that the register holding column j is known at compile time
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    if (q == (j % TPR) && r >= j) {
      double v = a[0];
#pragma unroll
      for (int u = 1; u < EPT; ++u)
        if (u == (j / TPR)) v = a[u];
      P[r][j] = v;
    }
    if (r == j) {
#pragma unroll
      for (int u = 0; u < EPT; ++u) trow[j & 1][TPR * u + q] = t[u];
    }
    __syncthreads();
    // all loads first and unconditionally (rows k < j of P[.][j] are not yet written:
    // their values are discarded by the select), so the reads share one wait
    const double pj = P[j][j];
    const double prj = P[r][j];
    double pk[EPT], tv[EPT];
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      pk[u] = P[TPR * u + q][j];
      tv[u] = trow[j & 1][TPR * u + q];
    }
    const bool badj = !(pj > double(0));  // non-positive or NaN pivot
    const double rp = recip64(badj ? double(1) : pj);
    const double f = r > j ? prj * rp : double(0);
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      const int k = TPR * u + q;
      const double upd = fma(-f, pk[u], a[u]);
      a[u] = (k > j && k <= r) ? upd : a[u];
      t[u] = fma(-f, tv[u], t[u]);   // T[j][c] = 0 for c > j: no change there
    }
    if (threadIdx.x == 0) {
      piv[j] = badj ? double(1) : pj;
      if (badj) bad = 1;
    }
  }
  // t[] holds T[r][q + TPR u]
#pragma unroll
  for (int u = 0; u < EPT; ++u) a[u] = t[u];
  __syncthreads();   // the last pivot (thread 0, after the last step's barrier)
  if (threadIdx.x < NB) {
    rsq[threadIdx.x] = 1.0 / sqrt(piv[threadIdx.x]);
  }
  __syncthreads();
  float* Li = Linv + ((size_t)l * (Np / NB) + kb) * NB * NB;
  const double rs = rsq[r];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int c = TPR * u + q;
    Li[r * NB + c] = (c <= r) ? (float)(a[u] * rs) : 0.0f;
  }
  if (threadIdx.x == 0 && bad) {
    atomicOr(&flags[kFlagNotPD], 1);
    atomicMin(&flags[kFlagNotPD + 1], l);
  }
}

// The diagonal block kb of every lambda factored in FP32, and (PANEL) the panel below it.
//
// The 128 x 64 matrix [A_kk; I] in LDS is eliminated by columns: the top half becomes L_kk and the
// bottom half W = inv(L_kk)^T (a row of either half takes the same column operations).  Four panels of
// 16 columns.  In a panel a lane holds one row's 16 entries; lanes 0-15 are the panel's diagonal rows
// (in both working waves), lanes 16-47 the four other 16-row blocks that are not zero (3 - b of A,
// b + 1 of W, at panel b).  Column j: the pivot and the multipliers are broadcast from the diagonal
// rows with v_readlane, so the 64 dependent column steps meet no LDS round trip and no barrier.
// Between panels the four 16 x 16 blocks of the next panel's columns are updated on the matrix cores,
// one per wave; the later columns' blocks by waves 2 and 3 during the next panel.
// Bound by the chain of column steps (about 105 cycles each, 1700 per panel measured; a broadcast by
// DPP with one wave for all rows took 2400).  The kernel this replaced published every column through
// LDS with a barrier per step: 19.2 us per block against 7.7 alone, 8.6 with the panel and 9.9 with
// the panel and its update (N = 4225).  Factorization at N = 4225: 2.25 -> 1.08 ms at one lambda, 12.3
// -> 11.2 ms at 64.  L_kk is not stored: the updates read finished panels only, the solves inv(L_kk).
//
// PANEL: the workgroups of a lambda (one per block row i >= kb) all factor the diagonal block
// themselves and then finish their own panel tile L[i][kb] = A[i][kb] W, which saves the launch of
// k_trsm_panel; row i = kb writes Linv.  UPD (with PANEL): the block column first takes its remaining
// term, A[i][kb] -= L[i][kb-1] L[kb][kb-1]^T (the diagonal tile in every workgroup), which saves the
// launch of k_left_update.  Wave w holds rows 16 w .. of the 64 x 64 tiles, as four 16 x 16
// accumulator blocks.
constexpr int LDP = NB + 4;   // row stride of the elimination's LDS matrix
template <bool PANEL, bool UPD>
__global__ __launch_bounds__(256) void k_factor_diag(float* __restrict__ A, int Np, int kb,
                                                     float* __restrict__ Linv, int nlam, int* flags) {
  __shared__ __align__(16) float S[2 * NB * LDP];
  static_assert(sizeof(S) >= 2 * sizeof(SplitTile), "the split tiles share the elimination's memory");
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  int l = blockIdx.x, i = 0;
  if constexpr (PANEL) xcd_place(Np / NB - kb, nlam, &l, &i);
  const int ib = kb + i;
  float* Al = A + (size_t)l * Np * Np;
  float* mine = Al + (size_t)ib * NB * Np + kb * NB;
  // the diagonal tile and this workgroup's own tile in accumulator layout: block cb, element v is
  // row 16 w + 4 lk + v, column 16 cb + li (blocks above the diagonal of the diagonal tile unused)
  floatx4 dg[4], own[4];
  {
    const float* src = Al + (size_t)kb * NB * Np + kb * NB;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const size_t o = (size_t)(16 * w + 4 * lk + v) * Np + 16 * cb + li;
        dg[cb][v] = src[o];
        if (PANEL) own[cb][v] = mine[o];
      }
  }
  if constexpr (UPD) {
    SplitTile& Ts = *reinterpret_cast<SplitTile*>(S);
    SplitTile& Ds = *(reinterpret_cast<SplitTile*>(S) + 1);
    const uint32_t* gi = reinterpret_cast<const uint32_t*>(Al + (size_t)ib * NB * Np + (kb - 1) * NB);
    const uint32_t* gd = reinterpret_cast<const uint32_t*>(Al + (size_t)kb * NB * Np + (kb - 1) * NB);
    uint4 ra[4], rb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = tid + q * 256, r = idx / (NB / 4), c = (idx % (NB / 4)) * 4;
      ra[q] = *reinterpret_cast<const uint4*>(gi + (size_t)r * Np + c);
      rb[q] = *reinterpret_cast<const uint4*>(gd + (size_t)r * Np + c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = tid + q * 256, r = idx / (NB / 4), c = (idx % (NB / 4)) * 4;
      split_stage(Ts, split_off(r, c), ra[q]);
      split_stage(Ds, split_off(r, c), rb[q]);
    }
    __syncthreads();
    floatx4 ad[4] = {}, adx[4] = {}, ao[4] = {}, aox[4] = {};
#pragma unroll
    for (int k = 0; k < NB; k += 32) {
      const int oa = split_off(16 * w + li, k + 8 * lk);
      const half8 th = *reinterpret_cast<const half8*>(&Ts.hi[oa]), tl = *reinterpret_cast<const half8*>(&Ts.lo[oa]);
      const half8 dh = *reinterpret_cast<const half8*>(&Ds.hi[oa]), dl = *reinterpret_cast<const half8*>(&Ds.lo[oa]);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int o = split_off(16 * cb + li, k + 8 * lk);
        const half8 bh = *reinterpret_cast<const half8*>(&Ds.hi[o]), bl = *reinterpret_cast<const half8*>(&Ds.lo[o]);
        ad[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(dh, bh, ad[cb], 0, 0, 0);
        ao[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(th, bh, ao[cb], 0, 0, 0);
        adx[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(dh, bl, adx[cb], 0, 0, 0);
        aox[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(th, bl, aox[cb], 0, 0, 0);
        adx[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(dl, bh, adx[cb], 0, 0, 0);
        aox[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(tl, bh, aox[cb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dg[cb][v] -= fmaf(adx[cb][v], 1.f / kSplitScale, ad[cb][v]);
        own[cb][v] -= fmaf(aox[cb][v], 1.f / kSplitScale, ao[cb][v]);
      }
    __syncthreads();   // the split tiles are read: their memory becomes the elimination's
  }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * w + 4 * lk + v, c = 16 * cb + li;
      S[r * LDP + c] = dg[cb][v];
      S[(NB + r) * LDP + c] = r == c ? 1.f : 0.f;
    }
  __syncthreads();
  // Block t of column block c takes its term of panel b: rows c.. of A (t < 4 - c), then rows 0 .. b
  // of W.  Lane group lk supplies k = 4 lk + e of both operands at product e.
  auto trail = [&](int b, int c, int t) {
    const int r0 = t < 4 - c ? 16 * (c + t) : NB + 16 * (t - (4 - c));
    const float4 av = *reinterpret_cast<const float4*>(S + (r0 + li) * LDP + 16 * b + 4 * lk);
    const float4 bv = *reinterpret_cast<const float4*>(S + (16 * c + li) * LDP + 16 * b + 4 * lk);
    float* cp = S + (r0 + 4 * lk) * LDP + 16 * c + li;
    floatx4 acc = {cp[0], cp[LDP], cp[2 * LDP], cp[3 * LDP]};
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.x, bv.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.y, bv.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.z, bv.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.w, bv.w, acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) cp[v * LDP] = acc[v];
  };
  bool bad = false;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    if (w < 2) {
      // lane's row: group 0 the diagonal rows, groups 1 and 2 the wave's two other blocks; group 3
      // repeats the diagonal rows and is not stored
      const int o = 2 * w + lk - 1;
      const int row = (lk == 0 || lk == 3) ? 16 * b + li
                                           : (o < 3 - b ? 16 * (b + 1 + o) + li : NB + 16 * (o - (3 - b)) + li);
      float* rp = S + row * LDP + 16 * b;
      float a[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(rp + 4 * q);
        a[4 * q] = v.x;
        a[4 * q + 1] = v.y;
        a[4 * q + 2] = v.z;
        a[4 * q + 3] = v.w;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float p = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a[j]), j));
        bad = bad || !(p > 0.f);   // non-positive or NaN pivot: reported, the values are not used
        // a[j] / sqrt(p): hardware 1 / sqrt (1 ulp) and one Newton step, applied to the product so
        // that it and the correction are computed side by side
        const float rs = __builtin_amdgcn_rsqf(p), l0 = a[j] * rs;
        a[j] = fmaf(l0, fmaf(-0.5f * p * rs, rs, 0.5f), l0);
#pragma unroll
        for (int k = j + 1; k < 16; ++k)
          a[k] = fmaf(-a[j], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a[j]), k)), a[k]);
      }
      if (lk == 1 || lk == 2 || (lk == 0 && w == 0)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(rp + 4 * q) = make_float4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
      }
    }
    if (w >= 2 && b >= 1) {
      int cnt = 0;
#pragma unroll
      for (int c = b + 1; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < 4 - c + b; ++t)
          if ((cnt++ & 1) == w - 2) trail(b - 1, c, t);
    }
    __syncthreads();
    if (b < 3) {
      trail(b, b + 1, w);   // the next panel's column block: four blocks, one per wave
      __syncthreads();
    }
  }
  const float* W = S + NB * LDP;
  if (!PANEL || i == 0) {
    float* Li = Linv + ((size_t)l * (Np / NB) + kb) * NB * NB;
#pragma unroll
    for (int u = 0; u < NB * NB / 256; ++u) {
      const int e = tid + 256 * u, r = e / NB, c = e % NB;
      Li[e] = c <= r ? W[c * LDP + r] : 0.f;
    }
    if (tid == 0 && bad) {
      atomicOr(&flags[kFlagNotPD], 1);
      atomicMin(&flags[kFlagNotPD + 1], l);
    }
    return;
  }
  if constexpr (PANEL) {
    // own tile into the top half (rows 16 w .. of it are written and read by wave w only), times W,
    // whose blocks below the diagonal are zero
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) S[(16 * w + 4 * lk + v) * LDP + 16 * cb + li] = own[cb][v];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    floatx4 acc[4] = {};
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) {
      const float4 av = *reinterpret_cast<const float4*>(S + (16 * w + li) * LDP + 16 * kq + 4 * lk);
      const float* wr = W + (16 * kq + 4 * lk) * LDP + li;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int cb = kq; cb < 4; ++cb)
          acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(e == 0 ? av.x : e == 1 ? av.y : e == 2 ? av.z : av.w,
                                                         wr[e * LDP + 16 * cb], acc[cb], 0, 0, 0);
    }
    uint32_t* dst = reinterpret_cast<uint32_t*>(mine);
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        dst[(size_t)(16 * w + 4 * lk + v) * Np + 16 * cb + li] = split_pack(acc[cb][v]);
  }
}

// Panel: L[i][kb] = A[i][kb] * inv(L_kk)^T for block rows i > kb.
__global__ __launch_bounds__(256) void k_trsm_panel(float* __restrict__ A, int Np, int kb,
                                                    const float* __restrict__ Linv, int nlam) {
  __shared__ float As[NB * LDT], Bs[NB * LDT];
  int l, ib;
  xcd_place(Np / NB - kb - 1, nlam, &l, &ib);
  ib += kb + 1;
  float* Al = A + (size_t)l * Np * Np;
  float* src = Al + (size_t)ib * NB * Np + kb * NB;
  const float* Li = Linv + ((size_t)l * (Np / NB) + kb) * NB * NB;
  load_tiles2(As, src, Np, Bs, Li, NB);
  __syncthreads();
  floatx4 acc[2][2] = {};
  mfma_tile64(As, Bs, acc);
  store_acc_split(src, Np, acc);   // finished: FP16 pairs for the updates and the solves
}

// Left-looking update of block column kb for every lambda (grid.y):
//   A[i][kb] -= sum_{k0 <= k < k1} L[i][k] L[kb][k]^T,   i = kb + blockIdx.x,
// the K loop over the finished panels (FP16 pairs, split tiles in LDS) with the next pair of
// tiles loaded into registers while the current pair is on the matrix cores.
__global__ __launch_bounds__(256) void k_left_update(float* __restrict__ A, int Np, int kb, int k0, int k1,
                                                     int nlam) {
  __shared__ __align__(16) SplitTile As;
  __shared__ __align__(16) SplitTile Bs;
  int l, i;
  xcd_place(Np / NB - kb, nlam, &l, &i);
  i += kb;
  float* Al = A + (size_t)l * Np * Np;
  const uint32_t* Ai = reinterpret_cast<const uint32_t*>(Al + (size_t)i * NB * Np);
  const uint32_t* Ak = reinterpret_cast<const uint32_t*>(Al + (size_t)kb * NB * Np);
  int off_g[4], off_s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int idx = threadIdx.x + q * 256, r = idx / (NB / 4), c = (idx % (NB / 4)) * 4;
    off_g[q] = r * Np + c;
    off_s[q] = split_off(r, c);
  }
  uint4 ra[4], rb[4];
  auto gload = [&](int k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ra[q] = *reinterpret_cast<const uint4*>(Ai + k * NB + off_g[q]);
      rb[q] = *reinterpret_cast<const uint4*>(Ak + k * NB + off_g[q]);
    }
  };
  floatx4 acc[1][2][2] = {}, accx[1][2][2] = {};
  gload(k0);
  for (int k = k0; k < k1; ++k) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      split_stage(As, off_s[q], ra[q]);
      split_stage(Bs, off_s[q], rb[q]);
    }
    __syncthreads();
    if (k + 1 < k1) gload(k + 1);
    mfma_split64<1>(As, Bs, Bs, acc, accx);
    __syncthreads();
  }
  store_split_update(Al + (size_t)i * NB * Np + kb * NB, Np, acc[0], accx[0]);
}

// ------------------------------------------------------------------ triangular solves (FP32)
// R, Y: [lambda][ncol][Np] (column-major per lambda: column t contiguous).

// MFMA product of a 64 x 64 LDS tile (or its transpose) with a 64 x (16*NCT) LDS
// block: wave w computes rows 16w..16w+15.  Lane layout as in mfma_tile64.
constexpr int LDB = 33;   // row stride of the 64 x ncol blocks (ncol <= 32)
template <bool TRANS, int NCT, bool ACC = false>
__device__ __forceinline__ void mfma_64xK(const float* Ls, const float (*Bs)[LDB], floatx4 acc[NCT]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  if (!ACC) {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll 4
  for (int k0 = 0; k0 < NB; k0 += 4) {
    const float a = TRANS ? Ls[(k0 + lk) * LDT + 16 * w + li] : Ls[(16 * w + li) * LDT + k0 + lk];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const float b = Bs[k0 + lk][ct * 16 + li];
      acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[ct], 0, 0, 0);
    }
  }
}

// One 64 x 64 tile of a finished panel (FP16 pairs) in four uint4 registers per thread
// (256 threads: thread t holds the four entries number t + 256 u of the row-major tile),
// for loading the next tile of a sweep while the current one is on the matrix cores; the
// staging into LDS unpacks it to FP32.
#define FK_TILE_FETCH_TO(src, ld, a0, a1, a2, a3)                                            \
  do {                                                                                       \
    _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_) {                                       \
      const int i_ = threadIdx.x + 256 * u_, r_ = i_ / (NB / 4), c_ = (i_ - r_ * (NB / 4)) * 4; \
      const uint4 v_ = *reinterpret_cast<const uint4*>((src) + r_ * (ld) + c_);            \
      if (u_ == 0) a0 = v_;                                                                  \
      if (u_ == 1) a1 = v_;                                                                  \
      if (u_ == 2) a2 = v_;                                                                  \
      if (u_ == 3) a3 = v_;                                                                  \
    }                                                                                        \
  } while (0)
#define FK_TILE_STAGE_FROM(T, a0, a1, a2, a3)                                                \
  do {                                                                                       \
    _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_) {                                       \
      const int i_ = threadIdx.x + 256 * u_, r_ = i_ / (NB / 4), c_ = (i_ - r_ * (NB / 4)) * 4; \
      const uint4 q_ = u_ == 0 ? a0 : u_ == 1 ? a1 : u_ == 2 ? a2 : a3;                     \
      *reinterpret_cast<float4*>((T) + r_ * LDT + c_) =                                      \
          make_float4(split_unpack(q_.x), split_unpack(q_.y), split_unpack(q_.z), split_unpack(q_.w)); \
    }                                                                                        \
  } while (0)
#define FK_TILE_FETCH(src, ld) FK_TILE_FETCH_TO(src, ld, nt0, nt1, nt2, nt3)
#define FK_TILE_STAGE(T) FK_TILE_STAGE_FROM(T, nt0, nt1, nt2, nt3)

// Forward step kb of L y = r for every lambda (grid.y): y_kb = inv(L_kk) r_kb, written
// by block 0; block x then updates rows ib = kb + 1 + x, kb + 1 + x + gridDim.x, ...:
// r_ib -= L[ib][kb] y_kb, with the next row's tile loaded while the current one is
// multiplied (two LDS buffers, one barrier per row).
template <int NCT>
__global__ __launch_bounds__(256) void k_fwd_mfma(const float* __restrict__ A, int Np, int kb,
                                                  const float* __restrict__ Linv, float* __restrict__ R,
                                                  float* __restrict__ Y, int ncol) {
  __shared__ float Ls[2][NB * LDT];
  __shared__ float Bs[NB][LDB];
  const int l = blockIdx.y;
  const int nb = Np / NB;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  float* Rl = R + (size_t)l * ncol * Np;
  const float* Al = A + (size_t)l * Np * Np;
  // every load of the prologue goes out before any is used
  int ib = kb + 1 + blockIdx.x;
  uint4 nt0, nt1, nt2, nt3;
  if (ib < nb) FK_TILE_FETCH(Al + (size_t)ib * NB * Np + kb * NB, Np);
  constexpr int NBS = NB * 16 * NCT / 256;   // right-hand-side entries per thread
  float bsv[NBS];
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / NB, k = i - t * NB;
    bsv[u] = t < ncol ? Rl[(size_t)t * Np + kb * NB + k] : 0.f;
  }
  float4 d0, d1, d2, d3;
  FK_F32_LOAD4(Linv + ((size_t)l * nb + kb) * NB * NB, NB, d0, d1, d2, d3);
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / NB, k = i - t * NB;
    Bs[k][t] = bsv[u];
  }
  FK_F32_STORE4(Ls[0], d0, d1, d2, d3);
  __syncthreads();
  floatx4 acc[NCT];
  mfma_64xK<false, NCT>(Ls[0], Bs, acc);
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[16 * w + 4 * lk + v][ct * 16 + li] = acc[ct][v];
  if (ib < nb) FK_TILE_STAGE(Ls[1]);
  __syncthreads();
  if (blockIdx.x == 0) {
    float* Yl = Y + (size_t)l * ncol * Np;
    for (int i = threadIdx.x; i < ncol * NB; i += blockDim.x) {
      const int t = i / NB, r = i - t * NB;
      Yl[(size_t)t * Np + kb * NB + r] = Bs[r][t];
    }
  }
  // this lane's part of the right-hand-side block of a row: 4 rows x NCT columns
  float rr[NCT][4];
#define FK_R_FETCH(RB)                                                                         \
  _Pragma("unroll") for (int ct = 0; ct < NCT; ++ct) {                                         \
    const int t_ = min(ct * 16 + li, ncol - 1);                                                \
    _Pragma("unroll") for (int v = 0; v < 4; ++v)                                              \
      rr[ct][v] = Rl[(size_t)t_ * Np + (RB) * NB + 16 * w + 4 * lk + v];                       \
  }
  if (ib < nb) FK_R_FETCH(ib)
  int cur = 1;
  for (; ib < nb; ib += gridDim.x) {
    const int nx = ib + gridDim.x;
    if (nx < nb) FK_TILE_FETCH(Al + (size_t)nx * NB * Np + kb * NB, Np);
    mfma_64xK<false, NCT>(Ls[cur], Bs, acc);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = ct * 16 + li;
        if (t < ncol) Rl[(size_t)t * Np + ib * NB + 16 * w + 4 * lk + v] = rr[ct][v] - acc[ct][v];
      }
    if (nx < nb) FK_R_FETCH(nx)
    if (nx < nb) FK_TILE_STAGE(Ls[cur ^ 1]);
    __syncthreads();
    cur ^= 1;
  }
#undef FK_R_FETCH
}

// Backward step kb of L^T x = y: x_kb = inv(L_kk)^T y_kb (block 0 writes X); block x
// then updates rows jb = x, x + gridDim.x, ... < kb: y_jb -= L[kb][jb]^T x_kb, the
// next row's tile loaded while the current one is multiplied.
template <int NCT>
__global__ __launch_bounds__(256) void k_bwd_mfma(const float* __restrict__ A, int Np, int kb,
                                                  const float* __restrict__ Linv, float* __restrict__ Yv,
                                                  float* __restrict__ X, int ncol) {
  __shared__ float Ls[2][NB * LDT];
  __shared__ float Bs[NB][LDB];
  const int l = blockIdx.y;
  const int nb = Np / NB;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  float* Yl = Yv + (size_t)l * ncol * Np;
  const float* Ak = A + (size_t)l * Np * Np + (size_t)kb * NB * Np;
  // every load of the prologue goes out before any is used
  int jb = blockIdx.x;
  uint4 nt0, nt1, nt2, nt3;
  if (jb < kb) FK_TILE_FETCH(Ak + jb * NB, Np);
  constexpr int NBS = NB * 16 * NCT / 256;   // right-hand-side entries per thread
  float bsv[NBS];
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / NB, k = i - t * NB;
    bsv[u] = t < ncol ? Yl[(size_t)t * Np + kb * NB + k] : 0.f;
  }
  float4 d0, d1, d2, d3;
  FK_F32_LOAD4(Linv + ((size_t)l * nb + kb) * NB * NB, NB, d0, d1, d2, d3);
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / NB, k = i - t * NB;
    Bs[k][t] = bsv[u];
  }
  FK_F32_STORE4(Ls[0], d0, d1, d2, d3);
  __syncthreads();
  floatx4 acc[NCT];
  mfma_64xK<true, NCT>(Ls[0], Bs, acc);
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[16 * w + 4 * lk + v][ct * 16 + li] = acc[ct][v];
  if (jb < kb) FK_TILE_STAGE(Ls[1]);
  __syncthreads();
  if (blockIdx.x == 0) {
    float* Xl = X + (size_t)l * ncol * Np;
    for (int i = threadIdx.x; i < ncol * NB; i += blockDim.x) {
      const int t = i / NB, r = i - t * NB;
      Xl[(size_t)t * Np + kb * NB + r] = Bs[r][t];
    }
  }
  float rr[NCT][4];
#define FK_R_FETCH(RB)                                                                         \
  _Pragma("unroll") for (int ct = 0; ct < NCT; ++ct) {                                         \
    const int t_ = min(ct * 16 + li, ncol - 1);                                                \
    _Pragma("unroll") for (int v = 0; v < 4; ++v)                                              \
      rr[ct][v] = Yl[(size_t)t_ * Np + (RB) * NB + 16 * w + 4 * lk + v];                       \
  }
  if (jb < kb) FK_R_FETCH(jb)
  int cur = 1;
  for (; jb < kb; jb += gridDim.x) {
    const int nx = jb + gridDim.x;
    if (nx < kb) FK_TILE_FETCH(Ak + nx * NB, Np);
    mfma_64xK<true, NCT>(Ls[cur], Bs, acc);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = ct * 16 + li;
        if (t < ncol) Yl[(size_t)t * Np + jb * NB + 16 * w + 4 * lk + v] = rr[ct][v] - acc[ct][v];
      }
    if (nx < kb) FK_R_FETCH(nx)
    if (nx < kb) FK_TILE_STAGE(Ls[cur ^ 1]);
    __syncthreads();
    cur ^= 1;
  }
#undef FK_R_FETCH
}


// Two forward steps kb, kb + 1 in one launch (kb + 1 < nb).  Every workgroup solves the 128-row
// diagonal part itself: y_kb = inv(L_kk) r_kb, then r_{kb+1} -= L[kb+1][kb] y_kb and y_{kb+1} =
// inv(L_{kb+1,kb+1}) r_{kb+1}; block 0 writes both blocks of Y.  Block x then updates rows ib = kb + 2
// + x, kb + 2 + x + gridDim.x, ...: r_ib -= L[ib][kb] y_kb + L[ib][kb+1] y_{kb+1}, the tiles streamed
// through the two LDS buffers in the order (ib, kb), (ib, kb + 1), (next ib, kb), ... (one barrier
// per tile).  Half the dependent launches of the one-step sweep.
template <int NCT>
__global__ __launch_bounds__(256) void k_fwd2_mfma(const float* __restrict__ A, int Np, int kb,
                                                   const float* __restrict__ Linv, float* __restrict__ R,
                                                   float* __restrict__ Y, int ncol) {
  __shared__ float Ls[2][NB * LDT];
  __shared__ float Bs[2 * NB][LDB];
  const int l = blockIdx.y;
  const int nb = Np / NB;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  float* Rl = R + (size_t)l * ncol * Np;
  const float* Al = A + (size_t)l * Np * Np;
  const int ib0 = kb + 2 + blockIdx.x;
  // Every global load of the two diagonal steps and of the first row goes out here, before any
  // is used: the prologue waits for memory once instead of three times.
  constexpr int NBS = 2 * NB * 16 * NCT / 256;   // right-hand-side entries per thread
  float bsv[NBS];
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / (2 * NB), k = i - t * (2 * NB);
    bsv[u] = t < ncol ? Rl[(size_t)t * Np + kb * NB + k] : 0.f;
  }
  float4 d00, d01, d02, d03, d10, d11, d12, d13;
  FK_F32_LOAD4(Linv + ((size_t)l * nb + kb) * NB * NB, NB, d00, d01, d02, d03);
  FK_F32_LOAD4(Linv + ((size_t)l * nb + kb + 1) * NB * NB, NB, d10, d11, d12, d13);
  uint4 nt0, nt1, nt2, nt3, ns0, ns1, ns2, ns3;
  FK_TILE_FETCH(Al + (size_t)(kb + 1) * NB * Np + kb * NB, Np);
  if (ib0 < nb) FK_TILE_FETCH_TO(Al + (size_t)ib0 * NB * Np + kb * NB, Np, ns0, ns1, ns2, ns3);
  // this lane's part of the right-hand-side block of a row: 4 rows x NCT columns
  float rr[NCT][4];
#define FK_R_FETCH(RB)                                                                         \
  _Pragma("unroll") for (int ct = 0; ct < NCT; ++ct) {                                         \
    const int t_ = min(ct * 16 + li, ncol - 1);                                                \
    _Pragma("unroll") for (int v = 0; v < 4; ++v)                                              \
      rr[ct][v] = Rl[(size_t)t_ * Np + (RB) * NB + 16 * w + 4 * lk + v];                       \
  }
  if (ib0 < nb) FK_R_FETCH(ib0)
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / (2 * NB), k = i - t * (2 * NB);
    Bs[k][t] = bsv[u];
  }
  FK_F32_STORE4(Ls[0], d00, d01, d02, d03);
  FK_TILE_STAGE(Ls[1]);
  __syncthreads();
  floatx4 acc[NCT];
  mfma_64xK<false, NCT>(Ls[0], Bs, acc);   // y_kb
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[16 * w + 4 * lk + v][ct * 16 + li] = acc[ct][v];
  __syncthreads();
  mfma_64xK<false, NCT>(Ls[1], Bs, acc);   // L[kb+1][kb] y_kb
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[NB + 16 * w + 4 * lk + v][ct * 16 + li] -= acc[ct][v];
  FK_F32_STORE4(Ls[0], d10, d11, d12, d13);
  __syncthreads();
  mfma_64xK<false, NCT>(Ls[0], Bs + NB, acc);   // y_{kb+1}
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[NB + 16 * w + 4 * lk + v][ct * 16 + li] = acc[ct][v];
  if (ib0 < nb) FK_TILE_STAGE_FROM(Ls[1], ns0, ns1, ns2, ns3);
  __syncthreads();
  if (blockIdx.x == 0) {
    float* Yl = Y + (size_t)l * ncol * Np;
    for (int i = threadIdx.x; i < ncol * 2 * NB; i += blockDim.x) {
      const int t = i / (2 * NB), r = i - t * (2 * NB);
      Yl[(size_t)t * Np + kb * NB + r] = Bs[r][t];
    }
  }
  int cur = 1;
  for (int ib = ib0; ib < nb; ib += gridDim.x) {
    // tile (ib, kb) is in Ls[cur]; (ib, kb + 1) comes next
    FK_TILE_FETCH(Al + (size_t)ib * NB * Np + (kb + 1) * NB, Np);
    mfma_64xK<false, NCT>(Ls[cur], Bs, acc);
    FK_TILE_STAGE(Ls[cur ^ 1]);
    __syncthreads();
    cur ^= 1;
    const int nx = ib + gridDim.x;
    if (nx < nb) FK_TILE_FETCH(Al + (size_t)nx * NB * Np + kb * NB, Np);
    mfma_64xK<false, NCT, true>(Ls[cur], Bs + NB, acc);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = ct * 16 + li;
        if (t < ncol) Rl[(size_t)t * Np + ib * NB + 16 * w + 4 * lk + v] = rr[ct][v] - acc[ct][v];
      }
    if (nx < nb) FK_R_FETCH(nx)
    if (nx < nb) FK_TILE_STAGE(Ls[cur ^ 1]);
    __syncthreads();
    cur ^= 1;
  }
#undef FK_R_FETCH
}

// Two backward steps kb, kb - 1 in one launch (kb >= 1): x_kb = inv(L_kk)^T y_kb, then y_{kb-1} -=
// L[kb][kb-1]^T x_kb and x_{kb-1} = inv(L_{kb-1,kb-1})^T y_{kb-1} in every workgroup (block 0 writes
// both blocks of X); block x then updates rows jb = x, x + gridDim.x, ... < kb - 1: y_jb -= L[kb][jb]^T
// x_kb + L[kb-1][jb]^T x_{kb-1}, the two tiles of a row streamed one after the other.
template <int NCT>
__global__ __launch_bounds__(256) void k_bwd2_mfma(const float* __restrict__ A, int Np, int kb,
                                                   const float* __restrict__ Linv, float* __restrict__ Yv,
                                                   float* __restrict__ X, int ncol) {
  __shared__ float Ls[2][NB * LDT];
  __shared__ float Bs[2 * NB][LDB];
  const int l = blockIdx.y;
  const int nb = Np / NB;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  float* Yl = Yv + (size_t)l * ncol * Np;
  const float* Ak = A + (size_t)l * Np * Np + (size_t)kb * NB * Np;         // block row kb
  const float* Ak1 = A + (size_t)l * Np * Np + (size_t)(kb - 1) * NB * Np;  // block row kb - 1
  const int jb0 = blockIdx.x;
  // every global load of the two diagonal steps and of the first row goes out here
  constexpr int NBS = 2 * NB * 16 * NCT / 256;   // right-hand-side entries per thread
  float bsv[NBS];
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / (2 * NB), k = i - t * (2 * NB);
    const int row = k < NB ? kb * NB + k : (kb - 1) * NB + (k - NB);
    bsv[u] = t < ncol ? Yl[(size_t)t * Np + row] : 0.f;
  }
  float4 d00, d01, d02, d03, d10, d11, d12, d13;
  FK_F32_LOAD4(Linv + ((size_t)l * nb + kb) * NB * NB, NB, d00, d01, d02, d03);
  FK_F32_LOAD4(Linv + ((size_t)l * nb + kb - 1) * NB * NB, NB, d10, d11, d12, d13);
  uint4 nt0, nt1, nt2, nt3, ns0, ns1, ns2, ns3;
  FK_TILE_FETCH(Ak + (kb - 1) * NB, Np);   // L[kb][kb-1]
  if (jb0 < kb - 1) FK_TILE_FETCH_TO(Ak + jb0 * NB, Np, ns0, ns1, ns2, ns3);
  float rr[NCT][4];
#define FK_R_FETCH(RB)                                                                         \
  _Pragma("unroll") for (int ct = 0; ct < NCT; ++ct) {                                         \
    const int t_ = min(ct * 16 + li, ncol - 1);                                                \
    _Pragma("unroll") for (int v = 0; v < 4; ++v)                                              \
      rr[ct][v] = Yl[(size_t)t_ * Np + (RB) * NB + 16 * w + 4 * lk + v];                       \
  }
  if (jb0 < kb - 1) FK_R_FETCH(jb0)
#pragma unroll
  for (int u = 0; u < NBS; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / (2 * NB), k = i - t * (2 * NB);
    Bs[k][t] = bsv[u];
  }
  FK_F32_STORE4(Ls[0], d00, d01, d02, d03);
  FK_TILE_STAGE(Ls[1]);
  __syncthreads();
  floatx4 acc[NCT];
  mfma_64xK<true, NCT>(Ls[0], Bs, acc);   // x_kb
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[16 * w + 4 * lk + v][ct * 16 + li] = acc[ct][v];
  __syncthreads();
  mfma_64xK<true, NCT>(Ls[1], Bs, acc);   // L[kb][kb-1]^T x_kb
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[NB + 16 * w + 4 * lk + v][ct * 16 + li] -= acc[ct][v];
  FK_F32_STORE4(Ls[0], d10, d11, d12, d13);
  __syncthreads();
  mfma_64xK<true, NCT>(Ls[0], Bs + NB, acc);   // x_{kb-1}
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) Bs[NB + 16 * w + 4 * lk + v][ct * 16 + li] = acc[ct][v];
  if (jb0 < kb - 1) FK_TILE_STAGE_FROM(Ls[1], ns0, ns1, ns2, ns3);
  __syncthreads();
  if (blockIdx.x == 0) {
    float* Xl = X + (size_t)l * ncol * Np;
    for (int i = threadIdx.x; i < ncol * 2 * NB; i += blockDim.x) {
      const int t = i / (2 * NB), k = i - t * (2 * NB);
      const int row = k < NB ? kb * NB + k : (kb - 1) * NB + (k - NB);
      Xl[(size_t)t * Np + row] = Bs[k][t];
    }
  }
  int cur = 1;
  for (int jb = jb0; jb < kb - 1; jb += gridDim.x) {
    // tile (kb, jb) is in Ls[cur]; (kb - 1, jb) comes next
    FK_TILE_FETCH(Ak1 + jb * NB, Np);
    mfma_64xK<true, NCT>(Ls[cur], Bs, acc);
    FK_TILE_STAGE(Ls[cur ^ 1]);
    __syncthreads();
    cur ^= 1;
    const int nx = jb + gridDim.x;
    if (nx < kb - 1) FK_TILE_FETCH(Ak + nx * NB, Np);
    mfma_64xK<true, NCT, true>(Ls[cur], Bs + NB, acc);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = ct * 16 + li;
        if (t < ncol) Yl[(size_t)t * Np + jb * NB + 16 * w + 4 * lk + v] = rr[ct][v] - acc[ct][v];
      }
    if (nx < kb - 1) FK_R_FETCH(nx)
    if (nx < kb - 1) FK_TILE_STAGE(Ls[cur ^ 1]);
    __syncthreads();
    cur ^= 1;
  }
#undef FK_R_FETCH
}


// ------------------------------------------------------------------ solves with inverted super-blocks
// The step-by-step sweeps above are a chain of dependent launches, one per two block columns, each of
// which must solve its 128 diagonal rows before it can update the others: 34 launches of 6 us per direction
// at N = 4225 and one lambda, most of it launch and load latency.  Here the 512 x 512 diagonal blocks (SB
// block columns) are inverted once after the factorization, in place: inv of [[P, 0], [L, Q]] has
// -inv(Q) L inv(P) below the diagonal, so three doublings of the block size (64 -> 128 -> 256 -> 512), two
// batched products each, take the 64 x 64 inverses to 512.  A solve step is then two plain products
// over the whole width of the chip: y_K = inv(L_KK) r_K and r_J -= L_JK y_K for the rows below.
// FP32 throughout (the panels below the diagonal blocks stay FP16 pairs, as for the sweeps).
constexpr int SB = 8;   // block columns per super-block

// acc += As Bs, both 64 x 64 row-major in LDS (wave layout of mfma_tile64).
__device__ __forceinline__ void mfma_tile64_nn(const float* As, const float* Bs, floatx4 acc[2][2]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll 4
  for (int k = 0; k < NB; k += 4) {
    const float a0 = As[(r0 + li) * LDT + k + lk], a1 = As[(r0 + 16 + li) * LDT + k + lk];
    const float b0 = Bs[(k + lk) * LDT + c0 + li], b1 = Bs[(k + lk) * LDT + c0 + 16 + li];
    acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
  }
}

// The FP32 inverses of the 64 x 64 diagonal blocks into their place in A (zeros above the diagonal), and
// the doubling to 128: one workgroup per pair of blocks, -inv(Q) (L inv(P)) with the inner product in LDS.
__global__ __launch_bounds__(256) void k_inv_pair(float* __restrict__ A, int Np, const float* __restrict__ Linv) {
  __shared__ __align__(16) float As[NB * LDT];
  __shared__ __align__(16) float Bs[NB * LDT];
  const int nb = Np / NB, np = (nb + 1) / 2, p = blockIdx.x % np, l = blockIdx.x / np;
  const int j = 2 * p, i = j + 1;
  float* Al = A + (size_t)l * Np * Np;
  float* dj = Al + (size_t)j * NB * Np + j * NB;
  const float* Lj = Linv + ((size_t)l * nb + j) * NB * NB;
  float4 v0, v1, v2, v3;
  FK_F32_LOAD4(Lj, NB, v0, v1, v2, v3);
#define FK_PUT(dst)                                                                          \
  _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_) {                                         \
    const int i_ = threadIdx.x + 256 * u_, r_ = i_ / (NB / 4), c_ = (i_ - r_ * (NB / 4)) * 4; \
    *reinterpret_cast<float4*>((dst) + (size_t)r_ * Np + c_) = u_ == 0 ? v0 : u_ == 1 ? v1 : u_ == 2 ? v2 : v3; \
  }
  FK_PUT(dj)
  if (i >= nb) return;
  uint32_t* lij = reinterpret_cast<uint32_t*>(Al + (size_t)i * NB * Np + j * NB);
  uint4 nt0, nt1, nt2, nt3;
  FK_TILE_FETCH(lij, Np);
  FK_F32_STORE4(Bs, v0, v1, v2, v3);
  FK_F32_LOAD4(Lj + NB * NB, NB, v0, v1, v2, v3);
  FK_TILE_STAGE(As);
  __syncthreads();
  floatx4 acc[2][2] = {};
  mfma_tile64_nn(As, Bs, acc);
  __syncthreads();
  store_acc(Bs, LDT, acc, false, 1.f);
  FK_F32_STORE4(As, v0, v1, v2, v3);
  FK_PUT(Al + (size_t)i * NB * Np + i * NB)
#undef FK_PUT
  __syncthreads();
  floatx4 acc2[2][2] = {};
  mfma_tile64_nn(As, Bs, acc2);
  store_acc(reinterpret_cast<float*>(lij), Np, acc2, false, -1.f);
}

// One product of a doubling from ht to 2 ht tiles.  A pair's first half is the tiles b0 .. b0 + ht - 1, its
// second half b0 + ht .. e - 1 (cut at the super-block's or the matrix's end); workgroup: one 64 x 64 tile
// (i, j), i in the second half, j in the first.
//   SECOND = false: T(i, j) = sum_{k >= j, first half} L(i, k) Inv(k, j), kept at tile (j, i), above the
//                   diagonal, where A holds nothing
//   SECOND = true:  X(i, j) = -sum_{k <= i, second half} Inv(i, k) T(k, j), over L(i, j)
template <bool SECOND>
__global__ __launch_bounds__(256) void k_inv_level(float* __restrict__ A, int Np, int ht) {
  __shared__ __align__(16) float As[NB * LDT];
  __shared__ __align__(16) float Bs[NB * LDT];
  const int nb = Np / NB, per = ht * ht;
  const int pairs_sb = SB / (2 * ht);   // pairs per super-block
  int b = blockIdx.x;
  const int t = b % per;
  b /= per;
  const int p = b % pairs_sb;
  b /= pairs_sb;
  const int nsb = (nb + SB - 1) / SB, sb = b % nsb, l = b / nsb;
  const int b0 = sb * SB + 2 * ht * p, mid = b0 + ht;
  const int i = mid + t / ht, j = b0 + t % ht;
  if (i >= nb) return;
  float* Al = A + (size_t)l * Np * Np;
  floatx4 acc[2][2] = {};
  const int k0 = SECOND ? mid : j, k1 = SECOND ? i + 1 : mid;
  for (int k = k0; k < k1; ++k) {
    float4 v0, v1, v2, v3;
    if constexpr (SECOND) {
      const float* a = Al + (size_t)i * NB * Np + k * NB;
      const float* c = Al + (size_t)j * NB * Np + k * NB;   // T(k, j) at tile (j, k)
      float4 w0, w1, w2, w3;
      FK_F32_LOAD4(a, Np, v0, v1, v2, v3);
      FK_F32_LOAD4(c, Np, w0, w1, w2, w3);
      __syncthreads();
      FK_F32_STORE4(As, v0, v1, v2, v3);
      FK_F32_STORE4(Bs, w0, w1, w2, w3);
    } else {
      const uint32_t* a = reinterpret_cast<const uint32_t*>(Al + (size_t)i * NB * Np + k * NB);
      const float* c = Al + (size_t)k * NB * Np + j * NB;
      uint4 nt0, nt1, nt2, nt3;
      FK_TILE_FETCH(a, Np);
      FK_F32_LOAD4(c, Np, v0, v1, v2, v3);
      __syncthreads();
      FK_TILE_STAGE(As);
      FK_F32_STORE4(Bs, v0, v1, v2, v3);
    }
    __syncthreads();
    mfma_tile64_nn(As, Bs, acc);
  }
  if constexpr (SECOND)
    store_acc(Al + (size_t)i * NB * Np + j * NB, Np, acc, false, -1.f);
  else
    store_acc(Al + (size_t)j * NB * Np + i * NB, Np, acc, false, 1.f);
}

// One product of a forward step for 16 rows and all columns: the four waves share the k range, their
// parts are added in a fixed order.  Lane (li, lk) of a wave holds, per 16 k, the matrix entries of row li
// at k = 4 lk + e and the vector entries of column li at the same k (e = 0..3, one matrix product each),
// straight from memory.  K: first row of the super-block, KE: its end.
//   INV:  out[r] = sum_{k <= r} Inv[r][k] v[k]   r in the super-block
//   else: out[r] -= sum_k L[r][k] v[k]           r >= KE
// v and out: [lambda][column][Np].
template <bool INV>
__device__ __forceinline__ float tri_entry(uint32_t x) { return INV ? __uint_as_float(x) : split_unpack(x); }

template <bool INV, int NCT>
__global__ __launch_bounds__(256) void k_tri_fwd(const float* __restrict__ A, int Np, int K, int KE,
                                                 const float* __restrict__ v, float* __restrict__ out, int ncol) {
  __shared__ float part[4][16][16 * NCT + 1];
  const int l = blockIdx.y;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int r0 = (INV ? K : KE) + 16 * blockIdx.x;
  const uint32_t* Al = reinterpret_cast<const uint32_t*>(A) + (size_t)l * Np * Np;
  const float* vl = v + (size_t)l * ncol * Np;
  // k range: whole 64-blocks (a diagonal block's zeros are stored), so that a wave's share is a multiple of 16
  const int len = ((INV ? r0 / NB * NB + NB : KE) - K) / 4, kw = K + w * len;
  floatx4 acc[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) acc[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int k = kw; k < kw + len; k += 16) {
    const uint4 m = *reinterpret_cast<const uint4*>(Al + (size_t)(r0 + li) * Np + k + 4 * lk);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const int t = min(ct * 16 + li, ncol - 1);
      const float4 b = *reinterpret_cast<const float4*>(vl + (size_t)t * Np + k + 4 * lk);
      acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m.x), b.x, acc[ct], 0, 0, 0);
      acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m.y), b.y, acc[ct], 0, 0, 0);
      acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m.z), b.z, acc[ct], 0, 0, 0);
      acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m.w), b.w, acc[ct], 0, 0, 0);
    }
  }
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int e = 0; e < 4; ++e) part[w][4 * lk + e][ct * 16 + li] = acc[ct][e];
  __syncthreads();
  float* ol = out + (size_t)l * ncol * Np;
#pragma unroll
  for (int u = 0; u < NCT; ++u) {
    const int i = threadIdx.x + 256 * u, t = i / 16, r = i % 16;
    if (t >= ncol) continue;
    const float s = (part[0][r][t] + part[1][r][t]) + (part[2][r][t] + part[3][r][t]);
    float* o = ol + (size_t)t * Np + r0 + r;
    *o = INV ? s : *o - s;
  }
}

// The transposed product of a backward step for 64 outputs (columns c of the matrix):
//   INV:  out[c] = sum_{k >= c} Inv[k][c] v[k]   c in the super-block
//   else: out[c] -= sum_k L[k][c] v[k]           c < K
// The eight waves share the 16-row groups of the k range.  A lane reads four consecutive columns 4 li ..
// of a row (rows whole: 256 contiguous bytes per 16 lanes; one column per lane took 10 us a launch, this
// 6); entry q of the four is the matrix operand of the product for the columns 4 li + q.
constexpr int TBW = 8;
template <bool INV, int NCT>
__global__ __launch_bounds__(64 * TBW) void k_tri_bwd(const float* __restrict__ A, int Np, int K, int KE,
                                                      const float* __restrict__ v, float* __restrict__ out, int ncol) {
  __shared__ float part[TBW][64][16 * NCT + 1];
  const int l = blockIdx.y;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int c0 = (INV ? K : 0) + 64 * blockIdx.x;
  const uint32_t* Al = reinterpret_cast<const uint32_t*>(A) + (size_t)l * Np * Np + c0 + 4 * li;
  const float* vl = v + (size_t)l * ncol * Np;
  const int ka = INV ? c0 : K, groups = (KE - ka) / 16;
  const int g0 = groups * w / TBW, g1 = groups * (w + 1) / TBW;
  floatx4 acc[NCT][4];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[ct][q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int g = g0; g < g1; ++g) {
    const int k = ka + 16 * g + 4 * lk;
    uint4 m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) m[j] = *reinterpret_cast<const uint4*>(Al + (size_t)(k + j) * Np);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const int t = min(ct * 16 + li, ncol - 1);
      const float4 b = *reinterpret_cast<const float4*>(vl + (size_t)t * Np + k);
      const float bj[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[ct][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m[j].x), bj[j], acc[ct][0], 0, 0, 0);
        acc[ct][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m[j].y), bj[j], acc[ct][1], 0, 0, 0);
        acc[ct][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m[j].z), bj[j], acc[ct][2], 0, 0, 0);
        acc[ct][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(tri_entry<INV>(m[j].w), bj[j], acc[ct][3], 0, 0, 0);
      }
    }
  }
  // row 4 lk + e of product q is column 4 (4 lk + e) + q
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[w][4 * (4 * lk + e) + q][ct * 16 + li] = acc[ct][q][e];
  __syncthreads();
  float* ol = out + (size_t)l * ncol * Np;
  for (int i = threadIdx.x; i < 64 * ncol; i += 64 * TBW) {
    const int t = i / 64, c = i % 64;
    float s = part[0][c][t];
#pragma unroll
    for (int u = 1; u < TBW; ++u) s += part[u][c][t];
    float* o = ol + (size_t)t * Np + c0 + c;
    *o = INV ? s : *o - s;
  }
}

// ------------------------------------------------------------------ FP64 residual
// Rres[l][t] = Bre[t] - (H64 + lambda_l diag(preal)) X[l][t], for all (l, t) at once:
// one FP64 GEMM H64 (Np x Np) times X (Np x ncolsTotal), then the diagonal and the
// subtraction.  Column c of X/Rres is (l, t) with l = c / ntgt.  With R32, the scaled residual in FP32 as
// well: the right-hand side of the next refinement step.
// On the FP64 matrix cores (v_mfma_f64_16x16x4f64): lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16]; element v of lane l's accumulator is D[l / 16 + 4 v][l % 16]
// (the FP32 form holds D[4 (l / 16) + v][l % 16] instead).  A workgroup computes 64 rows
// x 32 WN columns, its four waves 32 rows x 16 WN columns each (2 x WN blocks of
// 16 x 16).  The k dimension streams in chunks of 16 through double-buffered LDS (the
// next chunk in registers meanwhile).  Every operand value read from LDS feeds 16
// multiply-adds (a 4 x 4 register block on the vector units gets 2), so the kernel is
// bound by the FP64 matrix rate.
template <int WN>
__global__ __launch_bounds__(256) void k_resid64_mfma(const double* __restrict__ H, int N, int Np,
                                                      const double* __restrict__ X, int ncols, int ntgt,
                                                      int rhs_per_col, const double* __restrict__ Bre,
                                                      const double* __restrict__ preal,
                                                      const double* __restrict__ lams, double* __restrict__ Rres,
                                                      const double* __restrict__ scl, float* __restrict__ R32) {
  constexpr int TM = 64, TN = 32 * WN, KC = 16;
  constexpr int PH = TM * KC / 256, PX = TN * KC / 256;
  __shared__ double Hs[2][KC][TM + 4];  // Hs[k][row]
  __shared__ double Xs[2][KC][TN + 4];  // Xs[k][col]
  const int row0 = blockIdx.x * TM, col0 = blockIdx.y * TN;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wr = (w >> 1) * 32, wc = (w & 1) * 16 * WN;
  const int li = lane & 15, lk = lane >> 4;
  // global element e = tid + 256 u of a chunk: (row or column e / 16, k e % 16)
  const int gk = threadIdx.x & (KC - 1), gr = threadIdx.x >> 4;
  const int cmax = ncols - 1;
  double ph[PH], px[PX];
#define FK_RLOAD(k0)                                                                              \
  do {                                                                                            \
    _Pragma("unroll") for (int u = 0; u < PH; ++u)                                                \
      ph[u] = H[(size_t)(row0 + gr + 16 * u) * Np + (k0) + gk];                                  \
    _Pragma("unroll") for (int u = 0; u < PX; ++u)                                                \
      px[u] = X[(size_t)min(col0 + gr + 16 * u, cmax) * Np + (k0) + gk];                         \
  } while (0)
#define FK_RSTORE(buf)                                                                            \
  do {                                                                                            \
    _Pragma("unroll") for (int u = 0; u < PH; ++u) Hs[buf][gk][gr + 16 * u] = ph[u];              \
    _Pragma("unroll") for (int u = 0; u < PX; ++u)                                                \
      Xs[buf][gk][gr + 16 * u] = (col0 + gr + 16 * u <= cmax) ? px[u] : 0.0;                      \
  } while (0)
  doublex4 acc[2][WN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  FK_RLOAD(0);
  FK_RSTORE(0);
  __syncthreads();
  const int nk = Np / KC;
  for (int kc = 0; kc < nk; ++kc) {
    const int cur = kc & 1;
    if (kc + 1 < nk) FK_RLOAD((kc + 1) * KC);
#pragma unroll
    for (int ks = 0; ks < KC; ks += 4) {
      double a[2], b[WN];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = Hs[cur][ks + lk][wr + 16 * i + li];
#pragma unroll
      for (int j = 0; j < WN; ++j) b[j] = Xs[cur][ks + lk][wc + 16 * j + li];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kc + 1 < nk) FK_RSTORE(cur ^ 1);
    __syncthreads();
  }
#undef FK_RLOAD
#undef FK_RSTORE
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    const int c = col0 + wc + 16 * j + li;
    if (c >= ncols) continue;
    const int l = c / ntgt, t = c - l * ntgt;
    const double lam = lams[l];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = row0 + wr + 16 * i + lk + 4 * v;
        const double xv = X[(size_t)c * Np + r];
        const double ax = acc[i][j][v] + (r < N ? lam * preal[r] * xv : 0.0);
        const double bv = (r < N) ? Bre[(size_t)(rhs_per_col ? c : t) * Np + r] : 0.0;
        Rres[(size_t)c * Np + r] = bv - ax;
        if (R32) R32[(size_t)c * Np + r] = (float)((bv - ax) * scl[(size_t)l * Np + r]);
      }
  }
}

// The same residual for up to a few hundred columns, where the tiled kernel has too few tiles for the
// chip and each walks all of k alone: a workgroup takes 16 rows and 16 NCT columns, its eight waves share
// k, and their parts are added in a fixed order.  Operands straight from memory: lane (li, lk) holds row
// (column) li at k = 4 lk + e, e = 0..3, one matrix product each.  Bound by the read of H (147 MB in
// 46 us at N = 4225, one column); N = 1089: 15 columns 70 -> 5 us, N = 4225: 32 columns 200 -> 60 us.
// Tiled kernel against this, solve with one refinement step: N = 1089, 24 columns 292 / 176 us, N = 2401,
// 256 columns 671 / 644, N = 4225, 128 columns 1374 / 1329 and 1024 columns 4531 / 5488.
constexpr int kRowsCols = 256;
template <int NCT>
__global__ __launch_bounds__(512) void k_resid64_rows(const double* __restrict__ H, int N, int Np,
                                                      const double* __restrict__ X, int ncols, int ntgt,
                                                      int rhs_per_col, const double* __restrict__ Bre,
                                                      const double* __restrict__ preal,
                                                      const double* __restrict__ lams, double* __restrict__ Rres,
                                                      const double* __restrict__ scl, float* __restrict__ R32) {
  __shared__ double part[8][16][16 * NCT + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int r0 = blockIdx.x * 16, c0 = blockIdx.y * 16 * NCT;
  const int groups = Np / 16, g0 = groups * w / 8, g1 = groups * (w + 1) / 8;
  const double* h = H + (size_t)(r0 + li) * Np + 4 * lk;
  const double* x[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) x[ct] = X + (size_t)min(c0 + 16 * ct + li, ncols - 1) * Np + 4 * lk;
  doublex4 acc[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) acc[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int g = g0; g < g1; ++g) {
    const doublex4 a = *reinterpret_cast<const doublex4*>(h + 16 * g);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const doublex4 b = *reinterpret_cast<const doublex4*>(x[ct] + 16 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[e], acc[ct], 0, 0, 0);
    }
  }
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[w][lk + 4 * v][16 * ct + li] = acc[ct][v];
  __syncthreads();
  for (int i = threadIdx.x; i < 256 * NCT; i += 512) {
    const int r = r0 + i % 16, cc = i / 16, c = c0 + cc;
    if (c >= ncols) continue;
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) a += part[u][i % 16][cc];
    const int l = c / ntgt, t = c - l * ntgt;
    const double xv = X[(size_t)c * Np + r];
    const double ax = a + (r < N ? lams[l] * preal[r] * xv : 0.0);
    const double bv = (r < N) ? Bre[(size_t)(rhs_per_col ? c : t) * Np + r] : 0.0;
    Rres[(size_t)c * Np + r] = bv - ax;
    if (R32) R32[(size_t)c * Np + r] = (float)((bv - ax) * scl[(size_t)l * Np + r]);
  }
}

static void launch_resid(hipStream_t st, const double* H, int N, int Np, const double* X, int ncols, int ntgt,
                         int rhs_per_col, const double* Bre, const double* preal, const double* lams, double* R,
                         const double* scl, float* R32) {
  if (ncols <= kRowsCols) {
    const int nct = (ncols + 15) / 16;
#define FK_ROWS(NCT)                                                                                                \
  hipLaunchKernelGGL(k_resid64_rows<NCT>, dim3(Np / 16, (nct + NCT - 1) / NCT), dim3(512), 0, st, H, N, Np, X,       \
                     ncols, ntgt, rhs_per_col, Bre, preal, lams, R, scl, R32)
    if (nct == 1) FK_ROWS(1);
    else if (nct == 2) FK_ROWS(2);
    else if (nct == 3) FK_ROWS(3);
    else FK_ROWS(4);
#undef FK_ROWS
    return;
  }
  // Column tile of 32 WN: the one with the fewest tile columns per CU, counting every CU's last
  // round as full (ceil(tiles / 256 CUs) rounds x TN columns of work each); ties to the wider tile,
  // which reuses each loaded H value more.  For 1024 columns: WN = 3 (737 tiles, 3 rounds x 96)
  // against WN = 4 (536 tiles, 3 rounds x 128).
  int best_wn = 4;
  long best = -1;
  for (int wn = 4; wn >= 2; --wn) {
    const long tiles = (long)(Np / 64) * ((ncols + 32 * wn - 1) / (32 * wn));
    const long cost = (tiles + 255) / 256 * (32 * wn);
    if (best < 0 || cost < best) {
      best = cost;
      best_wn = wn;
    }
  }
  const int TN = 32 * best_wn;
  const dim3 grid(Np / 64, (ncols + TN - 1) / TN);
  if (best_wn == 4)
    hipLaunchKernelGGL(k_resid64_mfma<4>, grid, dim3(256), 0, st, H, N, Np, X, ncols, ntgt, rhs_per_col, Bre, preal,
                       lams, R, scl, R32);
  else if (best_wn == 3)
    hipLaunchKernelGGL(k_resid64_mfma<3>, grid, dim3(256), 0, st, H, N, Np, X, ncols, ntgt, rhs_per_col, Bre, preal,
                       lams, R, scl, R32);
  else
    hipLaunchKernelGGL(k_resid64_mfma<2>, grid, dim3(256), 0, st, H, N, Np, X, ncols, ntgt, rhs_per_col, Bre, preal,
                       lams, R, scl, R32);
}

// Sum over a workgroup of 256 threads, in thread 0.
__device__ __forceinline__ double sum256(double s, double* part) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  return (part[0] + part[1]) + (part[2] + part[3]);
}

// Column norms squared (one workgroup per column), FP64; the context's error flags behind them (as
// doubles at out[flag_at ..]), so that one copy brings both.
__global__ __launch_bounds__(256) void k_colnorm2(const double* __restrict__ V, int Np, double* __restrict__ out,
                                                  const int* __restrict__ flags, int flag_at) {
  __shared__ double part[4];
  const double* v = V + (size_t)blockIdx.x * Np;
  double s = 0.0;
  for (int i = threadIdx.x; i < Np; i += 256) s += v[i] * v[i];
  s = sum256(s, part);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
  if (blockIdx.x == 0 && threadIdx.x < kFlagCount) out[flag_at + threadIdx.x] = (double)flags[threadIdx.x];
}

// Start of a solve: R32 = S rhs in FP32 for every column (l, t) = (c / ntgt, c % ntgt), from per-target (or
// per-column) right-hand sides, and the norms squared of the right-hand sides.
__global__ __launch_bounds__(256) void k_refine_init(const double* __restrict__ rhs, int per_col,
                                                     const double* __restrict__ scl, int Np, int ntgt,
                                                     float* __restrict__ R32, double* __restrict__ norms) {
  __shared__ double part[4];
  const int c = blockIdx.x, l = c / ntgt;
  const double* v = rhs + (size_t)(per_col ? c : c - l * ntgt) * Np;
  double s = 0.0;
  for (int i = threadIdx.x; i < Np; i += 256) {
    const double x = v[i];
    R32[(size_t)c * Np + i] = (float)(x * scl[(size_t)l * Np + i]);
    s += x * x;
  }
  s = sum256(s, part);
  if (threadIdx.x == 0) norms[c] = s;
}

// X = (first ? 0 : X) + S d, with the per-lambda scaling; column blockIdx.y = (lambda, target).
__global__ void k_scale_axpy_f2d(const float* __restrict__ a, const double* __restrict__ scl, int Np, int ntgt,
                                 double* __restrict__ X, int first) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= Np) return;
  const size_t i = (size_t)blockIdx.y * Np + r;
  const double v = scl[(size_t)(blockIdx.y / ntgt) * Np + r] * (double)a[i];
  X[i] = first ? v : X[i] + v;
}

}  // namespace fk

// ==================================================================== host drivers
namespace fk {

static int round64(int n) { return (n + NB - 1) / NB * NB; }

SolveLayout solve_layout(int N, int nlam, int ntgt, void* base, size_t cap) {
  SolveLayout s;
  s.N = N;
  s.Np = round64(N);
  s.nlam = nlam;
  s.ntgt = ntgt;
  const size_t Np = s.Np;
  const size_t nc = (size_t)nlam * ntgt;
  Carve cv(base, cap);
  s.H64 = cv.take<double>(Np * Np);
  s.A32 = cv.take<float>((size_t)nlam * Np * Np);
  s.Linv = cv.take<float>((size_t)nlam * Np * NB);
  s.preal = cv.take<double>(Np);
  s.lams = cv.take<double>((size_t)nlam + N);   // and, behind them, the complex-mode weights: one upload
  s.pcx = s.lams ? s.lams + nlam : nullptr;
  s.Bre = cv.take<double>((size_t)ntgt * Np);
  s.X64 = cv.take<double>(nc * Np);
  s.R64 = cv.take<double>(nc * Np);
  s.U64 = cv.take<double>(nc * Np);
  s.G64 = cv.take<double>(nc * Np);
  s.Gadj = cv.take<double>(nc * Np);
  s.R32 = cv.take<float>(nc * Np);
  s.Y32 = cv.take<float>(nc * Np);
  s.D32 = cv.take<float>(nc * Np);
  s.norms = cv.take<double>(2 * nc + nlam + 64);
  s.Hv = cv.take<double>(Np * Np);
  s.Bv = cv.take<double>((size_t)ntgt * Np);
  s.scl = cv.take<double>((size_t)nlam * Np);
  s.dsym = cv.take<double>((size_t)2 * N);
  // parts of the split paired updates: 768 tiles of 64 x 128 at most (fewer for small systems)
  const int nb = (int)(Np / NB);
  s.part_tiles = (int)std::min<int64_t>(768, (int64_t)nb * nb * nlam);
  s.upart = cv.take<float>((size_t)s.part_tiles * NB * 2 * NB);
  s.bytes = ((cv.off + 255) & ~size_t(255)) + 256;   // a multiple of 256: what follows stays aligned
  return s;
}

// Splits of the paired update's sum over panels when its grid is small (few lambdas, or the last
// block columns): about three workgroups per CU in all, at least two panels per split, within the
// workspace's part tiles.  1 = no split.
static int update_split(int wgs, int kb, int part_tiles) {
  if (wgs >= 512 || kb < 4) return 1;
  int ns = std::min(std::min(kb / 2, kMaxSplit), 768 / wgs);
  ns = std::min(ns, part_tiles / wgs);
  return std::max(ns, 1);
}

// Most workgroups of a block column (rows x lambdas) whose panel is solved in the launch that factors
// the diagonal block, every workgroup factoring it for itself: up to four such workgroups fit a CU, so
// 1024 run at once and the launch costs one factorization, against two launches.  Whole factorization,
// fused up to 0 / 512 / 1024 / 8192 workgroups: N = 4225, one lambda 1401 / 1076 / 1078 / 1078 us; 8
// lambdas 2463 / 2198 / 2181 / 2182; N = 1089, 64 lambdas 601 / 573 / 561 / 569.  A block column that
// also takes the term of the panel before it is fused at any size: two launches saved and the panel
// tile read once (64 lambdas, N = 4225: 11.40 ms up to 1024 workgroups, 11.20 always).
constexpr int kFusedPanelWgs = 1024;

// Pairs of block columns that one unsplit update takes: two where the lower triangles of all lambdas are past what the
// caches hold (256 MB), and a pair's pass over the row panels comes from memory.  Whole factorization, one pair /
// two / four: N = 4225, 64 lambdas (2.3 GB) 11.17 / 10.46 / 10.55 ms, 16 lambdas (590 MB) 3.74 / 3.68 / 3.57, 8 lambdas
// (290 MB) 2.26 / 2.29 / 2.26; N = 2401, 16 lambdas (190 MB) 1.19 / 1.21 / 1.21; N = 1089, 64 lambdas 565 / 580 / 594 us.
static int update_pairs(const SolveLayout& s) { return 2.0 * s.Np * s.Np * s.nlam > 4e8 ? 2 : 1; }

// Factor A32[l] = L L^T for every lambda: left-looking blocked Cholesky, per block column an
// update with the finished panels (one pass over the column), the factorization of the
// diagonal block, the solve of the panel below it.
static fk_status factor_all(fk_ctx* ctx, const SolveLayout& s, const DenseShape& sh) {
  const int nb = s.Np / NB;
  // diagonal block and the panel below it; upd: block column kb first takes its term of panel kb - 1
  auto finish = [&](int kb, bool upd) {
    const int rem = nb - kb - 1;
    const bool fused = !sh.diag64 && (upd || (rem + 1) * s.nlam <= kFusedPanelWgs);
    if (upd && !fused)
      hipLaunchKernelGGL(k_left_update, dim3((nb - kb) * s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, kb - 1,
                         kb, s.nlam);
    if (fused) {
      if (upd)
        hipLaunchKernelGGL((k_factor_diag<true, true>), dim3((rem + 1) * s.nlam), dim3(256), 0, ctx->stream, s.A32,
                           s.Np, kb, s.Linv, s.nlam, ctx->flags);
      else
        hipLaunchKernelGGL((k_factor_diag<true, false>), dim3((rem + 1) * s.nlam), dim3(256), 0, ctx->stream, s.A32,
                           s.Np, kb, s.Linv, s.nlam, ctx->flags);
      return;
    }
    if (sh.diag64)
      hipLaunchKernelGGL(k_potrf_diag64, dim3(s.nlam), dim3(kPotrfThreads), 0, ctx->stream, s.A32, s.Np, kb, s.Linv,
                         ctx->flags);
    else
      hipLaunchKernelGGL((k_factor_diag<false, false>), dim3(s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb,
                         s.Linv, s.nlam, ctx->flags);
    if (rem > 0)
      hipLaunchKernelGGL(k_trsm_panel, dim3(rem * s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv,
                         s.nlam);
  };
  // Block columns in pairs (kb, kb + 1): one pass over the panels k < kb updates both,
  // then column kb is finished, then column kb + 1 takes its remaining term k = kb.
  for (int kb = 0; kb < nb;) {
    if (sh.pair && kb > 0 && kb + 1 < nb) {
      const int wgs = (nb - kb) * s.nlam;
      const int nsplit = update_split(wgs, kb, s.part_tiles);
      if (nsplit > 1) {
        hipLaunchKernelGGL(k_left_update2<true>, dim3(wgs * nsplit), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, 0, kb, 1,
                           s.nlam, nsplit, s.upart);
        hipLaunchKernelGGL(k_left_update2_sum, dim3(wgs * 8), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.nlam,
                           nsplit, s.upart);
      } else {
        // G pairs at once; inside the group, a pair then takes the panels of the pairs before it
        const int G = std::max(1, std::min(update_pairs(s), (nb - kb) / 2));
        hipLaunchKernelGGL(k_left_update2<false>, dim3(wgs * G), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, 0, kb, G,
                           s.nlam, 1, nullptr);
        for (int p = 0; p < G; ++p) {
          const int c = kb + 2 * p;
          if (p > 0)
            hipLaunchKernelGGL(k_left_update2<false>, dim3((nb - c) * s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, c,
                               kb, c, 1, s.nlam, 1, nullptr);
          finish(c, false);
          finish(c + 1, true);
        }
        kb += 2 * G;
        continue;
      }
      finish(kb, false);
      finish(kb + 1, true);
      kb += 2;
    } else {
      const bool one = kb == 1;   // a single panel before it: its term goes with the diagonal block
      if (kb > 1)
        hipLaunchKernelGGL(k_left_update, dim3((nb - kb) * s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, 0,
                           kb, s.nlam);
      finish(kb, one);
      kb += 1;
    }
  }
  FK_HIP(hipGetLastError());
  return FK_OK;
}

// Whether the solves of this shape go through inverted super-blocks: from three block columns on (two are
// one launch of the sweeps), and while the inverses, whose cost grows with nb nlam, cost less than the
// launches they save.  Factor + inverses and solves with one refinement step, sweeps / super-blocks:
// N = 4225 (nb = 67), 1 lambda and target 1952 / 1562 us, 16 lambdas x 8 targets 5505 / 5116, 64 x 16 16036
// / 16256; N = 2401, 16 x 16 2104 / 1873; N = 1089 (nb = 18), 5 x 3 656 / 579, 64 x 16 1252 / 1261; N = 289
// (nb = 5), 1 x 1 166 / 157.
static bool super_solve(const SolveLayout& s) {
  const int nb = s.Np / NB;
  return nb >= 3 && nb * s.nlam <= 1100;
}

// The super-blocks' inverses, after factor_all.
static fk_status invert_super(fk_ctx* ctx, const SolveLayout& s) {
  const int nb = s.Np / NB, nsb = (nb + SB - 1) / SB;
  hipLaunchKernelGGL(k_inv_pair, dim3((nb + 1) / 2 * s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, s.Linv);
  for (int ht = 2; ht < std::min(SB, nb); ht *= 2) {
    const dim3 grid(ht * ht * (SB / (2 * ht)) * nsb * s.nlam);
    hipLaunchKernelGGL(k_inv_level<false>, grid, dim3(256), 0, ctx->stream, s.A32, s.Np, ht);
    hipLaunchKernelGGL(k_inv_level<true>, grid, dim3(256), 0, ctx->stream, s.A32, s.Np, ht);
  }
  FK_HIP(hipGetLastError());
  return FK_OK;
}

template <int NCT>
static void super_steps(fk_ctx* ctx, const SolveLayout& s, float* R, float* Y, float* X) {
  const int W = SB * NB, nsb = (s.Np + W - 1) / W;
  for (int k = 0; k < nsb; ++k) {
    const int K = k * W, KE = std::min(s.Np, K + W);
    hipLaunchKernelGGL((k_tri_fwd<true, NCT>), dim3((KE - K) / 16, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, K,
                       KE, R, Y, s.ntgt);
    if (KE < s.Np)
      hipLaunchKernelGGL((k_tri_fwd<false, NCT>), dim3((s.Np - KE) / 16, s.nlam), dim3(256), 0, ctx->stream, s.A32,
                         s.Np, K, KE, Y, R, s.ntgt);
  }
  for (int k = nsb - 1; k >= 0; --k) {
    const int K = k * W, KE = std::min(s.Np, K + W);
    hipLaunchKernelGGL((k_tri_bwd<true, NCT>), dim3((KE - K) / 64, s.nlam), dim3(64 * TBW), 0, ctx->stream, s.A32,
                       s.Np, K, KE, Y, X, s.ntgt);
    if (K > 0)
      hipLaunchKernelGGL((k_tri_bwd<false, NCT>), dim3(K / 64, s.nlam), dim3(64 * TBW), 0, ctx->stream, s.A32, s.Np, K,
                         KE, X, Y, s.ntgt);
  }
}

// D32 = A^-1 R32 per lambda (ncol = ntgt columns each), through Y32.
static fk_status trsm_all(fk_ctx* ctx, const SolveLayout& s, const DenseShape& sh, float* R, float* Y, float* X) {
  const int nb = s.Np / NB;
  const bool two = s.ntgt > 16;
  if (super_solve(s)) {
    if (two) super_steps<2>(ctx, s, R, Y, X);
    else super_steps<1>(ctx, s, R, Y, X);
    FK_HIP(hipGetLastError());
    return FK_OK;
  }
  // workgroups per lambda: about sh.trsm_wg in all, each sweeping several rows
  const int gmax = std::max(1, sh.trsm_wg / s.nlam);
  // two block columns per launch (the last one alone when nb is odd)
  for (int kb = 0; kb < nb;) {
    if (kb + 1 < nb) {
      const int g = std::max(1, std::min(gmax, nb - kb - 2));
      if (two)
        hipLaunchKernelGGL(k_fwd2_mfma<2>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, R,
                           Y, s.ntgt);
      else
        hipLaunchKernelGGL(k_fwd2_mfma<1>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, R,
                           Y, s.ntgt);
      kb += 2;
    } else {
      const int g = std::max(1, std::min(gmax, nb - kb - 1));
      if (two)
        hipLaunchKernelGGL(k_fwd_mfma<2>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, R,
                           Y, s.ntgt);
      else
        hipLaunchKernelGGL(k_fwd_mfma<1>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, R,
                           Y, s.ntgt);
      kb += 1;
    }
  }
  for (int kb = nb - 1; kb >= 0;) {
    if (kb >= 1) {
      const int g = std::max(1, std::min(gmax, kb - 1));
      if (two)
        hipLaunchKernelGGL(k_bwd2_mfma<2>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, Y,
                           X, s.ntgt);
      else
        hipLaunchKernelGGL(k_bwd2_mfma<1>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, Y,
                           X, s.ntgt);
      kb -= 2;
    } else {
      const int g = std::max(1, std::min(gmax, kb));
      if (two)
        hipLaunchKernelGGL(k_bwd_mfma<2>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, Y,
                           X, s.ntgt);
      else
        hipLaunchKernelGGL(k_bwd_mfma<1>, dim3(g, s.nlam), dim3(256), 0, ctx->stream, s.A32, s.Np, kb, s.Linv, Y,
                           X, s.ntgt);
      kb -= 1;
    }
  }
  FK_HIP(hipGetLastError());
  return FK_OK;
}

// ------------------------------------------------------------------ small systems: refinement in one launch

// Up to 128 unknowns (one or two block columns) and 4 targets: a workgroup per lambda runs the FP32 solve with the
// factors, the FP64 update and the FP64 residual, `steps` times, and the norms, in place of ten launches of 1.5 to
// 3.6 us.  Bound by latency: 18 us (N = 101, one target, two steps).  Whole solves, ten launches / this: N = 41
// 111 / 71 us, N = 101 113 / 94, with 16 lambdas and 1, 4, 16 targets 129 / 108, 135 / 122 and 139 / 163 (the
// residual's columns, 16 at a time in registers, take longer than their own launch).
// Wave t owns column t of the FP32 solve, so its five products need no barrier.  NT: the
// columns of the residual's registers.
constexpr int kSmallCols = 4;
constexpr int CL = kSmallCols + 1;   // row stride of the right-hand sides in LDS
constexpr size_t kSmallLds = sizeof(float) * (3 * NB * (NB + 1) + 2 * NB * CL) +
                             sizeof(double) * (2 * NB * CL + 4 * kSmallCols + 2 * NB * 33);

template <int NT>
__global__ __launch_bounds__(256) void k_small_refine(const float* __restrict__ A, const float* __restrict__ Linv,
                                                      const double* __restrict__ H, int N, int Np,
                                                      const double* __restrict__ rhs, int per_col,
                                                      const double* __restrict__ scl, const double* __restrict__ preal,
                                                      const double* __restrict__ lams, int ntgt, int nc, int first,
                                                      int steps, double* __restrict__ X, float* __restrict__ R32,
                                                      double* __restrict__ norms, const int* __restrict__ flags) {
  extern __shared__ __align__(16) double lds_small[];
  double* Xs = lds_small;                                     // [128][CL]
  double* part = Xs + 2 * NB * CL;                            // [4][kSmallCols]
  double* Hc = part + 4 * kSmallCols;                         // the residual's chunk of H, [128][33]
  float* Bs = reinterpret_cast<float*>(Hc + 2 * NB * 33);     // [128][CL]
  float* Ls = Bs + 2 * NB * CL;                               // three blocks, rows of 65
  const int l = blockIdx.x, nb = Np / NB, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const double* sl = scl + (size_t)l * Np;
  // every load of the blocks and of the first chunk of H in flight together
  float4 tile[3][4];
#pragma unroll
  for (int blk = 0; blk < 3; ++blk)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = 4 * (tid + 256 * u), row = e / NB, col = e % NB;
      if (blk == 0 || nb == 2)
        tile[blk][u] = *reinterpret_cast<const float4*>(blk == 1 ? A + (size_t)l * Np * Np + (size_t)(NB + row) * Np + col
                                                                 : Linv + ((size_t)l * nb + blk / 2) * NB * NB + e);
    }
  double2 hc[8];
  auto fetch_h = [&](int k0) {   // thread: rows tid / 16 + 16 u, two columns
#pragma unroll
    for (int u = 0; u < 8; ++u)
      hc[u] = *reinterpret_cast<const double2*>(H + (size_t)min(tid / 16 + 16 * u, Np - 1) * Np + k0 + 2 * (tid & 15));
  };
  fetch_h(0);
#pragma unroll
  for (int blk = 0; blk < 3; ++blk)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = 4 * (tid + 256 * u);
      float* o = Ls + blk * NB * (NB + 1) + e / NB * (NB + 1) + e % NB;
      const float4 v = tile[blk][u];
      if (blk == 0 || nb == 2) {
        o[0] = blk == 1 ? split_unpack(__float_as_uint(v.x)) : v.x;   // the panel: FP16 pairs
        o[1] = blk == 1 ? split_unpack(__float_as_uint(v.y)) : v.y;
        o[2] = blk == 1 ? split_unpack(__float_as_uint(v.z)) : v.z;
        o[3] = blk == 1 ? split_unpack(__float_as_uint(v.w)) : v.w;
      }
    }
  auto rhs_at = [&](int t, int r) { return rhs[(size_t)(per_col ? l * ntgt + t : t) * Np + r]; };
  if (w < ntgt) {
    const int t = w, c = l * ntgt + t;
    double s = 0.0;
    for (int r = lane; r < Np; r += 64) {
      if (first) {
        const double x = rhs_at(t, r);
        Bs[r * CL + t] = (float)(x * sl[r]);
        Xs[r * CL + t] = 0.0;
        s += x * x;
      } else {
        Bs[r * CL + t] = R32[(size_t)c * Np + r];
        Xs[r * CL + t] = X[(size_t)c * Np + r];
      }
    }
    if (first) {
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (lane == 0) norms[nc + c] = s;
    }
  }
  // out = sum_k M[lane][k] b[k][w] (or M^T), M one of the staged blocks
  float out;
  auto product = [&](int blk, bool tr, int row0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const float* m = Ls + blk * NB * (NB + 1) + (tr ? lane : lane * (NB + 1));
    const int sm = tr ? NB + 1 : 1;
    const float* b = Bs + row0 * CL + w;
    out = 0.f;
#pragma unroll 16
    for (int k = 0; k < NB; ++k) out = fmaf(m[k * sm], b[k * CL], out);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto put = [&](int row0, bool sub) {
    float* o = Bs + (row0 + lane) * CL + w;
    *o = sub ? *o - out : out;
  };
  const int r = tid >> 1, h = tid & 1;   // of the residual: row, half of k
  for (int step = 0; step < steps; ++step) {
    __syncthreads();
    if (w < ntgt) {
      product(0, false, 0);   // y_0 = inv(L_00) r_0
      put(0, false);
      if (nb == 2) {
        product(1, false, 0);   // y_1 = inv(L_11) (r_1 - L_10 y_0)
        put(NB, true);
        product(2, false, NB);
        put(NB, false);
        product(2, true, NB);   // x_1 = inv(L_11)^T y_1
        put(NB, false);
        product(1, true, NB);   // x_0 = inv(L_00)^T (y_0 - L_10^T x_1)
        put(0, true);
      }
      product(0, true, 0);
      put(0, false);
      for (int q = lane; q < Np; q += 64) Xs[q * CL + w] += sl[q] * (double)Bs[q * CL + w];
    }
    __syncthreads();
    // residual: 32 columns of H at a time
    double acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = 0.0;
    for (int k0 = 0; k0 < Np; k0 += 32) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        double* o = Hc + (tid / 16 + 16 * u) * 33 + 2 * (tid & 15);
        o[0] = hc[u].x;
        o[1] = hc[u].y;
      }
      __syncthreads();
      fetch_h(k0 + 32 < Np ? k0 + 32 : 0);
      if (r < Np) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int k = 16 * h + q;
          const double a = Hc[r * 33 + k];
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t] = fma(a, Xs[(k0 + k) * CL + t], acc[t]);
        }
      }
      __syncthreads();
    }
    const double lp = r < N ? lams[l] * preal[r] : 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      double e = 0.0;
      acc[t] += __shfl_xor(acc[t], 1, 64);
      if (t < ntgt && r < Np) {
        e = (r < N ? rhs_at(t, r) : 0.0) - (acc[t] + lp * Xs[r * CL + t]);
        if (h == 0) Bs[r * CL + t] = (float)(e * sl[r]);
      }
      if (step == steps - 1) {
        double q = h == 0 ? e * e : 0.0;
        for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
        if (lane == 0) part[w * kSmallCols + t] = q;
      }
    }
    __syncthreads();
  }
  if (w < ntgt) {
    const int t = w, c = l * ntgt + t;
    for (int q = lane; q < Np; q += 64) {
      X[(size_t)c * Np + q] = Xs[q * CL + t];
      R32[(size_t)c * Np + q] = Bs[q * CL + t];
    }
    if (lane == 0) norms[c] = (part[t] + part[kSmallCols + t]) + (part[2 * kSmallCols + t] + part[3 * kSmallCols + t]);
  }
  if (l == 0 && tid < kFlagCount) norms[2 * nc + tid] = (double)flags[tid];
}

static bool small_solve(const SolveLayout& s) { return s.Np <= 2 * NB && s.ntgt <= kSmallCols; }

// Solve (H64 + lambda diag(preal)) X = RHS for all (lambda, target) with FP32
// factors and FP64 refinement.  RHS given per target (Bre) or per column (rhs_cols).
// Returns the number of refinement steps and the worst relative residual.
// With check_flags, every step's norm read-back also brings the context's error flags (the stages
// queued before the solve raised them: input NaN, range, not positive definite), and those are
// reported first: the caller then needs no synchronization of its own before the solve.
// after(): what the caller does with X, queued behind every step whose norms are checked, ahead of the
// host's wait for them (and queued again should a further step follow).
template <class After>
static fk_status refine_solve(fk_ctx* ctx, const SolveLayout& s, const DenseShape& sh, const double* rhs_cols,
                              double* X, int* iters_out, double* resid_out, int* bad_out, bool check_flags,
                              After after) {
  const int nc = s.nlam * s.ntgt;
  const double* rhs = rhs_cols ? rhs_cols : s.Bre;
  const int per_col = rhs_cols ? 1 : 0;
  const bool small = small_solve(s);
  if (!small)
    hipLaunchKernelGGL(k_refine_init, dim3(nc), dim3(256), 0, ctx->stream, rhs, per_col, s.scl, s.Np, s.ntgt, s.R32,
                       s.norms + nc);
  const int maxit = ctx->opt.max_refine;
  const double tol = ctx->opt.refine_tol;
  // the norms and flags come back through the context's pinned staging area (an asynchronous copy)
  const size_t back = (size_t)2 * nc + kFlagCount;
  double* nh = static_cast<double*>(stage_take(ctx, sizeof(double) * back));
  if (!nh) return FK_EHIP;
  int it = 0;
  double worst = 0.0;
  int bad = -1;
  for (;; ++it) {
    // Below 1e-8 the FP32-class first solve never meets the tolerance on its own: its check (a host
    // wait) is skipped and the first refinement step queued behind it; errors it would have found
    // (NaN, flags) are found by the next check with the same status.
    const bool unchecked = it == 0 && maxit > 0 && tol < 1e-8;
    fk_status st = FK_OK;
    if (small) {
      auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(s.nlam), dim3(256), kSmallLds, ctx->stream, s.A32, s.Linv, s.H64, s.N, s.Np, rhs,
                           per_col, s.scl, s.preal, s.lams, s.ntgt, nc, it == 0, unchecked ? 2 : 1, X, s.R32, s.norms,
                           ctx->flags);
      };
      if (s.ntgt == 1) run(k_small_refine<1>);
      else run(k_small_refine<kSmallCols>);
      FK_HIP(hipGetLastError());
      if (unchecked) ++it;
    } else {
      st = trsm_all(ctx, s, sh, s.R32, s.Y32, s.D32);
      if (st != FK_OK) return st;
      hipLaunchKernelGGL(k_scale_axpy_f2d, dim3((s.Np + 255) / 256, nc), dim3(256), 0, ctx->stream, s.D32, s.scl, s.Np,
                         s.ntgt, X, it == 0);
      // R64 = rhs - A X, and S R64 for the next step
      launch_resid(ctx->stream, s.H64, s.N, s.Np, X, nc, s.ntgt, per_col, rhs, s.preal, s.lams, s.R64, s.scl, s.R32);
      FK_HIP(hipGetLastError());
      if (unchecked) continue;
      hipLaunchKernelGGL(k_colnorm2, dim3(nc), dim3(256), 0, ctx->stream, s.R64, s.Np, s.norms, ctx->flags, 2 * nc);
    }
    FK_HIP(hipMemcpyAsync(nh, s.norms, sizeof(double) * back, hipMemcpyDeviceToHost, ctx->stream));
    st = after();
    if (st != FK_OK) return st;
    FK_HIP(hipStreamSynchronize(ctx->stream));
    if (check_flags) {
      for (int i = 0; i < kFlagCount; ++i) ctx->flags_host[i] = (int)nh[2 * nc + i];
      const fk_status fs = flag_status(ctx);
      if (fs != FK_OK) {
        *iters_out = it;
        *resid_out = 0.0;
        *bad_out = fs == FK_ENOTPD ? ctx->flags_host[kFlagNotPD + 1] : -1;
        return fs;
      }
    }
    worst = 0.0;
    bad = -1;
    for (int c = 0; c < nc; ++c) {
      // a NaN or Inf right-hand side (or one that the solve turned into one) is an input error,
      // not a refinement stall
      if (!std::isfinite(nh[c]) || !std::isfinite(nh[nc + c])) {
        *iters_out = it;
        *resid_out = nh[c];
        *bad_out = c / s.ntgt;
        return FK_ENAN;
      }
      double rel = nh[nc + c] > 0 ? std::sqrt(nh[c] / nh[nc + c]) : std::sqrt(nh[c]);
      if (!(rel <= worst)) {
        worst = rel;
        bad = c / s.ntgt;
      }
    }
    if (worst <= tol || it >= maxit) break;
  }
  *iters_out = it;
  *resid_out = worst;
  *bad_out = bad;
  return worst <= tol ? FK_OK : FK_ENOCONV;
}

static std::string dense_key(const fk_ctx* ctx, const SolveLayout& s) {
  char key[128];
  std::snprintf(key, sizeof(key), "%s dense Np=%d nlam=%d ntgt=%d", tune_arch(ctx->device).c_str(), s.Np, s.nlam,
                s.ntgt);
  return key;
}

static bool dense_tunable(const SolveLayout& s) { return (double)s.Np * s.Np * s.nlam >= (double)(1 << 28); }

// The table's launch shape of this dense shape (the defaults when there is none).
static DenseShape dense_shape(const fk_ctx* ctx, const SolveLayout& s) {
  DenseShape sh;
  std::map<std::string, double> v;
  if (tune_mode(ctx) == kTuneOff || !tune_lookup(dense_key(ctx, s), &v)) return sh;
  if (v.count("trsm_wg") && v["trsm_wg"] >= 64 && v["trsm_wg"] <= 4096) sh.trsm_wg = (int)v["trsm_wg"];
  if (v.count("pair")) sh.pair = v["pair"] != 0.0;
  if (v.count("diag64")) sh.diag64 = v["diag64"] != 0.0;
  return sh;
}

// Launch shape of the factorization and the triangular solves.  Tuning (large batched solves whose
// shape has no table entry): each pairing candidate rebuilds the FP32 matrices and factors them, and
// the chosen one's factors are left in place (*factored; rebuilt if another candidate ran last);
// each solve width is timed on zero right-hand sides.
static fk_status tune_dense(fk_ctx* ctx, const SolveLayout& s, DenseShape* out, bool* factored) {
  const int mode = tune_mode(ctx);
  *factored = false;
  *out = dense_shape(ctx, s);
  if (mode == kTuneOff || !dense_tunable(s)) return FK_OK;
  std::map<std::string, double> v;
  if (mode != kTuneForce && tune_lookup(dense_key(ctx, s), &v)) return FK_OK;
  // the trials synchronize anyway: no shape is measured on a system the earlier stages flagged
  fk_status fs = read_flags(ctx);
  if (fs != FK_OK) return fs;
  hipEvent_t e0 = ctx->ev[11], e1 = ctx->ev[12];
  DenseShape sh;
  float best_f = 0.f;
  for (int pair : {1, 0}) {
    DenseShape c = sh;
    c.pair = pair;
    hipLaunchKernelGGL(k_make_a32, dim3(a32_tiles(s.Np)), dim3(256), 0, ctx->stream, s.H64, s.preal, s.lams, s.scl, s.N, s.Np,
                       s.nlam, s.A32);
    FK_HIP(hipEventRecord(e0, ctx->stream));
    fk_status st = factor_all(ctx, s, c);
    if (st != FK_OK) return st;
    FK_HIP(hipEventRecord(e1, ctx->stream));
    FK_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    FK_HIP(hipEventElapsedTime(&ms, e0, e1));
    if (pair == 1 || ms < best_f) {
      best_f = ms;
      sh.pair = pair;
    }
  }
  // the factors the call goes on with are those of the chosen pairing, so that the first call of a
  // shape gives the same bits as the later ones
  if (sh.pair != 0) {
    hipLaunchKernelGGL(k_make_a32, dim3(a32_tiles(s.Np)), dim3(256), 0, ctx->stream, s.H64, s.preal, s.lams, s.scl,
                       s.N, s.Np, s.nlam, s.A32);
    fk_status st = factor_all(ctx, s, sh);
    if (st != FK_OK) return st;
  }
  *factored = true;
  const size_t nv = (size_t)s.nlam * s.ntgt * s.Np;
  FK_HIP(hipMemsetAsync(s.R32, 0, sizeof(float) * nv, ctx->stream));
  float best_t = 0.f;
  for (int wg : {512, 768, 256, 1024}) {
    if (super_solve(s)) break;   // no sweeps to tune
    DenseShape c = sh;
    c.trsm_wg = wg;
    FK_HIP(hipEventRecord(e0, ctx->stream));
    fk_status st = trsm_all(ctx, s, c, s.R32, s.Y32, s.D32);
    if (st != FK_OK) return st;
    FK_HIP(hipEventRecord(e1, ctx->stream));
    FK_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    FK_HIP(hipEventElapsedTime(&ms, e0, e1));
    if (wg == 512 || ms < best_t) {
      best_t = ms;
      sh.trsm_wg = wg;
    }
  }
  tune_store(dense_key(ctx, s), {{"pair", sh.pair}, {"trsm_wg", sh.trsm_wg}}, best_f + best_t);
  *out = sh;
  return FK_OK;
}

fk_status solve_impl(fk_ctx* ctx, const SolveProblem& P, const SolveLayout& s, double* theta_out,
                     fk_fit_info* info) {
  const int N = s.N, Np = s.Np;
  const int L = P.L;
  hipEvent_t* ev = ctx->ev;
  FK_HIP(hipEventRecord(ev[5], ctx->stream));
  // lambdas and penalty weights (complex modes) -> device, real-form weights and right-hand sides
  {
    double* h = static_cast<double*>(stage_take(ctx, sizeof(double) * ((size_t)s.nlam + N)));
    if (!h) return FK_EHIP;
    std::memcpy(h, P.lams.data(), sizeof(double) * s.nlam);
    std::memcpy(h + s.nlam, P.p.data(), sizeof(double) * N);
    FK_HIP(hipMemcpyAsync(s.lams, h, sizeof(double) * ((size_t)s.nlam + N), hipMemcpyHostToDevice, ctx->stream));
  }
  hipLaunchKernelGGL(k_real_inputs, dim3((Np + 255) / 256, s.ntgt + 1), dim3(256), 0, ctx->stream, s.pcx, P.b, N, L, Np,
                     s.preal, s.Bre);
  // FP64 real-form Gram (+ dense lambda-independent penalty)
  if (P.kind == SolveProblem::kToeplitz) {
    launch_assemble_pairs(ctx->stream, ToeplitzQ{P.M, P.m, P.d}, nullptr, N, Np, s.H64);
  } else if (P.kind == SolveProblem::kToeplitzPde) {
    const fk_status up = stage_upload(ctx, s.dsym, P.dsym.data(), sizeof(double) * 2 * N);
    if (up != FK_OK) return up;
    const PdeQ pq{s.dsym, P.m, P.d, P.mu, P.lo[0], P.hi[0], P.lo[1], P.hi[1]};
    launch_assemble_pairs(ctx->stream, ToeplitzQ{P.M, P.m, P.d}, &pq, N, Np, s.H64);
  } else {
    const int64_t tot2 = (int64_t)Np * Np;
    hipLaunchKernelGGL(k_assemble_real<DenseQ>, dim3((unsigned)((tot2 + 255) / 256)), dim3(256), 0, ctx->stream,
                       DenseQ{P.B, N}, N, L, Np, s.H64);
  }
  hipLaunchKernelGGL(k_make_scale, dim3((Np + 255) / 256, s.nlam), dim3(256), 0, ctx->stream, s.H64, s.preal,
                     s.lams, N, Np, s.scl);
  hipLaunchKernelGGL(k_make_a32, dim3(a32_tiles(Np)), dim3(256), 0, ctx->stream, s.H64, s.preal, s.lams, s.scl, N, Np,
                     s.nlam, s.A32);
  FK_HIP(hipGetLastError());
  DenseShape sh;
  bool factored = false;
  fk_status st = tune_dense(ctx, s, &sh, &factored);
  if (st != FK_OK) return st;
  FK_HIP(hipEventRecord(ev[6], ctx->stream));
  if (!factored) {
    st = factor_all(ctx, s, sh);
    if (st != FK_OK) return st;
  }
  if (super_solve(s)) {
    st = invert_super(ctx, s);
    if (st != FK_OK) return st;
  }
  FK_HIP(hipEventRecord(ev[7], ctx->stream));
  // the flags of the earlier stages and of the factorization come back with the first residual norms
  int iters = 0, bad = -1;
  double resid = 0.0;
  auto write_theta = [&]() -> fk_status {
    hipLaunchKernelGGL(k_theta_from_real, dim3((N + 255) / 256, s.nlam * s.ntgt), dim3(256), 0, ctx->stream, s.X64,
                       N, L, Np, s.ntgt, theta_out);
    FK_HIP(hipGetLastError());
    FK_HIP(hipEventRecord(ev[8], ctx->stream));
    return FK_OK;
  };
  st = refine_solve(ctx, s, sh, nullptr, s.X64, &iters, &resid, &bad, true, write_theta);
  if (st == FK_EHIP) return st;
  if (info) {
    info->refine_iters = iters;
    info->resid_rel = resid;
    if (st != FK_OK) info->bad_index = bad;
    float a = 0, f = 0, so = 0;
    hipEventElapsedTime(&a, ev[5], ev[6]);
    hipEventElapsedTime(&f, ev[6], ev[7]);
    hipEventElapsedTime(&so, ev[7], ev[8]);
    info->t_assemble_ms = a;
    info->t_factor_ms = f;
    info->t_solve_ms = so;
  }
  return st;
}

// ------------------------------------------------------------------ held-out loss and backward

// out[c] = x_c . v_c  (dot products of matching columns)
__global__ __launch_bounds__(256) void k_coldot(const double* __restrict__ A, const double* __restrict__ B,
                                                int Np, int bstride_cols, int ntgt, double* __restrict__ out) {
  __shared__ double part[256];
  const int c = blockIdx.x;
  const double* a = A + (size_t)c * Np;
  const double* b = B + (size_t)(bstride_cols ? c : (c % ntgt)) * Np;
  double s = 0.0;
  for (int i = threadIdx.x; i < Np; i += blockDim.x) s += a[i] * b[i];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[c] = part[0];
}

__global__ void k_mse_combine(const double* __restrict__ xg, const double* __restrict__ bx,
                              const double* __restrict__ yv2, int nc, int ntgt, double* __restrict__ mse) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nc) return;
  mse[c] = xg[c] - bx[c] + yv2[c % ntgt];   // x.(Hv x - bv) - x.bv + mean(Yv^2)
}

// G64[c] = Hv X[c] - Bv[t]   (gradient direction g in real form)
// (the residual kernels with lambda = 0:  Rres = Bv - Hv X  -> negate)
__global__ void k_negate(double* __restrict__ v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) v[i] = -v[i];
}

fk_status heldout_mse_impl(fk_ctx* ctx, const SolveLayout& s, int d, int m, const double* Mv, const double* bv,
                           const double* yv2, double* mse) {
  const int N = s.N, Np = s.Np, L = N;   // one real-form block of all N modes
  launch_assemble_pairs(ctx->stream, ToeplitzQ{Mv, m, d}, nullptr, N, Np, s.Hv);
  hipLaunchKernelGGL(k_real_inputs, dim3((Np + 255) / 256, s.ntgt + 1), dim3(256), 0, ctx->stream, nullptr, bv, N, L, Np,
                     nullptr, s.Bv);
  const int nc = s.nlam * s.ntgt;
  // zero "lambda" for the validation product: reuse norms scratch as a zero lambda array
  FK_HIP(hipMemsetAsync(s.norms, 0, sizeof(double) * (2 * nc + s.nlam + 64), ctx->stream));
  // R = Bv - Hv X   (lambda = 0 via a zero lambda array of length nlam in norms[2nc..])
  launch_resid(ctx->stream, s.Hv, N, Np, s.X64, nc, s.ntgt, 0, s.Bv, s.preal, s.norms + 2 * nc, s.G64,
               nullptr, nullptr);
  const int64_t tot = (int64_t)nc * Np;
  hipLaunchKernelGGL(k_negate, dim3((tot + 255) / 256), dim3(256), 0, ctx->stream, s.G64, tot);
  // xGx = x.(Hv x) = x.(g + bv) ; bx = bv.x
  hipLaunchKernelGGL(k_coldot, dim3(nc), dim3(256), 0, ctx->stream, s.X64, s.G64, Np, 1, s.ntgt, s.norms);
  hipLaunchKernelGGL(k_coldot, dim3(nc), dim3(256), 0, ctx->stream, s.X64, s.Bv, Np, 0, s.ntgt, s.norms + nc);
  // mse = x.g + x.bv - 2 x.bv + yv2 = x.g - x.bv + yv2
  hipLaunchKernelGGL(k_mse_combine, dim3((nc + 255) / 256), dim3(256), 0, ctx->stream, s.norms, s.norms + nc, yv2,
                     nc, s.ntgt, mse);
  FK_HIP(hipGetLastError());
  (void)L;
  return FK_OK;
}

// Adjoint right-hand sides in real form: Gadj[c] = gm[c] G64[c] + (1/2) d(Loss)/dc of the incoming
// Wirtinger gradient gin[c] = dLoss/dconj(theta_c) (complex, N modes).  With theta = U c (real c),
// dLoss/dc_r = 2 Re(gin^* dtheta/dc_r), so the real-form entry is Re gin_0 (constant),
// (Re gin_k + Re gin_-k)/sqrt2 (cosine of k) and (Im gin_-k - Im gin_k)/sqrt2 (sine of k): the
// projection onto Hermitian-symmetric theta, where every fitted theta lies.
__global__ void k_adjoint_rhs(const double* __restrict__ G64, const double* __restrict__ gm,
                              const double* __restrict__ gin, int N, int L, int Np, double* __restrict__ Gadj) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  const int c = blockIdx.y;
  if (r >= Np) return;
  double v = gm[c] * G64[(size_t)c * Np + r];
  if (gin && r < N) {
    int ty, k, nk;
    real_to_complex(r, L, &ty, &k, &nk);
    const double* g = gin + 2 * (size_t)c * N;
    const double rs2 = 0.70710678118654752440;
    v += ty == 0 ? g[2 * k] : (ty == 1 ? rs2 * (g[2 * k] + g[2 * nk]) : rs2 * (g[2 * nk + 1] - g[2 * k + 1]));
  }
  Gadj[(size_t)c * Np + r] = v;
}

// grad_loglam[l] = sum_t (-2 lambda_l) u.(preal o x), u the adjoint solution of the combined
// right-hand side;  grad_p (complex modes) likewise.
// One workgroup of 1024 threads per lambda (the sum runs over ntgt x Np terms).
__global__ __launch_bounds__(1024) void k_grad_loglam(const double* __restrict__ U, const double* __restrict__ X,
                                                      const double* __restrict__ preal, const double* __restrict__ lams,
                                                      int Np, int ntgt, double* __restrict__ out) {
  __shared__ double part[1024];
  const int l = blockIdx.x;
  double s = 0.0;
  for (int t = 0; t < ntgt; ++t) {
    const double* u = U + ((size_t)l * ntgt + t) * Np;
    const double* x = X + ((size_t)l * ntgt + t) * Np;
    double a = 0.0;
    for (int i = threadIdx.x; i < Np; i += blockDim.x) a += u[i] * preal[i] * x[i];
    s += a;
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[l] = -2.0 * lams[l] * part[0];
}

// grad_p over the (lambda, target) systems: blockIdx.y takes one slice of them, its four waves
// a quarter of the slice each, lane = real-form row; the slices' sums are added into gp, which
// k_zero_d cleared.
constexpr int kGradPSlices = 16;
__global__ void k_zero_d(double* __restrict__ x, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.0;
}

__global__ __launch_bounds__(256) void k_grad_p(const double* __restrict__ U, const double* __restrict__ X,
                                                const double* __restrict__ lams, int N, int L, int Np, int nlam,
                                                int ntgt, double* __restrict__ gp) {
  __shared__ double part[4][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = blockIdx.x * 64 + lane;
  const int nc = nlam * ntgt;
  const int c0 = (int)((int64_t)nc * blockIdx.y / gridDim.y), c1 = (int)((int64_t)nc * (blockIdx.y + 1) / gridDim.y);
  int ty = 2, k = 0, nk = 0;
  if (r < N) real_to_complex(r, L, &ty, &k, &nk);
  double s = 0.0;
  if (ty != 2)
    for (int c = c0 + wv; c < c1; c += 4) {
      const int l = c / ntgt;
      const size_t o = (size_t)c * Np;
      const double v = ty == 0 ? U[o + r] * X[o + r] : 0.5 * (U[o + r] * X[o + r] + U[o + r + 1] * X[o + r + 1]);
      s += (-2.0 * lams[l]) * v;
    }
  part[wv][lane] = s;
  __syncthreads();
  if (wv == 0 && ty != 2) {
    const double t = part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane];
    atomicAdd(&gp[k], t);
    if (ty == 1) atomicAdd(&gp[nk], t);
  }
}

__global__ void k_scale_cols_cplx(double* __restrict__ th, const double* __restrict__ gm, int N) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  int c = blockIdx.y;
  if (i >= 2 * N) return;
  th[(size_t)c * 2 * N + i] *= gm[c];
}

fk_status backward_impl(fk_ctx* ctx, const SolveLayout& s, int d, const double* gm, const double* gin,
                        double* grad_loglam, double* grad_p, double* grad_theta) {
  const int N = s.N, Np = s.Np, L = N;   // one real-form block of all N modes
  const int nc = s.nlam * s.ntgt;
  int iters = 0, bad = -1;
  double resid = 0.0;
  // u = A^-1 (gm g + gin) for every (lambda, target)
  hipLaunchKernelGGL(k_adjoint_rhs, dim3((Np + 255) / 256, nc), dim3(256), 0, ctx->stream, s.G64, gm, gin, N, L, Np,
                     s.Gadj);
  fk_status st = refine_solve(ctx, s, dense_shape(ctx, s), s.Gadj, s.U64, &iters, &resid, &bad, false,
                              []() -> fk_status { return FK_OK; });
  if (st != FK_OK && st != FK_ENOCONV) return st;
  hipLaunchKernelGGL(k_grad_loglam, dim3(s.nlam), dim3(1024), 0, ctx->stream, s.U64, s.X64, s.preal, s.lams, Np,
                     s.ntgt, grad_loglam);
  if (grad_p) {
    hipLaunchKernelGGL(k_zero_d, dim3((N + 255) / 256), dim3(256), 0, ctx->stream, grad_p, N);
    hipLaunchKernelGGL(k_grad_p, dim3((N + 63) / 64, kGradPSlices), dim3(256), 0, ctx->stream, s.U64, s.X64, s.lams,
                       N, L, Np, s.nlam, s.ntgt, grad_p);
  }
  if (grad_theta) {
    hipLaunchKernelGGL(k_theta_from_real, dim3((N + 255) / 256, nc), dim3(256), 0, ctx->stream, s.G64, N, L, Np,
                       s.ntgt, grad_theta);
    hipLaunchKernelGGL(k_scale_cols_cplx, dim3((2 * N + 255) / 256, nc), dim3(256), 0, ctx->stream, grad_theta, gm,
                       N);
  }
  FK_HIP(hipGetLastError());
  return st;
}

}  // namespace fk
