// 3-D binned spread of the type-1 stage (the records of sort3, in the order of their bins).
//
// Bins are 8^3 window-start cells (nbx = nf / 8 per axis): the whole window of a bin's point lies in the
// bin's subgrid of S = 8 + w - 1 cells per axis, kept in LDS in FP64 and added into the FP64 grid at the
// end.  Every product w_c psi1 psi2 psi3 is rounded to FP32 and summed in FP64.
//
// Widths up to 8 (k_spread3_reg): w^3 FP64 LDS additions per point and channel are what bounded the spread
// (4.67 ms for 1e7 points and two channels, w = 7, 2.4 additions per clock and CU).  Points whose windows
// start in the same E x E cells of the (x, y) plane share an 8 x 8 patch of it (E + w - 1 <= 8), one
// patch cell per lane: the lane sums its column over z in registers, and only the patch's columns are
// added into LDS, once per E x E group of a batch of points instead of once per point.  Batches are
// ordered by group and z start, so that the loop over a z start knows its registers.  Bound by the
// conversions and FP64 additions of the products (three vector instructions each) and by the latency of a
// point's table reads: 2.17 ms (the additions into the grid 0.2 of it); 1e6 points and five channels 9.9
// -> 3.5 ms.  Sums on the FP32 matrix cores are not used: they would round what is summed in FP64 here.
// Larger widths (k_spread3_atomic): one LDS addition per cell and point.
#include "fk_internal.h"

#include <algorithm>

namespace fk {

namespace {

constexpr int B3 = 8;       // bin edge in cells
constexpr int NP3 = 256;    // points per batch at most
constexpr int NT3 = 512;    // threads of the register kernel

// psi(s) = exp(beta (sqrt(1 - (2s/w)^2) - 1)) with beta pre-multiplied by log2(e): exponent in
// [-beta log2 e, 0], so the hardware exp2 and square root need no range handling.
struct Es3 {
  float beta_log2e, two_over_w;
};
__device__ __forceinline__ float psi3(float s, Es3 es) {
  const float z = s * es.two_over_w;
  const float r = fmaxf(fmaf(-z, z, 1.0f), 0.0f);
  return __builtin_amdgcn_exp2f(fmaf(es.beta_log2e, __builtin_amdgcn_sqrtf(r), -es.beta_log2e));
}

// i0 = ceil(u - w/2) and s0 = i0 - u for the fixed-point coordinate U = u 2^fb.
__device__ __forceinline__ void window3(uint32_t U, int fb, int w, int* i0, float* s0) {
  const int64_t V = (int64_t)U - ((int64_t)w << (fb - 1)), one = (int64_t)1 << fb;
  const int64_t c = (V >= 0) ? ((V + one - 1) >> fb) : -((-V) >> fb);
  *i0 = (int)c;
  *s0 = (float)((double)((c << fb) - (int64_t)U) * (1.0 / (double)one));
}

// The slice of a bin that a workgroup takes: blockIdx.x = (bin * slices + slice) * groups + channel group.
struct Slice3 {
  int bin, c0, o[3];
  uint64_t q0, q1;
};
__device__ __forceinline__ Slice3 slice3(const uint64_t* __restrict__ start, int nbx, int slices, int groups, int nc) {
  Slice3 r;
  int b = blockIdx.x;
  r.c0 = (b % groups) * nc;
  b /= groups;
  const int sl = b % slices;
  r.bin = b / slices;
  const uint64_t p0 = start[r.bin], len = start[r.bin + 1] - p0;
  r.q0 = p0 + len * sl / slices;
  r.q1 = p0 + len * (sl + 1) / slices;
  r.o[2] = r.bin % nbx * B3;
  r.o[1] = r.bin / nbx % nbx * B3;
  r.o[0] = r.bin / (nbx * nbx) * B3;
  return r;
}

// The LDS subgrid [c][x][y][z] (z rows of ZP doubles) into the grid: 16 (or 32) lanes per row of S cells.
template <int S, int ZP, int NT>
__device__ __forceinline__ void flush3(const double* sub, int nc, int c0, int C, const int* o, int nf,
                                       double* __restrict__ grid) {
  constexpr int LZ = S <= 16 ? 4 : 5;
  const int z = threadIdx.x & ((1 << LZ) - 1);
  if (z >= S) return;
  int gz = o[2] + z;
  gz -= gz >= nf ? nf : 0;
  for (int row = threadIdx.x >> LZ; row < nc * S * S; row += NT >> LZ) {
    const double v = sub[row * ZP + z];
    const int y = row % S, u = row / S, x = u % S, c = u / S;
    if (v == 0.0 || c0 + c >= C) continue;
    int gx = o[0] + x, gy = o[1] + y;
    gx -= gx >= nf ? nf : 0;
    gy -= gy >= nf ? nf : 0;
    atomicAdd(&grid[(((int64_t)(c0 + c) * nf + gx) * nf + gy) * nf + gz], v);
  }
}

template <int W, int NC>
__global__ __launch_bounds__(NT3) void k_spread3_reg(const uint32_t* __restrict__ rec, int nw,
                                                     const uint64_t* __restrict__ start, int nbx, int nf, int fb,
                                                     Es3 es, int slices, int groups, double* __restrict__ grid) {
  constexpr int E = W <= 7 ? 2 : 1, PE = E + W - 1;     // patch edge
  constexpr int S = B3 + W - 1, ZP = S | 1;             // odd rows: a patch's lanes spread over the banks
  constexpr int G1 = B3 / E, NG = G1 * G1, NK = NG * B3;   // groups per axis and in all; keys (group, z start)
  constexpr int ROW = 24 + 4;                           // psi1[8], psi2[8], psi3[8], weights
  static_assert(PE <= 8 && W <= 8 && NC <= 4, "one patch cell per lane");
  extern __shared__ __align__(16) unsigned char smem3[];
  double* sub = reinterpret_cast<double*>(smem3);               // NC S S ZP
  float* tab = reinterpret_cast<float*>(sub + NC * S * S * ZP);  // NP3 rows
  uint32_t* ofs = reinterpret_cast<uint32_t*>(tab + NP3 * ROW);  // NK + 1 key starts
  uint32_t* hist = ofs + NK + 4;                                 // NK counts
  const int C = nw + 1, R = 3 + nw, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const Slice3 s = slice3(start, nbx, slices, groups, NC);
  if (s.q0 == s.q1) return;
  for (int i = tid; i < NC * S * S * ZP; i += NT3) sub[i] = 0.0;
  const int px = lane >> 3, py = lane & 7;
  // batches of equal size: a bin of 305 points takes two of 153, not 256 and 49
  const uint32_t len = (uint32_t)(s.q1 - s.q0), nbat = (len + NP3 - 1) / NP3;
  for (uint32_t bt = 0; bt < nbat; ++bt) {
    const uint32_t b0 = (uint32_t)((uint64_t)len * bt / nbat), b1 = (uint32_t)((uint64_t)len * (bt + 1) / nbat);
    for (int i = tid; i < NK; i += NT3) hist[i] = 0;
    __syncthreads();   // also: the last batch's table is read
    // one point per thread: kernel values, weights and key
    const bool ok = b0 + tid < b1;
    float k[3][W], wt[NC];
    int rel[3], key = 0;
    uint32_t rank = 0;
    if (ok) {
      const uint32_t* r = rec + (s.q0 + b0 + tid) * R;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        int i0;
        float s0;
        window3(r[a], fb, W, &i0, &s0);
        rel[a] = (i0 & (nf - 1)) - s.o[a];
#pragma unroll
        for (int t = 0; t < W; ++t) k[a][t] = psi3(s0 + (float)t, es);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int ch = s.c0 + c;
        wt[c] = ch == 0 ? 1.0f : (ch < C ? __uint_as_float(r[2 + ch]) : 0.f);
      }
      key = ((rel[0] / E) * G1 + rel[1] / E) * B3 + rel[2];
      rank = atomicAdd(&hist[key], 1u);
    }
    __syncthreads();
    if (tid < 64) {   // exclusive sums of the NK counts
      constexpr int PER = NK / 64;
      uint32_t v[PER], sum = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        v[i] = hist[tid * PER + i];
        sum += v[i];
      }
      uint32_t x = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (tid >= o) x += y;
      }
      uint32_t run = x - sum;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        ofs[tid * PER + i] = run;
        run += v[i];
      }
      if (tid == 63) ofs[NK] = run;
    }
    __syncthreads();
    if (ok) {
      float* row = tab + (ofs[key] + rank) * ROW;
      float4* r4 = reinterpret_cast<float4*>(row);
#pragma unroll
      for (int q = 0; q < 4; ++q) r4[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      const int ex = rel[0] % E, ey = rel[1] % E;
#pragma unroll
      for (int t = 0; t < W; ++t) {
        row[ex + t] = k[0][t];
        row[8 + ey + t] = k[1][t];
        row[16 + t] = k[2][t];
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) row[24 + c] = wt[c];
    }
    __syncthreads();
    for (int g = w; g < NG; g += NT3 / 64) {
      if (ofs[g * B3] == ofs[g * B3 + B3]) continue;
      double acc[NC][S];
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int z = 0; z < S; ++z) acc[c][z] = 0.0;
#pragma unroll
      for (int z0 = 0; z0 < B3; ++z0) {
        const uint32_t p1 = ofs[g * B3 + z0 + 1];
        for (uint32_t p = ofs[g * B3 + z0]; p < p1; ++p) {
          const float* row = tab + p * ROW;
          const float a = row[px], b = row[8 + py];
          float kz[8];
          *reinterpret_cast<float4*>(kz) = *reinterpret_cast<const float4*>(row + 16);
          *reinterpret_cast<float4*>(kz + 4) = *reinterpret_cast<const float4*>(row + 20);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const float v = (row[24 + c] * a) * b;
#pragma unroll
            for (int t = 0; t < W; ++t) acc[c][z0 + t] += (double)(v * kz[t]);
          }
        }
      }
      if (px < PE && py < PE) {
        double* d = sub + (((g / G1) * E + px) * S + (g % G1) * E + py) * ZP;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int z = 0; z < S; ++z) atomicAdd(&d[c * S * S * ZP + z], acc[c][z]);
      }
    }
  }
  __syncthreads();
  flush3<S, ZP, NT3>(sub, NC, s.c0, C, s.o, nf, grid);
}

// One LDS addition per cell and point, one channel per workgroup.
template <int W>
__global__ __launch_bounds__(256) void k_spread3_atomic(const uint32_t* __restrict__ rec, int nw,
                                                        const uint64_t* __restrict__ start, int nbx, int nf, int fb,
                                                        Es3 es, int slices, int groups, double* __restrict__ grid) {
  constexpr int S = B3 + W - 1;
  extern __shared__ __align__(16) unsigned char smem3[];
  double* sub = reinterpret_cast<double*>(smem3);
  const int R = 3 + nw;
  const Slice3 s = slice3(start, nbx, slices, groups, 1);
  if (s.q0 == s.q1) return;
  for (int i = threadIdx.x; i < S * S * S; i += 256) sub[i] = 0.0;
  __syncthreads();
  for (uint64_t q = s.q0 + threadIdx.x; q < s.q1; q += 256) {
    const uint32_t* r = rec + q * R;
    float k[3][W];
    int rel[3];
    for (int a = 0; a < 3; ++a) {
      int i0;
      float s0;
      window3(r[a], fb, W, &i0, &s0);
      rel[a] = (i0 & (nf - 1)) - s.o[a];
#pragma unroll
      for (int t = 0; t < W; ++t) k[a][t] = psi3(s0 + (float)t, es);
    }
    const float wc = s.c0 == 0 ? 1.0f : __uint_as_float(r[2 + s.c0]);
    for (int a1 = 0; a1 < W; ++a1) {
      const float v1 = wc * k[0][a1];
      for (int a2 = 0; a2 < W; ++a2) {
        const float v12 = v1 * k[1][a2];
        double* row = sub + ((rel[0] + a1) * S + (rel[1] + a2)) * S + rel[2];
#pragma unroll
        for (int a3 = 0; a3 < W; ++a3) atomicAdd(&row[a3], (double)(v12 * k[2][a3]));
      }
    }
  }
  __syncthreads();
  flush3<S, S, 256>(sub, 1, s.c0, nw + 1, s.o, nf, grid);
}

template <int W, int NC>
void launch_reg(hipStream_t st, int64_t blocks, const uint32_t* rec, int nw, const uint64_t* start, int nbx, int nf,
                int fb, Es3 es, int slices, int groups, double* grid) {
  constexpr int S = B3 + W - 1, ZP = S | 1, E = W <= 7 ? 2 : 1, NK = (B3 / E) * (B3 / E) * B3;
  const size_t lds = sizeof(double) * NC * S * S * ZP + sizeof(float) * NP3 * 28 + sizeof(uint32_t) * (2 * NK + 4);
  hipLaunchKernelGGL((k_spread3_reg<W, NC>), dim3((unsigned)blocks), dim3(NT3), lds, st, rec, nw, start, nbx, nf, fb,
                     es, slices, groups, grid);
}

template <int W>
fk_status launch_w3(hipStream_t st, const uint32_t* rec, int nw, const uint64_t* start, int nf, int fb, Es3 es,
                    int64_t n, double* grid) {
  const int nbx = nf / B3, C = nw + 1;
  const int64_t nb = (int64_t)nbx * nbx * nbx, per_bin = (n + nb - 1) / nb;
  const int slices = (int)std::max<int64_t>(1, std::min<int64_t>(256, (per_bin + 2047) / 2048));
  // channels of a workgroup: at most four (registers, and LDS for two workgroups per CU or nearly)
  const int groups = W <= 8 ? (C + 3) / 4 : C, nc = (C + groups - 1) / groups;
  const int64_t blocks = nb * slices * groups;
  if (blocks > 0x7fffffff) return FK_EINVAL;
  if constexpr (W <= 8) {
    switch (nc) {
      case 1: launch_reg<W, 1>(st, blocks, rec, nw, start, nbx, nf, fb, es, slices, groups, grid); break;
      case 2: launch_reg<W, 2>(st, blocks, rec, nw, start, nbx, nf, fb, es, slices, groups, grid); break;
      case 3: launch_reg<W, 3>(st, blocks, rec, nw, start, nbx, nf, fb, es, slices, groups, grid); break;
      default: launch_reg<W, 4>(st, blocks, rec, nw, start, nbx, nf, fb, es, slices, groups, grid); break;
    }
  } else {
    constexpr int S = B3 + W - 1;
    hipLaunchKernelGGL(k_spread3_atomic<W>, dim3((unsigned)blocks), dim3(256), sizeof(double) * S * S * S, st, rec, nw,
                       start, nbx, nf, fb, es, slices, groups, grid);
  }
  return hipGetLastError() == hipSuccess ? FK_OK : FK_EHIP;
}

}  // namespace

fk_status launch_spread3(hipStream_t st, int W, const uint32_t* rec, int nw, const uint64_t* start, int nf, int fb,
                         double beta, int64_t n, double* grid) {
  if (nf % B3 || nf < 2 * B3 || nw < 0 || nw > 8) return FK_EINVAL;
  const Es3 es{(float)(beta * 1.44269504088896340736), 2.0f / (float)W};
#define FK_W3(WW) \
  case WW: return launch_w3<WW>(st, rec, nw, start, nf, fb, es, n, grid);
  switch (W) {
    FK_W3(4) FK_W3(5) FK_W3(6) FK_W3(7) FK_W3(8) FK_W3(9) FK_W3(10) FK_W3(11) FK_W3(12) FK_W3(13) FK_W3(14) FK_W3(15)
    FK_W3(16)
  }
#undef FK_W3
  return FK_EINVAL;
}

}  // namespace fk
