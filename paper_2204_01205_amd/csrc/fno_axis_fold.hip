// Pruned complex transforms along the middle axis of [outer][N][inner] (the x and y axes of F and of its
// inverse, eq. (3) of arXiv 2204.01205) for axis lengths without a large power of two, as real matrix
// products on the matrix cores.
//
// Folded about the middle of the axis (nu = n + 1/2; rows n and N - 1 - n, frequencies k and -k):
//   forward   X[+-k] = exp(+-i pi k / N) (C[k] -+ i S[k]),  C[k] = sum_n cos(2 pi k nu / N) (x[n] + x[N-1-n]),
//                                                            S[k] = sum_n sin(2 pi k nu / N) (x[n] - x[N-1-n]);
//   inverse   Y[+-k] turned by exp(-+i pi k / N) and added to P[k], subtracted to Q[k]; then
//             x[n] = E + i O,  x[N-1-n] = E - i O,  E = sum_k cos(..) P[k],  O = sum_k sin(..) Q[k].
// The matrices are real, so real and imaginary parts are just columns, as they lie in memory, and the complex
// sum's multiply-adds fall to a quarter.  v_mfma_f32_16x16x4 (full fp32): lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and holds rows 4 (l/16) + v of column l%16.  The data are the right operand, read from memory
// into registers (16 lanes take 64 contiguous bytes of a row); the table (FoldPlan) is the left one, in LDS.
// A wave owns CT tiles of 16 floats and needs no other wave.
//
// Bound by memory (one read and one write of the tensor): y stage of 68 x 118 x 263 x 16 with 32 of 118 frequencies,
// 0.63 GB, inverse 507 -> 148 us = 4.2 TB/s, forward 340 -> 208 us, against the kernels with a two-point FFT and a
// dense sum over the 59 residue classes, which waited for two LDS reads per complex multiply-add.
#include "fno_device.h"

namespace fno {

namespace {

constexpr size_t kAxisFoldLds = 40 * 1024;     // four resident blocks per CU
// Axes that go to these kernels rather than to those with an M-point FFT in registers: all with a small power of two
// in their length, and all short ones.  Two stages there and back, FFT kernels against these: 50 x 45 points 354 ->
// 116 us, 68 x 118 960 -> 437 us, 60 x 60 175 -> 88 us, 64 x 64 (M = 32) 224 -> 190 us; but the products grow with N
// times the kept frequencies: 256 x 256 (M = 32) 1.97 -> 2.51 ms.
constexpr int kAxisFoldMaxM = 8, kAxisFoldMaxN = 64;

__device__ __forceinline__ float swap_pair(float v) {      // the value of lane ^ 1: the other part of a complex number
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}

__device__ __forceinline__ void stage_table(const float* __restrict__ tab, float* smem, int floats) {
  for (int i = threadIdx.x; i < (floats >> 2); i += kThreads)
    reinterpret_cast<float4*>(smem)[i] = reinterpret_cast<const float4*>(tab)[i];
  __syncthreads();
}

// MT: row tiles of 16 frequencies; inner2: floats per row; ntile: tiles of 16 floats per row
template <int MT, int CT, bool STREAM>
__global__ __launch_bounds__(kThreads, MT == 4 ? 3 : 4) void axis_fwd_fold_kernel(
    const float* __restrict__ in, float* __restrict__ out, const float* __restrict__ tab, int N, int L, int npos,
    int inner2, int ntile, int ntiles, int pairs, int stride) {
  HIP_DYNAMIC_SHARED(float, smem)
  constexpr int rows = 16 * MT;
  stage_table(tab, smem, 2 * rows * stride + 2 * rows);
  const float* COS = smem;
  const float* SIN = smem + rows * stride;
  const float2* ROT = reinterpret_cast<const float2*>(smem + 2 * rows * stride);
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const float sg = (c & 1) ? -1.f : 1.f;
  const int steps = (pairs + 15) >> 4;
  for (int t = CT * (blockIdx.x * (kThreads / 64) + wave); t < ntiles; t += CT * (kThreads / 64) * gridDim.x) {
    const float* src[CT];
    float* dst[CT];
    bool ok[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int tt = min(t + ct, ntiles - 1), o = tt / ntile;
      const int col = 16 * (tt - o * ntile) + c;
      ok[ct] = t + ct < ntiles && col < inner2;
      src[ct] = in + (long long)o * N * inner2 + (col < inner2 ? col : (c & 1));
      dst[ct] = out + (long long)o * L * inner2 + col;
    }
    v4f accC[MT][CT], accS[MT][CT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) accC[m][ct] = accS[m][ct] = v4f{0.f, 0.f, 0.f, 0.f};
    float lo[CT][4], hi[CT][4];
    auto load = [&](int s) {                     // row pairs 16 s + 4 g + u; past the last one: pair 0, dropped below
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = 16 * s + 4 * g + u, nc = n < pairs ? n : 0;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          lo[ct][u] = ld_once<STREAM>(src[ct] + nc * inner2);
          hi[ct][u] = ld_once<STREAM>(src[ct] + (N - 1 - nc) * inner2);
        }
      }
    };
    load(0);
    for (int s = 0; s < steps; ++s) {
      float E[CT][4], O[CT][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool live = 16 * s + 4 * g + u < pairs;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          E[ct][u] = live ? lo[ct][u] + hi[ct][u] : 0.f;
          O[ct][u] = live ? lo[ct][u] - hi[ct][u] : 0.f;
        }
      }
      if (s + 1 < steps) load(s + 1);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const v4f cs = *reinterpret_cast<const v4f*>(COS + (16 * m + c) * stride + 16 * s + 4 * g);
        const v4f sn = *reinterpret_cast<const v4f*>(SIN + (16 * m + c) * stride + 16 * s + 4 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            accC[m][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs[u], E[ct][u], accC[m][ct], 0, 0, 0);
            accS[m][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(sn[u], O[ct][u], accS[m][ct], 0, 0, 0);
          }
      }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = 16 * m + 4 * g + v;
        const float2 r = ROT[k];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const float is = sg * swap_pair(accS[m][ct][v]);       // -i S
          const float a = accC[m][ct][v] + is, b = accC[m][ct][v] - is;
          const float xp = fmaf(a, r.x, -sg * r.y * swap_pair(a));
          const float xm = fmaf(b, r.x, sg * r.y * swap_pair(b));
          if (ok[ct] && k < npos) dst[ct][k * inner2] = xp;
          if (ok[ct] && k >= 1 && k <= L - npos) dst[ct][(L - k) * inner2] = xm;
        }
      }
  }
}

// KS: steps of four frequencies k = 4 s + g
template <int KS, int CT, bool STREAM>
__global__ __launch_bounds__(kThreads, KS > 8 ? 3 : 4) void axis_inv_fold_kernel(
    const float* __restrict__ in, float* __restrict__ out, const float* __restrict__ tab, int N, int L, int npos,
    int inner2, int ntile, int ntiles, int rows, int pairs, int stride) {
  HIP_DYNAMIC_SHARED(float, smem)
  stage_table(tab, smem, 2 * rows * stride + 2 * rows);
  const float* COS = smem;
  const float* SIN = smem + rows * stride;
  const float2* ROT = reinterpret_cast<const float2*>(smem + 2 * rows * stride);
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const float sg = (c & 1) ? -1.f : 1.f;
  for (int t = CT * (blockIdx.x * (kThreads / 64) + wave); t < ntiles; t += CT * (kThreads / 64) * gridDim.x) {
    float* dst[CT];
    bool ok[CT];
    float P[CT][KS], Q[CT][KS];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int tt = min(t + ct, ntiles - 1), o = tt / ntile;
      const int col = 16 * (tt - o * ntile) + c;
      ok[ct] = t + ct < ntiles && col < inner2;
      const float* src = in + (long long)o * L * inner2 + (col < inner2 ? col : (c & 1));
      dst[ct] = out + (long long)o * N * inner2 + col;
#pragma unroll
      for (int s = 0; s < KS; ++s) {             // frequencies that are not kept read row 0, dropped below
        const int k = 4 * s + g;
        P[ct][s] = src[(k < npos ? k : 0) * inner2];
        Q[ct][s] = src[(k >= 1 && k <= L - npos ? L - k : 0) * inner2];
      }
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int k = 4 * s + g;
      const float2 r = ROT[k];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const float yp = k < npos ? P[ct][s] : 0.f;
        const float ym = k >= 1 && k <= L - npos ? Q[ct][s] : 0.f;
        const float a = fmaf(yp, r.x, sg * r.y * swap_pair(yp));
        const float b = fmaf(ym, r.x, -sg * r.y * swap_pair(ym));
        P[ct][s] = a + b;
        Q[ct][s] = a - b;
      }
    }
    for (int n0 = 0; n0 < pairs; n0 += 16) {
      v4f E[CT], O[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) E[ct] = O[ct] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const float cs = COS[(4 * s + g) * stride + n0 + c], sn = SIN[(4 * s + g) * stride + n0 + c];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          E[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs, P[ct][s], E[ct], 0, 0, 0);
          O[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(sn, Q[ct][s], O[ct], 0, 0, 0);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = n0 + 4 * g + v;
        const bool middle = 2 * n + 1 == N;      // its cosines stand in the table at half their value
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const float io = sg * swap_pair(O[ct][v]);             // -i O
          const float e = middle ? 2.f * E[ct][v] : E[ct][v];
          if (ok[ct] && n < pairs) {
            st_once<STREAM>(dst[ct] + n * inner2, e - io);
            if (!middle) st_once<STREAM>(dst[ct] + (N - 1 - n) * inner2, e + io);
          }
        }
      }
    }
  }
}

struct Tiles { int ntile, ntiles, ct, blocks; };

// Two tiles per wave share each table entry read from LDS; one where that would leave CUs without work
Tiles axis_tiles(int64_t outer, int64_t inner) {
  Tiles t;
  t.ntile = (int)((2 * inner + 15) / 16);
  t.ntiles = (int)(outer * t.ntile);
  t.ct = t.ntiles >= 2 * 4 * 1024 ? 2 : 1;
  const int waves = (t.ntiles + t.ct - 1) / t.ct;
  t.blocks = (waves + kThreads / 64 - 1) / (kThreads / 64);
  if (t.blocks > 2048) t.blocks = 2048;
  return t;
}

int folded_count(AxisPlan ax) { return (ax.npos - 1 > ax.L - ax.npos ? ax.npos - 1 : ax.L - ax.npos) + 1; }

}  // namespace

bool axis_fold_fits(AxisPlan ax, int64_t outer, int64_t inner) {
  if ((ax.M > kAxisFoldMaxM && ax.N > kAxisFoldMaxN) || folded_count(ax) > 48) return false;
  if (inner <= 0 || 2 * inner * ax.N >= (1ll << 30) || outer * ((2 * inner + 15) / 16) >= (1ll << 30)) return false;
  return fold_plan(ax).floats * 4 <= kAxisFoldLds;
}

hipError_t launch_axis_fwd_fold(const float2* in, float2* out, const float* tab, int64_t outer, AxisPlan ax,
                                int64_t inner, hipStream_t s) {
  const FoldPlan f = fold_plan(ax);
  const Tiles t = axis_tiles(outer, inner);
  const size_t lds = f.floats * 4;
  const bool stream = outer * ax.N * inner * 8 >= kStreamBytes;
#define FNO_AXF(MTV, CTV, STV)                                                                                    \
  hipLaunchKernelGGL((axis_fwd_fold_kernel<MTV, CTV, STV>), dim3((unsigned)t.blocks), dim3(kThreads), lds, s,     \
                     reinterpret_cast<const float*>(in), reinterpret_cast<float*>(out), tab, ax.N, ax.L, ax.npos, \
                     (int)(2 * inner), t.ntile, t.ntiles, f.pairs, f.stride)
#define FNO_AXF_C(MTV)                                                                                            \
  do { if (t.ct == 1) FNO_AXF(MTV, 1, false); else if (stream) FNO_AXF(MTV, 2, true); else FNO_AXF(MTV, 2, false); } while (0)
  switch (f.rows) {
    case 16: FNO_AXF_C(1); break;
    case 32: FNO_AXF_C(2); break;
    case 64: FNO_AXF_C(4); break;
    default: return hipErrorInvalidValue;
  }
#undef FNO_AXF_C
#undef FNO_AXF
  return hipGetLastError();
}

hipError_t launch_axis_inv_fold(const float2* in, float2* out, const float* tab, int64_t outer, AxisPlan ax,
                                int64_t inner, hipStream_t s) {
  const FoldPlan f = fold_plan(ax);
  const Tiles t = axis_tiles(outer, inner);
  const size_t lds = f.floats * 4;
  const bool stream = outer * ax.N * inner * 8 >= kStreamBytes;
  const int ks = (folded_count(ax) + 3) / 4;
#define FNO_AXI(KSV, CTV, STV)                                                                                    \
  hipLaunchKernelGGL((axis_inv_fold_kernel<KSV, CTV, STV>), dim3((unsigned)t.blocks), dim3(kThreads), lds, s,     \
                     reinterpret_cast<const float*>(in), reinterpret_cast<float*>(out), tab, ax.N, ax.L, ax.npos, \
                     (int)(2 * inner), t.ntile, t.ntiles, f.rows, f.pairs, f.stride)
#define FNO_AXI_C(KSV)                                                                                            \
  do { if (t.ct == 1) FNO_AXI(KSV, 1, false); else if (stream) FNO_AXI(KSV, 2, true); else FNO_AXI(KSV, 2, false); } while (0)
  switch (ks) {
    case 1: FNO_AXI_C(1); break;
    case 2: FNO_AXI_C(2); break;
    case 3: FNO_AXI_C(3); break;
    case 4: FNO_AXI_C(4); break;
    case 5: FNO_AXI_C(5); break;
    case 6: FNO_AXI_C(6); break;
    case 7: FNO_AXI_C(7); break;
    case 8: FNO_AXI_C(8); break;
    case 9: case 10: FNO_AXI_C(10); break;
    default: FNO_AXI_C(12); break;
  }
#undef FNO_AXI_C
#undef FNO_AXI
  return hipGetLastError();
}

}  // namespace fno
