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
// sum's multiply-adds fall to a quarter.  v_mfma_f64_16x16x4 (lane l supplies A[l%16][l/16] and B[l/16][l%16] and
// holds rows 4 v + l/16 of column l%16) takes the float data and table and adds in double, and the turn by the phase
// follows in double, so that the only roundings are the table's entries and the result: 3 to 5e-8 of the norm on every
// length.  The same sums in fp32 chains of N / 2 terms were off by 6.4e-8 (12 points) to 1.6e-7 (150), more than the
// FFT kernels they took over from (5.4e-8 to 1.2e-7).  The data are the right operand, read from memory into
// registers (16 lanes take 64 contiguous bytes of a row); the table (FoldPlan) is the left one, in LDS.  A wave owns
// CT tiles of 16 floats and needs no other wave.
//
// Bound by memory (one read and one write of the tensor), with the fp64 products (64 cycles each) close behind: y stage
// of 68 x 118 x 64 x 16 with 32 of 118 frequencies, 20 channels, 0.62 GB, inverse 477 -> 148 us = 4.2 TB/s, forward
// 352 -> 197 us, against the kernels with a two-point FFT and a dense sum over the 59 residue classes, which wait for
// two LDS reads per complex multiply-add (fp32 products in this kernel: 158 and 205 us).
#include "fno_device.h"

namespace fno {

namespace {

constexpr size_t kAxisFoldLds = 40 * 1024;     // four resident blocks per CU
// Axes that go to these kernels rather than to those with an M-point FFT in registers: M <= 4, and 32 points, which the
// FFT kernels hold in one thread.  Both stages there and back on 20 channels, z and t of 64 x 16 with 24 x 8 kept, us,
// FFT kernels against these: 50 x 45 points 361 -> 134 (t of 24), 68 x 118 941 -> 438, 60 x 60 182 -> 117 (t of 30),
// 32 x 32 127 -> 108; but 64 x 64 118 and 126, 48 x 48 113 and 136, 16 x 16 126 and 175, 72 x 88 358 and 386,
// 120 x 104 410 and 410, 64 x 64 with 40 kept 315 and 370.
//
// A short axis leaves most of the 16 pairs of a step and of the 16 frequencies of a tile empty, while a 2- or 4-point FFT
// with few residues and few frequencies is next to nothing.  One axis there and back, 20 x 64 slabs of rows of 192 floats,
// us, FFT kernels and these: 4 points 22 and 34, 6 points 24 and 35, 10 points with 2 and 4 kept 28 and 35, 29 and 35, 12
// points with 4 and 10 kept 27 and 36, 31 and 40, 14 points with 2 kept 30 and 36, 20 and 28 points with 4 kept 32 and
// 37, 37 and 38; 20 points with 8 kept 38 and 40, with 18 49 and 45.  Rows of 96 floats: 12 points with 4 kept 23 and 25,
// 20 points with 4 kept 26 and 26, 28 points 28 and 27; of 12 floats: equal.
bool axis_fold_pays(AxisPlan ax, int64_t inner) {
  const int terms = ax.P * ax.L;
  if (ax.M > 1 && terms <= 32 && inner >= (terms <= 16 ? 48 : 80)) return false;
  return ax.M <= 4 || ax.N == 32;
}

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void stage_table(const float* __restrict__ tab, float* smem, int floats) {
  for (int i = threadIdx.x; i < (floats >> 2); i += kThreads)
    reinterpret_cast<float4*>(smem)[i] = reinterpret_cast<const float4*>(tab)[i];
  __syncthreads();
}

// MT: row tiles of 16 frequencies; inner2: floats per row; ntile: tiles of 16 floats per row.  MT = 4 keeps 16 of its
// registers in scratch
template <int MT, int CT, bool STREAM>
__global__ __launch_bounds__(kThreads, MT == 4 ? 2 : (MT * CT == 2 ? 3 : 4)) void axis_fwd_fold_kernel(
    const float* __restrict__ in, float* __restrict__ out, const float* __restrict__ tab, int N, int L, int npos,
    int inner2, int ntile, int ntiles, int pairs, int stride) {
  HIP_DYNAMIC_SHARED(float, smem)
  constexpr int rows = 16 * MT;
  stage_table(tab, smem, 2 * rows * stride + 4 * rows);
  const float* COS = smem;
  const float* SIN = smem + rows * stride;
  const double2* ROT = reinterpret_cast<const double2*>(smem + 2 * rows * stride);
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const double sg = (c & 1) ? -1.0 : 1.0;
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
    v4d accC[MT][CT], accS[MT][CT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) accC[m][ct] = accS[m][ct] = v4d{0.0, 0.0, 0.0, 0.0};
    float lo[CT][4], hi[CT][4];
    auto load = [&](int s) {                     // row pairs 16 s + 4 g + u; past the last one: pair 0, against zeros in the table
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
      double E[CT][4], O[CT][4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const double a = lo[ct][u], b = hi[ct][u];
          E[ct][u] = a + b;
          O[ct][u] = a - b;
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
            accC[m][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(cs[u], E[ct][u], accC[m][ct], 0, 0, 0);
            accS[m][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(sn[u], O[ct][u], accS[m][ct], 0, 0, 0);
          }
      }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = 16 * m + 4 * v + g;
        const double2 r = ROT[k];
        const double ry = sg * r.y;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const double is = sg * swap_pair(accS[m][ct][v]);      // -i S
          const double a = accC[m][ct][v] + is, b = accC[m][ct][v] - is;
          const double xp = fma(a, r.x, -ry * swap_pair(a));
          const double xm = fma(b, r.x, ry * swap_pair(b));
          if (ok[ct] && k < npos) dst[ct][k * inner2] = (float)xp;
          if (ok[ct] && k >= 1 && k <= L - npos) dst[ct][(L - k) * inner2] = (float)xm;
        }
      }
  }
}

// KS: steps of four frequencies k = 4 s + g
template <int KS, int CT, bool STREAM>
__global__ __launch_bounds__(kThreads, KS >= 10 ? 2 : (KS >= 8 ? 3 : 4)) void axis_inv_fold_kernel(
    const float* __restrict__ in, float* __restrict__ out, const float* __restrict__ tab, int N, int L, int npos,
    int inner2, int ntile, int ntiles, int rows, int pairs, int stride) {
  HIP_DYNAMIC_SHARED(float, smem)
  stage_table(tab, smem, 2 * rows * stride + 4 * rows);
  const float* COS = smem;
  const float* SIN = smem + rows * stride;
  const double2* ROT = reinterpret_cast<const double2*>(smem + 2 * rows * stride);
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const double sg = (c & 1) ? -1.0 : 1.0;
  for (int t = CT * (blockIdx.x * (kThreads / 64) + wave); t < ntiles; t += CT * (kThreads / 64) * gridDim.x) {
    float* dst[CT];
    bool ok[CT];
    float yp[CT][KS], ym[CT][KS];
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
        yp[ct][s] = src[(k < npos ? k : 0) * inner2];
        ym[ct][s] = src[(k >= 1 && k <= L - npos ? L - k : 0) * inner2];
      }
    }
    double P[CT][KS], Q[CT][KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int k = 4 * s + g;
      const double2 r = ROT[k];
      const double ry = sg * r.y;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const double p = k < npos ? yp[ct][s] : 0.f, q = k >= 1 && k <= L - npos ? ym[ct][s] : 0.f;
        const double a = fma(p, r.x, ry * swap_pair(p));
        const double b = fma(q, r.x, -ry * swap_pair(q));
        P[ct][s] = a + b;
        Q[ct][s] = a - b;
      }
    }
    for (int n0 = 0; n0 < pairs; n0 += 16) {
      v4d E[CT], O[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) E[ct] = O[ct] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const float cs = COS[(4 * s + g) * stride + n0 + c], sn = SIN[(4 * s + g) * stride + n0 + c];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          E[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(cs, P[ct][s], E[ct], 0, 0, 0);
          O[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(sn, Q[ct][s], O[ct], 0, 0, 0);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = n0 + 4 * v + g;
        const bool middle = 2 * n + 1 == N;      // its cosines stand in the table at half their value
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const double io = sg * swap_pair(O[ct][v]);            // -i O
          const double e = middle ? 2.0 * E[ct][v] : E[ct][v];
          if (ok[ct] && n < pairs) {
            st_once<STREAM>(dst[ct] + n * inner2, (float)(e - io));
            if (!middle) st_once<STREAM>(dst[ct] + (N - 1 - n) * inner2, (float)(e + io));
          }
        }
      }
    }
  }
}

struct Tiles { int ntile, ntiles, ct, blocks; };

// Up to max_ct tiles per wave share each table entry read from LDS; one where that would leave CUs without work
Tiles axis_tiles(int64_t outer, int64_t inner, int max_ct) {
  Tiles t;
  t.ntile = (int)((2 * inner + 15) / 16);
  t.ntiles = (int)(outer * t.ntile);
  t.ct = t.ntiles >= 2 * 4 * 1024 ? max_ct : 1;
  const int waves = (t.ntiles + t.ct - 1) / t.ct;
  t.blocks = (waves + kThreads / 64 - 1) / (kThreads / 64);
  if (t.blocks > 2048) t.blocks = 2048;
  return t;
}

// Slabs of [N][inner] per launch: the kernels count tiles of 16 floats in 32 bits.  The rule of axis_fold_fits() cannot
// ask for that, since one set of tables in a workspace serves every batch.
int64_t slabs_per_launch(int64_t inner) { return ((1ll << 30) - 1) / ((2 * inner + 15) / 16); }

int folded_count(AxisPlan ax) { return (ax.npos - 1 > ax.L - ax.npos ? ax.npos - 1 : ax.L - ax.npos) + 1; }

}  // namespace

bool axis_fold_fits(AxisPlan ax, int64_t inner) {
  if (!axis_fold_pays(ax, inner) || folded_count(ax) > 48) return false;
  if (inner <= 0 || 2 * inner * ax.N >= (1ll << 30)) return false;
  return fold_plan(ax).floats * 4 <= kAxisFoldLds;
}

hipError_t launch_axis_fwd_fold(const float2* in, float2* out, const float* tab, int64_t outer, AxisPlan ax,
                                int64_t inner, hipStream_t s) {
  const int64_t most = slabs_per_launch(inner);
  if (outer > most) {
    const hipError_t err = launch_axis_fwd_fold(in, out, tab, most, ax, inner, s);
    if (err != hipSuccess) return err;
    return launch_axis_fwd_fold(in + most * ax.N * inner, out + most * ax.L * inner, tab, outer - most, ax, inner, s);
  }
  const FoldPlan f = fold_plan(ax);
  const Tiles t = axis_tiles(outer, inner, f.rows == 16 ? 2 : 1);
  const size_t lds = f.floats * 4;
  const bool stream = outer * ax.N * inner * 8 >= kStreamBytes;
#define FNO_AXF(MTV, CTV, STV)                                                                                    \
  hipLaunchKernelGGL((axis_fwd_fold_kernel<MTV, CTV, STV>), dim3((unsigned)t.blocks), dim3(kThreads), lds, s,     \
                     reinterpret_cast<const float*>(in), reinterpret_cast<float*>(out), tab, ax.N, ax.L, ax.npos, \
                     (int)(2 * inner), t.ntile, t.ntiles, f.pairs, f.stride)
#define FNO_AXF_S(MTV, CTV) do { if (stream) FNO_AXF(MTV, CTV, true); else FNO_AXF(MTV, CTV, false); } while (0)
  switch (f.rows) {
    case 16: if (t.ct == 2) FNO_AXF_S(1, 2); else FNO_AXF_S(1, 1); break;
    case 32: FNO_AXF_S(2, 1); break;
    case 64: FNO_AXF_S(4, 1); break;
    default: return hipErrorInvalidValue;
  }
#undef FNO_AXF_S
#undef FNO_AXF
  return hipGetLastError();
}

hipError_t launch_axis_inv_fold(const float2* in, float2* out, const float* tab, int64_t outer, AxisPlan ax,
                                int64_t inner, hipStream_t s) {
  const int64_t most = slabs_per_launch(inner);
  if (outer > most) {
    const hipError_t err = launch_axis_inv_fold(in, out, tab, most, ax, inner, s);
    if (err != hipSuccess) return err;
    return launch_axis_inv_fold(in + most * ax.L * inner, out + most * ax.N * inner, tab, outer - most, ax, inner, s);
  }
  const FoldPlan f = fold_plan(ax);
  const int ks = (folded_count(ax) + 3) / 4;
  const Tiles t = axis_tiles(outer, inner, ks <= 4 ? 2 : 1);
  const size_t lds = f.floats * 4;
  const bool stream = outer * ax.N * inner * 8 >= kStreamBytes;
#define FNO_AXI(KSV, CTV, STV)                                                                                    \
  hipLaunchKernelGGL((axis_inv_fold_kernel<KSV, CTV, STV>), dim3((unsigned)t.blocks), dim3(kThreads), lds, s,     \
                     reinterpret_cast<const float*>(in), reinterpret_cast<float*>(out), tab, ax.N, ax.L, ax.npos, \
                     (int)(2 * inner), t.ntile, t.ntiles, f.rows, f.pairs, f.stride)
#define FNO_AXI_S(KSV, CTV) do { if (stream) FNO_AXI(KSV, CTV, true); else FNO_AXI(KSV, CTV, false); } while (0)
#define FNO_AXI_C(KSV) do { if (t.ct == 2) FNO_AXI_S(KSV, 2); else FNO_AXI_S(KSV, 1); } while (0)
  switch (ks) {
    case 1: FNO_AXI_C(1); break;
    case 2: FNO_AXI_C(2); break;
    case 3: FNO_AXI_C(3); break;
    case 4: FNO_AXI_C(4); break;
    case 5: FNO_AXI_S(5, 1); break;
    case 6: FNO_AXI_S(6, 1); break;
    case 7: FNO_AXI_S(7, 1); break;
    case 8: FNO_AXI_S(8, 1); break;
    case 9: case 10: FNO_AXI_S(10, 1); break;
    default: FNO_AXI_S(12, 1); break;
  }
#undef FNO_AXI_C
#undef FNO_AXI_S
#undef FNO_AXI
  return hipGetLastError();
}

}  // namespace fno
