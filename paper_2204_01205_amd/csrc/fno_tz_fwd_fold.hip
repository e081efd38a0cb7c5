// Forward (t, z) stage of the transform chain (F of eq. (3) of arXiv 2204.01205 along the last two
// axes) for any axis lengths, as two chained real matrix products on the matrix cores.
//
// A plane of Nz x Nt reals goes to its kept bins in two contractions.  Over t: T[n][c] =
// sum_t x[n][t] cs[t][c], c running over the cos and -sin columns of the kept bins.  Over z, folded
// about the middle of the axis: with nu = n + 1/2 and the row pairs E[n] = T[n] + T[Nz-1-n],
// O[n] = T[n] - T[Nz-1-n],
//   X[+-k] = exp(+-i pi k / Nz) (C[k] -+ i S[k]),   C[k] = sum_n cos(2 pi k nu / Nz) E[n],
//                                                    S[k] = sum_n sin(2 pi k nu / Nz) O[n],
// n over the ceil(Nz / 2) pairs: both matrices are real, every pair of rows and every pair of
// frequencies shares its products (a quarter of the multiply-adds of the plain complex sum), and no
// row is special (an odd Nz pairs its middle row with itself, at half the weight).
//
// Both run on v_mfma_f32_16x16x4 (full fp32; lane l supplies A[l%16][l/16] and B[l/16][l%16] and holds
// rows 4 (l/16) + v of column l%16).  One wave owns a plane: it folds 16 row pairs as they arrive from
// memory (four lanes read 64 contiguous bytes of a row), turns them over t, and the accumulator
// registers of that product are, as they stand, the right operand of the product over z (register v of
// lane group g is row 4 g + v of the contraction, so the table operand is read in that order).  No
// tile of the plane passes through LDS, no wave waits for another; LDS holds only the z table, which
// a block's waves share over all planes they walk.
//
// The sums stay in fp32 but in short chains: two over t, blocks of eight pairs over z that are added up as they come,
// and the turn by the phase is in double.  One chain of Nz / 2 terms was off by up to 1.7 times what the FFT over z
// that these kernels replaced is off by (128 x 20: 1.18e-7 with the FFT, 1.75e-7 in one chain, 1.07e-7 now).
//
// What bounds it: the matrix cores at 32 cycles per instruction (a 263 x 16 plane with 49 frequencies and
// 8 bins: 9 tiles of 8 + 16 instructions) next to one read of the field.  Measured against the kernels it
// replaced (mixed-radix and dense complex sums on tiles staged in LDS), us on 1536 columns: 64 x 20, 20 channels, 93 -> 53;
// 128 x 24 202 -> 179; 80 x 40 375 -> 145; 263 x 16, 6 channels, 293 -> 102; two entries of 8 x 40 113 -> 44.
#include "fno_device.h"

namespace fno {

namespace {

// registers of a variant (two row tiles in flight and folded, the t table, the accumulators, the z
// table's operands and the addresses), and the waves per SIMD they allow; one variant, <1, 3, 2, 1, 1>, needs five more
// than its 128 and keeps them in scratch
constexpr int fold_regs(int KS, int CT, int MT, int PP) {
  return KS * (4 + CT) + 8 * MT * CT * PP + (CT == 2 ? 16 : 6) * MT + 48;
}
constexpr int fold_waves(int KS, int CT, int MT, int PP) {
  const int regs = fold_regs(KS, CT, MT, PP);
  return regs <= 64 ? 8 : (regs <= 72 ? 6 : (regs <= 96 ? 5 : (regs <= 128 ? 4 : (regs <= 168 ? 3 : 2))));
}

// A row of Nt = 16 J + r floats (1 <= r <= 16): J runs of 16 (four per lane group) and a tail in which
// lane group g takes W = ceil(r / 4) floats from min(W g, r - W), so that no lane reads past its row;
// entries a lower group has already taken meet zeros in the t table.
// PP planes of at most 16 / PP row pairs share a tile: row 4 g + v of it is pair (4 / PP) g + v % (4 / PP) of
// plane v / (4 / PP), so that each register of the first product belongs to one plane.
template <int J, int W, int CT, int MT, int PP, bool STREAM>
__global__ __launch_bounds__(kThreads, fold_waves(4 * J + W, CT, MT, PP)) void tz_fwd_fold_kernel(
    const float* __restrict__ x, float* __restrict__ out, const float2* __restrict__ twt,
    const float* __restrict__ ztab, long long planes, int Nz, int Nt, int Lz, int npos, int mt, int mrows,
    int pairs, int stride, int ngroups, int mgroups) {
  HIP_DYNAMIC_SHARED(float, smem)
  constexpr int KS = 4 * J + W;                 // K steps of the product over t
  float* COS = smem;                            // [16 MT][stride]
  float* SIN = smem + 16 * MT * stride;         // [16 MT][stride]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // uniform: plane addresses stay scalar
  const int c = lane & 15, g = lane >> 4;
  // blocks that share planes but not frequencies or columns sit on one XCD next to each other
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const int grp = local % ngroups;
  const int m0 = 16 * MT * (grp % mgroups), c0 = 16 * CT * (grp / mgroups);
  {
    const float4* cs = reinterpret_cast<const float4*>(ztab + (long long)m0 * stride);
    const float4* sn = reinterpret_cast<const float4*>(ztab + (long long)(mrows + m0) * stride);
    const int n4 = (16 * MT * stride) >> 2;
    for (int i = tid; i < n4; i += kThreads) {
      reinterpret_cast<float4*>(COS)[i] = cs[i];
      reinterpret_cast<float4*>(SIN)[i] = sn[i];
    }
  }
  double2* ROT = reinterpret_cast<double2*>(SIN + 16 * MT * stride);    // [16 MT]
  if (tid < 16 * MT) ROT[tid] = reinterpret_cast<const double2*>(ztab + (long long)2 * mrows * stride)[m0 + tid];
  const int r = Nt - 16 * J;
  const int t0 = min(W * g, r - W);             // start of this lane group's tail
  float tb[CT][KS];                             // t table, the right operand of every K step
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int col = c0 + 16 * ct + c, kt = col >> 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int t = s < 4 * J ? 16 * (s >> 2) + 4 * g + (s & 3) : 16 * J + t0 + (s - 4 * J);
      const bool dup = s >= 4 * J && t < 16 * J + W * g;
      float v = 0.f;
      if (kt < mt && !dup) {
        const float2 w = twt[kt * Nt + t];
        v = (col & 1) ? w.y : w.x;
      }
      tb[ct][s] = v;
    }
  }
  const double sgn = (c & 1) ? -1.0 : 1.0;
  __syncthreads();

  // each XCD walks a contiguous eighth of the planes, its waves interleaved inside it
  const long long per_x = (planes + 7) >> 3;
  const long long pe = min(planes, (long long)(xcd + 1) * per_x);
  const long long nwl = (long long)((gridDim.x >> 3) / ngroups) * (kThreads / 64) * PP;
  long long p = (long long)xcd * per_x + ((long long)(local / ngroups) * (kThreads / 64) + wave) * PP;
  if (p >= pe) return;
  const int ntile = PP > 1 ? 1 : (pairs + 15) >> 4;
  constexpr int VP = 4 / PP;                    // registers of a lane that belong to one plane
  const int lp = (c & 3) / VP, ln = VP * (c >> 2) + (c & (VP - 1));      // plane and pair of tile row c (PP > 1)

  float va[KS], vb[KS];                         // this lane's part of row n and of row Nz - 1 - n
  auto load_tile = [&](long long plane, int tile) {
    const int n = min(PP > 1 ? ln : 16 * tile + c, pairs - 1);
    const int first = PP > 1 ? min(lp, (int)min((long long)PP, planes - plane) - 1) * Nz : 0;      // row of the lane's plane
    const float* base = x + plane * (Nz * Nt);
    const float* ra = base + (first + n) * Nt;
    const float* rb = base + (first + Nz - 1 - n) * Nt;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      float qa[4], qb[4];
      load_run<4, STREAM>(ra + 16 * j + 4 * g, qa);
      load_run<4, STREAM>(rb + 16 * j + 4 * g, qb);
#pragma unroll
      for (int u = 0; u < 4; ++u) { va[4 * j + u] = qa[u]; vb[4 * j + u] = qb[u]; }
    }
    float qa[W], qb[W];
    load_run<W, STREAM>(ra + 16 * J + t0, qa);
    load_run<W, STREAM>(rb + 16 * J + t0, qb);
#pragma unroll
    for (int u = 0; u < W; ++u) { va[4 * J + u] = qa[u]; vb[4 * J + u] = qb[u]; }
  };
  load_tile(p, 0);
  for (; p < pe; p += nwl) {
    v4f accC[PP][MT][CT], accS[PP][MT][CT];
#pragma unroll
    for (int q = 0; q < PP; ++q)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          accC[q][m][ct] = v4f{0.f, 0.f, 0.f, 0.f};
          accS[q][m][ct] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    for (int tile = 0; tile < ntile; ++tile) {
      float e[KS], o[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) { e[s] = va[s] + vb[s]; o[s] = va[s] - vb[s]; }
      if (tile + 1 < ntile) load_tile(p, tile + 1);
      else if (p + nwl < pe) load_tile(p + nwl, 0);
      float ca[MT][VP], sa[MT][VP];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        typedef typename run_of<VP>::type vec;
        const int at = (16 * m + c) * stride + 16 * tile + VP * g;
        const vec cq = *reinterpret_cast<const vec*>(COS + at), sq = *reinterpret_cast<const vec*>(SIN + at);
#pragma unroll
        for (int v = 0; v < VP; ++v) {
          if constexpr (VP == 1) { ca[m][v] = cq; sa[m][v] = sq; }
          else { ca[m][v] = cq[v]; sa[m][v] = sq[v]; }
        }
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const v4f zero = {0.f, 0.f, 0.f, 0.f};
        v4f dE = zero, dO = zero, dE1 = zero, dO1 = zero;        // two chains each: even and odd steps
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          v4f& E = s & 1 ? dE1 : dE;
          v4f& O = s & 1 ? dO1 : dO;
          E = __builtin_amdgcn_mfma_f32_16x16x4f32(e[s], tb[ct][s], E, 0, 0, 0);
          O = __builtin_amdgcn_mfma_f32_16x16x4f32(o[s], tb[ct][s], O, 0, 0, 0);
        }
        if constexpr (KS > 1) { dE += dE1; dO += dO1; }
        if constexpr (PP > 1) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            v4f& C = accC[v / VP][0][ct];
            v4f& S = accS[v / VP][0][ct];
            C = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[0][v % VP], dE[v], C, 0, 0, 0);
            S = __builtin_amdgcn_mfma_f32_16x16x4f32(sa[0][v % VP], dO[v], S, 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            v4f pc[2], ps[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              pc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[m][2 * h], dE[2 * h], zero, 0, 0, 0);
              ps[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(sa[m][2 * h], dO[2 * h], zero, 0, 0, 0);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              pc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[m][2 * h + 1], dE[2 * h + 1], pc[h], 0, 0, 0);
              ps[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(sa[m][2 * h + 1], dO[2 * h + 1], ps[h], 0, 0, 0);
            }
            accC[0][m][ct] += pc[0] + pc[1];
            accS[0][m][ct] += ps[0] + ps[1];
          }
        }
      }
    }
    // X[+-k] from C, S: real and imaginary parts sit in neighbouring lanes
    // the phases and the store offsets are worked out again for every plane, not kept in registers
    int g4 = 4 * g;
    asm volatile("" : "+v"(g4)::"memory");
#pragma unroll
    for (int q = 0; q < PP; ++q) {
      if (PP > 1 && p + q >= pe) break;
      float* dst = out + (p + q) * (Lz * mt * 2);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int kl = 16 * m + g4 + v, k = m0 + kl;
          const double2 w = ROT[kl];
          const double ws = sgn * w.y;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const int col = c0 + 16 * ct + c;
            const float fc = accC[q][m][ct][v], fs = accS[q][m][ct][v];
            const double C = fc, is = sgn * swap_pair(fs);       // this part of C and -i S, and the other part
            const double D = swap_pair(fc), it = sgn * fs;
            const double yp = fma(C + is, w.x, -ws * (D - it));
            const double ym = fma(C - is, w.x, ws * (D + it));
            if (col < 2 * mt) {
              if (k < npos) dst[k * mt * 2 + col] = (float)yp;
              if (k >= 1 && k <= Lz - npos) dst[(Lz - k) * mt * 2 + col] = (float)ym;
            }
          }
        }
    }
  }
}

constexpr size_t kFoldLds = 78 * 1024;      // two blocks per CU

size_t fold_lds(const FoldPlan& f, int MT) { return (size_t)(2 * 16 * MT * f.stride + 4 * 16 * MT) * 4; }

}  // namespace

FoldPlan fold_plan(AxisPlan az) {
  FoldPlan f;
  const int kmax = az.npos - 1 > az.L - az.npos ? az.npos - 1 : az.L - az.npos;
  f.rows = kmax + 1 <= 16 ? 16 : (kmax + 1 + 31) / 32 * 32;    // whole groups of the kernel's row tiles
  f.pairs = (az.N + 1) / 2;
  f.stride = (f.pairs + 15) / 16 * 16 + 4;      // 4 floats beside whole tiles: rows spread over the LDS banks
  f.floats = (size_t)2 * f.rows * f.stride + 4 * f.rows;
  return f;
}

// Whether these kernels are the faster ones, against the mixed-radix kernel for a z axis with a power of two in its
// length (M = 4: the four-point FFT leaves long residue sums, so the line lies further out there).
//
// Short rows: a wave has few bytes to ask for per load and mostly empty K steps.  us on 4096 columns of 8 channels,
// mixed radix against this one: z of 24 (two entries), t of 5, 8, 12, 14: 19, 27, 35, 49 and 40, 40, 45, 49; z of 48,
// t of 5, 9, 12: 19, 30, 43 and 32, 36, 38; z of 72, t of 7, 8, 12: 33, 40, 55 and 42, 43, 50; z of 120, t of 5, 9, 12:
// 51, 82, 101 and 78, 84, 85.  With few planes the chip is not full and the tiles that the other kernel stages in LDS are
// its longer chain: us, mixed radix against this one, z of 24 with 3 kept, t of 4, 8, 12: 2048 planes 7.2, 8.7, 10.8 and
// 6.7, 7.2, 7.2; 4608 planes 7.2, 8.6, 10.9 and 8.2, 8.5, 8.9; 9216 planes 7.5, 9.3, 11.4 and 9.8, 10.7, 11.1.  Of 588
// shapes with z of 8 to 64 points and t of 4 to 12 that differ on 512 and 2048 planes, 466 are more than a tenth faster here
// and 1 more than a tenth slower; on 4608 planes, with at most 32 points of z and more than 7 of t, 58 and 1 of 96.
//
// Many frequencies: the product over z is worked for every group of 32 rows of the table, and the one over t is worked
// again for each, where the FFT costs the same for any number of frequencies.  us on 576 columns of 4 channels, mixed
// radix against this one: z of 128 with t of 10 and 5 bins, 7, 19, 32, 64 kept per side: 11.9, 13.6, 15.0, 20.1 and
// 10.8, 14.5, 20.6, 28.2; z of 256 with t of 24 and 12 bins, 15, 38, 128 per side: 48, 53, 77 and 30, 56, 125; z of 160
// with t of 48 and 16 bins, 9, 20, 80 per side: 88, 92, 106 and 33, 39, 81.  Over 10.8 thousand shapes on 576 columns (z
// of 8 to 512, t of 8 to 48, 4 to 32 channels) 15 % were more than a tenth slower here than mixed radix without this part
// of the rule, 2 % are with it (and 2 % more than a tenth slower than here); over 2.9 thousand on 4096 columns 11 and 3 %
// (1 %).
bool tz_fwd_fold_pays(AxisPlan az, int Nt, int mt, int64_t planes) {
  if (az.M < 4) return true;
  const bool few = (planes <= 3072 && az.N <= 64) || (planes <= 6144 && az.N <= 32 && Nt > 7);
  if (!few && (Nt <= 7 || (Nt <= 9 && (az.N <= 48 || az.N > 96)) || (Nt <= 12 && az.N <= 24))) return false;
  const int rows = fold_plan(az).rows;
  if (az.M == 4) return rows <= 32 || mt > 4;
  return rows <= 16 || Nt > 36 || (rows <= 32 && mt > 4);
}

// Nt up to 64 in registers; one or two row tiles of frequencies and column tiles of bins per block (one, where the table
// of two does not leave room for two blocks on a CU: z axes of more than 608 points)
bool tz_fwd_fold_fits(AxisPlan az, int Nt, int mt) {
  return Nt <= 64 && mt <= 64 && fold_lds(fold_plan(az), 1) <= kFoldLds;
}

hipError_t launch_tz_fwd_fold(const float* x, float2* out, const float2* twt, const float* ztab, int64_t planes,
                              AxisPlan az, int Nt, int mt, hipStream_t s) {
  const FoldPlan f = fold_plan(az);
  const int CT = 2 * mt <= 16 ? 1 : 2, MT = f.rows >= 32 && fold_lds(f, 2) <= kFoldLds ? 2 : 1;
  const int mgroups = (f.rows + 16 * MT - 1) / (16 * MT), cgroups = (2 * mt + 16 * CT - 1) / (16 * CT);
  const int ngroups = mgroups * cgroups;
  const size_t lds = fold_lds(f, MT);
  // resident blocks only: each loads the z table once and walks planes
  const int J = (Nt - 1) / 16, r = Nt - 16 * J, W = (r + 3) / 4;
  const int PP = f.pairs <= 4 ? 4 : (f.pairs <= 8 ? 2 : 1);      // then also MT = 1: no more frequencies than rows
  int64_t per_cu = fold_waves(4 * J + W, CT, MT, PP);
  if (per_cu > (int64_t)(160 * 1024 / lds)) per_cu = (int64_t)(160 * 1024 / lds);
  int64_t per_x = ((planes + 7) / 8 + 4 * PP - 1) / (4 * PP);
  if (per_x > 32 * per_cu) per_x = 32 * per_cu;
  const dim3 grid((unsigned)(8 * per_x * ngroups));
  const bool stream = planes * (int64_t)az.N * Nt * 4 >= kStreamBytes;
#define FNO_TZD_S(JV, WV, CTV, MTV, PPV, STRV)                                                                  \
  hipLaunchKernelGGL((tz_fwd_fold_kernel<JV, WV, CTV, MTV, PPV, STRV>), grid, dim3(kThreads), lds, s, x,         \
                     reinterpret_cast<float*>(out), twt, ztab, (long long)planes, az.N, Nt, az.L, az.npos, mt,  \
                     f.rows, f.pairs, f.stride, ngroups, mgroups)
#define FNO_TZD_M(JV, WV, CTV, MTV, PPV)                                                                \
  do {                                                                                                  \
    if (stream) FNO_TZD_S(JV, WV, CTV, MTV, PPV, true); else FNO_TZD_S(JV, WV, CTV, MTV, PPV, false);   \
  } while (0)
#define FNO_TZD_P(JV, WV, CTV)                                                                          \
  do {                                                                                                  \
    if (PP == 4) FNO_TZD_M(JV, WV, CTV, 1, 4); else if (PP == 2) FNO_TZD_M(JV, WV, CTV, 1, 2);          \
    else if (MT == 1) FNO_TZD_M(JV, WV, CTV, 1, 1); else FNO_TZD_M(JV, WV, CTV, 2, 1);                  \
  } while (0)
  // more than eight bins (CT = 2) need 16 points of t at least: no variant of shorter rows
#define FNO_TZD_C(JV, WV)                                                           \
  do {                                                                              \
    if constexpr ((JV) > 0 || (WV) == 4) { if (CT == 2) { FNO_TZD_P(JV, WV, 2); break; } } \
    FNO_TZD_P(JV, WV, 1);                                                           \
  } while (0)
#define FNO_TZD_W(JV)                                                                         \
  do {                                                                                        \
    if (W == 1) FNO_TZD_C(JV, 1); else if (W == 2) FNO_TZD_C(JV, 2);                          \
    else if (W == 3) FNO_TZD_C(JV, 3); else FNO_TZD_C(JV, 4);                                 \
  } while (0)
  if (J == 0) FNO_TZD_W(0); else if (J == 1) FNO_TZD_W(1); else if (J == 2) FNO_TZD_W(2); else FNO_TZD_W(3);
#undef FNO_TZD_W
#undef FNO_TZD_C
#undef FNO_TZD_P
#undef FNO_TZD_M
#undef FNO_TZD_S
  return hipGetLastError();
}

}  // namespace fno
