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
// The fp32 products' sums are in short chains: two over t, blocks of eight pairs over z that are added up as they come,
// and the turn by the phase is in double.  One chain of Nz / 2 terms was off by up to 1.7 times what the FFT over z
// that these kernels replaced is off by (128 x 20: 1.18e-7 with the FFT, 1.75e-7 in one chain, 1.07e-7 now).
//
// Most shapes run both products on v_mfma_f32_16x16x32_bf16 instead (fold_split), with every float the exact sum of three
// bf16 values and the six of nine products that count (what is left out is below 2^-25 of a product): fp32 matrix
// instructions and vector instructions share one datapath, the 16-bit ones run beside it, and take 32 terms per rounding.
// Splitting a value costs five and a half vector instructions.  A K step holds 32 values: of four values (KS <= 4, and
// the rows of a tile) two parts each, so that three instructions make the six products, of eight one part.
//
// A tile's rows become sums and differences before the next tile is asked for, and those are made behind the stores of the
// plane before, whose number does not vary: the loads of a tile are on their way over the products of the one before it,
// and no wait is for stores.  (Left alone, the compiler put the sums behind the next loads, and a wave waited for these
// first.)  us, before and after: 50 x 45 columns of 40 x 24, 32 channels, 95 -> 80; 21 x 14, 24 fields of 810 columns 19 ->
// 17; 64 x 20, 20 channels, 4096 columns 123 and 122; 263 x 16 666 and 678.  Planes that share a tile have many stores
// without a lane to store, which are left out there; a wave's first tile is asked for behind its tables, since the waits
// for these would be for the tile as well.  (8 x 40, 16 bins, 3726 planes 9.9 us, 11.5 in the order before all of this.)
//
// What bounds it: in fp32 the matrix cores at 32 cycles per instruction (a 263 x 16 plane with 49 frequencies and
// 8 bins: 9 tiles of 8 + 16 instructions) next to one read of the field (20 channels, 68 x 118 columns: 0.85 ms); in parts
// the vector unit's splits, 0.68 ms = 4.7 TB/s with the bins written.  Measured against the kernels it
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
// on bf16 parts: two row tiles in flight, the parts of the t table, the accumulators, the parts of a tile, addresses
constexpr int split_regs(int KS, int CT, int MT) {
  return KS * 2 + CT * (KS <= 4 ? 6 : 12 * ((KS + 7) / 8)) + 8 * MT * CT + (KS <= 4 ? 40 : 56) + 40;
}
constexpr int fold_waves(int KS, int CT, int MT, int PP, bool split) {
  const int regs = split ? split_regs(KS, CT, MT) : fold_regs(KS, CT, MT, PP);
  return regs <= 64 ? 8 : (regs <= 72 ? 6 : (regs <= 96 ? 5 : (regs <= 128 ? 4 : (regs <= 168 ? 3 : 2))));
}
// words of a row of the table in parts (three bf16 a value): 4 modulo 8, so that the rows that a read covers spread over
// all banks
__host__ __device__ constexpr int split_stride(int stride) { return (6 * (stride >> 2) + 3) / 8 * 8 + 4; }
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v4f mfma_split(u32x4 a, u32x4 b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// Four values in parts p[0] (large) to p[2], as the operands of the six products that count: against a table's (third,
// first) parts (p0, p2), against its (first, second) ones (p1, p1) and (p0, p0).
struct Quad { u32x4 p02, p11, p00; };
template <int N>
__device__ __forceinline__ void split_quad(const float (&v)[N], Quad& q) {
  unsigned a[3], b[3];
  bf16_split(v[0], N > 1 ? v[N > 1 ? 1 : 0] : 0.f, a);
  bf16_split(N > 2 ? v[N > 2 ? 2 : 0] : 0.f, N > 3 ? v[N > 3 ? 3 : 0] : 0.f, b);
  q.p02 = u32x4{a[0], b[0], a[2], b[2]};
  q.p11 = u32x4{a[1], b[1], a[1], b[1]};
  q.p00 = u32x4{a[0], b[0], a[0], b[0]};
}
// t: third, first and second parts of four entries of a table
template <class F>
__device__ __forceinline__ v4f quad_product(const u32x2 (&t)[3], const Quad& q, F mfma) {
  const u32x4 t20 = {t[0][0], t[0][1], t[1][0], t[1][1]}, t01 = {t[1][0], t[1][1], t[2][0], t[2][1]};
  v4f a = mfma(t20, q.p02, v4f{0.f, 0.f, 0.f, 0.f});
  a = mfma(t01, q.p11, a);
  return mfma(t01, q.p00, a);
}
// values s0 .. s0 + 7 of N in parts, zeros past the end
template <int N>
__device__ __forceinline__ void split_octet(const float (&v)[N], int s0, u32x4 (&p)[3]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    unsigned q[3];
    const int s = s0 + 2 * j;
    bf16_split(s < N ? v[s < N ? s : 0] : 0.f, s + 1 < N ? v[s + 1 < N ? s + 1 : 0] : 0.f, q);
#pragma unroll
    for (int h = 0; h < 3; ++h) p[h][j] = q[h];
  }
}

// A row of Nt = 16 J + r floats (1 <= r <= 16): J runs of 16 (four per lane group) and a tail in which
// lane group g takes W = ceil(r / 4) floats from min(W g, r - W), so that no lane reads past its row;
// entries a lower group has already taken meet zeros in the t table.
// PP planes of at most 16 / PP row pairs share a tile: row 4 g + v of it is pair (4 / PP) g + v % (4 / PP) of
// plane v / (4 / PP), so that each register of the first product belongs to one plane.
// SPLIT: 1 the products on bf16 parts, 2 the same in blocks of eight waves.
template <int J, int W, int CT, int MT, int PP, int SPLIT, bool STREAM>
__global__ __launch_bounds__(SPLIT > 1 ? 2 * kThreads : kThreads, fold_waves(4 * J + W, CT, MT, PP, SPLIT > 0)) void tz_fwd_fold_kernel(
    const float* __restrict__ x, float* __restrict__ out, const float2* __restrict__ twt,
    const float* __restrict__ ztab, long long planes, int field, int Nz, int Nt, int Lz, int npos, int mt, int mrows,
    int pairs, int stride, int ngroups, int mgroups) {
  HIP_DYNAMIC_SHARED(float, smem)
  constexpr int TH = SPLIT > 1 ? 2 * kThreads : kThreads;
  constexpr int KS = 4 * J + W;                 // K steps of the product over t
  const int row = SPLIT ? split_stride(stride) : stride;       // words of a row of the table in LDS
  float* COS = smem;                            // [16 MT][row]
  float* SIN = smem + 16 * MT * row;            // [16 MT][row]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // uniform: plane addresses stay scalar
  const int c = lane & 15, g = lane >> 4;
  // blocks that share planes but not frequencies or columns sit on one XCD next to each other
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const int grp = local % ngroups;
  const int m0 = 16 * MT * (grp % mgroups), c0 = 16 * CT * (grp / mgroups);
  const int r = Nt - 16 * J;
  const int t0 = min(W * g, r - W);             // start of this lane group's tail
  // each XCD walks a contiguous eighth of the planes, its waves interleaved inside it
  const long long per_x = (planes + 7) >> 3;
  const long long pe = min(planes, (long long)(xcd + 1) * per_x);
  const long long nwl = (long long)((gridDim.x >> 3) / ngroups) * (TH / 64) * PP;
  long long p = (long long)xcd * per_x + ((long long)(local / ngroups) * (TH / 64) + wave) * PP;
  const int ntile = PP > 1 ? 1 : (pairs + 15) >> 4;
  constexpr int VP = 4 / PP;                    // registers of a lane that belong to one plane
  const int lp = (c & 3) / VP, ln = VP * (c >> 2) + (c & (VP - 1));      // plane and pair of tile row c (PP > 1)

  float va[KS], vb[KS];                         // this lane's part of row n and of row Nz - 1 - n
  // (there: else nothing is read and the values are zeros)
  auto load_tile = [&](long long plane, int tile, bool there) {
    const int n = min(PP > 1 ? ln : 16 * tile + c, pairs - 1);
    const int first = PP > 1 ? min(lp, (int)min((long long)PP, planes - plane) - 1) * Nz : 0;      // row of the lane's plane
    const __amdgpu_buffer_rsrc_t base = buffer_of(x + plane * (Nz * Nt), there ? PP * Nz * Nt * 4 : 0);
    const unsigned ra = (unsigned)((first + n) * Nt) * 4u, rb = (unsigned)((first + Nz - 1 - n) * Nt) * 4u;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      float qa[4], qb[4];
      buffer_load<4, STREAM>(base, ra + 64u * j + 16u * g, qa);
      buffer_load<4, STREAM>(base, rb + 64u * j + 16u * g, qb);
#pragma unroll
      for (int u = 0; u < 4; ++u) { va[4 * j + u] = qa[u]; vb[4 * j + u] = qb[u]; }
    }
    float qa[W], qb[W];
    buffer_load<W, STREAM>(base, ra + 64u * J + 4u * t0, qa);
    buffer_load<W, STREAM>(base, rb + 64u * J + 4u * t0, qb);
#pragma unroll
    for (int u = 0; u < W; ++u) { va[4 * J + u] = qa[u]; vb[4 * J + u] = qb[u]; }
  };
  {
    const float4* cs = reinterpret_cast<const float4*>(ztab + (long long)m0 * stride);
    const float4* sn = reinterpret_cast<const float4*>(ztab + (long long)(mrows + m0) * stride);
    const int n4 = (16 * MT * stride) >> 2;
    if constexpr (SPLIT) {
      // four pairs of a row at a time: their third, first and second parts
      const int quads = stride >> 2;
      for (int i = tid; i < n4; i += TH) {
        const int r = i / quads, at = r * row + 6 * (i - r * quads);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 v = h ? sn[i] : cs[i];
          unsigned a[3], b[3];
          bf16_split(v.x, v.y, a);
          bf16_split(v.z, v.w, b);
          u32x2* d = reinterpret_cast<u32x2*>((h ? SIN : COS) + at);
          d[0] = u32x2{a[2], b[2]};
          d[1] = u32x2{a[0], b[0]};
          d[2] = u32x2{a[1], b[1]};
        }
      }
    } else {
      for (int i = tid; i < n4; i += TH) {
        reinterpret_cast<float4*>(COS)[i] = cs[i];
        reinterpret_cast<float4*>(SIN)[i] = sn[i];
      }
    }
  }
  double2* ROT = reinterpret_cast<double2*>(SIN + 16 * MT * row);       // [16 MT]
  if (tid < 16 * MT) ROT[tid] = reinterpret_cast<const double2*>(ztab + (long long)2 * mrows * stride)[m0 + tid];
  float tb[CT][KS];                             // t table, the right operand of every K step
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int col = c0 + 16 * ct + c, kt = col >> 1;
    const float* part = reinterpret_cast<const float*>(twt + min(kt, mt - 1) * Nt) + (col & 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int t = s < 4 * J ? 16 * (s >> 2) + 4 * g + (s & 3) : 16 * J + t0 + (s - 4 * J);
      const bool dup = s >= 4 * J && t < 16 * J + W * g;
      tb[ct][s] = 0.f;
      if (kt < mt && !dup) tb[ct][s] = part[2 * t];
    }
  }
  // the same in parts: KS <= 4 third, first and second part of four values; else eight values a part
  constexpr int KB = (KS + 7) / 8;
  u32x2 t4[SPLIT && KS <= 4 ? CT : 1][3];
  u32x4 t8[SPLIT && KS > 4 ? CT : 1][KB][3];
  if constexpr (SPLIT) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      auto part2 = [&](int s0, unsigned (&q)[3]) { bf16_split(s0 < KS ? tb[ct][s0 < KS ? s0 : 0] : 0.f, s0 + 1 < KS ? tb[ct][s0 + 1 < KS ? s0 + 1 : 0] : 0.f, q); };
      if constexpr (KS <= 4) {
        unsigned a[3], b[3];
        part2(0, a);
        part2(2, b);
        t4[ct][0] = u32x2{a[2], b[2]};
        t4[ct][1] = u32x2{a[0], b[0]};
        t4[ct][2] = u32x2{a[1], b[1]};
      } else {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            unsigned q[3];
            part2(8 * kb + 2 * j, q);
#pragma unroll
            for (int p = 0; p < 3; ++p) t8[ct][kb][p][j] = q[p];
          }
      }
    }
  }
  const double sgn = (c & 1) ? -1.0 : 1.0;
  __syncthreads();
  if (p >= pe) return;
  load_tile(p, 0, true);                        // (behind the tables, whose waits would be for it too)

  int at_field = SPLIT > 0 ? (int)(p % field) : 0;         // of the plane in its (batch, channel) field
  const int step_field = SPLIT > 0 ? (int)(nwl % field) : 0;
  // Sums and differences of the tile's rows.  They are made behind the stores of the plane before, of which there are
  // always as many, so that the wait for the tile's loads is not one for stores; and here and now, so that the next loads
  // take the places of these values.
  float e[KS], o[KS];
  bool neg;
  auto fold_rows = [&]() {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      float sum = neg ? -va[s] - vb[s] : va[s] + vb[s], diff = neg ? vb[s] - va[s] : va[s] - vb[s];
      asm volatile("" : "+v"(sum), "+v"(diff));
      e[s] = sum;
      o[s] = diff;
    }
  };
  neg = SPLIT > 0 && (__builtin_popcount((unsigned)at_field) & 1);
  fold_rows();
  for (; p < pe; p += nwl) {
    // The 16-bit instructions cut their sums towards minus infinity some bits below the rounding (0.004 units of the last
    // place on average).  Planes add up over y and x, where the lowest frequencies of 48 x 32 planes of 108 x 33 were off
    // by 3.3e-6 of a bin's size, fp32 products 8e-7.  Planes with an odd number of ones in their index within the field are
    // worked with the other sign, which takes it out (6.5e-7).
    const bool turned = neg;                     // neg is the next plane's from the last tile on
    if constexpr (SPLIT > 0) {
      at_field += step_field;
      if (at_field >= field) at_field -= field;
    }
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
    // the products of a tile's rows, while the next tile's are on their way
    auto products = [&](int tile) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (SPLIT) {
        const v4f zero = {0.f, 0.f, 0.f, 0.f};
        v4f dE[CT], dO[CT];
        if constexpr (KS <= 4) {
          Quad qe, qo;
          split_quad<KS>(e, qe);
          split_quad<KS>(o, qo);
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            dE[ct] = quad_product(t4[ct], qe, [](u32x4 t, u32x4 d, v4f a) { return mfma_split(d, t, a); });
            dO[ct] = quad_product(t4[ct], qo, [](u32x4 t, u32x4 d, v4f a) { return mfma_split(d, t, a); });
          }
        } else {
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) dE[ct] = dO[ct] = zero;
          u32x4 pe[KB][3], po[KB][3];
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            split_octet<KS>(e, 8 * kb, pe[kb]);
            split_octet<KS>(o, 8 * kb, po[kb]);
          }
          constexpr int A[6] = {2, 0, 1, 1, 0, 0}, Bp[6] = {0, 2, 1, 0, 1, 0};       // the small products first
#pragma unroll
          for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
              for (int ct = 0; ct < CT; ++ct) {
                dE[ct] = mfma_split(pe[kb][A[r]], t8[ct][kb][Bp[r]], dE[ct]);
                dO[ct] = mfma_split(po[kb][A[r]], t8[ct][kb][Bp[r]], dO[ct]);
              }
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          Quad qe, qo;
          const float ve[4] = {dE[ct][0], dE[ct][1], dE[ct][2], dE[ct][3]}, vo[4] = {dO[ct][0], dO[ct][1], dO[ct][2], dO[ct][3]};
          split_quad<4>(ve, qe);
          split_quad<4>(vo, qo);
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const u32x2* zc = reinterpret_cast<const u32x2*>(COS + (16 * m + c) * row + 6 * (4 * tile + g));
            const u32x2* zs = reinterpret_cast<const u32x2*>(SIN + (16 * m + c) * row + 6 * (4 * tile + g));
            const u32x2 tc[3] = {zc[0], zc[1], zc[2]}, ts[3] = {zs[0], zs[1], zs[2]};
            accC[0][m][ct] += quad_product(tc, qe, [](u32x4 t, u32x4 d, v4f a) { return mfma_split(t, d, a); });
            accS[0][m][ct] += quad_product(ts, qo, [](u32x4 t, u32x4 d, v4f a) { return mfma_split(t, d, a); });
          }
        }
        return;
      }
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
    };
    // the plane's last tile apart: on its way the next plane's first is asked for, and stores come between
    if constexpr (PP == 1) {
#pragma unroll 1
      for (int tile = 0; tile + 1 < ntile; ++tile) {
        load_tile(p, tile + 1, true);
        products(tile);
        fold_rows();
      }
    }
    load_tile(p + nwl < pe ? p + nwl : p, 0, p + nwl < pe);
    products(ntile - 1);
    // X[+-k] from C, S: real and imaginary parts sit in neighbouring lanes
    // the phases and the store offsets are worked out again for every plane, not kept in registers
    int g4 = 4 * g;
    asm volatile("" : "+v"(g4)::"memory");
#pragma unroll
    for (int q = 0; q < PP; ++q) {
      // lanes and planes without a place have an offset past the end
      const __amdgpu_buffer_rsrc_t dst = buffer_of(out + (p + q) * (Lz * mt * 2), PP == 1 || p + q < pe ? Lz * mt * 8 : 0);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          // no lane has a frequency (with one plane a tile, whose wait for the next loads counts the stores, these stay)
          if (PP > 1 && m0 + 16 * m + v >= npos && m0 + 16 * m + v > Lz - npos) continue;
          const int kl = 16 * m + g4 + v, k = m0 + kl;
          double2 w = ROT[kl];
          if (turned) w = make_double2(-w.x, -w.y);
          const double ws = sgn * w.y;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const int col = c0 + 16 * ct + c;
            const float fc = accC[q][m][ct][v], fs = accS[q][m][ct][v];
            const double C = fc, is = sgn * swap_pair(fs);       // this part of C and -i S, and the other part
            const double D = swap_pair(fc), it = sgn * fs;
            const double yp = fma(C + is, w.x, -ws * (D - it));
            const double ym = fma(C - is, w.x, ws * (D + it));
            const float p1[1] = {(float)yp}, m1[1] = {(float)ym};
            buffer_store<1, false>(dst, col < 2 * mt && k < npos ? (unsigned)(k * mt * 2 + col) * 4u : kNowhere, p1);
            buffer_store<1, false>(dst, col < 2 * mt && k >= 1 && k <= Lz - npos ? (unsigned)((Lz - k) * mt * 2 + col) * 4u : kNowhere, m1);
          }
        }
    }
    if constexpr (SPLIT > 0) neg = __builtin_popcount((unsigned)at_field) & 1;
    fold_rows();
  }
}

constexpr size_t kFoldLds = 78 * 1024;      // two blocks per CU

size_t fold_lds(const FoldPlan& f, int MT, int split = 0) {
  return (size_t)(2 * 16 * MT * (split ? split_stride(f.stride) : f.stride) + 4 * 16 * MT) * 4;
}

// Which products: 0 fp32, 1 bf16 parts, 2 the same in blocks of eight waves.  The parts pay where the matrix work is what
// a wave waits for: two tiles of bins or of frequencies, or whole K steps of the product over t (KS: a quarter of 16
// points, or most of 32 and more).  Their table takes half as much LDS again, so that above 40 KiB a block has eight waves,
// and only where four values a lane make a K step.  us, fp32 and parts, 8 channels, 24 x 24 columns: z of 118, 20 kept a
// side, t of 8, 16, 24 and 48 with 3, 8, 12 and 16 bins 17.0, 20.2, 34.3, 47.4 and 15.1, 17.6, 25.0, 37.7; 64 x 64
// columns: z of 60, 12 kept, t of 16, 24, 30 with 8, 12, 8 bins 40.2, 78.5, 85.5 and 38.3, 70.5, 76.9, but t of 8 and 10
// with 3 and 4 bins 29.6, 32.4 and 31.2, 34.4; z of 263, 24 kept, t of 10 and 14 with 4 and 6 bins 162, 173 and 137, 146
// (in blocks of four waves 181, 192), but 24 x 24 columns of 20 and 30 points of t 33 and 41 and, in blocks of eight, 39
// and 47.  Blocks of eight waves need a plane for every wave of a chip full of them; with fewer, blocks of four take their
// place: 263 x 16, 24 kept, 8 bins on 64, 256, 1024 and 2304 planes 12.6, 12.7, 14.1, 21.1 with eight waves, 11.1, 10.4, 12.2
// with four (fp32 11.0, 11.0, 13.6, 21.4).
int fold_split(const FoldPlan& f, int KS, int CT, int MT, int PP, int64_t planes) {
  const size_t lds = fold_lds(f, MT, 1);
  if (PP > 1 || lds > kFoldLds) return 0;
  if (CT == 2) return 1;
  if (lds > 40 * 1024) return MT == 2 && KS <= 4 ? (planes >= 2048 ? 2 : 1) : 0;
  return MT == 2 || (f.pairs > 16 && (KS == 4 || KS >= 7)) ? 1 : 0;
}

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
                              int field, AxisPlan az, int Nt, int mt, hipStream_t s) {
  const FoldPlan f = fold_plan(az);
  const int PP = f.pairs <= 4 ? 4 : (f.pairs <= 8 ? 2 : 1);      // more than one: also MT = 1, no more frequencies than rows
  const int CT = 2 * mt <= 16 ? 1 : 2, MT = f.rows >= 32 && fold_lds(f, 2) <= kFoldLds ? 2 : 1;
  const int J = (Nt - 1) / 16, r = Nt - 16 * J, W = (r + 3) / 4;
  const int split = fold_split(f, 4 * J + W, CT, MT, PP, planes), threads = split > 1 ? 2 * kThreads : kThreads;
  const int mgroups = (f.rows + 16 * MT - 1) / (16 * MT), cgroups = (2 * mt + 16 * CT - 1) / (16 * CT);
  const int ngroups = mgroups * cgroups;
  const size_t lds = fold_lds(f, MT, split);
  // resident blocks only: each loads the z table once and walks planes
  int64_t per_cu = fold_waves(4 * J + W, CT, MT, PP, split > 0) * kThreads / threads;
  if (per_cu > (int64_t)(160 * 1024 / lds)) per_cu = (int64_t)(160 * 1024 / lds);
  const int64_t per_block = threads / 64 * PP;
  int64_t per_x = ((planes + 7) / 8 + per_block - 1) / per_block;
  if (per_x > 32 * per_cu) per_x = 32 * per_cu;
  const dim3 grid((unsigned)(8 * per_x * ngroups));
  const bool stream = planes * (int64_t)az.N * Nt * 4 >= kStreamBytes;
#define FNO_TZD_S(JV, WV, CTV, MTV, PPV, SPV, STRV)                                                             \
  hipLaunchKernelGGL((tz_fwd_fold_kernel<JV, WV, CTV, MTV, PPV, SPV, STRV>), grid, dim3(threads), lds, s, x,    \
                     reinterpret_cast<float*>(out), twt, ztab, (long long)planes, field, az.N, Nt, az.L, az.npos, mt,  \
                     f.rows, f.pairs, f.stride, ngroups, mgroups)
#define FNO_TZD_M(JV, WV, CTV, MTV, PPV, SPV)                                                                    \
  do {                                                                                                           \
    if (stream) FNO_TZD_S(JV, WV, CTV, MTV, PPV, SPV, true); else FNO_TZD_S(JV, WV, CTV, MTV, PPV, SPV, false);  \
  } while (0)
#define FNO_TZD_P(JV, WV, CTV)                                                                                   \
  do {                                                                                                           \
    if (PP == 4) FNO_TZD_M(JV, WV, CTV, 1, 4, 0);                                                                \
    else if (PP == 2) FNO_TZD_M(JV, WV, CTV, 1, 2, 0);                                                           \
    else if (MT == 1) {                                                                                          \
      if constexpr ((CTV) == 2 || 4 * (JV) + (WV) == 4 || 4 * (JV) + (WV) >= 7) {                                \
        if (split) { FNO_TZD_M(JV, WV, CTV, 1, 1, 1); break; }                                                   \
      }                                                                                                          \
      FNO_TZD_M(JV, WV, CTV, 1, 1, 0);                                                                           \
    } else if (split == 1) FNO_TZD_M(JV, WV, CTV, 2, 1, 1);                                                      \
    else {                                                                                                       \
      if constexpr ((CTV) == 1 && (JV) == 0) { if (split) { FNO_TZD_M(JV, WV, 1, 2, 1, 2); break; } }            \
      FNO_TZD_M(JV, WV, CTV, 2, 1, 0);                                                                           \
    }                                                                                                            \
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
