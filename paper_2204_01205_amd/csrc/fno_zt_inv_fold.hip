// Inverse (z, t) + block epilogue for any axis lengths (see fno_zt_inv.hip for what the stage computes), as
// chained matrix products on the matrix cores: the counterpart of fno_tz_fwd_fold.hip.
//
// With nu = n + 1/2 and the kept frequencies k = 0 .. kmax of the z axis folded into
//   E[k] = a'[k] + a'[-k],  O[k] = i (a'[k] - a'[-k]),  a'[+-k] = exp(-+i pi k / Nz) a[+-k],
// the rows of a pair are V[n] = C[n] + S[n] and V[Nz-1-n] = C[n] - S[n] with
//   C[n] = sum_k cos(2 pi k nu / Nz) E[k],   S[n] = sum_k sin(2 pi k nu / Nz) O[k]:
// both matrices are real, and a pair of rows shares its products.  A row's points then follow as
// sum_c cs[t][c] V[n][c] over the 2 mt - 1 real columns c (the imaginary part of bin 0 does not enter).
//
// Both products run on v_mfma_f32_16x16x4 (full fp32; lane l supplies A[l%16][l/16] and B[l/16][l%16] and
// holds rows 4 (l/16) + v of column l%16).  Four output channels share a tile of the first: its row 4 g + v is
// column c = 4 tau + g of channel v, its columns are 16 row pairs.  Register v of the result then holds, as it
// stands, one K step of channel v's product over c, whose result gives a lane W consecutive t of one row: the
// layout in which u is read and the output written.  The channel-linear term joins in that layout too:
// v_mfma_f32_4x4x1 with W[4T+i][.] as the left and a lane's own point as the right operand leaves four output
// channels of that point in the lane.
//
// Rounding: E and O are folded and turned in double, once per column; the sums over k run from the highest frequency
// down, in four chains where no u is held (a convolution; the channel-linear term outweighs them in a block).  With an
// fp32 phase and one chain a 128 x 20 plane was off by 1.31e-7, against 1.06e-7 for the FFT over z that these kernels
// replaced and 1.10e-7 now, at 1 % more time; after all axes a convolution is no further off than it was with the FFTs.
//
// One wave works a tile of 16 row pairs x 4 W points of t for all output channels, its u values in registers; or, where t
// takes two tiles, 16 rows x 8 W points, so that its accesses are whole rows: with one tile of t per task the lines that
// two tiles share were read twice, and a third of the writes were halves of lines that had left the L2 before the other
// wave's half came (64 x 30, forward of a training block: 24.3 million writes for 17.3 million lines' worth).
// LDS holds E and O of the block's columns, folded once per column by the waves that share it, and per wave the
// cos / sin entries of its row pairs.  After the fold no wave waits for another.  A last tile of at most eight
// pairs puts the second rows of its pairs into the idle half of the lanes.
//
// The next task's u and table are asked for when the last group of channels has used u, and no wait in between is for
// them or for stores: accesses go through buffer resources (loads through a pointer without an address space are flat
// ones, which count as LDS accesses too, so that every LDS wait waited for them), lanes without a point have an offset
// past the end instead of a branch, and the table goes to LDS by itself.
//
// What bounds it: issue where many frequencies are kept (263 x 16, 24 kept: matrix instructions in 43 % of a SIMD's cycles,
// vector instructions in 31 %; fp32 matrix instructions and vector instructions share one datapath, measured: their times
// add up, within a wave and between waves), else its traffic in part (64 x 30, three streams: 28 and 25 %, 3.8 TB/s): u
// in registers allows two waves per SIMD; streaming u past accumulators for all output channels takes as many, and one
// row at a time, with three waves, was no faster.  us before and after the whole rows and the waits: 64 x 30, 3600 columns of 20
// channels, forward with the pre-activation 495 -> 435, adjoint 372 -> 332; 263 x 16, 8024 columns, 1730 -> 1650.
// Measured against the kernels that this one replaced (mixed-radix or dense sums with LDS staging, and
// 4x4x1 tiles of one residue class), milliseconds: 20 channels, 68 x 118 columns of 263 x 16 3.95 -> 1.68; one block
// forward and back: 20 channels, 64^3 x 20 0.89 -> 0.68, x 30 0.95 -> 0.81, 32 channels, 50 x 45 x 40 x 24
// 1.19 -> 0.54, 16 channels, 64^3 x 16 0.42 -> 0.33, 12 channels, 64 x 64 x 48 x 16 0.52 -> 0.21.
#include "fno_zt_inv.h"

#include <type_traits>

namespace fno {

namespace {

struct FoldInv {
  long long ncols, Npts;
  int Co, NxNy, Nz, Nt, Lz, npos, mt;
  int K1, ks;            // folded frequencies, K steps of the product over them
  int R;                 // tiles of columns: ceil((2 mt - 1) / 4)
  int pairs, stride, mrows;      // of the folded table (FoldPlan)
  int ntile, tt;         // tiles of row pairs and of t
  int two_t;             // a task takes both tiles of t and one row of each pair (two tiles of t in all)
  int half_last;         // both rows of the last tile's pairs fit its 16 columns
  int ntask;             // tiles of t inside tiles of row pairs; one row at a time: rows n, then rows Nz-1-n of whole tiles
  int ct, nchunk;        // groups of four output channels per block, blocks per column
  int wc_shift;          // log2 of the waves that share a column
  unsigned items;        // blocks with work
  unsigned inv_mt;       // ceil(2^32 / mt): division by multiplication, exact for the counts here
};

constexpr int fold_inv_ns(int W, int CI) { return 2 * W * CI <= 160 ? 2 : 1; }
// smallest channel count that runs with CI register slots: the slots from there on may be empty
constexpr int fold_inv_low(int CI) { return CI <= 8 ? 1 : (CI == 32 ? 25 : CI - 3); }

// Where a lane's points of one task lie: NU runs of W points, of the two rows of a pair or of one row.
template <int NU> struct FoldTile {
  int n;                 // pair of rows
  bool second;           // one row per lane: it is Nz-1-n
  bool half;             // both rows of the pairs in one set of 16 columns (uniform)
  int ti;                // tile of t of the first run
  unsigned at[NU];       // byte offsets of the runs inside a column of one channel; kNowhere: no such points, or another lane's
};
template <int NU, int W>
__device__ __forceinline__ FoldTile<NU> fold_inv_place(const FoldInv& f, int task, bool active) {
  FoldTile<NU> q;
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  const bool two_t = NU == 2 && f.two_t;
  const int t1 = two_t ? task : task / f.tt, rt = t1 < f.ntile ? t1 : t1 - f.ntile;
  q.ti = two_t ? 0 : task - t1 * f.tt;
  q.half = f.half_last && rt == f.ntile - 1;
  q.second = q.half ? c >= 8 : t1 >= f.ntile;
  q.n = 16 * rt + (q.half ? c & 7 : c);
  const bool own = 2 * q.n + 1 == f.Nz;        // the middle row of an odd axis: stored once
  const bool there = active && q.n < f.pairs;
  auto run = [&](int row, int ti) {
    const int t = W * (4 * ti + g);
    return t < f.Nt ? (unsigned)(row * f.Nt + min(t, f.Nt - W)) * 4u : kNowhere;
  };
  const int row = q.second ? f.Nz - 1 - q.n : q.n;
  const bool once = there && !(q.second && own);
  q.at[0] = once ? run(row, q.ti) : kNowhere;
  if constexpr (NU == 2)
    q.at[1] = two_t ? (once ? run(row, 1) : kNowhere) : (once && !own && !q.half ? run(f.Nz - 1 - q.n, q.ti) : kNowhere);
  return q;
}

// the waves of a block meet once their LDS accesses are done; what is on its way from and to memory stays so
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// u of the lane's points, every input channel (up: channel 0 of the column)
template <int NU, int W, int CI, bool STREAM>
__device__ __forceinline__ void fold_inv_load_u(const unsigned (&at)[NU], const char* up, unsigned bytes, int Cu, long long chan_bytes,
                                                float (&u)[CI > 0 ? CI : 1][NU][W]) {
#pragma unroll
  for (int i = 0; i < CI; ++i) {
    // channels past the last: nothing to read, zeros
    const __amdgpu_buffer_rsrc_t r = buffer_of(up, i < fold_inv_low(CI) || i < Cu ? bytes : 0);
#pragma unroll
    for (int s = 0; s < NU; ++s) buffer_load<W, STREAM>(r, at[s], u[i][s]);
    up += chan_bytes;
    asm volatile("" : "+s"(up));                 // one running base, not one per channel
  }
}

// C and S of NR tiles of columns (stride R1 float2 apart), each in CH chains: the operands of the next K step are read
// while this one's products run.  From the highest frequencies down, so that the large low ones join the sums last.
// last: the lane's entry of the last K step, which may reach past the folded frequencies (its lanes there read the last
// one again, and in_last is false).
template <int NR, int CH>
__device__ __forceinline__ void fold_inv_z(const float2* eo, int R1, const float* zt, int ks, int last, bool in_last,
                                           v4f (&C)[NR], v4f (&S)[NR]) {
  const int lane = threadIdx.x & 63;
  v4f c[CH][NR], s[CH][NR];
  auto entry = [&](int k) { return make_float2(zt[128 * k + lane], zt[128 * k + 64 + lane]); };
  float2 e[NR], z = entry(ks - 1);
  z = in_last ? z : make_float2(0.f, 0.f);
#pragma unroll
  for (int h = 0; h < NR; ++h) {
    e[h] = eo[h * R1 + last];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) c[ch][h] = s[ch][h] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  auto step = [&](v4f (&cc)[NR], v4f (&ss)[NR], int k) {
    const int at = 64 * max(k - 1, 0) + lane;
    const float2 zn = entry(max(k - 1, 0));
    float2 en[NR];
#pragma unroll
    for (int h = 0; h < NR; ++h) en[h] = eo[h * R1 + at];
#pragma unroll
    for (int h = 0; h < NR; ++h) {
      cc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(e[h].x, z.x, cc[h], 0, 0, 0);
      ss[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(e[h].y, z.y, ss[h], 0, 0, 0);
    }
    z = zn;
#pragma unroll
    for (int h = 0; h < NR; ++h) e[h] = en[h];
  };
  int k = ks - 1;
  if constexpr (CH == 1) {
#pragma unroll 2
    for (; k > 0; --k) step(c[0], s[0], k);
  } else {
    for (; k >= CH; k -= CH)
#pragma unroll
      for (int ch = 0; ch < CH; ++ch) step(c[ch], s[ch], k - ch);
#pragma unroll
    for (int ch = 0; ch + 1 < CH; ++ch)
      if (k > 0) step(c[ch], s[ch], k--);
  }
#pragma unroll
  for (int h = 0; h < NR; ++h) {                 // the lowest frequencies: nothing left to read
    c[CH - 1][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(e[h].x, z.x, c[CH - 1][h], 0, 0, 0);
    s[CH - 1][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(e[h].y, z.y, s[CH - 1][h], 0, 0, 0);
    C[h] = c[0][h];
    S[h] = s[0][h];
#pragma unroll
    for (int ch = 1; ch < CH; ++ch) { C[h] += c[ch][h]; S[h] += s[ch][h]; }
  }
}

// One K step of the four channels' products over t, for the lane's first run and (both) its second one.
template <int NS>
__device__ __forceinline__ void fold_inv_t(const float (&tb)[NS], v4f C, v4f S, const float (&sign)[NS], bool both,
                                           v4f (&d2)[4][NS]) {
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s == 0 || both)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        d2[v][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(tb[s], fmaf(sign[s], S[v], C[v]), d2[v][s], 0, 0, 0);
}

// The cos / sin entries of a task's row pairs, K step by K step: straight to the wave's LDS.
template <int NS>
__device__ __forceinline__ void fold_inv_load_z(const FoldInv& f, const float* ztab, const FoldTile<NS>& q, float* ZT) {
  const int g = (threadIdx.x & 63) >> 4, plane = f.mrows * f.stride * 4, at = (g * f.stride + q.n) * 4;
  const __amdgpu_buffer_rsrc_t r = buffer_of(ztab, 2 * plane);
  for (int s = 0; s < f.ks; ++s) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(ZT + 128 * s), 4, at,
                                             16 * s * f.stride, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(ZT + 128 * s + 64), 4, at,
                                             16 * s * f.stride + plane, 0, 0);
  }
}

// What a task needs from memory.  u comes after the table, in fold_inv_asked() instructions.
template <int NS, int CI> constexpr int fold_inv_asked() { return NS * CI; }
template <int NS, int W, int CI, bool STREAM>
__device__ __forceinline__ void fold_inv_ask(const FoldInv& f, const float* ztab, const FoldTile<NS>& q, float* ZT,
                                             const char* up, int Cu, float (&u)[CI > 0 ? CI : 1][NS][W]) {
  asm volatile("" ::: "memory");
  fold_inv_load_z<NS>(f, ztab, q, ZT);
  asm volatile("" ::: "memory");
  if constexpr (CI > 0) fold_inv_load_u<NS, W, CI, STREAM>(q.at, up, f.Nz * f.Nt * 4, Cu, f.Npts * 4, u);
  asm volatile("" ::: "memory");
}
// all but the last n memory instructions of the wave are done (n: fewer are still allowed)
template <int n>
__device__ __forceinline__ void wait_vm() {
  constexpr int v = n < 63 ? n : 63;
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((v & 15) | 7 << 4 | 15 << 8 | (v >> 4) << 14);
  asm volatile("" ::: "memory");
}

// One task: NS runs of a lane's points.
template <int NS, int W, int CI, bool STREAM>
__device__ __forceinline__ void fold_inv_tile(const FoldInv& f, const EpiArgs& ep, float* __restrict__ out,
                                              const float* __restrict__ ztab, const float2* EO, float* ZT,
                                              const float* TB, const float* WL, const float4* BL, long long first,
                                              int o0, const FoldTile<NS>& q,
                                              float (&u)[CI > 0 ? CI : 1][NS][W], const char* up,
                                              int task_next, bool active) {
  const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  // the middle row of an odd axis is its own pair, in the table at half weight
  const float weight = 2 * q.n + 1 == f.Nz ? 2.f : 1.f;
  const bool two_t = NS == 2 && f.two_t, both = NS == 2 && (two_t || !q.half);       // uniform
  float sign[NS];                                // of S in the run's row
  sign[0] = q.second ? -1.f : 1.f;
  if constexpr (NS == 2) sign[1] = two_t ? sign[0] : -1.f;
  const int last = min(4 * (f.ks - 1) + g, f.K1 - 1) * 16 + c;
  const bool in_last = 4 * (f.ks - 1) + g < f.K1;
  const int R1 = f.K1 * 16;
  const float* tbp = TB + q.ti * f.R * 64 + lane;
  const int tb_next = two_t ? f.R * 64 : 0;
  auto tables = [&](int r, float (&tb)[NS]) {
    tb[0] = tbp[64 * r];
    if constexpr (NS == 2) tb[1] = tbp[tb_next + 64 * r];
  };
  for (int T = 0; T < f.ct; ++T) {
    const int o = o0 + 4 * T;
    v4f d2[4][NS];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int s = 0; s < NS; ++s) d2[v][s] = v4f{0.f, 0.f, 0.f, 0.f};
    const float2* eot = EO + T * f.R * R1;
    int r = f.R;                                 // from the highest bins of t down
    if (CI == 0 || (r & 1)) {
      for (; r > (CI == 0 ? 0 : f.R - 1); --r) {
        v4f C[1], S[1];
        float tb[NS];
        tables(r - 1, tb);
        fold_inv_z<1, CI == 0 ? 4 : 1>(eot + (r - 1) * R1, R1, ZT, f.ks, last, in_last, C, S);
        fold_inv_t<NS>(tb, C[0], S[0], sign, both, d2);
      }
    }
    if constexpr (CI > 0) {
      for (; r >= 2; r -= 2) {
        v4f C[2], S[2];
        float tb0[NS], tb1[NS];
        tables(r - 2, tb0);
        tables(r - 1, tb1);
        fold_inv_z<2, 1>(eot + (r - 2) * R1, R1, ZT, f.ks, last, in_last, C, S);
        fold_inv_t<NS>(tb1, C[1], S[1], sign, both, d2);
        fold_inv_t<NS>(tb0, C[0], S[0], sign, both, d2);
      }
    }
    // four channels of a point side by side, the bias, and the channel-linear term on top
    const float4 bias = BL[T];
    v4f acc[NS][W];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int v = 0; v < W; ++v)
        acc[s][v] = v4f{fmaf(weight, d2[0][s][v], bias.x), fmaf(weight, d2[1][s][v], bias.y),
                        fmaf(weight, d2[2][s][v], bias.z), fmaf(weight, d2[3][s][v], bias.w)};
    if constexpr (CI > 0) {
      const float* wl = WL + T * (CI * 4) + (lane & 3);
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s == 0 || both)
#pragma unroll
          for (int i = 0; i < CI; ++i) {
            const float wv = wl[4 * i];
#pragma unroll
            for (int v = 0; v < W; ++v)
              acc[s][v] = __builtin_amdgcn_mfma_f32_4x4x1f32(wv, u[i][s][v], acc[s][v], 0, 0, 0);
          }
    }
    // the next task's table and u are on their way while this one's last channels are finished
    if (T + 1 == f.ct && task_next < f.ntask)
        fold_inv_ask<NS, W, CI, STREAM>(f, ztab, fold_inv_place<NS, W>(f, task_next, active), ZT, up, ep.Cu, u);
    const long long base = first + o * f.Npts;
    auto store4 = [&](float* dst) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        // the column of one channel; nothing for a channel past the last
        const __amdgpu_buffer_rsrc_t r = buffer_of(dst + base + w * f.Npts, o + w < f.Co ? f.Nz * f.Nt * 4 : 0);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          float y[W];
#pragma unroll
          for (int v = 0; v < W; ++v) y[v] = acc[s][v][w];
          buffer_store<W, STREAM>(r, q.at[s], y);
        }
      }
    };
    if (ep.zsave != nullptr) store4(ep.zsave);
    if (ep.act) {
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s == 0 || both)
#pragma unroll
          for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int v = 0; v < W; ++v) acc[s][v][w] = gelu_fast_f(acc[s][v][w]);
    }
    store4(out);
  }
}

// waves per SIMD: u, the two accumulator sets and about 50 registers of operands and addresses
constexpr int fold_inv_waves(int W, int CI) {
  const int ns = fold_inv_ns(W, CI), regs = ns * W * CI + ns * 16 + ns * W * 4 + 50;
  return regs <= 128 ? 4 : (regs <= 168 ? 3 : 2);
}

template <int W, int CI, bool STREAM>
__global__ __launch_bounds__(kThreads, fold_inv_waves(W, CI)) void zt_inv_fold_kernel(
    const float2* __restrict__ a, float* __restrict__ out, const float2* __restrict__ twt,
    const float* __restrict__ ztab, FoldInv f, EpiArgs ep) {
  HIP_DYNAMIC_SHARED(float4, smem4)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long long item = xcd_contiguous_item(blockIdx.x, gridDim.x);      // grid: a multiple of 8
  if (item >= (long long)f.items) return;
  // the blocks of one column follow each other on one XCD, whose L2 serves their second read of u
  const long long group = item / f.nchunk;
  const int chunk = (int)(item - group * f.nchunk);
  const int o0 = chunk * f.ct * 4;
  const int wc = 1 << f.wc_shift, cb = 4 >> f.wc_shift;
  const int cl = wave >> f.wc_shift, wl = wave & (wc - 1);
  const bool active = group * cb + cl < f.ncols;
  const long long col = min(group * cb + cl, f.ncols - 1);

  const int eo_col = f.ct * f.R * f.K1 * 16;                     // float2 per column
  float2* EO = reinterpret_cast<float2*>(smem4);                 // [cb][ct][R][K1][16]
  float* ZT = reinterpret_cast<float*>(EO + cb * eo_col);        // [4][ks][2][64]
  float* TB = ZT + 4 * f.ks * 128;                               // [tt][R][64]
  float* BL = TB + f.tt * f.R * 64;                              // [ct][4]
  float* WL = BL + 4 * f.ct;                                     // [ct][CI][4]
  EO += cl * eo_col;
  ZT += wave * f.ks * 128;

  constexpr int NS = fold_inv_ns(W, CI);
  const long long b = col / f.NxNy, xy = col - b * f.NxNy;
  const long long first = b * f.Co * f.Npts + xy * f.Nz * (long long)f.Nt;      // the column in channel 0 of out
  const char* up = CI > 0 ? reinterpret_cast<const char*>(ep.u + b * ep.Cu * f.Npts + xy * f.Nz * (long long)f.Nt) : nullptr;
  float u[CI > 0 ? CI : 1][NS][W];
  // Tables for the whole block: asked for first, kept in LDS while the spectrum below is on its way.  Entry (tile, r,
  // lane) of the product over t is cs[t][4 r + lane / 16] at the t of tile row lane % 16.
  {
    const int ntb = f.tt * f.R * 64, nwl = CI > 0 ? f.ct * CI * 4 : 0;
    auto entries = [&](int i0, auto count) {
      constexpr int TU = count.value;
      float2 w[TU];
      float wv[TU];
      int kind[TU];                              // of the entry: 0 zero, 1 cos, 2 sin
#pragma unroll
      for (int j = 0; j < TU; ++j) {
        const int i = min(i0 + j * kThreads, ntb - 1), l = i & 63, q = i >> 6;
        const int ti = q / f.R, r = q - ti * f.R;
        const int m = l & 15, cc = 4 * r + (l >> 4), kt = (cc + 1) >> 1;
        const int t = min(W * (4 * ti + (m >> 2)), f.Nt - W) + (m & 3);
        kind[j] = cc < 2 * f.mt - 1 && (m & 3) < W ? ((cc & 1) || cc == 0 ? 1 : 2) : 0;
        w[j] = twt[kind[j] ? kt * f.Nt + t : 0];
        wv[j] = 0.f;
        if constexpr (CI > 0) {
          const int e = min(i0 + j * kThreads, nwl - 1);
          const int T = e / (4 * CI), ii = (e >> 2) - T * CI, o = o0 + 4 * T + (e & 3);
          const bool in = ii < ep.Cu && o < f.Co;
          const float v = ep.W[in ? o * ep.w_so + ii * ep.w_si : 0];
          wv[j] = in ? v : 0.f;
        }
      }
#pragma unroll
      for (int j = 0; j < TU; ++j) {
        const int i = i0 + j * kThreads;
        if (i < ntb) TB[i] = kind[j] == 0 ? 0.f : (kind[j] == 1 ? w[j].x : w[j].y);
        if (CI > 0 && i < nwl) WL[i] = wv[j];
      }
    };
    int i0 = tid;                                // four at a time, one where no more are left
    for (; i0 - tid + kThreads < max(ntb, nwl); i0 += 4 * kThreads) entries(i0, std::integral_constant<int, 4>{});
    if (i0 - tid < max(ntb, nwl)) entries(i0, std::integral_constant<int, 1>{});
    for (int i = tid; i < 4 * f.ct; i += kThreads) BL[i] = (ep.bias != nullptr && o0 + i < f.Co) ? ep.bias[o0 + i] : 0.f;
  }
  // E and O of this wave's channels of its column; a lane takes one (k, kt), both parts, four channels a round, and
  // asks for up to four rounds at a time, no more than there are: small spectra have one, and reading it four times over
  // showed (one channel, 6512 columns of 10 x 10, 3 kept, 5 bins: 15.9 us, 19.7 with four always here and above, 16.5 one
  // after the other).
  // Columns of the tile past the 2 mt - 1 real ones, and channels past the last, are zeros.
  if (wl < f.ct) {
    const float2* src = a + ((b * f.Co + o0) * f.NxNy + xy) * (long long)(f.Lz * f.mt);
    const long long ostride = (long long)f.NxNy * f.Lz * f.mt;
    const double2* rot = reinterpret_cast<const double2*>(ztab + (long long)2 * f.mrows * f.stride);
    const int R1 = f.K1 * 16, real = 2 * f.mt - 1, n = f.K1 * f.mt;
    constexpr int UB = 4;
    // lanes past the end repeat the last entry
    auto index = [&](int i0, int& k, int& kt, bool& has_p, bool& has_q) {
      const int idx = min(i0 + lane, n - 1);
      k = f.mt > 1 ? (int)__umulhi((unsigned)idx, f.inv_mt) : idx;
      kt = idx - k * f.mt;
      has_p = k < f.npos;
      has_q = k >= 1 && k <= f.Lz - f.npos;
      return idx;
    };
    auto advance = [&](int& i0, int& T) {
      T += wc;
      if (T >= f.ct) { T = wl; i0 += 64; }
    };
    int la = 0, lT = wl, pa = 0, pT = wl;
    auto rounds = [&](auto count) {
      constexpr int NB = count.value;
      float2 p[NB][UB], q[NB][UB];
      double2 w[NB];
#pragma unroll
      for (int r = 0; r < NB; ++r) {             // rounds past the last: the last entry again
        int k, kt;
        bool has_p, has_q;
        const int idx = index(la, k, kt, has_p, has_q);
        const int off_p = has_p ? idx : 0, off_q = has_q ? (f.Lz - k) * f.mt + kt : 0;
        w[r] = rot[k];
#pragma unroll
        for (int h = 0; h < UB; ++h) {
          const float2* so = src + min(4 * lT + h, f.Co - 1 - o0) * ostride;
          p[r][h] = so[off_p];
          q[r][h] = so[off_q];
        }
        advance(la, lT);
      }
#pragma unroll
      for (int r = 0; r < NB; ++r) {
        if (pa >= n) break;
        int k, kt;
        bool has_p, has_q;
        index(pa, k, kt, has_p, has_q);
        // bin 0 has no imaginary part: its place takes the first padding column
        const int c_re = kt == 0 ? 0 : 2 * kt - 1, c_im = kt == 0 ? real : 2 * kt;
        float2* d = EO + pT * f.R * R1;
        float2* d_re = d + (c_re >> 2) * R1 + 16 * k + 4 * (c_re & 3);
        float2* d_im = d + (c_im >> 2) * R1 + 16 * k + 4 * (c_im & 3);
#pragma unroll
        for (int h = 0; h < UB; ++h) {
          const bool in = o0 + 4 * pT + h < f.Co, ip = in && has_p, iq = in && has_q;
          // folded and turned in double: one rounding each
          const double px = ip ? p[r][h].x : 0.f, py = ip ? p[r][h].y : 0.f;
          const double qx = iq ? q[r][h].x : 0.f, qy = iq ? q[r][h].y : 0.f;
          const double sx = px + qx, dx = px - qx, sy = py + qy, dy = py - qy;
          float2 im = make_float2((float)fma(-w[r].y, dx, w[r].x * sy), (float)fma(w[r].y, sy, w[r].x * dx));
          if (kt == 0) im = make_float2(0.f, 0.f);
          d_re[h] = make_float2((float)fma(w[r].y, dy, w[r].x * sx), (float)fma(w[r].y, sx, -w[r].x * dy));
          d_im[h] = im;
          if (4 * f.R > real + 1 && kt == 0) {   // two more padding columns
            d[h + (f.R - 1) * R1 + 16 * k + 8] = make_float2(0.f, 0.f);
            d[h + (f.R - 1) * R1 + 16 * k + 12] = make_float2(0.f, 0.f);
          }
        }
        advance(pa, pT);
      }
    };
    int left = ((n + 63) >> 6) * ((f.ct - wl + wc - 1) >> f.wc_shift);
    for (; left >= 3; left -= 4) rounds(std::integral_constant<int, 4>{});
    if (left == 2) rounds(std::integral_constant<int, 2>{});
    else if (left == 1) rounds(std::integral_constant<int, 1>{});
  }
  // the first task's table and u are on their way over the barrier
  fold_inv_ask<NS, W, CI, STREAM>(f, ztab, fold_inv_place<NS, W>(f, min(wl, f.ntask - 1), active), ZT, up, ep.Cu, u);
  lds_barrier();
  // The number of memory instructions that a wait may leave open is the smallest over all ways to its place.  On the way
  // from the last task there are a group's stores after u; here, as many that store nothing.
  const __amdgpu_buffer_rsrc_t none = buffer_of(out, 0);
#pragma unroll
  for (int s = 0; s < 4 * NS; ++s) {
    __builtin_amdgcn_raw_buffer_store_b32(0u, none, 4 * s, 0, 0);
    asm volatile("" ::: "memory");                         // all of them: two alike would be one
  }

  const float4* BL4 = reinterpret_cast<const float4*>(BL);
  for (int task = wl; task < f.ntask; task += wc) {
    wait_vm<fold_inv_asked<NS, CI>() + 4 * NS>();          // the table; u and a group's stores came after it
    fold_inv_tile<NS, W, CI, STREAM>(f, ep, out, ztab, EO, ZT, TB, WL, BL4, first, o0,
                                     fold_inv_place<NS, W>(f, task, active), u, up, task + wc, active);
  }
}

int fold_inv_bucket(int Cu) { return Cu <= 0 ? 0 : (Cu <= 8 ? 8 : (Cu <= 20 ? (Cu + 3) / 4 * 4 : (Cu <= 24 ? 24 : 32))); }
int fold_inv_run(int Nt, int tt) { return (Nt + 4 * tt - 1) / (4 * tt); }      // points of t per lane

// everything but the number of columns, which only has a say in how many waves share one (0: any); false where no split
// fits the LDS
bool fold_inv_geometry(AxisPlan az, int Nt, int mt, int Co, int Cu, int64_t ncols, FoldInv* out, size_t* lds) {
  if (Co > kMaxCo || Cu > 32 || (int64_t)az.N * Nt > (1 << 28) || !tz_fwd_fold_fits(az, Nt, mt)) return false;
  const FoldPlan fp = fold_plan(az);
  FoldInv f{};
  f.Co = Co; f.Nz = az.N; f.Nt = Nt; f.Lz = az.L; f.npos = az.npos; f.mt = mt;
  f.K1 = 1 + (az.npos - 1 > az.L - az.npos ? az.npos - 1 : az.L - az.npos);
  f.ks = (f.K1 + 3) / 4;
  f.R = (2 * mt - 1 + 3) / 4;
  f.pairs = fp.pairs; f.stride = fp.stride; f.mrows = fp.rows;
  f.ntile = (f.pairs + 15) / 16;
  f.tt = (Nt + 15) / 16;
  const int W = fold_inv_run(Nt, f.tt), CI = fold_inv_bucket(Cu);
  f.inv_mt = mt > 1 ? (unsigned)((0x100000000ull + mt - 1) / mt) : 0;
  f.half_last = f.pairs - 16 * (f.ntile - 1) <= 8;
  // Two tiles of t: one task takes whole rows, so that the lines of memory that the tiles share are read once and written
  // whole.
  f.two_t = fold_inv_ns(W, CI) == 2 && f.tt == 2;
  f.ntask = (f.ntile + (fold_inv_ns(W, CI) == 1 || f.two_t ? f.ntile - f.half_last : 0)) * (f.two_t ? 1 : f.tt);
  const int CT = (Co + 3) / 4;
  // Waves per column: two tasks each, so that the second one's u values load under the first (64 x 20, one block
  // forward and back: 0.71 ms with one task per wave, 0.68 with two); more waves when the columns of a block then
  // fit the LDS share of its resident waves; then fewer output channels per block.  A short last tile over both tiles of t
  // counts as two (us, 20 channels with the linear term, 220 columns of 40 x 18: its three tasks on one wave 58, on two 41;
  // up to 2400 columns of 33 to 48 points of z 3 to 19 % faster on two, from 2500 on 1 % slower), but not where three tasks on
  // one wave a column fill the chip once and twice the waves would come to little less than two rounds (us on one and on two,
  // 16 channels, 40 x 20: 1280 columns 66 and 63, 1664 67 and 77, 2000 75 and 81, 2208 past one round 108 and 101).
  const auto share = [](int tasks) { return tasks >= 8 ? 2 : (tasks >= 4 ? 1 : 0); };
  const int64_t room = (int64_t)256 * 4 * fold_inv_waves(W, CI);
  const bool once = f.ntask == 3 && ncols <= room && 4 * ncols > 3 * room;
  const int wc0 = share(f.ntask + (f.two_t && !once ? f.half_last : 0));
  for (int nchunk = 1; nchunk <= CT; ++nchunk) {
    f.ct = (CT + nchunk - 1) / nchunk;
    f.nchunk = (CT + f.ct - 1) / f.ct;
    for (const size_t cap : {(size_t)160 * 1024 / fold_inv_waves(W, CI), (size_t)80 * 1024})
      for (f.wc_shift = wc0; f.wc_shift <= 2; ++f.wc_shift) {
        const size_t fl = (size_t)(4 >> f.wc_shift) * f.ct * f.R * f.K1 * 32 + (size_t)4 * f.ks * 128 +
                          (size_t)f.tt * f.R * 64 + 4 * f.ct + (size_t)f.ct * CI * 4;
        if (fl * 4 > cap) continue;
        *out = f;
        *lds = fl * 4;
        return true;
      }
  }
  return false;
}

}  // namespace

bool zt_inv_fold_fits(AxisPlan az, int Nt, int mt, int Co, int Cu) {
  FoldInv f;
  size_t lds;
  return fold_inv_geometry(az, Nt, mt, Co, Cu, 0, &f, &lds);
}

FoldInvLoad zt_inv_fold_load(AxisPlan az, int Nt, int mt, int Co, int Cu) {
  FoldInv f;
  size_t lds;
  if (!fold_inv_geometry(az, Nt, mt, Co, Cu, 0, &f, &lds)) return {0, 0};
  const int waves = fold_inv_waves(fold_inv_run(Nt, f.tt), fold_inv_bucket(Cu)), room = (int)((size_t)160 * 1024 / lds);
  // A block's short last tile over both tiles of t counts as two tasks, which it is with u for both.  us, 4096 columns of 16 x
  // 24, 24 channels with the linear term, 5 kept, 12 bins: per tile 235, folded 167; 16 x 22, 12 channels, 8 kept, 11 bins
  // 115 and 79; but convolutions, 20 channels, 16 x 22, 9 and 11 bins, 79 and 84 per tile, 108 and 123 folded.
  const int wc = 1 << f.wc_shift, tasks = f.ntask + (f.two_t && Cu > 0 ? f.half_last : 0);
  return {(room < waves ? room : waves) * (4 / wc) * (tasks < wc ? tasks : wc),
          (2 * mt + 2) / 4 * (2 * f.ks + 8) * f.nchunk};
}

hipError_t launch_zt_inv_fold(const float2* a, float* out, const float2* twt, const float* ztab, int64_t ncols, int Co,
                              int NxNy, AxisPlan az, int Nt, int mt, EpiArgs e, hipStream_t s) {
  FoldInv f{};
  size_t lds = 0;
  const int Cu = e.u != nullptr ? e.Cu : 0;
  if (!fold_inv_geometry(az, Nt, mt, Co, Cu, ncols, &f, &lds)) return hipErrorInvalidValue;
  f.ncols = ncols; f.NxNy = NxNy; f.Npts = (int64_t)NxNy * az.N * Nt;
  const int W = fold_inv_run(Nt, f.tt), CI = fold_inv_bucket(Cu);
  const int cb = 4 >> f.wc_shift;
  const int64_t items = (ncols + cb - 1) / cb * f.nchunk;
  const int64_t nblk = (items + 7) / 8 * 8;
  if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
  f.items = (unsigned)items;
  // Whole rows per tile: its 16 rows are one run of memory, and streams pay as everywhere (263 x 16: 6.9 -> 6.7 ms
  // over four blocks).  Rows in two tiles of t are whole lines together but not by the instruction, which plain stores
  // let the L2 complete (64 x 30, four blocks forward and back: 3.0 ms streamed, 2.2 ms plain), parts of rows even more.
  const bool stream = f.tt == 1 && ncols * (int64_t)Co * az.N * Nt * 4 >= kStreamBytes;
#define FNO_ZF_S(WV, CIV, STRV)                                                                                      \
  hipLaunchKernelGGL((zt_inv_fold_kernel<WV, CIV, STRV>), dim3((unsigned)nblk), dim3(kThreads), lds, s, a, out, twt, \
                     ztab, f, e)
#define FNO_ZF_C(WV, CIV) do { if (stream) FNO_ZF_S(WV, CIV, true); else FNO_ZF_S(WV, CIV, false); } while (0)
#define FNO_ZF_W(WV)                                                              \
  switch (CI) {                                                                   \
    case 0: FNO_ZF_C(WV, 0); break;                                               \
    case 8: FNO_ZF_C(WV, 8); break;                                               \
    case 12: FNO_ZF_C(WV, 12); break;                                             \
    case 16: FNO_ZF_C(WV, 16); break;                                             \
    case 20: FNO_ZF_C(WV, 20); break;                                             \
    case 24: FNO_ZF_C(WV, 24); break;                                             \
    default: FNO_ZF_C(WV, 32); break;                                             \
  }
  if (W == 1) FNO_ZF_W(1) else if (W == 2) FNO_ZF_W(2) else if (W == 3) FNO_ZF_W(3) else FNO_ZF_W(4)
#undef FNO_ZF_W
#undef FNO_ZF_C
#undef FNO_ZF_S
  return hipGetLastError();
}

}  // namespace fno
