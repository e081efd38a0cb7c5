// Kernels of libfno for gfx950 that act point by point over the grid (arXiv 2204.01205): the
// activation/loss gradient with the sum-reductions that are the adjoint of broadcasting W and b
// (Sec. 2.1), the channel lift and the projection of Sec. 2.4 with their adjoints, the time lift
// (eqs. (8)-(9)) with its adjoint, the relative L2 misfit and the Adam update of Sec. 4.
#include "fno_device.h"

namespace fno {

namespace {

// ------------------------------------------------------------------------------------------
// Backward pointwise: gz = g * act'(z); partial sums for gb and gW
// ------------------------------------------------------------------------------------------
// Widths that are a multiple of 4 (up to 20) and N a multiple of 64, streaming
// and without LDS: lane (blk, j) of a wave owns channels j, 4+j, ... at the four consecutive
// points 4*blk .. 4*blk+3 of a 64-point step, so every z / g / x access is a float4 and gz is
// computed exactly once per element.  gW[o][i] = sum_p gz[o][p] x[i][p] is a dense contraction
// over points and runs on the matrix cores: v_mfma_f32_4x4x1 block blk adds the outer product
// gz[4To..4To+3][p] x[4Ti..4Ti+3][p] of its point p to its own 4x4 partial tile; the 16 blocks,
// the waves and the thread blocks are summed at the end (per-wave partials in double, fixed order).
// GELU and its slope: with a = |z| and t = 1 / (1 + 0.4 a) the upper tail is exp(-a^2 / 2) t P(t), the form of Abramowitz &
// Stegun 7.1.26, whose exponential is the density up to a constant.  P has degree 5 (7.1.26: 4) and is fitted over [0, 13]
// to 3.5e-8 of max(a, 1) T(a) and to 1.7e-3 of the tail T itself, whichever is less, so that units that are all but off
// keep their slope.  Against float64, of the norm, with 7.1.26 in brackets: under N(0, 1) 4.8e-8 on z Phi(z) and 6.9e-8 on
// the slope (8.8e-8, 1.1e-7), at z = -5 7e-6 and 5e-7 (1.1e-3, 5e-5), at -9 5e-4 and 7e-6 (1.2e-2, 1.7e-4).  A polynomial
// for the tail's logarithm, fitted in absolute error, was off by 7e-3 and 3e-4 at -5, by more than the value at -9, and
// grew with |z| beyond 1e20.
__device__ __forceinline__ void gelu_and_grad_f(float z, float& val, float& grad) {
  const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(z), 0.4f, 1.0f));
  float q = fmaf(t, 5.5231631e-02f, -2.5018391e-01f);
  q = fmaf(t, q, 3.3274594e-01f);
  q = fmaf(t, q, 1.8495135e-02f);
  q = fmaf(t, q, 1.8670905e-01f);
  q = fmaf(t, q, 1.5700214e-01f);
  q *= t;
  const float e = __builtin_amdgcn_exp2f((z * z) * -0.72134752044f);    // exp(-z^2 / 2)
  const float tail = q * e;
  const float cdf = z < 0.f ? tail : 1.0f - tail;
  val = z * cdf;
  grad = fmaf(z, 0.39894228040143267794f * e, cdf);
}

// The same closer to float64 around zero: log2 of twice the tail is a q(a), q of degree 9 (largest
// error of max(a, 1) T(a) 1.9e-10; a q(a) falls from 0 to minus infinity), so that its rounding shrinks with a.  20
// instructions, where erff and expf took over 100 (both branches of erff run in a wave); against float64, of the norm under
// N(0, 1): the slope 3.9e-8, value times slope 6.6e-8 (erff and expf 4.0e-8 and 7.2e-8); at z = -5 the slope 2e-6 (5e-4).
__device__ __forceinline__ void gelu_and_grad_fine_f(float z, float& val, float& grad) {
  const float a = fabsf(z);
  float q = fmaf(a, -5.62642732e-08f, 1.38986923e-06f);
  q = fmaf(a, q, -1.52123248e-05f);
  q = fmaf(a, q, 9.45571737e-05f);
  q = fmaf(a, q, -3.24071734e-04f);
  q = fmaf(a, q, 6.31522853e-05f);
  q = fmaf(a, q, 6.89695915e-03f);
  q = fmaf(a, q, -5.24215102e-02f);
  q = fmaf(a, q, -4.59223896e-01f);
  q = fmaf(a, q, -1.15110409e+00f);
  const float t = __builtin_amdgcn_exp2f(a * q);
  const float pdf = __builtin_amdgcn_exp2f(fmaf(z * z, -0.72134752044f, -1.3257480647f));     // log2 of 1 / sqrt(2 pi)
  const float cdf = z < 0.f ? 0.5f * t : fmaf(-0.5f, t, 1.0f);
  val = z * cdf;
  grad = fmaf(z, pdf, cdf);
}

template <int CT, bool STREAM>
__global__ __launch_bounds__(kThreads) void bwd_pointwise_mfma_kernel(
    const float* __restrict__ z, const float* __restrict__ gout, const float* __restrict__ x,
    float* __restrict__ gz_out, double* __restrict__ part, int B, long long N, int act, int mse_target,
    float mse_scale) {
  constexpr int C = 4 * CT;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int j4 = lane & 3, blk = lane >> 2;
  v4f acc[CT][CT];
#pragma unroll
  for (int a = 0; a < CT; ++a)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[a][c] = v4f{0.f, 0.f, 0.f, 0.f};
  float gbacc[CT];
#pragma unroll
  for (int a = 0; a < CT; ++a) gbacc[a] = 0.f;

  const long long steps_per_b = N >> 6;
  const long long steps = steps_per_b * B;
  const long long wave_id = (long long)blockIdx.x * (kThreads / 64) + wave;
  // Thread blocks are dealt to the eight XCDs round robin (the grid is a multiple of 8 blocks): each
  // XCD walks a contiguous eighth of the steps, its waves interleaved inside it (1-6 % faster than
  // all waves interleaved over the whole range, measured on the same allocations)
  const long long per_x = (steps + 7) >> 3;
  const long long xs = (long long)(blockIdx.x & 7) * per_x;
  const long long xe = xs + per_x < steps ? xs + per_x : steps;
  const long long wl = (long long)(blockIdx.x >> 3) * (kThreads / 64) + wave;
  const long long nwl = (long long)(gridDim.x >> 3) * (kThreads / 64);
  for (long long s = xs + wl; s < xe; s += nwl) {
    const long long bb = s / steps_per_b;
    const long long p0 = (s - bb * steps_per_b) * 64 + 4 * blk;
    float4 gzv[CT], xv[CT];
#pragma unroll
    for (int T = 0; T < CT; ++T) {
      const long long e = (bb * C + 4 * T + j4) * N + p0;
      const v4f zq = ld_once<STREAM>(reinterpret_cast<const v4f*>(z + e));
      const v4f gq = ld_once<STREAM>(reinterpret_cast<const v4f*>(gout + e));
      const v4f xq = ld_once<STREAM>(reinterpret_cast<const v4f*>(x + e));
      const float4 zv = make_float4(zq[0], zq[1], zq[2], zq[3]);
      float4 g = make_float4(gq[0], gq[1], gq[2], gq[3]);
      xv[T] = make_float4(xq[0], xq[1], xq[2], xq[3]);
      if (act) {
        float v0, v1, v2, v3, d0, d1, d2, d3;
        gelu_and_grad_f(zv.x, v0, d0); gelu_and_grad_f(zv.y, v1, d1);
        gelu_and_grad_f(zv.z, v2, d2); gelu_and_grad_f(zv.w, v3, d3);
        if (mse_target) g = make_float4(mse_scale * (v0 - g.x), mse_scale * (v1 - g.y),
                                        mse_scale * (v2 - g.z), mse_scale * (v3 - g.w));
        g = make_float4(g.x * d0, g.y * d1, g.z * d2, g.w * d3);
      } else if (mse_target) {
        g = make_float4(mse_scale * (zv.x - g.x), mse_scale * (zv.y - g.y), mse_scale * (zv.z - g.z),
                        mse_scale * (zv.w - g.w));
      }
      st_once<STREAM>(reinterpret_cast<v4f*>(gz_out + e), v4f{g.x, g.y, g.z, g.w});
      gbacc[T] += (g.x + g.y) + (g.z + g.w);
      gzv[T] = g;
    }
#pragma unroll
    for (int a = 0; a < CT; ++a) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        acc[a][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(gzv[a].x, xv[c].x, acc[a][c], 0, 0, 0);
        acc[a][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(gzv[a].y, xv[c].y, acc[a][c], 0, 0, 0);
        acc[a][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(gzv[a].z, xv[c].z, acc[a][c], 0, 0, 0);
        acc[a][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(gzv[a].w, xv[c].w, acc[a][c], 0, 0, 0);
      }
    }
  }
  // sum the 16 blocks of the wave (lanes with equal j4), then lanes 0..3 write the wave's partial
  const int npairs = C * C + C;
  double* dst = part + wave_id * npairs;
#pragma unroll
  for (int a = 0; a < CT; ++a) {
#pragma unroll
    for (int c = 0; c < CT; ++c) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = acc[a][c][i];
        v += __shfl_xor(v, 4); v += __shfl_xor(v, 8); v += __shfl_xor(v, 16); v += __shfl_xor(v, 32);
        if (blk == 0) dst[(4 * a + i) * C + 4 * c + j4] = double(v);
      }
    }
    float gsum = gbacc[a];
    gsum += __shfl_xor(gsum, 4); gsum += __shfl_xor(gsum, 8); gsum += __shfl_xor(gsum, 16); gsum += __shfl_xor(gsum, 32);
    if (blk == 0) dst[C * C + 4 * a + j4] = double(gsum);
  }
}

// The same step for every other width up to 32, any point count and alignment, and c_in != c_out (the adjoint of the
// lift).  The kernel above keeps all of gW in a wave's accumulators, which 32 channels do not fit; here the output
// channels are dealt to `ngrp` waves of a block (OT tiles of 4 each).  Layout and products are those of the kernel above;
// rows need not be aligned (4-byte aligned 16-byte loads), points past the end of a batch entry and channels past the last
// count as zero.  The fp32 accumulators take kBwdChain steps (128 terms of a lane block) and then go to doubles, which are
// added over the wave's 16 lane blocks, half of them sent away at each level: every lane keeps a sixteenth.
//
// Where the waves of a step are two or four (NG), each reads its share of x and leaves it in LDS, double buffered, one
// barrier a step; that takes half to three quarters of a step's loads off every wave, and the registers they took hold
// the next step's, asked for a step ahead.  (With all of x in every wave there is no room for that: 0.45 ms in the first
// case below, with spills.)  What bounds it: memory at 32 channels, 4.7 TB/s (0.21 ms at the 5.2 of a large copy).  At
// 2.16 M points with GELU and a target, us: 32, 27, 25, 24, 22, 17 channels 236, 215, 200, 181, 166, 139; with a ragged
// step, a last step and channels past the last on ways of their own, where the loads of the next step were waited for as
// they were sent, 268, 253, 245, 184, 172, 144.  (Below 16 MB a tensor and without activation, with one or two turns a
// wave, 25 channels and more are 1 us slower than so, of 10 to 20.)  9 and 10 (one wave a step) 88, 91; 5 -> 20 at 33.5 M
// points, no activation, 655 (754 where values of z that are not needed were set to zero one by one, which waited for the
// loads between them).
constexpr int kBwdChain = 32;

template <bool STREAM>
__device__ __forceinline__ v4f load4(const float* p) {
  float v[4];
  load_run<4, STREAM>(p, v);
  return v4f{v[0], v[1], v[2], v[3]};
}

// one level of the sum over lane blocks, in double: N values per lane to N / 2 (an odd N: all are added, both lanes keep
// them)
template <int N, class T>
__device__ __forceinline__ void fold_level(const T* v, double* out, bool upper, int mask) {
  if constexpr (N % 2 == 0) {
#pragma unroll
    for (int q = 0; q < N / 2; ++q) {
      const T keep = upper ? v[q + N / 2] : v[q], send = upper ? v[q] : v[q + N / 2];
      out[q] = (double)keep + (double)__shfl_xor(send, mask);
    }
  } else {
#pragma unroll
    for (int q = 0; q < N; ++q) out[q] = (double)v[q] + (double)__shfl_xor(v[q], mask);
  }
}
constexpr int fold_count(int n) { return n % 2 == 0 ? n / 2 : n; }

// NG: waves that share x through LDS, or 0, where every wave reads all of it.
constexpr int kBwdXS = 80;               // row stride of staged x: 16 banks, so that four channels by four points spread over all
template <int OT, int IT, int NG, bool STREAM>
__global__ __launch_bounds__(kThreads, 2) void bwd_pointwise_wide_kernel(
    const float* __restrict__ z, const float* __restrict__ gout, const float* __restrict__ x,
    float* __restrict__ gz_out, double* __restrict__ part, int B, int Ci, int Co, long long N, int act,
    int mse_target, float mse_scale, int ngrp) {
  constexpr int R0 = 4 * OT * IT, R1 = fold_count(R0), R2 = fold_count(R1), R3 = fold_count(R2), R4 = fold_count(R3);
  // scalar where buffer loads need it; alone it costs: with scalar branches the loads of a step (5 -> 20 channels) wait for
  // one another, 662 -> 702 us
  const int tid = threadIdx.x, wave = NG > 0 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int lane = tid & 63;
  const int j4 = lane & 3, blk = lane >> 2;
  const int per_block = (kThreads / 64) / ngrp;            // point ranges per block
  const int o0 = (wave % ngrp) * 4 * OT;
  const bool need_z = act || mse_target;
  long long orow[OT], irow[NG > 0 ? IT / NG : IT];
  bool olive[OT], ilive[NG > 0 ? IT / NG : IT];
#pragma unroll
  for (int T = 0; T < OT; ++T) {
    const int o = o0 + 4 * T + j4;
    olive[T] = o < Co;
    orow[T] = (long long)(olive[T] ? o : Co - 1) * N;
  }
#pragma unroll
  for (int T = 0; T < (NG > 0 ? IT / NG : IT); ++T) {
    const int i = 4 * (NG > 0 ? wave % NG * (IT / NG) + T : T) + j4;
    ilive[T] = i < Ci;
    irow[T] = (long long)(ilive[T] ? i : Ci - 1) * N;
  }
  v4f acc[OT][IT];
  float gbacc[OT];
  double sum[R4], gbsum[OT];
#pragma unroll
  for (int q = 0; q < R4; ++q) sum[q] = 0.0;
#pragma unroll
  for (int a = 0; a < OT; ++a) {
    gbacc[a] = 0.f;
    gbsum[a] = 0.0;
#pragma unroll
    for (int c = 0; c < IT; ++c) acc[a][c] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  auto flush = [&]() {
    float v[R0];
#pragma unroll
    for (int a = 0; a < OT; ++a) {
      gbsum[a] += (double)gbacc[a];
      gbacc[a] = 0.f;
#pragma unroll
      for (int c = 0; c < IT; ++c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[(a * IT + c) * 4 + i] = acc[a][c][i];
        acc[a][c] = v4f{0.f, 0.f, 0.f, 0.f};
      }
    }
    double w[R1];
    fold_level<R0>(v, w, blk & 1, 4);
    fold_level<R1>(w, w, blk & 2, 8);
    fold_level<R2>(w, w, blk & 4, 16);
    fold_level<R3>(w, w, blk & 8, 32);
#pragma unroll
    for (int q = 0; q < R4; ++q) sum[q] += w[q];
  };

  const long long steps_per_b = (N + 63) >> 6;
  const long long steps = steps_per_b * B;
  // as above: each XCD walks a contiguous eighth of the steps
  const long long per_x = (steps + 7) >> 3;
  const long long xs = (long long)(blockIdx.x & 7) * per_x;
  const long long xe = xs + per_x < steps ? xs + per_x : steps;
  const long long wl = (long long)(blockIdx.x >> 3) * per_block + wave / ngrp;
  const long long nwl = (long long)(gridDim.x >> 3) * per_block;
  constexpr int XT = NG > 0 ? IT / NG : IT;      // tiles of x that a wave reads
  constexpr int XS = 4 * IT * kBwdXS;
  __shared__ float XL[NG > 0 ? 2 * (kThreads / 64 / NG) * XS : 1];       // [parity][point range][4 IT][kBwdXS]
  const int member = NG > 0 ? wave % NG : 0;
  float* own = XL + (NG > 0 ? wave / NG * XS : 0);
  // the values of step s, whole or ragged
  auto fetch = [&](long long s, long long& ob, long long& p0, v4f (&zn)[OT], v4f (&gn)[OT], v4f (&xn)[XT]) {
    const long long bb = s / steps_per_b;
    p0 = (s - bb * steps_per_b) * 64;
    ob = bb * Co * N;
    const long long p = p0 + 4 * blk, ib = bb * Ci * N;
    const bool whole = p0 + 64 <= N;                       // the same for the whole wave
    if (whole) {
      if (need_z)                                          // else z is nowhere used: zeros here would wait for other loads
#pragma unroll
        for (int T = 0; T < OT; ++T) zn[T] = load4<STREAM>(z + ob + orow[T] + p);
#pragma unroll
      for (int T = 0; T < OT; ++T) gn[T] = load4<STREAM>(gout + ob + orow[T] + p);
#pragma unroll
      for (int T = 0; T < XT; ++T) xn[T] = load4<STREAM && (NG > 0)>(x + ib + irow[T] + p);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const long long pu = p + u < N ? p + u : N - 1;
#pragma unroll
        for (int T = 0; T < OT; ++T) {
          if (need_z) zn[T][u] = z[ob + orow[T] + pu];
          gn[T][u] = gout[ob + orow[T] + pu];
        }
#pragma unroll
        for (int T = 0; T < XT; ++T) xn[T][u] = p + u < N ? x[ib + irow[T] + pu] : 0.f;
      }
    }
    return whole;
  };
  // the cotangent of the pre-activation, in gq's place
  auto cotangent_of = [&](const v4f (&zq)[OT], v4f (&gq)[OT]) {
    if (act) {
#pragma unroll
      for (int T = 0; T < OT; ++T)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float val, slope;
          gelu_and_grad_fine_f(zq[T][u], val, slope);
          if (mse_target) gq[T][u] = mse_scale * (val - gq[T][u]);
          gq[T][u] *= slope;
        }
    } else if (mse_target) {
#pragma unroll
      for (int T = 0; T < OT; ++T)
#pragma unroll
        for (int u = 0; u < 4; ++u) gq[T][u] = mse_scale * (zq[T][u] - gq[T][u]);
    }
  };
  // and stored
  auto cotangent = [&](long long ob, long long p0, bool whole, const v4f (&zq)[OT], v4f (&gq)[OT]) {
    const long long p = p0 + 4 * blk;
    cotangent_of(zq, gq);
#pragma unroll
    for (int T = 0; T < OT; ++T) {
      v4f g = gq[T];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (!olive[T] || (!whole && p + u >= N)) g[u] = 0.f;
      if (gz_out != nullptr && olive[T]) {
        float* dst = gz_out + ob + orow[T] + p;
        if (whole) {
          const float gs[4] = {g[0], g[1], g[2], g[3]};
          store_run<4, STREAM>(dst, gs);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (p + u < N) dst[u] = g[u];
        }
      }
      gbacc[T] += (g[0] + g[1]) + (g[2] + g[3]);
      gq[T] = g;
    }
  };
  // gq against XN tiles of x from c0 on
  auto products = [&](const v4f (&gq)[OT], const auto& xv, auto c0) {
    constexpr int XN = sizeof(xv) / sizeof(v4f);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int a = 0; a < OT; ++a)
#pragma unroll
        for (int c = 0; c < XN; ++c)
          acc[a][c0.value + c] = __builtin_amdgcn_mfma_f32_4x4x1f32(gq[a][u], xv[c][u], acc[a][c0.value + c], 0, 0, 0);
  };
  // the waves of a block meet once their LDS accesses are done; what is on its way from and to memory stays so
  auto lds_meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  int chain = 0;
  using std::integral_constant;
  if constexpr (NG == 0) {
    for (long long s = xs + wl; s < xe; s += nwl) {
      long long ob, p0;
      v4f zq[OT], gq[OT], xq[XT];
      const bool whole = fetch(s, ob, p0, zq, gq, xq);
      cotangent(ob, p0, whole, zq, gq);
#pragma unroll
      for (int T = 0; T < XT; ++T)
        if (!ilive[T]) xq[T] = v4f{0.f, 0.f, 0.f, 0.f};
      products(gq, xq, integral_constant<int, 0>{});
      if (++chain == kBwdChain) { chain = 0; flush(); }
    }
  } else {
    // All waves of a block take as many turns; the values of a step are asked for a step ahead.  One way through a turn, with
    // as many loads and stores whatever the step: where a ragged step's loads, a last step without a next one or channels
    // past the last were ways of their own, the values met in copies that waited for them at once.  So of a step past the last
    // nothing is there to be read, a lane past the row's last four points takes those and shifts them when they are there,
    // and what is not to be stored has an offset past the end.  (N from 4 to 2^27: 32-bit offsets over four rows.)
    // The step that is asked for next, as entry and step in it.  Divisions are long chains: two of 64 bits a turn took 3 % of
    // the time with GELU at any size, two before the first turn 1.5 % of 10 us.  (Counts of steps fit 32 bits: a step holds
    // four points at least, and more than 2^31 of these, at nine channels and more, no memory.)
    long long entry = (unsigned)(xs + wl) / (unsigned)steps_per_b, inside = xs + wl - entry * steps_per_b;
    const long long skip_entries = (unsigned)nwl / (unsigned)steps_per_b, skip = nwl - skip_entries * steps_per_b;
    const long long Nall = (long long)B * N;
    // rows first .. first + 3 of a tensor of C channels, from point p0 of an entry on: a base and the lane's offset
    auto tile_of = [&](const float* t, long long base, int C, int first, long long p0, bool there) {
      const int row = first < C ? first : C - 1;
      const long long at = base + row * N + p0, left = (Nall * C - at) * 4;
      return buffer_of(t + at, there ? (unsigned)(left < 0x7fffffffLL ? left : 0x7fffffffLL) : 0u);
    };
    auto offset_of = [&](int C, int first, int point) {
      const int row = first < C ? first : C - 1, mine = first + j4 < C ? first + j4 : C - 1;
      return ((unsigned)(mine - row) * (unsigned)N + (unsigned)point) * 4u;
    };
    auto four = [&](__amdgpu_buffer_rsrc_t r, unsigned at) {
      float q[4];
      buffer_load<4, STREAM>(r, at, q);
      return v4f{q[0], q[1], q[2], q[3]};
    };
    const int i0 = 4 * member * XT;
    v4f zn[OT], gn[OT], xn[XT];
    long long asked_ob, asked_p0;
    auto ask = [&](bool there) {
      const long long ob = entry * Co * N, ib = entry * Ci * N, p0 = inside * 64;
      const long long from = p0 > 0 ? p0 - 4 : 0;          // the last four points start at p0 - 3 at the earliest
      const int at = (int)(min(p0 + 4 * blk, N - 4) - from);
      if (need_z)
#pragma unroll
        for (int T = 0; T < OT; ++T) zn[T] = four(tile_of(z, ob, Co, o0 + 4 * T, from, there), offset_of(Co, o0 + 4 * T, at));
#pragma unroll
      for (int T = 0; T < OT; ++T) gn[T] = four(tile_of(gout, ob, Co, o0 + 4 * T, from, there), offset_of(Co, o0 + 4 * T, at));
#pragma unroll
      for (int T = 0; T < XT; ++T) xn[T] = four(tile_of(x, ib, Ci, i0 + 4 * T, from, there), offset_of(Ci, i0 + 4 * T, at));
      asked_ob = ob;
      asked_p0 = p0;
      entry += skip_entries;
      inside += skip;
      if (inside >= steps_per_b) { inside -= steps_per_b; ++entry; }
    };
    long long s = xs + wl;
    ask(s < xe);
    int turn = 0;
    for (long long s0 = xs + (long long)(blockIdx.x >> 3) * per_block; s0 < xe; s0 += nwl, s += nwl, turn ^= 1) {
      float* buf = own + turn * (kThreads / 64 / NG) * XS;
      const bool live = s < xe;
      const long long ob = asked_ob, p0 = asked_p0;
      const bool whole = p0 + 64 <= N;
      if (!whole) {
        // the lane's first point is `d` further on in what it read
        const int d = (int)(4 * blk - min((long long)(4 * blk), N - 4 - p0));
        auto shift = [&](v4f& v) {
          const v4f q = v;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float r = d == 0 ? q[u] : 0.f;
#pragma unroll
            for (int e = 1; u + e < 4; ++e) r = d == e ? q[u + e] : r;
            v[u] = r;
          }
        };
#pragma unroll
        for (int T = 0; T < OT; ++T) {
          if (need_z) shift(zn[T]);
          shift(gn[T]);
        }
#pragma unroll
        for (int T = 0; T < XT; ++T) shift(xn[T]);
      }
      v4f gq[OT];
#pragma unroll
      for (int T = 0; T < XT; ++T)
        *reinterpret_cast<v4f*>(buf + (4 * (member * XT + T) + j4) * kBwdXS + 4 * blk) = ilive[T] ? xn[T] : v4f{0.f, 0.f, 0.f, 0.f};
      // the slopes before the next step's values are asked for, which take the places of these
      cotangent_of(zn, gn);
#pragma unroll
      for (int T = 0; T < OT; ++T) {
        gq[T] = gn[T];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float v = gq[T][u];
          asm volatile("" : "+v"(v));
          gq[T][u] = v;
        }
      }
      ask(s + nwl < xe);
#pragma unroll
      for (int T = 0; T < OT; ++T) {
        const int row = o0 + 4 * T;
        const __amdgpu_buffer_rsrc_t r = tile_of(gz_out, ob, Co, row, p0, live && gz_out != nullptr && row < Co);
        const unsigned to = olive[T] ? offset_of(Co, row, 4 * blk) : kNowhere;
        if (whole) {
          const float gs[4] = {gq[T][0], gq[T][1], gq[T][2], gq[T][3]};
          buffer_store<4, STREAM>(r, to, gs);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float g1[1] = {gq[T][u]};
            buffer_store<1, false>(r, p0 + 4 * blk + u < N ? to + 4u * u : kNowhere, g1);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (!live || !olive[T] || p0 + 4 * blk + u >= N) gq[T][u] = 0.f;
        gbacc[T] += (gq[T][0] + gq[T][1]) + (gq[T][2] + gq[T][3]);
      }
      lds_meet();
      if (live) {
        constexpr int XN = IT == 6 ? 3 : IT;               // tiles of x in registers at a time: as many as leave no spills
        auto piece = [&](auto c0) {
          v4f xq[XN];
#pragma unroll
          for (int c = 0; c < XN; ++c)
            xq[c] = *reinterpret_cast<const v4f*>(buf + (4 * (c0.value + c) + j4) * kBwdXS + 4 * blk);
          products(gq, xq, c0);
        };
        piece(integral_constant<int, 0>{});
        if constexpr (XN < IT) piece(integral_constant<int, IT - XN>{});
        if (++chain == kBwdChain) { chain = 0; flush(); }
      }
    }
  }
  flush();
  // where this lane's sums stand in (tile row, tile column, row in the tile); lanes that share them write the same
  const int base = (R0 % 2 == 0 && (blk & 1) ? R0 / 2 : 0) + (R1 % 2 == 0 && (blk & 2) ? R1 / 2 : 0) +
                   (R2 % 2 == 0 && (blk & 4) ? R2 / 2 : 0) + (R3 % 2 == 0 && (blk & 8) ? R3 / 2 : 0);
  double* dst = part + ((long long)blockIdx.x * per_block + wave / ngrp) * (Co * Ci + Co);
#pragma unroll
  for (int q = 0; q < R4; ++q) {
    const int r = base + q, tile = r >> 2;
    const int o = o0 + 4 * (tile / IT) + (r & 3), i = 4 * (tile % IT) + j4;
    if (o < Co && i < Ci) dst[o * Ci + i] = sum[q];
  }
#pragma unroll
  for (int a = 0; a < OT; ++a) {
    double t = gbsum[a];
    t += __shfl_xor(t, 4); t += __shfl_xor(t, 8); t += __shfl_xor(t, 16); t += __shfl_xor(t, 32);
    if (blk == 0 && olive[a]) dst[Co * Ci + o0 + 4 * a + j4] = t;
  }
}

// Sum over the partial slots part[slot][q] in a fixed order (same bits on every run): kRedPairs sums per block, the
// slots dealt round-robin to kRedGroups threads per sum, whose sums are added in group order.  Returns the total in
// group 0.  What bounds it is the latency of a thread's chain of loads, so the chain is short: 4096 slots of 420 sums
// take 12 us (31 us with 64 sums and 16 groups per block), 512 slots of 2945 sums 8 us (126 us with one thread per sum).
constexpr int kRedPairs = 16, kRedGroups = 64;
__device__ __forceinline__ double sum_slots(const double* __restrict__ part, int nslots, int n, int q) {
  __shared__ double sums[kRedGroups][kRedPairs];
  const int c = threadIdx.x % kRedPairs, grp = threadIdx.x / kRedPairs;
  double s = 0.0;
  if (q < n) {
    const double* p = part + q;
    int slot = grp;
    for (; slot + 7 * kRedGroups < nslots; slot += 8 * kRedGroups) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(long long)(slot + u * kRedGroups) * n];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; slot < nslots; slot += kRedGroups) s += p[(long long)slot * n];
  }
  sums[grp][c] = s;
  __syncthreads();
  double t = 0.0;
  if (grp == 0)
#pragma unroll
    for (int g = 0; g < kRedGroups; ++g) t += sums[g][c];
  return t;
}

__global__ __launch_bounds__(kRedPairs * kRedGroups) void reduce_partials_kernel(
    const double* __restrict__ part, int nblk, int Co, int Ci, float* __restrict__ gW,
    float* __restrict__ gb, int accumulate) {
  const int q = blockIdx.x * kRedPairs + threadIdx.x % kRedPairs;
  const int npairs = Co * Ci + Co;
  const double t = sum_slots(part, nblk, npairs, q);
  if (threadIdx.x < kRedPairs && q < npairs) {
    // accumulate: the sums are added to what gW and gb hold (a step over several calls)
    if (q < Co * Ci) { if (gW != nullptr) gW[q] = float(accumulate ? t + double(gW[q]) : t); }
    else if (gb != nullptr) gb[q - Co * Ci] = float(accumulate ? t + double(gb[q - Co * Ci]) : t);
  }
}

// ------------------------------------------------------------------------------------------
// Pointwise lift and projection (Sec. 2.4)
// ------------------------------------------------------------------------------------------
template <int CO>
__global__ __launch_bounds__(kThreads) void pointwise_linear_kernel(
    int Ci, int Co, long long np, const float* __restrict__ x, const float* __restrict__ W,
    const float* __restrict__ bias, float* __restrict__ y) {
  const long long p = (long long)blockIdx.x * kThreads + threadIdx.x;
  const long long b = blockIdx.y;
  if (p >= np) return;
  float acc[CO];
#pragma unroll
  for (int o = 0; o < CO; ++o) acc[o] = (bias != nullptr && o < Co) ? bias[o] : 0.f;
  for (int i = 0; i < Ci; ++i) {
    const float xv = x[(b * Ci + i) * np + p];
#pragma unroll
    for (int o = 0; o < CO; ++o)
      if (o < Co) acc[o] = fmaf(W[o * Ci + i], xv, acc[o]);
  }
#pragma unroll
  for (int o = 0; o < CO; ++o)
    if (o < Co) y[(b * Co + o) * np + p] = acc[o];
}

// Four consecutive points per thread (16-byte loads and stores); the arithmetic of a point is
// the scalar kernel's, term by term.  For point counts that are multiples of 4 and 16-byte
// aligned tensors.
template <int CO>
__global__ __launch_bounds__(kThreads) void pointwise_linear_v4_kernel(
    int Ci, int Co, long long np4, const v4f* __restrict__ x, const float* __restrict__ W,
    const float* __restrict__ bias, v4f* __restrict__ y) {
  const long long p = (long long)blockIdx.x * kThreads + threadIdx.x;
  const long long b = blockIdx.y;
  if (p >= np4) return;
  v4f acc[CO];
#pragma unroll
  for (int o = 0; o < CO; ++o) {
    const float bo = (bias != nullptr && o < Co) ? bias[o] : 0.f;
    acc[o] = v4f{bo, bo, bo, bo};
  }
  for (int i = 0; i < Ci; ++i) {
    const v4f xv = __builtin_nontemporal_load(&x[(b * Ci + i) * np4 + p]);
#pragma unroll
    for (int o = 0; o < CO; ++o)
      if (o < Co) {
        const float w = W[o * Ci + i];
        acc[o].x = fmaf(w, xv.x, acc[o].x);
        acc[o].y = fmaf(w, xv.y, acc[o].y);
        acc[o].z = fmaf(w, xv.z, acc[o].z);
        acc[o].w = fmaf(w, xv.w, acc[o].w);
      }
  }
#pragma unroll
  for (int o = 0; o < CO; ++o)
    if (o < Co) y[(b * Co + o) * np4 + p] = acc[o];
}

// ------------------------------------------------------------------------------------------
// Adjoints of the lift and of the projection (what a whole-network backward needs around the
// blocks): sums over all points in a fixed order, per-block partials in double
// ------------------------------------------------------------------------------------------
__global__ void transpose_kernel(const float* __restrict__ w, float* __restrict__ wt, int rows, int cols) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < rows * cols) wt[(idx % cols) * rows + idx / cols] = w[idx];
}

// The totals over the slots go to four destinations by ranges of q (any of them may be null).
__global__ __launch_bounds__(kRedPairs * kRedGroups) void reduce_ranges_kernel(
    const double* __restrict__ part, int nblk, int n0, int n1, int n2, int n3, float* __restrict__ d0,
    float* __restrict__ d1, float* __restrict__ d2, float* __restrict__ d3) {
  const int q = blockIdx.x * kRedPairs + threadIdx.x % kRedPairs;
  const int npairs = n0 + n1 + n2 + n3;
  const double s = sum_slots(part, nblk, npairs, q);
  if (threadIdx.x >= kRedPairs || q >= npairs) return;
  if (q < n0) { if (d0 != nullptr) d0[q] = (float)s; }
  else if (q < n0 + n1) { if (d1 != nullptr) d1[q - n0] = (float)s; }
  else if (q < n0 + n1 + n2) { if (d2 != nullptr) d2[q - n0 - n1] = (float)s; }
  else if (d3 != nullptr) d3[q - n0 - n1 - n2] = (float)s;
}

// Adjoint of u = W2 gelu(W1 x + b1) + b2 per point.  One block: tiles of 256 points.  The hidden
// units are taken kMlpChunk at a time: every thread computes, for its point, h, a = gelu(h) and
// gh = (W2^T g) gelu'(h) of the chunk into LDS and adds W1^T gh to its gx; then the threads take
// one (row, row) pair each of the chunk's sums -- gW1[k][i] = sum gh_k x_i, gb1[k] = sum gh_k,
// gW2[o][k] = sum g_o a_k -- as a 256-term inner product in float, added to the block's double
// accumulator of that pair in LDS (one owner per pair: no atomics, fixed order).
constexpr int kMlpChunk = 8;
constexpr int kMlpBlocks = 512;     // blocks (= partial-sum slots) of the projection's backward
template <int CI>
__global__ __launch_bounds__(kThreads) void mlp2_bwd_kernel(
    int B, int Ci, int H, int Co, long long N, const float* __restrict__ x, const float* __restrict__ W1,
    const float* __restrict__ b1, const float* __restrict__ W2, const float* __restrict__ g,
    float* __restrict__ gx, double* __restrict__ part) {
  HIP_DYNAMIC_SHARED(float, smem)
  constexpr int sR = kThreads + 1;
  float* XS = smem;                          // [Ci][sR]
  float* GS = XS + Ci * sR;                  // [Co][sR]
  float* GH = GS + Co * sR;                  // [kMlpChunk][sR]
  float* AA = GH + kMlpChunk * sR;           // [kMlpChunk][sR]
  const int nsum = H * (Ci + 1) + Co * H + Co;       // gW1 | gb1 | gW2 | gb2
  int acc_off = (Ci + Co + 2 * kMlpChunk) * sR;
  acc_off += acc_off & 1;
  double* ACC = reinterpret_cast<double*>(smem + acc_off);   // [nsum]
  const int tid = threadIdx.x;
  for (int q = tid; q < nsum; q += kThreads) ACC[q] = 0.0;
  const long long tiles_per_b = (N + kThreads - 1) / kThreads;
  const long long ntiles = tiles_per_b * B;
  const int per_k = Ci + 1 + Co;             // sums per hidden unit
  for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const long long b = tile / tiles_per_b;
    const long long p = (tile % tiles_per_b) * kThreads + tid;
    const bool live = p < N;
    float xr[CI], gxr[CI], gr[4];
#pragma unroll
    for (int i = 0; i < CI; ++i) {
      xr[i] = (live && i < Ci) ? x[(b * Ci + i) * N + p] : 0.f;
      gxr[i] = 0.f;
      if (i < Ci) XS[i * sR + tid] = xr[i];
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      gr[o] = (live && o < Co) ? g[(b * Co + o) * N + p] : 0.f;
      if (o < Co) GS[o * sR + tid] = gr[o];
    }
    for (int k0 = 0; k0 < H; k0 += kMlpChunk) {
      __syncthreads();                         // the previous chunk's pair sums have read GH, AA
      for (int kk = 0; kk < kMlpChunk; ++kk) {
        const int k = k0 + kk;
        float ghv = 0.f, av = 0.f;
        if (k < H) {
          float h = b1 != nullptr ? b1[k] : 0.f;
#pragma unroll
          for (int i = 0; i < CI; ++i)
            if (i < Ci) h = fmaf(W1[k * Ci + i], xr[i], h);
          float t = 0.f;
#pragma unroll
          for (int o = 0; o < 4; ++o)
            if (o < Co) t = fmaf(W2[o * H + k], gr[o], t);
          av = gelu_f(h);
          ghv = t * gelu_prime_f(h);
#pragma unroll
          for (int i = 0; i < CI; ++i)
            if (i < Ci) gxr[i] = fmaf(W1[k * Ci + i], ghv, gxr[i]);
        }
        GH[kk * sR + tid] = ghv;
        AA[kk * sR + tid] = av;
      }
      __syncthreads();
      for (int q = tid; q < kMlpChunk * per_k; q += kThreads) {
        const int kk = q / per_k, r = q - kk * per_k;
        const int k = k0 + kk;
        if (k >= H) continue;
        const float* u = r <= Ci ? GH + kk * sR : GS + (r - Ci - 1) * sR;
        float sum = 0.f;
        int dst;
        if (r < Ci) {
          const float* w = XS + r * sR;
          for (int t = 0; t < kThreads; ++t) sum = fmaf(u[t], w[t], sum);
          dst = k * Ci + r;
        } else if (r == Ci) {
          for (int t = 0; t < kThreads; ++t) sum += u[t];
          dst = H * Ci + k;
        } else {
          const float* w = AA + kk * sR;
          for (int t = 0; t < kThreads; ++t) sum = fmaf(u[t], w[t], sum);
          dst = H * (Ci + 1) + (r - Ci - 1) * H + k;
        }
        ACC[dst] += (double)sum;
      }
    }
    // gb2[o] = sum g_o
    if (tid < Co) {
      const float* u = GS + tid * sR;
      float sum = 0.f;
      for (int t = 0; t < kThreads; ++t) sum += u[t];
      ACC[H * (Ci + 1) + Co * H + tid] += (double)sum;
    }
    if (gx != nullptr && live) {
#pragma unroll
      for (int i = 0; i < CI; ++i)
        if (i < Ci) gx[(b * Ci + i) * N + p] = gxr[i];
    }
    __syncthreads();                           // XS, GS are rewritten by the next tile
  }
  __syncthreads();
  for (int q = tid; q < nsum; q += kThreads) part[(long long)blockIdx.x * nsum + q] = ACC[q];
}

// ------------------------------------------------------------------------------------------
// The two-layer projection and its adjoint on the matrix cores
// ------------------------------------------------------------------------------------------
// Accumulators are 32 x 32: register v of lane l holds the element in row mfma_row(v, l/32), column l%32.
typedef float v16f __attribute__((ext_vector_type(16)));
__device__ __forceinline__ int mfma_row(int v, int half) { return 8 * (v >> 2) + 4 * half + (v & 3); }

// fp32 products on the bf16 matrix instructions: a float is the exact sum of three bf16 values (hi and mid rounded to nearest, lo what is left: 3 x 8 bits), and six of
// the nine products of two such sums, added up in fp32, leave out less than 2^-25 of the product: less than one fp32
// rounding.  v_mfma_f32_32x32x16_bf16 takes half the cycles of v_mfma_f32_32x32x2 for eight times the terms, so the six
// cost three eighths of the fp32 instruction, and unlike it they run beside the vector unit's work.
// Lane l supplies A[l%32][8 (l/32) + j] and B[8 (l/32) + j][l%32], j < 8; the accumulator is laid out as mfma_row says.
__device__ __forceinline__ v16f mfma_bf16(u32x4 a, u32x4 b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// the six products, the small ones first
constexpr int kSplitA[6] = {0, 2, 1, 0, 1, 0}, kSplitB[6] = {2, 0, 1, 1, 0, 0};

// u = W2 gelu(W1 x + b1) + b2.  A wave takes 32 points at a time through all hidden units, 32 of them per accumulator:
// its x values are loaded in operand order straight from memory (slot s of lane l is channel 2 s + l/32, the bias a
// channel of ones after the last), split once, and used against every group of hidden units, whose split weights the
// block keeps in LDS.  Waves meet nowhere after the weights are there.
//
// What bounds it: the vector unit, 13.5 instructions a hidden value (GELU 10, the product with W2 one, else loads and
// splits); it issues in all of the cycles, the products' matrix instructions in 39 % of them run beside it, and the chip
// holds 1.8 GHz.  20 -> 128 -> 1 at 4 million points 442 -> 312 us, off the measured rms error of the fp32 instruction
// (2.2e-7, 1.1e-7 now); against the scalar kernel, which took the hidden and channel widths that one did not fit,
// 20 -> 64 -> 1 862 -> 179 us, 32 -> 128 -> 1 at 2 million points 1352 -> 192 us.
template <int NS, int CO>
__global__ __launch_bounds__(kThreads, 4) void mlp2_fwd_split_kernel(
    int B, int Ci, int H, int Co, long long N, const float* __restrict__ x, const float* __restrict__ W1,
    const float* __restrict__ b1, const float* __restrict__ W2, const float* __restrict__ b2,
    float* __restrict__ y) {
  HIP_DYNAMIC_SHARED(float4, smem4)
  constexpr int KB = (NS + 7) / 8;
  constexpr int LOW = NS == 18 ? 32 : 2 * NS - 8;          // fewest channels that run with NS slots: those below are all there
  const int NH = (H + 31) / 32;
  u32x4* A = reinterpret_cast<u32x4*>(smem4);              // [NH][KB][3][64]
  float4* W2S = reinterpret_cast<float4*>(A + NH * KB * 3 * 64);     // [CO][NH][8]: hidden units in order
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, c = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int e = tid; e < NH * KB * 64; e += kThreads) {
    const int l = e & 63, g = e >> 6, kb = g % KB, k = (g / KB) * 32 + (l & 31);
    unsigned part[4][3];
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      float v[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int i = 2 * (8 * kb + j + q) + (l >> 5);
        v[q] = k < H ? (i < Ci ? W1[k * Ci + i] : (i == Ci && b1 != nullptr ? b1[k] : 0.f)) : 0.f;
      }
      bf16_split(v[0], v[1], part[j / 2]);
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) A[(g * 3 + p) * 64 + l] = u32x4{part[0][p], part[1][p], part[2][p], part[3][p]};
  }
  for (int e = tid; e < CO * NH * 32; e += kThreads) {
    const int o = e / (NH * 32), k = e - o * NH * 32;
    reinterpret_cast<float*>(W2S)[e] = (o < Co && k < H) ? W2[o * H + k] : 0.f;
  }
  __syncthreads();

  unsigned keep[NS], one[NS];                              // (v & keep) | one: what a slot past LOW holds
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = 2 * s + half;
    keep[s] = i < Ci ? ~0u : 0u;
    one[s] = i == Ci ? 0x3f800000u : 0u;
  }
  float bias[CO];
#pragma unroll
  for (int o = 0; o < CO; ++o) bias[o] = (b2 != nullptr && o < Co) ? b2[o] : 0.f;
  // tiles of 32 points, the last of a batch entry ragged; lanes past its end repeat its last point
  const long long tiles_per_b = (N + 31) >> 5;
  long long t = (long long)blockIdx.x * (kThreads / 64) + wave;
  const long long step = (long long)gridDim.x * (kThreads / 64);
  long long b = t / tiles_per_b;
  t -= b * tiles_per_b;
  float v[NS];
  auto load = [&](long long bb, long long tt) {
    const long long p0 = tt << 5, col = min((long long)c, N - 1 - p0);
    const float* xb = x + bb * Ci * N + p0;
    const float *xh = xb + half * N + col, *xc = xb + col;
#pragma unroll
    for (int s = 0; s < NS; ++s)                           // past the last channel: the last one, masked below
      v[s] = (2 * s + 1 < LOW || 2 * s + 1 < Ci) ? xh[2 * s * N] : xc[min(2 * s, Ci - 1) * N];
  };
  if (b < B) load(b, t);
  while (b < B) {
    u32x4 xs[KB][3];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        unsigned part[3] = {0u, 0u, 0u};
        const int s = 8 * kb + j;
        if (s < NS) {
          float q[2];
#pragma unroll
          for (int h = 0; h < 2; ++h)
            q[h] = 2 * (s + h) + 1 < LOW ? v[s + h]
                                         : __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, v[s + h]) & keep[s + h]) | one[s + h]);
          bf16_split(q[0], q[1], part);
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) xs[kb][p][j / 2] = part[p];
      }
    const long long bo = b, to = t;
    for (t += step; t >= tiles_per_b && b < B; t -= tiles_per_b) ++b;
    if (b < B) load(b, t);
    float sum[CO];
#pragma unroll
    for (int o = 0; o < CO; ++o) sum[o] = 0.f;
    auto hidden = [&](int hb) {
      u32x4 a[KB][3];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int p = 0; p < 3; ++p) a[kb][p] = A[((hb * KB + kb) * 3 + p) * 64 + lane];
      v16f acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) acc = mfma_bf16(a[kb][kSplitA[r]], xs[kb][kSplitB[r]], acc);
      return acc;
    };
#pragma unroll 1
    for (int hb = 0; hb < NH; ++hb) {
      const v16f acc = hidden(hb);
      float part[CO];
#pragma unroll
      for (int o = 0; o < CO; ++o) part[o] = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {                        // rows 8 q + 4 half + 0 .. 3
        float g[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) g[w] = gelu_fast_f(acc[4 * q + w]);
#pragma unroll
        for (int o = 0; o < CO; ++o) {
          const float4 w2 = W2S[(o * NH + hb) * 8 + 2 * q + half];
          part[o] = fmaf(w2.x, g[0], part[o]);
          part[o] = fmaf(w2.y, g[1], part[o]);
          part[o] = fmaf(w2.z, g[2], part[o]);
          part[o] = fmaf(w2.w, g[3], part[o]);
        }
      }
#pragma unroll
      for (int o = 0; o < CO; ++o) sum[o] += part[o];
    }
    const long long p = (to << 5) + c;
#pragma unroll
    for (int o = 0; o < CO; ++o) {
      sum[o] += __shfl_xor(sum[o], 32);
      if (half == 0 && o < Co && p < N) y[(bo * Co + o) * N + p] = sum[o] + bias[o];
    }
  }
}

// 16-bit elements of LDS turned in reading: with rows of `stride` elements, lane l gets column l % 32 of rows
// row0 + 8 (l/32) + 0 .. 7, two ds_read_b64_tr_b16 of four rows each (a group of 16 lanes reads 4 rows x 16 columns,
// lane j of it the address of four elements of row j / 4, and keeps column j).
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4 lds_turned(const unsigned short* base, int row0, int stride) {
  const int lane = threadIdx.x & 63;
  const unsigned short* p = base + (row0 + 8 * (lane >> 5) + ((lane & 15) >> 2)) * stride + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
  const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * stride)));
  return u32x4{a[0], a[1], b[0], b[1]};
}

// Adjoint of the projection to one channel.  A block walks over tiles of 64 points, staged split in LDS; wave (wh, wp)
// takes 32 hidden units, whose split weights stay in its registers, and both column blocks of 32 points or (two waves
// per group of hidden units) one of them.  With d = gelu'(h), M = diag(W2) W1 and Y = g [x ; 1],
//   h   = [W1 | b1] [x ; 1]
//   gx  = g M^T d                      K runs over the hidden units in accumulator order: the parts of d are the right
//                                      operand as they are packed
//   gW1 | gb1 = diag(W2) d Y^T         K runs over the points; the parts of d are turned through LDS
// so that neither g nor W2 multiplies anything per hidden value.  All products are sums of three bf16 parts, which have
// fp32's exponents: d of a unit that is off, a weight far below the largest and points with small values keep their 24
// bits.  (Two fp16 parts with a scale for every channel of M and Y took 907 us where this takes 1000, but have 2^-35 of the
// largest value, and of d 2^-25, as their last place: hidden values of -5 gave gx off by 6e-4, of -7 by its whole size.)
//
// The products for gW1 of a column block go to an accumulator of their own, which is added to the fp32 accumulator of the
// tiles (vector additions, 64 between two flushes), and that to doubles.  Y has the other sign every other time: the matrix
// instruction's sums are rounded to nearest after a cut towards minus infinity some bits below (measured: 0.004 units of
// the accumulator's last place on average; single products rounded in fp32 show none), which adds up over millions of
// points (4 million: gW1 off by 4.2e-6), and cancels in the difference (1.7e-7; with fp32 instructions 5.4e-7).  With one
// wave per group of hidden units the doubles stand in the block's slot of partial sums, in L2: 32 registers that the parts of d
// need, at 2 % for a flush every 32 tiles (9 % every four).
// The lanes' fp32 sums for gW2, with 32 channels also those for gb1, go to doubles at the same time: 64 terms at most.
//
// What bounds it: issue at two waves per SIMD (the parts of d, of the weights and of x, and LDS, allow no more), 1050 vector
// instructions (64 of them transcendental, at half rate) and 72 matrix instructions of 32 cycles a wave and tile.  Equal
// priorities left the vector unit idle in 32 % of the cycles, both units in 13 %.  20 -> 128 -> 1 at 4 million points: 1370
// us with both ways' products on the fp32 instruction, 945 with sums for gW2 that the compiler kept back to the tile's
// end (64 registers), a select of every value of x as it was asked for (which waited for it) and one priority, now 870;
// 16, 24, 32 channels at 2 million 422, 522, 582 and 376, 430, 521; against the scalar kernel (hidden or channel widths
// that the fp32 one did not fit) 20 -> 64 -> 1 5815 and 540 us, 32 -> 128 -> 1 at 2 million points 23050 and 521 us.
constexpr int kMlpTS = 36;               // row stride of turned tiles, in 16-bit elements: 18 banks, so that rows spread over all
struct MlpBwd {
  int B, Ci, H, nwh;                     // nwh: groups of 32 hidden units
  long long N;
};
constexpr int kMlpFlush = 32;            // tiles between flushes of the fp32 weight-gradient accumulators
constexpr int mlp_rows(int NS) { return NS == 4 ? 8 : (NS == 8 ? 16 : (NS == 12 ? 24 : 32)); }      // rows of gx
// LDS floats of a wave: the parts of d of its column blocks, then in the same place its share of gx (32 channels, one column
// block after the other: beside it)
constexpr int mlp_buffers(int NS, int NPG) { return NPG == 2 || NS == 18 ? 1 : 2; }
constexpr int mlp_region(int NS, int NPG) {
  const int parts = mlp_buffers(NS, NPG) * 48 * kMlpTS, share = mlp_rows(NS) * 64;
  return NS == 18 && NPG == 1 ? parts + share : (share > parts ? share : parts);
}
constexpr size_t mlp_bwd_lds(int NS, int NPG, int nw) {
  return (size_t)(NS > 8 ? 2 : 1) * 6 * 64 * 16 + 3 * 64 * kMlpTS * 2 + 2 * 64 * 4 + (NS == 18 ? 256 * 4 : 0) +
         (size_t)nw * mlp_region(NS, NPG) * 4;
}
// most pairs of channels that a wave of nw (or more) stages
constexpr int mlp_stage(int NS, int nw) { return ((NS < 16 ? NS : 16) + nw - 1) / nw; }
// NPG: waves per group of hidden units; SR: most pairs of channels that a wave stages
template <int NS, int NPG, int SR>
__global__ __launch_bounds__(512, 2) void mlp2_bwd_split_kernel(
    MlpBwd f, const float* __restrict__ x, const float* __restrict__ W1, const float* __restrict__ b1,
    const float* __restrict__ W2, const float* __restrict__ g, float* __restrict__ gx, double* __restrict__ part) {
  HIP_DYNAMIC_SHARED(float4, smem4)
  constexpr int KB = NS > 8 ? 2 : 1, ROWS = mlp_rows(NS), REG = mlp_region(NS, NPG);
  constexpr bool ALL = NS == 18;           // 32 input channels: no column left for gb1, the bias is where h starts
  constexpr int BUF = mlp_buffers(NS, NPG);                // column blocks that a wave works on at a time
  const int Ci = f.Ci, H = f.H;
  const long long N = f.N;
  const int nthreads = blockDim.x, nw = nthreads >> 6;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, c = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = w / f.nwh, wh = w - wp * f.nwh;
  u32x4* XS = reinterpret_cast<u32x4*>(smem4);                               // [KB][3][2][64]: octets of channels of a point
  unsigned short* YS = reinterpret_cast<unsigned short*>(XS + KB * 6 * 64);  // [3][64][kMlpTS]: channels of a point
  float* GS2 = reinterpret_cast<float*>(YS + 3 * 64 * kMlpTS);               // [2][64] cotangents, tile by tile in turn
  float* BS = GS2 + 2 * 64;                                                  // [256] b1
  float* regions = BS + (ALL ? 256 : 0);
  float* own = regions + w * REG;
  unsigned short* T = reinterpret_cast<unsigned short*>(own);                // [BUF][3][32][kMlpTS]
  float* share = own + (ALL && NPG == 1 ? BUF * 48 * kMlpTS : 0);            // [ROWS][64] of gx
  const int nsum = H * (Ci + 1) + H + 1;
  const int np = ALL ? 16 : Ci / 2 + 1;    // pairs with the channel of ones
  double* dst = part + (long long)blockIdx.x * nsum;       // gW1 | gb1 | gW2 | gb2
  for (int e = tid; e < KB * 6 * 64; e += nthreads) XS[e] = u32x4{0u, 0u, 0u, 0u};
  for (int e = tid; e < 3 * 64 * kMlpTS / 2; e += nthreads) reinterpret_cast<unsigned*>(YS)[e] = 0u;
  if constexpr (ALL)
    for (int e = tid; e < 256; e += nthreads) BS[e] = b1 != nullptr && e < H ? b1[e] : 0.f;
  // M holds W2 by a power of two that makes the largest 1 .. 2 (the products with W1 keep W1's range); g takes it back
  int w2_exp = 0;
  {
    float m = 0.f;
    for (int k = lane; k < H; k += 64) m = fmaxf(m, fabsf(W2[k]));
#pragma unroll
    for (int j = 1; j < 64; j <<= 1) m = fmaxf(m, __shfl_xor(m, j));
    w2_exp = (int)(__builtin_bit_cast(unsigned, m) >> 23 & 255u) - 127;
  }
  u32x4 a1[KB][3], am[2][3];
  {
    const int k = wh * 32 + c;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        float v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int i = 16 * kb + 8 * half + j + q;
          v[q] = k < H ? (i < Ci ? W1[k * Ci + i] : (i == Ci && b1 != nullptr ? b1[k] : 0.f)) : 0.f;
        }
        unsigned pt[3];
        bf16_split(v[0], v[1], pt);
#pragma unroll
        for (int p = 0; p < 3; ++p) a1[kb][p][j / 2] = pt[p];
      }
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      float m[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int kk = wh * 32 + mfma_row(v + q, half);
        m[q] = (c < Ci && kk < H) ? W1[kk * Ci + c] * ldexpf(W2[kk], -w2_exp) : 0.f;
      }
      unsigned pt[3];
      bf16_split(m[0], m[1], pt);
#pragma unroll
      for (int p = 0; p < 3; ++p) am[v >> 3][p][(v & 7) / 2] = pt[p];
    }
  }
  v16f accw;
  double accg = 0.0;
  float acc2[16], accb[ALL ? 16 : 1];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc2[v] = accw[v] = 0.f;
#pragma unroll
  for (int v = 0; v < (ALL ? 16 : 1); ++v) accb[v] = 0.f;
  // the doubles of accw: with two waves per group of hidden units in registers, else in the block's slot, of which every
  // lane owns its entries
  double accd[NPG == 2 ? 16 : 1];
#pragma unroll
  for (int v = 0; v < (NPG == 2 ? 16 : 1); ++v) accd[v] = 0.0;
  const int slot_step = c < Ci ? Ci : 1;
  double* slot = dst + (c < Ci ? c : H * Ci) + (wh * 32 + 4 * half) * slot_step;
  auto in_slot = [&](int v) { return c <= Ci && wh * 32 + mfma_row(v, half) < H; };
  bool begun = false;                      // the slot holds something

  const long long tiles_per_b = (N + 63) >> 6;
  long long t = blockIdx.x, b = t / tiles_per_b;
  t -= b * tiles_per_b;
  // a wave stages pairs of channels w, w + nw, ..; its lanes are the points
  float pv[SR][2], pg;
  // (lanes past the last point read it again, under g = 0; pairs past the last channel are not used).  Nothing is done
  // with the values before they are staged, a tile later: a select here waits for them here.
  auto load = [&]() {
    const long long p = (t << 6) + lane, pc = min(p, N - 1);
    const float* xb = x + b * Ci * N + pc;
#pragma unroll
    for (int r = 0; r < SR; ++r) {
      const int i = 2 * (r * nw + w);
      pv[r][0] = xb[min(i, Ci - 1) * N];
      pv[r][1] = xb[min(i + 1, Ci - 1) * N];
    }
    pg = g[b * N + pc];
  };
  if (b < f.B) load();
  __syncthreads();                         // XS is clear
  float sign = blockIdx.x & 1 ? -1.f : 1.f;                // of Y
  // sums that only a flush reads are added to here and now: left alone they move behind the tile's last barrier, and
  // hidden values, distribution values and products stay in 80 registers until then
  auto now = [](float& v) { asm volatile("" : "+v"(v)); };
  // a value that a flush forms its addresses from: these would be kept over the loop otherwise
  auto anew = [](int v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  // accw to its doubles; at the end these, times W2, go to the slot
  auto flush = [&](bool last) {
    double sum[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = (double)(sign * accw[v]);
    if constexpr (NPG == 2) {
#pragma unroll
      for (int v = 0; v < 16; ++v) accd[v] += sum[v];
    } else {
      const int step = anew(slot_step);
      if (begun)
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] += in_slot(v) ? slot[mfma_row(v, 0) * step] : 0.0;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (in_slot(v)) slot[mfma_row(v, 0) * step] = last ? sum[v] * (double)W2[wh * 32 + mfma_row(v, half)] : sum[v];
      begun = true;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) accw[v] = 0.f;
    sign = -sign;
  };
  // acc2 and accb to doubles, kept as those of accw: in lane l, over the lanes of register l / 2, half l % 2
  double sum2 = 0.0, sumb = 0.0;
  auto row_sum = [&](float (&a)[16]) {
    const int at = anew(c);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      own[66 * v + 33 * half + at] = a[v];
      a[v] = 0.f;
    }
    __builtin_amdgcn_wave_barrier();
    double sum = 0.0;
    for (int j = 0; j < 32; ++j) sum += (double)own[33 * at + j];
    return sum;
  };
  auto row_of = [&](int q) { return wh * 32 + mfma_row(q >> 1, q & 1); };
  auto flush_rows = [&](bool last) {       // before flush()
    __syncthreads();                       // the shares of gx have been read
    if constexpr (NPG == 2) {
      sum2 += row_sum(acc2);
      if constexpr (ALL) sumb += row_sum(accb);
      return;
    }
    const int row = row_of(anew(c));
    const bool mine = half == 0 && row < H;
    auto add = [&](double* at, double v, double factor) {
      if (mine) *at = (begun ? *at + v : v) * factor;
    };
    add(dst + H * (Ci + 1) + row, row_sum(acc2), 1.0);
    if constexpr (ALL) add(dst + H * Ci + row, row_sum(accb), last && mine ? (double)W2[row] : 1.0);
  };
  int pass = 0;
  static_assert(kMlpFlush % 2 == 0, "passes take the two halves of GS2 in turn");
  while (b < f.B) {
    const long long bo = b, to = t;
    // The cotangents are read after the tile's last barrier, when wave 0 may be at the next tile already: that one has the
    // other half.  This half is written again a tile later, behind the next tile's first barrier, which every wave reaches
    // with its reads done.  (One array: a wave held up took another tile's cotangents.)
    float* GS = GS2 + 64 * (pass & 1);
    const float gp = (to << 6) + lane < N ? pg : 0.f, gs = gp * sign;
#pragma unroll
    for (int r = 0; r < SR; ++r) {
      const int q = r * nw + w;
      if (q < np) {
        const float v0 = 2 * q == Ci ? 1.f : pv[r][0], v1 = 2 * q + 1 == Ci ? 1.f : pv[r][1];
        unsigned pt[3], py[3];
        bf16_split(v0, v1, pt);
        bf16_split(gs * v0, gs * v1, py);
        unsigned* xd = reinterpret_cast<unsigned*>(XS + ((q >> 3) * 6 + ((q >> 2) & 1)) * 64 + lane) + (q & 3);
        unsigned* yd = reinterpret_cast<unsigned*>(YS + lane * kMlpTS) + q;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          xd[p * 2 * 64 * 4] = pt[p];
          yd[p * 64 * (kMlpTS / 2)] = py[p];
        }
      }
    }
    if (w == 0) GS[lane] = gp;
    __syncthreads();
    for (t += gridDim.x; t >= tiles_per_b && b < f.B; t -= tiles_per_b) ++b;
    const bool more = b < f.B;
    // The next tile's values are asked for when the slopes are done, which need all registers: the last products and what
    // follows them are as long as the loads take.
    auto ask = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      if (more) load();
      __builtin_amdgcn_sched_barrier(0);
    };
    // Column block by column block.  The matrix instructions of one are dealt between the vector instructions of the
    // other by hand: left alone, the compiler keeps them together, and a wave waits for its own chain of products.
    v16f ga[BUF], hacc[BUF], gw_part;
    u32x4 xs[KB][3], dp[BUF][2][3], dt[3], yt[3];
    auto turn_buffer = [&](int u) { return T + u * 3 * 32 * kMlpTS; };
    auto read_x = [&](int col) {
      const int pc = col * 32 + c;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int p = 0; p < 3; ++p) xs[kb][p] = XS[((kb * 3 + p) * 2 + half) * 64 + pc];
    };
    auto clear = [](v16f& a) {
#pragma unroll
      for (int v = 0; v < 16; ++v) a[v] = 0.f;
    };
    auto hidden = [&](int nb, int r0, int r1) {            // products r0 .. r1 - 1 of 6 KB
#pragma unroll
      for (int r = 0; r < 6 * KB; ++r)
        if (r >= r0 && r < r1) {
          if (r == 0) {
            if constexpr (ALL) {
#pragma unroll
              for (int v = 0; v < 16; v += 4) {
                const float4 q = *reinterpret_cast<const float4*>(BS + wh * 32 + mfma_row(v, half));
                hacc[nb][v] = q.x; hacc[nb][v + 1] = q.y; hacc[nb][v + 2] = q.z; hacc[nb][v + 3] = q.w;
              }
            } else {
              clear(hacc[nb]);
            }
          }
          hacc[nb] = mfma_bf16(a1[r % KB][kSplitA[r / KB]], xs[r % KB][kSplitB[r / KB]], hacc[nb]);
        }
    };
    auto turned = [&](int nb, int col, int m) {
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        dt[p] = lds_turned(turn_buffer(nb) + p * 32 * kMlpTS, 16 * m, kMlpTS);
        yt[p] = lds_turned(YS + p * 64 * kMlpTS, col * 32 + 16 * m, kMlpTS);
      }
    };
    auto products = [&](int nb, int col, int step) {       // eighth `step` of the 24 products with d
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if (s != step) continue;
        if (s == 0) clear(ga[nb]);
        if (s == 2) turned(nb, col, 0);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          if (s < 4) {
            const int r = (3 * s + j) / 2, m = (3 * s + j) % 2;
            ga[nb] = mfma_bf16(am[m][kSplitA[r]], dp[nb][m][kSplitB[r]], ga[nb]);
          } else {
            const int r = 3 * (s & 1) + j;
            if (s == 4 && j == 0) clear(gw_part);
            gw_part = mfma_bf16(dt[kSplitA[r]], yt[kSplitB[r]], gw_part);
          }
        }
        if (s == 5) turned(nb, col, 1);
        if (s == 7) {
          accw += gw_part;
#pragma unroll
          for (int v = 0; v < 16; ++v) asm volatile("" : "+v"(accw[v]));
        }
      }
    };
    auto slopes = [&](int nb, int col, auto&& beside) {
      const float gl = GS[col * 32 + c];
      accg += half == 0 ? (double)gl : 0.0;
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        beside(v / 2);
        float d[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          float a;
          gelu_and_grad_f(hacc[nb][v + q], a, d[q]);
          acc2[v + q] = fmaf(gl, a, acc2[v + q]);
          now(acc2[v + q]);
          if constexpr (ALL) {
            accb[v + q] = fmaf(gl, d[q], accb[v + q]);
            now(accb[v + q]);
          }
        }
        unsigned pt[3];
        bf16_split(d[0], d[1], pt);
#pragma unroll
        for (int p = 0; p < 3; ++p) dp[nb][v >> 3][p][(v & 7) / 2] = pt[p];
        if ((v & 3) == 2) {                // rows 8 q + 4 half + 0 .. 3 of point c
          const int q = v >> 2;
#pragma unroll
          for (int p = 0; p < 3; ++p)
            *reinterpret_cast<uint2*>(turn_buffer(nb) + (p * 32 + c) * kMlpTS + 8 * q + 4 * half) =
                make_uint2(dp[nb][q >> 1][p][2 * (q & 1)], dp[nb][q >> 1][p][2 * (q & 1) + 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto share_gx = [&](int nb, int col) {
      __builtin_amdgcn_wave_barrier();
      float* dst = share + 4 * half * 64 + col * 32 + c;
      if (gx != nullptr)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (mfma_row(v, 0) < ROWS) dst[mfma_row(v, 0) * 64] = ga[nb][v];
    };
    if constexpr (BUF == 1) {              // one by one: 32 channels leave no registers for two
#pragma unroll 1
      for (int col = NPG == 2 ? wp : 0; col < (NPG == 2 ? wp + 1 : 2); ++col) {
        read_x(col);
        hidden(0, 0, 6 * KB);
        __builtin_amdgcn_s_setprio(1);
        slopes(0, col, [](int) {});
        __builtin_amdgcn_s_setprio(0);
        if (NPG == 2 || col == 1) ask();
#pragma unroll
        for (int u = 0; u < 8; ++u) products(0, col, u);
        share_gx(0, col);
      }
    } else {
      read_x(0);
      hidden(0, 0, 6 * KB);
      read_x(1);
      __builtin_amdgcn_sched_barrier(0);
      // The wave with slopes to work goes before the one (of the other block) in its chains of products, which wait for
      // one another anyhow: 10 % over equal priorities, which leave the products ahead as often as not.
      __builtin_amdgcn_s_setprio(1);
      slopes(0, 0, [&](int u) { hidden(1, 6 * KB * u / 8, 6 * KB * (u + 1) / 8); });
      slopes(1, 1, [&](int u) { products(0, 0, u); });
      ask();
      __builtin_amdgcn_s_setprio(0);
#pragma unroll
      for (int u = 0; u < 8; ++u) products(1, 1, u);
      share_gx(0, 0);
      share_gx(1, 1);
    }
    __syncthreads();
    const int point = __lane_id();         // made anew: kept over the products it would be in scratch, whose wait is for x too
    if (gx != nullptr && (to << 6) + point < N) {
      const float* src = regions + (share - own) + (NPG == 2 ? (point >> 5) * f.nwh * REG : 0) + point;
      const float gw = ldexpf(GS[point], w2_exp);
      // the channels of this wave, two shares of all of them at a time: the reads go out together
      float sum[2 * SR];
#pragma unroll
      for (int r = 0; r < 2 * SR; ++r) sum[r] = 0.f;
#pragma unroll 1
      for (int ww = 0; ww < f.nwh; ww += 2) {
        float one[2 * SR], two[2 * SR];
        const float* s1 = src + ww * REG;
        const float* s2 = src + min(ww + 1, f.nwh - 1) * REG;
#pragma unroll
        for (int r = 0; r < 2 * SR; ++r) {
          const int i = min(w + r * nw, Ci - 1) * 64;
          one[r] = s1[i];
          two[r] = s2[i];
        }
#pragma unroll
        for (int r = 0; r < 2 * SR; ++r) {
          sum[r] += one[r];
          if (ww + 1 < f.nwh) sum[r] += two[r];
        }
      }
      float* tile = gx + bo * Ci * N + (to << 6);
#pragma unroll
      for (int r = 0; r < 2 * SR; ++r)
        if (w + r * nw < Ci) tile[(w + r * nw) * N + point] = sum[r] * gw;
    }
    if (++pass == kMlpFlush) {
      pass = 0;
      flush_rows(false);
      flush(false);
    }
  }
  flush_rows(true);
  flush(true);
  // the lanes of a row, then two waves with the same hidden units, meet in LDS in a fixed order
  __syncthreads();
  double* meet = reinterpret_cast<double*>(smem4) + wh * 64;
  auto joined = [&](double v) {
    if (NPG == 1) return v;
    __syncthreads();
    if (wp == 1) meet[lane] = v;
    __syncthreads();
    return wp == 0 ? v + meet[lane] : 0.0;
  };
  if constexpr (NPG == 2) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const double sum = joined(accd[v]);
      if (wp == 0 && in_slot(v)) slot[mfma_row(v, 0) * slot_step] = sum * (double)W2[wh * 32 + mfma_row(v, half)];
    }
    const int row = row_of(c);
    const bool mine = wp == 0 && half == 0 && row < H;
    const double s2 = joined(sum2);
    if (mine) dst[H * (Ci + 1) + row] = s2;
    if constexpr (ALL) {
      const double sb = joined(sumb);
      if (mine) dst[H * Ci + row] = sb * (double)W2[row];
    }
  }
  double sg = accg;
#pragma unroll
  for (int m = 1; m < 32; m <<= 1) sg += __shfl_xor(sg, m);
  sg = joined(sg);
  if (tid == 0) dst[H * (Ci + 1) + H] = sg;
}

// The adjoint of a projection to two to four channels, in fp32 throughout: v_mfma_f32_32x32x2, lane l supplies A[l%32][l/32]
// and B[l/32][l%32].  As above, but gh = (W2^T g) gelu'(h) stands in the place of d and is not split.
constexpr int kMlpTile = 64;             // points per pass of a block
constexpr int kMlpStage = 6;             // values a thread stages per pass
constexpr int kMlpXS = kMlpTile + 1;     // row stride of the staged tile (odd: column reads spread over the banks)
constexpr int kMlpFlush32 = 16;          // passes between flushes of the fp32 weight-gradient accumulator
constexpr int kMlpTurn = 33;               // row stride of a wave's 32x32 turn buffer

template <int KS>
__global__ __launch_bounds__(512) void mlp2_bwd_mfma_kernel(
    int B, int Ci, int H, int Co, long long N, const float* __restrict__ x, const float* __restrict__ W1,
    const float* __restrict__ b1, const float* __restrict__ W2, const float* __restrict__ g,
    float* __restrict__ gx, double* __restrict__ part) {
  HIP_DYNAMIC_SHARED(float, smem)
  constexpr int CO = 4;
  const int nthreads = blockDim.x, nw = nthreads >> 6;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, half = lane >> 5, c = lane & 31;
  float* XS = smem;                                      // [32][kMlpXS]: tile, ones, zeros as above
  float* GS = XS + 32 * kMlpXS;                          // [CO][kMlpTile] upstream gradient of the tile
  float* T = GS + CO * kMlpTile + w * (32 * kMlpTurn);     // this wave's [32][kMlpTurn] turn buffer
  float* GXP = GS + CO * kMlpTile + nw * (32 * kMlpTurn);  // [nw][Ci][kMlpXS] partial gx of the waves
  float* W2S = GXP + nw * Ci * kMlpXS;                   // [CO][H]
  int acc_off = 32 * kMlpXS + CO * kMlpTile + nw * (32 * kMlpTurn) + nw * Ci * kMlpXS + CO * H;
  acc_off += acc_off & 1;
  double* ACC = reinterpret_cast<double*>(smem + acc_off);   // [nsum] gW1 | gb1 | gW2 | gb2
  const int nsum = H * (Ci + 1) + Co * H + Co;
  for (int q = tid; q < nsum; q += nthreads) ACC[q] = 0.0;
  for (int e = tid; e < (32 - Ci) * kMlpXS; e += nthreads) XS[Ci * kMlpXS + e] = e < kMlpXS ? 1.f : 0.f;
  for (int e = tid; e < CO * H; e += nthreads) W2S[e] = e < Co * H ? W2[e] : 0.f;
  float A1[KS], A2[16];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int i = 2 * s + half, k = w * 32 + c;
    A1[s] = i < Ci ? W1[k * Ci + i] : ((i == Ci && b1 != nullptr) ? b1[k] : 0.f);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int k = w * 32 + mfma_row(v, half);
    A2[v] = c < Ci ? W1[k * Ci + c] : 0.f;
  }
  const long long tiles_per_b = (N + kMlpTile - 1) / kMlpTile;
  const long long ntiles = tiles_per_b * B;
  const int nstage = (Ci + Co) * kMlpTile;
  v16f accw = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float acc2[CO][16], accg[CO];
#pragma unroll
  for (int o = 0; o < CO; ++o) {
    accg[o] = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc2[o][v] = 0.f;
  }
  float pf[kMlpStage];
  {
    const long long t = blockIdx.x;
    const long long b = t / tiles_per_b, p0 = (t - b * tiles_per_b) * kMlpTile;
#pragma unroll
    for (int r = 0; r < kMlpStage; ++r) {
      const int e = tid + r * nthreads, row = e >> 6, col = e & 63;
      float val = 0.f;
      if (t < ntiles && e < nstage && p0 + col < N)
        val = row < Ci ? x[(b * Ci + row) * N + p0 + col] : g[(b * Co + (row - Ci)) * N + p0 + col];
      pf[r] = val;
    }
  }
  int pass = 0;
  for (long long t = blockIdx.x; t < ntiles; t += gridDim.x) {
#pragma unroll
    for (int r = 0; r < kMlpStage; ++r) {
      const int e = tid + r * nthreads, row = e >> 6, col = e & 63;
      if (e < nstage) {
        if (row < Ci) XS[row * kMlpXS + col] = pf[r];
        else GS[(row - Ci) * kMlpTile + col] = pf[r];
      }
    }
    __syncthreads();
    {
      const long long tn = t + gridDim.x;
      const long long b = tn / tiles_per_b, p0 = (tn - b * tiles_per_b) * kMlpTile;
#pragma unroll
      for (int r = 0; r < kMlpStage; ++r) {
        const int e = tid + r * nthreads, row = e >> 6, col = e & 63;
        float val = 0.f;
        if (tn < ntiles && e < nstage && p0 + col < N)
          val = row < Ci ? x[(b * Ci + row) * N + p0 + col] : g[(b * Co + (row - Ci)) * N + p0 + col];
        pf[r] = val;
      }
    }
    const long long b = t / tiles_per_b, p0 = (t - b * tiles_per_b) * kMlpTile;
#pragma unroll 1
    for (int nb = 0; nb < 2; ++nb) {
      const int pc = nb * 32 + c;
      v16f hacc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s)
        hacc = __builtin_amdgcn_mfma_f32_32x32x2f32(A1[s], XS[(2 * s + half) * kMlpXS + pc], hacc, 0, 0, 0);
      float gl[CO];
#pragma unroll
      for (int o = 0; o < CO; ++o) {
        gl[o] = o < Co ? GS[o * kMlpTile + pc] : 0.f;
        if (half == 0) accg[o] += gl[o];
      }
      float gh[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float a, d;
        gelu_and_grad_f(hacc[v], a, d);
        float tt = 0.f;
#pragma unroll
        for (int o = 0; o < CO; ++o) {
          const float w2v = W2S[o * H + w * 32 + mfma_row(v, half)];
          tt = fmaf(w2v, gl[o], tt);
          acc2[o][v] = fmaf(gl[o], a, acc2[o][v]);
        }
        gh[v] = tt * d;
        T[mfma_row(v, half) * kMlpTurn + c] = gh[v];
      }
      v16f gacc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 16; ++v) gacc = __builtin_amdgcn_mfma_f32_32x32x2f32(A2[v], gh[v], gacc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = mfma_row(v, half);
        if (row < Ci) GXP[(w * Ci + row) * kMlpXS + pc] = gacc[v];
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int s = 0; s < 16; ++s)
        accw = __builtin_amdgcn_mfma_f32_32x32x2f32(T[c * kMlpTurn + 2 * s + half],
                                                    XS[c * kMlpXS + nb * 32 + 2 * s + half], accw, 0, 0, 0);
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (gx != nullptr) {
      for (int e = tid; e < Ci * kMlpTile; e += nthreads) {
        const int i = e >> 6, col = e & 63;
        float sum = 0.f;
        for (int ww = 0; ww < nw; ++ww) sum += GXP[(ww * Ci + i) * kMlpXS + col];
        if (p0 + col < N) gx[(b * Ci + i) * N + p0 + col] = sum;
      }
    }
    if (++pass == kMlpFlush32) {
      pass = 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int k = w * 32 + mfma_row(v, half);
        if (c < Ci) ACC[k * Ci + c] += (double)accw[v];
        else if (c == Ci) ACC[H * Ci + k] += (double)accw[v];
        accw[v] = 0.f;
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int k = w * 32 + mfma_row(v, half);
    if (c < Ci) ACC[k * Ci + c] += (double)accw[v];
    else if (c == Ci) ACC[H * Ci + k] += (double)accw[v];
  }
  // gW2[o][k]: the lanes' sums over their points, added over the 32 lanes of a row through T
#pragma unroll
  for (int o = 0; o < CO; ++o) {
    if (o < Co) {
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v) T[mfma_row(v, half) * kMlpTurn + c] = acc2[o][v];
      __syncthreads();
      if (half == 0) {
        double sum = 0.0;
        for (int cc = 0; cc < 32; ++cc) sum += (double)T[c * kMlpTurn + cc];
        ACC[H * (Ci + 1) + o * H + w * 32 + c] = sum;
      }
      float sg = accg[o];
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) sg += __shfl_xor(sg, m);
      if (tid == 0) ACC[H * (Ci + 1) + Co * H + o] = (double)sg;
    }
  }
  __syncthreads();
  for (int q = tid; q < nsum; q += nthreads) part[(long long)blockIdx.x * nsum + q] = ACC[q];
}

// ------------------------------------------------------------------------------------------
// Training pieces outside the block (Sec. 4): relative L2 misfit and the Adam update
// ------------------------------------------------------------------------------------------
constexpr int kLossBlocks = 1024;      // partial sums of the loss (two doubles each)

// part[blk] = (sum (pred - target)^2, sum target^2) over the block's strided share, in double,
// combined in a fixed order (lane tree, then waves in order): same bits on every run.
__global__ __launch_bounds__(kThreads) void rel_l2_partial_kernel(
    long long n, const float* __restrict__ pred, const float* __restrict__ target, double* __restrict__ part) {
  __shared__ double sd[kThreads / 64], sy[kThreads / 64];
  double d2 = 0.0, y2 = 0.0;
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads) {
    const double y = target[i];
    const double d = (double)pred[i] - y;
    d2 += d * d;
    y2 += y * y;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    d2 += __shfl_xor(d2, off);
    y2 += __shfl_xor(y2, off);
  }
  if ((threadIdx.x & 63) == 0) { sd[threadIdx.x >> 6] = d2; sy[threadIdx.x >> 6] = y2; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int w = 0; w < kThreads / 64; ++w) { a += sd[w]; b += sy[w]; }
    part[2 * blockIdx.x] = a;
    part[2 * blockIdx.x + 1] = b;
  }
}

// loss = sqrt(Sd) / sqrt(Sy); scale = 1 / (sqrt(Sd) sqrt(Sy)) for the gradient (0 when Sd = 0).  One block; the
// partials in a fixed order (a thread's share, then lanes as a tree, then waves): 5 us, 83 us with a single thread.
__global__ __launch_bounds__(kThreads) void rel_l2_final_kernel(const double* __restrict__ part, int nblk,
                                                                float* __restrict__ loss, double* __restrict__ scale) {
  __shared__ double sd[kThreads / 64], sy[kThreads / 64];
  double a = 0.0, b = 0.0;
#pragma unroll
  for (int u = 0; u < kLossBlocks / kThreads; ++u) {
    const int i = threadIdx.x + u * kThreads;
    if (i < nblk) { a += part[2 * i]; b += part[2 * i + 1]; }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
  }
  if ((threadIdx.x & 63) == 0) { sd[threadIdx.x >> 6] = a; sy[threadIdx.x >> 6] = b; }
  __syncthreads();
  if (threadIdx.x != 0) return;
  a = 0.0; b = 0.0;
  for (int w = 0; w < kThreads / 64; ++w) { a += sd[w]; b += sy[w]; }
  const double nd = sqrt(a), ny = sqrt(b);
  if (loss != nullptr) *loss = (float)(nd / ny);
  *scale = nd > 0.0 ? 1.0 / (nd * ny) : 0.0;
}

__global__ __launch_bounds__(kThreads) void rel_l2_grad_kernel(
    long long n, const float* __restrict__ pred, const float* __restrict__ target,
    const double* __restrict__ scale, float* __restrict__ grad) {
  const float sc = (float)*scale;
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads)
    grad[i] = (pred[i] - target[i]) * sc;
}

// Adam (Kingma & Ba, Algorithm 1), one step in place; c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t)
__global__ __launch_bounds__(kThreads) void adam_kernel(
    long long n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
    float* __restrict__ v, float lr, float beta1, float omb1, float beta2, float omb2, float eps, float c1,
    float c2) {
  // omb = 1 - beta, rounded from double on the host (1 - beta in float would lose five digits)
  // every element is read and written once per step: nontemporal accesses
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads) {
    const float gi = __builtin_nontemporal_load(g + i);
    const float mi = fmaf(beta1, __builtin_nontemporal_load(m + i), omb1 * gi);
    const float vi = fmaf(beta2, __builtin_nontemporal_load(v + i), omb2 * gi * gi);
    __builtin_nontemporal_store(mi, m + i);
    __builtin_nontemporal_store(vi, v + i);
    __builtin_nontemporal_store(__builtin_nontemporal_load(p + i) - lr * (mi * c1) / (sqrtf(vi * c2) + eps), p + i);
  }
}

// Input lifts of Sec. 2.4 (eqs. (8)-(9)) in one sweep: a_1 = W_t a + b_t along a time axis of
// length one, then nu = W_c a_1 + b_c along the channels, i.e.
//   nu[b][c][p][t] = W_t[t] s_c(p) + b_t[t] r_c + b_c[c],  s_c(p) = sum_j W_c[c][j] a[b][j][p],
//   r_c = sum_j W_c[c][j].
// One thread: one spatial point and four consecutive t; the output (the only large tensor) is
// written once, a is read through the cache by the threads that share a point.
template <int CO, bool STREAM>
__global__ __launch_bounds__(kThreads) void time_lift_kernel(
    int Ci, int Co, long long np, int Nt, const float* __restrict__ a, const float* __restrict__ wt,
    const float* __restrict__ bt, const float* __restrict__ wc, const float* __restrict__ bc,
    float* __restrict__ out) {
  const int nt4 = (Nt + 3) >> 2;
  const long long e = (long long)blockIdx.x * kThreads + threadIdx.x;
  const long long b = blockIdx.y;
  if (e >= np * nt4) return;
  const long long p = e / nt4;
  const int t0 = 4 * (int)(e - p * nt4);
  float sc[CO], rc[CO];
#pragma unroll
  for (int c = 0; c < CO; ++c) { sc[c] = 0.f; rc[c] = 0.f; }
  for (int j = 0; j < Ci; ++j) {
    const float av = a[(b * Ci + j) * np + p];
#pragma unroll
    for (int c = 0; c < CO; ++c) {
      if (c < Co) {
        const float w = wc[c * Ci + j];
        sc[c] = fmaf(w, av, sc[c]);
        rc[c] += w;
      }
    }
  }
  float w4[4], b4[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    w4[u] = t0 + u < Nt ? wt[t0 + u] : 0.f;
    b4[u] = (bt != nullptr && t0 + u < Nt) ? bt[t0 + u] : 0.f;
  }
  const bool vec = (Nt & 3) == 0;      // rows of whole float4s (the base pointer is checked on the host)
#pragma unroll
  for (int c = 0; c < CO; ++c) {
    if (c < Co) {
      const float bias = bc != nullptr ? bc[c] : 0.f;
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = fmaf(w4[u], sc[c], fmaf(b4[u], rc[c], bias));
      float* dst = out + ((b * Co + c) * np + p) * Nt + t0;
      if (vec) {
        st_once<STREAM>(reinterpret_cast<v4f*>(dst), v4f{v[0], v[1], v[2], v[3]});
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (t0 + u < Nt) dst[u] = v[u];
      }
    }
  }
}

// Adjoint of the fused lifts (eqs. (8)-(9)) with respect to their parameters.  With
//   G0[o][t] = sum_{b,s} g[b][o][s][t]   and   G1[i][o][t] = sum_{b,s} g[b][o][s][t] a[b][i][s]
// every gradient is a small contraction:  gbc[o] = sum_t G0,  gWc[o][i] = sum_t (Wt[t] G1 + bt[t] G0),
// gWt[t] = sum_{o,i} Wc[o][i] G1,  gbt[t] = sum_{o,i} Wc[o][i] G0.  The sweep over g (the only large
// tensor) keeps one (o, t) pair per thread, so a wave reads whole 128-byte runs of t and the input
// value a[b][i][s] is the same for all its lanes; a chunk of space positions per block row, fp32
// sums of 64 terms added into doubles, one partial per (chunk, pair) in a fixed order.
constexpr int kLiftChunks = 1024;      // partial-sum slots of the sweep
template <int CI, bool STREAM>
__global__ __launch_bounds__(kThreads) void time_lift_bwd_kernel(
    int Ci, int Co, long long S, int Nt, int cpb, const float* __restrict__ a, const float* __restrict__ g,
    double* __restrict__ part) {
  const int pair = blockIdx.x * kThreads + threadIdx.x;
  const int npair = Co * Nt;
  const long long b = blockIdx.y / cpb;
  const int c = blockIdx.y - (int)b * cpb;
  const long long len = (S + cpb - 1) / cpb;
  const long long s0 = c * len, s1 = min(S, s0 + len);
  const bool live = pair < npair;
  const int o = live ? pair / Nt : 0, t = live ? pair - o * Nt : 0;
  const float* gp = g + ((b * Co + o) * S) * Nt + t;
  const float* ap = a + (b * Ci) * S;
  double d0 = 0.0, d1[CI];
#pragma unroll
  for (int i = 0; i < CI; ++i) d1[i] = 0.0;
  for (long long sb = s0; sb < s1; sb += 64) {
    float f0 = 0.f, f1[CI];
#pragma unroll
    for (int i = 0; i < CI; ++i) f1[i] = 0.f;
    const long long se = min(s1, sb + 64);
    long long sp = sb;
    for (; sp + 8 <= se; sp += 8) {              // eight positions per pass: their loads go out together
      float gv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) gv[u] = live ? ld_once<STREAM>(&gp[(sp + u) * Nt]) : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        f0 += gv[u];
#pragma unroll
        for (int i = 0; i < CI; ++i)
          if (i < Ci) f1[i] = fmaf(gv[u], ap[i * S + sp + u], f1[i]);
      }
    }
    for (; sp < se; ++sp) {
      const float gv = live ? gp[sp * Nt] : 0.f;
      f0 += gv;
#pragma unroll
      for (int i = 0; i < CI; ++i)
        if (i < Ci) f1[i] = fmaf(gv, ap[i * S + sp], f1[i]);
    }
    d0 += (double)f0;
#pragma unroll
    for (int i = 0; i < CI; ++i) d1[i] += (double)f1[i];
  }
  if (live) {
    double* dst = part + ((long long)blockIdx.y * (Ci + 1)) * npair + pair;
    dst[0] = d0;
#pragma unroll
    for (int i = 0; i < CI; ++i)
      if (i < Ci) dst[(long long)(i + 1) * npair] = d1[i];
  }
}

// G[k][pair] = sum over the chunks: 32 entries per block, the chunks dealt to 8 thread groups whose
// sums are added in a fixed order
__global__ __launch_bounds__(kThreads) void time_lift_bwd_reduce_kernel(const double* __restrict__ part, int nchunk,
                                                                        int nent, double* __restrict__ G) {
  __shared__ double P[8][32];
  const int el = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int e = blockIdx.x * 32 + el;
  double sum = 0.0;
  if (e < nent)
    for (int c = grp; c < nchunk; c += 8) sum += part[(long long)c * nent + e];
  P[grp][el] = sum;
  __syncthreads();
  if (grp == 0 && e < nent) {
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) tot += P[k][el];
    G[e] = tot;
  }
}

// the four small contractions, one output per thread
__global__ __launch_bounds__(kThreads) void time_lift_bwd_final_kernel(
    int Ci, int Co, int Nt, const double* __restrict__ G, const float* __restrict__ wt,
    const float* __restrict__ bt, const float* __restrict__ wc, float* __restrict__ gwt,
    float* __restrict__ gbt, float* __restrict__ gwc, float* __restrict__ gbc) {
  const int npair = Co * Nt;
  const int nout = 2 * Nt + Co * Ci + Co;
  for (int q = threadIdx.x; q < nout; q += kThreads) {
    double sum = 0.0;
    if (q < 2 * Nt) {                            // gWt[t] (q < Nt) or gbt[t]
      const int t = q < Nt ? q : q - Nt;
      for (int o = 0; o < Co; ++o)
        for (int i = 0; i < Ci; ++i)
          sum += (double)wc[o * Ci + i] * (q < Nt ? G[(long long)(i + 1) * npair + o * Nt + t] : G[o * Nt + t]);
      float* dst = q < Nt ? gwt : gbt;
      if (dst != nullptr) dst[t] = (float)sum;
    } else if (q < 2 * Nt + Co * Ci) {           // gWc[o][i]
      const int oi = q - 2 * Nt, o = oi / Ci, i = oi - o * Ci;
      for (int t = 0; t < Nt; ++t)
        sum += (double)wt[t] * G[(long long)(i + 1) * npair + o * Nt + t] +
               (bt != nullptr ? (double)bt[t] * G[o * Nt + t] : 0.0);
      if (gwc != nullptr) gwc[oi] = (float)sum;
    } else {                                     // gbc[o]
      const int o = q - 2 * Nt - Co * Ci;
      for (int t = 0; t < Nt; ++t) sum += G[o * Nt + t];
      if (gbc != nullptr) gbc[o] = (float)sum;
    }
  }
}

template <int CI>
__global__ __launch_bounds__(kThreads) void pointwise_mlp2_kernel(
    int Ci, int H, int Co, long long np, const float* __restrict__ x, const float* __restrict__ W1,
    const float* __restrict__ b1, const float* __restrict__ W2, const float* __restrict__ b2,
    float* __restrict__ y) {
  const long long p = (long long)blockIdx.x * kThreads + threadIdx.x;
  const long long b = blockIdx.y;
  if (p >= np) return;
  float xv[CI];
#pragma unroll
  for (int i = 0; i < CI; ++i) xv[i] = (i < Ci) ? x[(b * Ci + i) * np + p] : 0.f;
  float acc[4];
#pragma unroll
  for (int o = 0; o < 4; ++o) acc[o] = (b2 != nullptr && o < Co) ? b2[o] : 0.f;
  for (int h = 0; h < H; ++h) {
    float s = (b1 != nullptr) ? b1[h] : 0.f;
#pragma unroll
    for (int i = 0; i < CI; ++i)
      if (i < Ci) s = fmaf(W1[h * Ci + i], xv[i], s);
    const float gh = gelu_f(s);
#pragma unroll
    for (int o = 0; o < 4; ++o)
      if (o < Co) acc[o] = fmaf(W2[o * H + h], gh, acc[o]);
  }
#pragma unroll
  for (int o = 0; o < 4; ++o)
    if (o < Co) y[(b * Co + o) * np + p] = acc[o];
}

}  // namespace

// number of partial-sum slots the workspace must hold (one per wave of the streaming kernel)
int bwd_pointwise_blocks(int B, int64_t N) {
  (void)B; (void)N;
  return 4096;
}

// The tiles of the wide kernel for these widths, at most max_slots point ranges of partial sums.  The waves of a block
// share out gW so that a wave's accumulators, the values of a step and the sums in doubles fit 256 registers (4 x 8
// tiles per wave spilled 82 of them).
hipError_t launch_bwd_wide(const float* z, const float* gout, const float* x, float* gz_out, double* part, int* nslots,
                           int max_slots, int B, int Ci, int Co, int64_t N, int act, int mse_target, double mse_scale,
                           hipStream_t s) {
  if (Ci > 32 || Co > 32) return hipErrorInvalidValue;
  const int ot = Ci <= 8 ? (Co <= 8 ? 2 : Co <= 20 ? 5 : 4) : (Ci <= 24 && Co <= 24 ? 3 : 2);
  const int it = Ci <= 8 ? 2 : (ot == 3 ? 6 : 8);
  const int ngrp = Co <= 4 * ot ? 1 : Co <= 8 * ot ? 2 : 4, per_block = 4 / ngrp;
  const int64_t steps = ((N + 63) / 64) * B;
  int64_t nb = ((steps + per_block - 1) / per_block + 7) / 8 * 8;       // a multiple of 8: the kernel's step ranges
  if (nb > max_slots / per_block) nb = max_slots / per_block;
  if (nb > 1024) nb = 1024;
  *nslots = (int)nb * per_block;
  const bool stream = (int64_t)B * Co * N * 4 >= kStreamBytes;
  // a lane's four points within an entry, and 32-bit offsets over four rows of one: else every wave reads all of x
  const bool ahead = N >= 4 && N <= (1ll << 27);
#define FNO_BPX(OTV, ITV, NGV)                                                                                         \
  do {                                                                                                                 \
    if (stream)                                                                                                        \
      hipLaunchKernelGGL((bwd_pointwise_wide_kernel<OTV, ITV, NGV, true>), dim3((unsigned)nb), dim3(kThreads), 0, s,   \
                         z, gout, x, gz_out, part, B, Ci, Co, (long long)N, act, mse_target, (float)mse_scale, ngrp);  \
    else                                                                                                               \
      hipLaunchKernelGGL((bwd_pointwise_wide_kernel<OTV, ITV, NGV, false>), dim3((unsigned)nb), dim3(kThreads), 0, s,  \
                         z, gout, x, gz_out, part, B, Ci, Co, (long long)N, act, mse_target, (float)mse_scale, ngrp);  \
  } while (0)
  if (it == 2) { if (ot == 2) FNO_BPX(2, 2, 0); else if (ot == 5) FNO_BPX(5, 2, 0); else FNO_BPX(4, 2, 0); }
  else if (it == 6) { if (ngrp == 2 && ahead) FNO_BPX(3, 6, 2); else FNO_BPX(3, 6, 0); }
  else if (ngrp == 4 && ahead) FNO_BPX(2, 8, 4);
  else FNO_BPX(2, 8, 0);
#undef FNO_BPX
  return hipGetLastError();
}

hipError_t launch_bwd_pointwise(const float* z, const float* gout, const float* x, float* gz_out,
                                double* part, int* nslots, int B, int Ci, int Co, int64_t N, int act,
                                int mse_target, double mse_scale, hipStream_t s) {
  const bool aligned = ((reinterpret_cast<uintptr_t>(z) | reinterpret_cast<uintptr_t>(gout) |
                         reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(gz_out)) & 15) == 0;
  if (Ci == Co && Co % 4 == 0 && Co <= 20 && N % 64 == 0 && aligned) {
    const int64_t steps = (N / 64) * B;
    int64_t nb = ((steps + 3) / 4 + 7) / 8 * 8;      // a multiple of 8: see the kernel's step ranges
    if (nb > 1024) nb = 1024;
    *nslots = (int)nb * 4;
    const dim3 grid((unsigned)nb);
    const bool stream = (int64_t)B * Co * N * 4 >= kStreamBytes;      // each tensor is touched once
    switch (Co / 4) {
#define FNO_BPW(CTV)                                                                               \
  case CTV:                                                                                        \
    if (stream)                                                                                    \
      hipLaunchKernelGGL((bwd_pointwise_mfma_kernel<CTV, true>), grid, dim3(kThreads), 0, s, z, gout, x,  \
                         gz_out, part, B, (long long)N, act, mse_target, (float)mse_scale);        \
    else                                                                                           \
      hipLaunchKernelGGL((bwd_pointwise_mfma_kernel<CTV, false>), grid, dim3(kThreads), 0, s, z, gout, x, \
                         gz_out, part, B, (long long)N, act, mse_target, (float)mse_scale);        \
    break;
      FNO_BPW(1) FNO_BPW(2) FNO_BPW(3) FNO_BPW(4) FNO_BPW(5)
#undef FNO_BPW
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  return launch_bwd_wide(z, gout, x, gz_out, part, nslots, bwd_pointwise_blocks(B, N), B, Ci, Co, N, act, mse_target,
                         mse_scale, s);
}

hipError_t launch_reduce_partials(const double* part, int nblk, int Co, int Ci, float* gW,
                                  float* gb, int accumulate, hipStream_t s) {
  const int npairs = Co * Ci + Co;
  hipLaunchKernelGGL(reduce_partials_kernel, dim3((npairs + kRedPairs - 1) / kRedPairs),
                     dim3(kRedPairs * kRedGroups), 0, s, part, nblk, Co, Ci, gW, gb, accumulate);
  return hipGetLastError();
}

hipError_t launch_pointwise_linear(int B, int Ci, int Co, int64_t np, const float* x, const float* W,
                                   const float* bias, float* y, hipStream_t s) {
  const int64_t nb = (np + kThreads - 1) / kThreads;
  if (nb > 0x7fffffffLL || B > 65535 || Co > 32) return hipErrorInvalidValue;
  if (nb == 0 || B == 0) return hipSuccess;
  if (np % 4 == 0 && Co <= 20 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & 15) == 0) {
    const int64_t np4 = np / 4;
    dim3 grid4((unsigned)((np4 + kThreads - 1) / kThreads), (unsigned)B);
    if (Co <= 8)
      hipLaunchKernelGGL((pointwise_linear_v4_kernel<8>), grid4, dim3(kThreads), 0, s, Ci, Co,
                         (long long)np4, reinterpret_cast<const v4f*>(x), W, bias,
                         reinterpret_cast<v4f*>(y));
    else
      hipLaunchKernelGGL((pointwise_linear_v4_kernel<20>), grid4, dim3(kThreads), 0, s, Ci, Co,
                         (long long)np4, reinterpret_cast<const v4f*>(x), W, bias,
                         reinterpret_cast<v4f*>(y));
    return hipGetLastError();
  }
  dim3 grid((unsigned)nb, (unsigned)B);
  if (Co <= 8)
    hipLaunchKernelGGL((pointwise_linear_kernel<8>), grid, dim3(kThreads), 0, s, Ci, Co,
                       (long long)np, x, W, bias, y);
  else if (Co <= 20)
    hipLaunchKernelGGL((pointwise_linear_kernel<20>), grid, dim3(kThreads), 0, s, Ci, Co,
                       (long long)np, x, W, bias, y);
  else
    hipLaunchKernelGGL((pointwise_linear_kernel<32>), grid, dim3(kThreads), 0, s, Ci, Co,
                       (long long)np, x, W, bias, y);
  return hipGetLastError();
}

// The fp32 adjoint of the projection takes hidden widths that are whole 32-row blocks, one wave
// each, and tiles whose (c_in + c_out) x 64 values the block's threads stage in kMlpStage loads.
bool mlp2_mfma_fits(int Ci, int H, int Co) {
  if (H % 32 != 0 || H < 32 || H > 256 || Ci > 31 || Co > 4 || Ci < 1 || Co < 1) return false;
  return Ci + Co <= kMlpStage * (H / 32);
}

size_t mlp2_bwd_mfma_lds(int Ci, int H, int Co) {
  const int nw = H / 32;
  size_t floats = (size_t)32 * kMlpXS + (size_t)4 * kMlpTile + (size_t)nw * 32 * kMlpTurn + (size_t)nw * Ci * kMlpXS +
                  (size_t)4 * H;
  floats += floats & 1;
  return floats * 4 + ((size_t)H * (Ci + 1) + (size_t)Co * H + Co) * 8;
}

// LDS of the projection: the weights' three parts in operand order (a channel of ones joins the input channels) and W2
size_t mlp2_split_lds(int Ci, int H, int Co) {
  const size_t nh = (H + 31) / 32;
  return nh * ((Ci + 16) / 16) * 3 * 64 * 16 + (size_t)(Co == 1 ? 1 : 4) * nh * 32 * 4;
}

hipError_t launch_pointwise_mlp2(int B, int Ci, int H, int Co, int64_t np, const float* x,
                                 const float* W1, const float* b1, const float* W2,
                                 const float* b2, float* y, hipStream_t s) {
  const int64_t nb = (np + kThreads - 1) / kThreads;
  if (nb > 0x7fffffffLL || B > 65535 || Co > 4 || Ci > 32) return hipErrorInvalidValue;
  if (nb == 0 || B == 0) return hipSuccess;
  if (mlp2_split_lds(Ci, H, Co) <= (size_t)(150 * 1024)) {
    const size_t lds = mlp2_split_lds(Ci, H, Co);
    const int64_t tiles = (int64_t)B * ((np + 31) / 32), room = (int64_t)(160 * 1024 / lds);
    const int64_t most = 256 * (room < 4 ? room : 4);
    const unsigned nblk = (unsigned)((tiles + 3) / 4 < most ? (tiles + 3) / 4 : most);
#define FNO_MLPF(NSV, COV)                                                                              \
  hipLaunchKernelGGL((mlp2_fwd_split_kernel<NSV, COV>), dim3(nblk), dim3(kThreads), lds, s, B, Ci, H, Co, \
                     (long long)np, x, W1, b1, W2, b2, y)
#define FNO_MLPF_C(NSV) do { if (Co == 1) FNO_MLPF(NSV, 1); else FNO_MLPF(NSV, 4); } while (0)
    if (Ci < 8) FNO_MLPF_C(4);
    else if (Ci < 16) FNO_MLPF_C(8);
    else if (Ci < 24) FNO_MLPF_C(12);
    else if (Ci < 32) FNO_MLPF_C(16);
    else FNO_MLPF_C(18);
#undef FNO_MLPF_C
#undef FNO_MLPF
    return hipGetLastError();
  }
  dim3 grid((unsigned)nb, (unsigned)B);
  if (Ci <= 20)
    hipLaunchKernelGGL((pointwise_mlp2_kernel<20>), grid, dim3(kThreads), 0, s, Ci, H, Co,
                       (long long)np, x, W1, b1, W2, b2, y);
  else
    hipLaunchKernelGGL((pointwise_mlp2_kernel<32>), grid, dim3(kThreads), 0, s, Ci, H, Co,
                       (long long)np, x, W1, b1, W2, b2, y);
  return hipGetLastError();
}

hipError_t launch_time_lift(int B, int Ci, int Co, int64_t np, int Nt, const float* a, const float* wt,
                            const float* bt, const float* wc, const float* bc, float* out, hipStream_t s) {
  const int nt4 = (Nt + 3) / 4;
  const int64_t nb = (np * nt4 + kThreads - 1) / kThreads;
  if (nb > 0x7fffffffLL || B > 65535 || Co > 32) return hipErrorInvalidValue;
  if (nb == 0 || B == 0) return hipSuccess;
  // float4 stores need whole quads per row and an aligned tensor
  if ((Nt & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) != 0) return hipErrorInvalidValue;
  dim3 grid((unsigned)nb, (unsigned)B);
  // the lifted tensor is written once: as a stream when it is larger than the caches
  const bool stream = (int64_t)B * Co * np * Nt * 4 >= kStreamBytes;
#define FNO_TL(COV)                                                                                          \
  do {                                                                                                       \
    if (stream)                                                                                              \
      hipLaunchKernelGGL((time_lift_kernel<COV, true>), grid, dim3(kThreads), 0, s, Ci, Co, (long long)np, Nt, a, \
                         wt, bt, wc, bc, out);                                                               \
    else                                                                                                     \
      hipLaunchKernelGGL((time_lift_kernel<COV, false>), grid, dim3(kThreads), 0, s, Ci, Co, (long long)np, Nt, a, \
                         wt, bt, wc, bc, out);                                                               \
  } while (0)
  if (Co <= 8) FNO_TL(8); else if (Co <= 20) FNO_TL(20); else FNO_TL(32);
#undef FNO_TL
  return hipGetLastError();
}

size_t time_lift_bwd_workspace_bytes(int Ci, int Co, int Nt) {
  return ((size_t)kLiftChunks + 1) * (size_t)(Ci + 1) * Co * Nt * sizeof(double);
}

hipError_t launch_time_lift_bwd(int B, int Ci, int Co, int64_t S, int Nt, const float* a, const float* wt,
                                const float* bt, const float* wc, const float* g, float* gwt, float* gbt,
                                float* gwc, float* gbc, void* ws, hipStream_t s) {
  if (Ci > 8 || B > kLiftChunks || S <= 0) return hipErrorInvalidValue;
  const int npair = Co * Nt, nent = (Ci + 1) * npair;
  int cpb = (int)((S + 511) / 512);               // chunks per batch entry: at least 512 positions each
  if (cpb > kLiftChunks / B) cpb = kLiftChunks / B;
  if (cpb < 1) cpb = 1;
  const int nchunk = B * cpb;
  double* part = static_cast<double*>(ws);
  double* G = part + (size_t)kLiftChunks * nent;
  const dim3 grid((unsigned)((npair + kThreads - 1) / kThreads), (unsigned)nchunk);
  // the cotangent of the lifted tensor is read once: as a stream when it is larger than the caches
  const bool stream = (int64_t)B * Co * S * Nt * 4 >= kStreamBytes;
#define FNO_TLB(CIV)                                                                                         \
  do {                                                                                                       \
    if (stream)                                                                                              \
      hipLaunchKernelGGL((time_lift_bwd_kernel<CIV, true>), grid, dim3(kThreads), 0, s, Ci, Co, (long long)S, Nt, \
                         cpb, a, g, part);                                                                   \
    else                                                                                                     \
      hipLaunchKernelGGL((time_lift_bwd_kernel<CIV, false>), grid, dim3(kThreads), 0, s, Ci, Co, (long long)S, Nt, \
                         cpb, a, g, part);                                                                   \
  } while (0)
  if (Ci == 1) FNO_TLB(1); else if (Ci == 2) FNO_TLB(2); else if (Ci <= 4) FNO_TLB(4); else FNO_TLB(8);
#undef FNO_TLB
  hipLaunchKernelGGL(time_lift_bwd_reduce_kernel, dim3((nent + 31) / 32), dim3(kThreads), 0, s, part, nchunk,
                     nent, G);
  hipLaunchKernelGGL(time_lift_bwd_final_kernel, dim3(1), dim3(kThreads), 0, s, Ci, Co, Nt, G, wt, bt, wc, gwt,
                     gbt, gwc, gbc);
  return hipGetLastError();
}

size_t rel_l2_workspace_bytes() { return (size_t)(2 * kLossBlocks + 1) * sizeof(double); }

hipError_t launch_rel_l2(int64_t n, const float* pred, const float* target, float* loss, float* grad,
                         double* ws, hipStream_t s) {
  if (n <= 0) return hipErrorInvalidValue;
  int nblk = (int)((n + kThreads - 1) / kThreads);
  if (nblk > kLossBlocks) nblk = kLossBlocks;
  double* scale = ws + 2 * kLossBlocks;
  hipLaunchKernelGGL(rel_l2_partial_kernel, dim3(nblk), dim3(kThreads), 0, s, (long long)n, pred, target, ws);
  hipLaunchKernelGGL(rel_l2_final_kernel, dim3(1), dim3(kThreads), 0, s, ws, nblk, loss, scale);
  if (grad != nullptr) {
    int64_t gb = (n + kThreads - 1) / kThreads;
    if (gb > 65536) gb = 65536;
    hipLaunchKernelGGL(rel_l2_grad_kernel, dim3((unsigned)gb), dim3(kThreads), 0, s, (long long)n, pred, target,
                       scale, grad);
  }
  return hipGetLastError();
}

hipError_t launch_adam(int64_t n, float* p, const float* g, float* m, float* v, double lr, double beta1,
                       double beta2, double eps, int step, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const float c1 = (float)(1.0 / (1.0 - pow(beta1, (double)step)));
  const float c2 = (float)(1.0 / (1.0 - pow(beta2, (double)step)));
  int64_t nb = (n + kThreads - 1) / kThreads;
  if (nb > 65536) nb = 65536;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)nb), dim3(kThreads), 0, s, (long long)n, p, g, m, v, (float)lr,
                     (float)beta1, (float)(1.0 - beta1), (float)beta2, (float)(1.0 - beta2), (float)eps, c1, c2);
  return hipGetLastError();
}

// doubles of partial sums + floats of a transposed weight
size_t pointwise_bwd_workspace_bytes(int Ci, int H, int Co) {
  const size_t lin = (size_t)2048 * ((size_t)Co * Ci + Co) * 8 + (size_t)Co * Ci * 4 + 64;
  const size_t mlp = (size_t)kMlpBlocks * ((size_t)H * (Ci + 1) + (size_t)Co * H + Co) * 8 + 64;
  return lin > mlp ? lin : mlp;
}

hipError_t launch_pointwise_linear_bwd(int B, int Ci, int Co, int64_t N, const float* x, const float* W,
                                       const float* g, float* gx, float* gW, float* gb, void* ws,
                                       hipStream_t s) {
  if (N <= 0) return hipErrorInvalidValue;
  double* part = static_cast<double*>(ws);
  if (gW != nullptr || gb != nullptr) {
    int nblk = 0;
    const hipError_t e = launch_bwd_wide(g, g, x, nullptr, part, &nblk, 2048, B, Ci, Co, N, 0, 0, 0.0, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((Co * Ci + Co + kRedPairs - 1) / kRedPairs),
                       dim3(kRedPairs * kRedGroups), 0, s, part, nblk, Co, Ci, gW, gb, 0);
  }
  if (gx != nullptr) {
    float* wt = reinterpret_cast<float*>(part + (size_t)2048 * (Co * Ci + Co));
    hipLaunchKernelGGL(transpose_kernel, dim3((Co * Ci + 255) / 256), dim3(256), 0, s, W, wt, Co, Ci);
    const hipError_t e = launch_pointwise_linear(B, Co, Ci, N, g, wt, nullptr, gx, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t launch_pointwise_mlp2_bwd(int B, int Ci, int H, int Co, int64_t N, const float* x, const float* W1,
                                     const float* b1, const float* W2, const float* g, float* gx, float* gW1,
                                     float* gb1, float* gW2, float* gb2, void* ws, hipStream_t s) {
  if (Ci > 32 || Co > 4 || N <= 0) return hipErrorInvalidValue;
  const int nsum = H * (Ci + 1) + Co * H + Co;
  if (Co == 1 && H <= 256) {
    const MlpBwd f{B, Ci, H, (H + 31) / 32, (long long)N};
    // two waves where groups of hidden units are few, and with 32 channels, whose wave takes its two column blocks one by one,
    // as far as blocks of eight waves go: 32 -> 128 -> 1 at 2 million points 572 us, with one wave a group 776 (20 channels
    // 545 and 500; before the sums were kept in place)
    const int npg = f.nwh <= 2 || (Ci == 32 && f.nwh <= 4) ? 2 : 1, nw = f.nwh * npg;
    const int64_t tiles = (int64_t)B * ((N + 63) / 64);
    const int nblk = (int)(tiles < kMlpBlocks ? tiles : kMlpBlocks);
    double* part = static_cast<double*>(ws);
#define FNO_MLPB(NSV, NPGV, NWV)                                                                                  \
  hipLaunchKernelGGL((mlp2_bwd_split_kernel<NSV, NPGV, mlp_stage(NSV, NWV)>), dim3((unsigned)nblk), dim3(64 * nw), \
                     mlp_bwd_lds(NSV, NPGV, nw), s, f, x, W1, b1, W2, g, gx, part)
#define FNO_MLPB_N(NSV) \
  do { if (npg == 2) FNO_MLPB(NSV, 2, 2); else if (nw == 3) FNO_MLPB(NSV, 1, 3); else FNO_MLPB(NSV, 1, 4); } while (0)
    if (Ci < 8) FNO_MLPB_N(4);
    else if (Ci < 16) FNO_MLPB_N(8);
    else if (Ci < 24) FNO_MLPB_N(12);
    else if (Ci < 32) FNO_MLPB_N(16);
    else if (npg == 2 && nw >= 6) FNO_MLPB(18, 2, 6);
    else FNO_MLPB_N(18);
#undef FNO_MLPB_N
#undef FNO_MLPB
    hipLaunchKernelGGL(reduce_ranges_kernel, dim3((nsum + kRedPairs - 1) / kRedPairs),
                       dim3(kRedPairs * kRedGroups), 0, s, part, nblk, H * Ci, H, Co * H, Co, gW1, gb1, gW2, gb2);
    return hipGetLastError();
  }
  if (Co > 1 && mlp2_mfma_fits(Ci, H, Co) && mlp2_bwd_mfma_lds(Ci, H, Co) <= (size_t)(150 * 1024)) {
    const int nw = H / 32;
    const size_t lds = mlp2_bwd_mfma_lds(Ci, H, Co);
    const int64_t tiles = (int64_t)B * ((N + kMlpTile - 1) / kMlpTile);
    const int nblk = (int)(tiles < kMlpBlocks ? tiles : kMlpBlocks);
    double* part = static_cast<double*>(ws);
    if (Ci <= 21)
      hipLaunchKernelGGL((mlp2_bwd_mfma_kernel<11>), dim3((unsigned)nblk), dim3(64 * nw), lds, s, B, Ci, H, Co, (long long)N,
                         x, W1, b1, W2, g, gx, part);
    else
      hipLaunchKernelGGL((mlp2_bwd_mfma_kernel<16>), dim3((unsigned)nblk), dim3(64 * nw), lds, s, B, Ci, H, Co, (long long)N,
                         x, W1, b1, W2, g, gx, part);
    hipLaunchKernelGGL(reduce_ranges_kernel, dim3((nsum + kRedPairs - 1) / kRedPairs),
                       dim3(kRedPairs * kRedGroups), 0, s, part, nblk, H * Ci, H, Co * H, Co, gW1, gb1, gW2, gb2);
    return hipGetLastError();
  }
  size_t lds_floats = (size_t)(Ci + Co + 2 * kMlpChunk) * (kThreads + 1);
  lds_floats += lds_floats & 1;
  const size_t lds = lds_floats * 4 + (size_t)nsum * 8;
  if (lds > (size_t)(150 * 1024)) return hipErrorInvalidValue;
  const int64_t tiles = (int64_t)B * ((N + kThreads - 1) / kThreads);
  const int nblk = (int)(tiles < kMlpBlocks ? tiles : kMlpBlocks);
  double* part = static_cast<double*>(ws);
  if (Ci <= 20)
    hipLaunchKernelGGL((mlp2_bwd_kernel<20>), dim3((unsigned)nblk), dim3(kThreads), lds, s, B, Ci, H, Co,
                       (long long)N, x, W1, b1, W2, g, gx, part);
  else
    hipLaunchKernelGGL((mlp2_bwd_kernel<32>), dim3((unsigned)nblk), dim3(kThreads), lds, s, B, Ci, H, Co,
                       (long long)N, x, W1, b1, W2, g, gx, part);
  hipLaunchKernelGGL(reduce_ranges_kernel, dim3((nsum + kRedPairs - 1) / kRedPairs),
                     dim3(kRedPairs * kRedGroups), 0, s, part, nblk, H * Ci, H, Co * H, Co, gW1, gb1, gW2, gb2);
  return hipGetLastError();
}


}  // namespace fno
