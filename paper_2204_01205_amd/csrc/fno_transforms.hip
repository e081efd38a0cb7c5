// HIP kernels of libfno for gfx950 (wave64).  What they compute, in the paper's terms
// (arXiv 2204.01205): the transform F of eq. (3) restricted to the kept low-frequency modes,
// applied axis by axis (separability, Sec. 2.3); the per-mode weight multiplication of R_phi;
// the inverse transform; and the pointwise part of the block update of eq. (2) / Sec. 2.4,
// sigma(W x + b + K x), fused into the last inverse stage.  The adjoint kernels implement the
// transposed chain (eq. (7)) and the sum-reductions that are the adjoint of broadcasting W
// and b (Sec. 2.1).
//
// Every axis of length N is split N = P * M: M-point FFTs held in registers (fft_reg.h) over
// the residue classes n = P*n1 + n2, then a P-term twiddle combine evaluated only at the kept
// frequencies.  M = 1 degenerates to a dense truncated DFT and covers any axis length.
//
// This file: twiddle tables, the forward (t, z) kernels, the pruned transforms along y and x,
// and the per-mode channel mix with its adjoint.
#include "fno_device.h"

namespace fno {

namespace {

// ------------------------------------------------------------------------------------------
// Twiddle tables (double-precision sincospi, rounded once to float)
// ------------------------------------------------------------------------------------------
// All tables of a plan in one launch: blockIdx.y picks the table.  An axis table holds
// w_N^(k_j n2) for the kept frequencies k_j and the residue classes n2 < P; the t table (L = 0)
// holds w_Nt^(kt n) for kt < npos (= mt), n < N (= Nt); the folded table is described at FoldPlan.
__global__ void plan_tables_kernel(TableSet ts) {
  const TableDesc t = ts.t[blockIdx.y];
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (t.L > 0) {
    if (idx >= t.L * t.P) return;
    const int j = idx / t.P, n2 = idx % t.P;
    const long long k = kfreq(j, t.L, t.npos);
    long long r = (k * n2) % t.N;
    if (r < 0) r += t.N;
    double s, c;
    sincospi(-2.0 * double(r) / double(t.N), &s, &c);
    t.tw[idx] = make_float2(float(c), float(s));
  } else if (t.L < 0) {
    const int rows = -t.L, stride = t.P;
    if (idx >= rows * (stride + 1)) return;
    const bool phase = idx >= rows * stride;             // the last `rows` entries: exp(i pi k / N)
    const int k = phase ? idx - rows * stride : idx / stride, n = phase ? 0 : idx - k * stride;
    float* f = reinterpret_cast<float*>(t.tw);
    double s = 0.0, c = 0.0;
    if (2 * n < t.N) {
      // angle pi r / N; k and 2 n + 1 are below 2^13
      const unsigned r = ((unsigned)k * (phase ? 1u : 2u * n + 1u)) % (2u * t.N);
      sincospi(double(r) / double(t.N), &s, &c);
      if (2 * n + 1 == t.N && !phase) c *= 0.5;
    }
    if (phase) {
      reinterpret_cast<double2*>(f + 2 * rows * stride)[k] = make_double2(c, s);
    } else {
      f[idx] = float(c);
      f[rows * stride + idx] = float(s);
    }
  } else {
    if (idx >= t.N * t.npos) return;
    const int kt = idx / t.N, n = idx % t.N;
    const long long r = ((long long)kt * n) % t.N;
    double s, c;
    sincospi(-2.0 * double(r) / double(t.N), &s, &c);
    t.tw[idx] = make_float2(float(c), float(s));
  }
}

// ------------------------------------------------------------------------------------------
// Forward (t, z): one block transforms `ppb` contiguous (b,c,nx,ny) planes of Nz x Nt reals
// ------------------------------------------------------------------------------------------
// sum_i w[i] * x[i * xs] over n terms, eight at a time so that their reads are issued together
// (a term-by-term loop waits for every read before the next one goes out)
__device__ __forceinline__ float2 combine_terms(const float2* w, const float2* x, int xs, int n) {
  float2 acc0 = make_float2(0.f, 0.f), acc1 = make_float2(0.f, 0.f);
  int i = 0;
  for (; i + 8 <= n; i += 8) {
    float2 wv[8], xv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      wv[u] = w[i + u];
      xv[u] = x[(i + u) * xs];
    }
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      acc0 = cfma(wv[u], xv[u], acc0);
      acc1 = cfma(wv[u + 1], xv[u + 1], acc1);
    }
  }
  for (; i < n; ++i) acc0 = cfma(w[i], x[i * xs], acc0);
  return make_float2(acc0.x + acc1.x, acc0.y + acc1.y);
}

// Row stride of the z-rows in LDS, in complex values: 1 mod 16, so that the rows of the kt bins
// that adjacent lanes combine start 2 banks apart.
__host__ __device__ inline int tz_row_stride(int Nz) { return Nz + ((17 - (Nz & 15)) & 15); }

template <int MZ>
__global__ __launch_bounds__(kThreads) void tz_fwd_kernel(
    const float* __restrict__ x, float2* __restrict__ out, const float2* __restrict__ twt,
    const float2* __restrict__ twz, long long planes, int Nz, int Nt, int Lz, int nposz, int mt,
    int ppb) {
  HIP_DYNAMIC_SHARED(float, smem)
  const int Pz = Nz / MZ;
  const int sS = Nt + 1;                       // row stride of S in floats
  const int sT = tz_row_stride(Nz);            // row stride of T in float2
  float* S = smem;                             // [ppb][Nz][sS]
  int s_floats = ppb * Nz * sS;
  s_floats += (s_floats & 1);
  float2* T = reinterpret_cast<float2*>(smem + s_floats);   // [ppb][mt][sT]
  const int tid = threadIdx.x;
  const long long plane0 = xcd_contiguous_item(blockIdx.x, gridDim.x) * ppb;   // grid: a multiple of 8
  if (plane0 >= planes) return;
  const int np = (int)min((long long)ppb, planes - plane0);
  const int plane_elems = Nz * Nt;

  // 1. coalesced load of the planes
  const float* src = x + plane0 * plane_elems;
  const int nelem = np * plane_elems;
  for (int i0 = tid; i0 < nelem; i0 += 8 * kThreads) {     // eight loads in flight per thread
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = i0 + u * kThreads;
      v[u] = idx < nelem ? src[idx] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = i0 + u * kThreads;
      if (idx < nelem) {
        const int row = idx / Nt, t = idx - row * Nt;
        S[row * sS + t] = v[u];
      }
    }
  }
  __syncthreads();

  // 2. real-to-complex transform over t, kept bins only: one thread per z-row
  for (int row = tid; row < np * Nz; row += kThreads) {
    const int p = row / Nz, z = row - p * Nz;
    const float* srow = S + row * sS;
    for (int kt0 = 0; kt0 < mt; kt0 += 4) {
      float2 acc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = make_float2(0.f, 0.f);
      int n = 0;
      for (; n + 4 <= Nt; n += 4) {         // four points per pass: their reads go out together
        float v[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) v[h] = srow[n + h];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (kt0 + u < mt) {
            float2 w[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) w[h] = twt[(kt0 + u) * Nt + n + h];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
              acc[u].x = fmaf(v[h], w[h].x, acc[u].x);
              acc[u].y = fmaf(v[h], w[h].y, acc[u].y);
            }
          }
        }
      }
      for (; n < Nt; ++n) {
        const float v = srow[n];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (kt0 + u < mt) {
            const float2 w = twt[(kt0 + u) * Nt + n];
            acc[u].x = fmaf(v, w.x, acc[u].x);
            acc[u].y = fmaf(v, w.y, acc[u].y);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (kt0 + u < mt) T[(p * mt + kt0 + u) * sT + z] = acc[u];
    }
  }
  __syncthreads();

  // 3. MZ-point FFTs over the residue classes of z, in place
  if constexpr (MZ > 1) {
    for (int idx = tid; idx < np * mt * Pz; idx += kThreads) {
      const int n2 = idx % Pz, col = idx / Pz;          // col = p*mt + kt
      float2* base = T + col * sT + n2;
      float2 a[MZ];
#pragma unroll
      for (int n1 = 0; n1 < MZ; ++n1) a[n1] = base[Pz * n1];
      fft_reg<MZ, -1>(a);
#pragma unroll
      for (int m = 0; m < MZ; ++m) base[Pz * m] = a[bitrev<MZ>(m)];
    }
    __syncthreads();
  }

  // 4. twiddle combine at the kept z-frequencies
  for (int idx = tid; idx < np * Lz * mt; idx += kThreads) {
    const int kt = idx % mt;
    const int jz = (idx / mt) % Lz;
    const int p = idx / (mt * Lz);
    const int mj = posmod(kfreq(jz, Lz, nposz), MZ);
    const float2* base = T + (p * mt + kt) * sT + Pz * mj;
    const float2* w = twz + jz * Pz;
    out[((plane0 + p) * Lz + jz) * mt + kt] = combine_terms(w, base, 1, Pz);
  }
}

// ------------------------------------------------------------------------------------------
// Forward (t, z) for power-of-two Nt (16, 32, 64): float4 loads issued up front, the t stage as
// a real-input FFT of one z-row per thread (an NT/2-point complex FFT of the even/odd samples
// plus the split step), z twiddles in LDS.
// ------------------------------------------------------------------------------------------
// X[K] = E[K] + w^K O[K],  E = (Z[K] + conj Z[H-K]) / 2,  O = (Z[K] - conj Z[H-K]) / (2i)
template <int NT, int K>
__device__ __forceinline__ void rfft_bin(const float2 (&zc)[NT / 2], int mt, float2 (&X)[NT / 2 + 1]) {
  constexpr int H = NT / 2;
  if (K < mt) {
    const float2 zk = zc[bitrev<H>(K % H)];
    const float2 zm = zc[bitrev<H>((H - K) % H)];
    const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    const float2 od = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
    X[K] = cadd(e, mul_root<NT, K, -1>(od));
  }
}

template <int NT, int... Ks>
__device__ __forceinline__ void rfft_bins(const float2 (&zc)[NT / 2], int mt, float2 (&X)[NT / 2 + 1],
                                          std::integer_sequence<int, Ks...>) {
  (rfft_bin<NT, Ks>(zc, mt, X), ...);
}

// Bins 0..mt-1 of the real-input transform of one row of NT floats held as NT/4 float4 quads.
template <int NT>
__device__ __forceinline__ void rfft_row_bins(const float4 (&quads)[NT / 4], int mt, float2 (&X)[NT / 2 + 1]) {
  constexpr int H = NT / 2;
  float2 zc[H];
#pragma unroll
  for (int m4 = 0; m4 < NT / 4; ++m4) {
    zc[2 * m4] = make_float2(quads[m4].x, quads[m4].y);
    zc[2 * m4 + 1] = make_float2(quads[m4].z, quads[m4].w);
  }
  fft_reg<H, -1>(zc);
  rfft_bins<NT>(zc, mt, X, std::make_integer_sequence<int, H + 1>{});
}

// The same bins by a radix-4 split in time, for NT = 16 and 32: with n = 4 m + p,
//   X[K] = sum_{p<4} w_NT^{pK} D_p[K mod R],   D_p[q] = sum_{m<R} x[4m+p] w_R^{qm},  R = NT / 4,
// where each D_p is the transform of R real samples (the p-th component of the row's quads): only
// its bins 0..R/2 are computed, the others are their conjugates, and bins 0 and R/2 are real.
// About half the arithmetic of the packed complex transform above when few bins are kept.
// Forward transform of 4 / 8 real samples, bins 0..R/2 (w = exp(-2 pi i / R)).
__device__ __forceinline__ void real_dft(const float (&a)[4], float2 (&D)[3]) {
  const float s02 = a[0] + a[2], d02 = a[0] - a[2], s13 = a[1] + a[3], d13 = a[1] - a[3];
  D[0] = make_float2(s02 + s13, 0.f);
  D[1] = make_float2(d02, -d13);
  D[2] = make_float2(s02 - s13, 0.f);
}
__device__ __forceinline__ void real_dft(const float (&a)[8], float2 (&D)[5]) {
  constexpr float r = 0.70710678118654752440f;
  const float s04 = a[0] + a[4], d04 = a[0] - a[4], s26 = a[2] + a[6], d26 = a[2] - a[6];
  const float s15 = a[1] + a[5], d15 = a[1] - a[5], s37 = a[3] + a[7], d37 = a[3] - a[7];
  const float e0 = s04 + s26, e1 = s04 - s26, o0 = s15 + s37, o1 = s15 - s37;
  const float u = (d15 - d37) * r, v = (d15 + d37) * r;
  D[0] = make_float2(e0 + o0, 0.f);
  D[1] = make_float2(d04 + u, -d26 - v);
  D[2] = make_float2(e1, -o1);
  D[3] = make_float2(d04 - u, d26 - v);
  D[4] = make_float2(e0 - o0, 0.f);
}

// acc += exp(-2 pi i IDX / NT) * v, v complex or (REAL) real-valued
template <int NT, int IDX, bool REAL>
__device__ __forceinline__ float2 add_rooted(float2 acc, float2 v) {
  constexpr int idx = ((IDX % NT) + NT) % NT;
  constexpr float c = float(ct_cos_frac(idx, NT));
  constexpr float s = float(-ct_sin_frac(idx, NT));
  if constexpr (idx == 0) {
    acc.x += v.x;
    if constexpr (!REAL) acc.y += v.y;
  } else if constexpr (2 * idx == NT) {
    acc.x -= v.x;
    if constexpr (!REAL) acc.y -= v.y;
  } else if constexpr (4 * idx == NT) {            // * (-i)
    if constexpr (!REAL) acc.x += v.y;
    acc.y -= v.x;
  } else if constexpr (4 * idx == 3 * NT) {        // * (+i)
    if constexpr (!REAL) acc.x -= v.y;
    acc.y += v.x;
  } else {
    acc.x = fmaf(c, v.x, acc.x);
    acc.y = fmaf(s, v.x, acc.y);
    if constexpr (!REAL) {
      acc.x = fmaf(-s, v.y, acc.x);
      acc.y = fmaf(c, v.y, acc.y);
    }
  }
  return acc;
}

template <int NT, int K>
__device__ __forceinline__ void rfft4_bin(const float2 (&D)[4][NT / 8 + 1], int mt, float2 (&X)[NT / 2 + 1]) {
  constexpr int R = NT / 4;
  constexpr int q = K % R;
  constexpr bool real_bin = (q == 0) || (2 * q == R);
  constexpr bool conj_bin = 2 * q > R;
  constexpr int qi = conj_bin ? R - q : q;
  if (K < mt) {
    float2 acc = make_float2(D[0][qi].x, real_bin ? 0.f : (conj_bin ? -D[0][qi].y : D[0][qi].y));
    acc = add_rooted<NT, 1 * K, real_bin>(acc, make_float2(D[1][qi].x, conj_bin ? -D[1][qi].y : D[1][qi].y));
    acc = add_rooted<NT, 2 * K, real_bin>(acc, make_float2(D[2][qi].x, conj_bin ? -D[2][qi].y : D[2][qi].y));
    acc = add_rooted<NT, 3 * K, real_bin>(acc, make_float2(D[3][qi].x, conj_bin ? -D[3][qi].y : D[3][qi].y));
    X[K] = acc;
  }
}

template <int NT, int... Ks>
__device__ __forceinline__ void rfft4_bins(const float2 (&D)[4][NT / 8 + 1], int mt, float2 (&X)[NT / 2 + 1],
                                           std::integer_sequence<int, Ks...>) {
  (rfft4_bin<NT, Ks>(D, mt, X), ...);
}

template <int NT>
__device__ __forceinline__ void rfft_row_bins_r4(const float4 (&quads)[NT / 4], int mt, float2 (&X)[NT / 2 + 1]) {
  constexpr int R = NT / 4;
  float2 D[4][R / 2 + 1];
  float a[R];
#pragma unroll
  for (int m = 0; m < R; ++m) a[m] = quads[m].x;
  real_dft(a, D[0]);
#pragma unroll
  for (int m = 0; m < R; ++m) a[m] = quads[m].y;
  real_dft(a, D[1]);
#pragma unroll
  for (int m = 0; m < R; ++m) a[m] = quads[m].z;
  real_dft(a, D[2]);
#pragma unroll
  for (int m = 0; m < R; ++m) a[m] = quads[m].w;
  real_dft(a, D[3]);
  rfft4_bins<NT>(D, mt, X, std::make_integer_sequence<int, NT / 2 + 1>{});
}

// Bins 0..mt-1 of the real-input transform of one row of NT floats for an even NT that is no
// power of two: the plain sums, with x[n] and x[NT-n] folded (cos is even, sin odd in n), all
// twiddles compile-time constants.
//   Re X[k] = x[0] + (-1)^k x[NT/2] + sum_{0<n<NT/2} (x[n] + x[NT-n]) cos(2 pi k n / NT)
//   Im X[k] =                       - sum_{0<n<NT/2} (x[n] - x[NT-n]) sin(2 pi k n / NT)
template <int NT, int IDX> constexpr float kCosFrac = float(ct_cos_frac(IDX, NT));      // cos(2 pi IDX / NT)
template <int NT, int IDX> constexpr float kNegSinFrac = float(-ct_sin_frac(IDX, NT)); // -sin(2 pi IDX / NT)

template <int NT, int K, int... Ns>
__device__ __forceinline__ float2 dense_bin(const float (&sm)[NT / 2], const float (&df)[NT / 2], float x0, float xh,
                                            std::integer_sequence<int, Ns...>) {
  float re = (K % 2 == 0) ? x0 + xh : x0 - xh, im = 0.f;
  ((Ns > 0 ? (void)(re = fmaf(kCosFrac<NT, (K * Ns) % NT>, sm[Ns], re),
                    im = fmaf(kNegSinFrac<NT, (K * Ns) % NT>, df[Ns], im))
           : (void)0),
   ...);
  return make_float2(re, im);
}

template <int NT, int... Ks>
__device__ __forceinline__ void dense_bins(const float (&sm)[NT / 2], const float (&df)[NT / 2], float x0, float xh, int mt,
                                           float2 (&X)[NT / 2 + 1], std::integer_sequence<int, Ks...>) {
  ((Ks < mt ? (void)(X[Ks] = dense_bin<NT, Ks>(sm, df, x0, xh, std::make_integer_sequence<int, NT / 2>{})) : (void)0), ...);
}

template <int NT>
__device__ __forceinline__ void rdft_row_bins_dense(const float (&x)[NT], int mt, float2 (&X)[NT / 2 + 1]) {
  constexpr int H = NT / 2;
  float sm[H], df[H];
  sm[0] = 0.f; df[0] = 0.f;
#pragma unroll
  for (int n = 1; n < H; ++n) { sm[n] = x[n] + x[NT - n]; df[n] = x[n] - x[NT - n]; }
  dense_bins<NT>(sm, df, x[0], x[H], mt, X, std::make_integer_sequence<int, H + 1>{});
}

// One thread per z-row (blockDim.x >= ppb * Nz).  The planes and the z twiddles go straight to
// LDS (16 bytes per lane, 1 KiB per wave instruction, nothing staged in registers).  Inside a
// row the quads are stored rotated by the row number so that the row-per-thread reads of the
// t stage spread over all banks; a wave's load still covers whole 128-byte lines.  The t-stage
// results wait in registers over a barrier so the complex tile T can reuse the LDS of S.
// Pz is a power of two and inv_mt = ceil(2^16 / mt) (shifts and a multiply instead of divisions).
// FULL: every bin of t is kept, so that the t stage needs no guards (128 x 16, 9 bins, 32 kept, 10.7 GB: 2530 us, 2626 with
// them).  PZC: log2 Pz at compile time (-1: taken from the arguments), where the LDS reads of the combine go out together:
// rows of more than 16 points (64 x 64, 32 kept, 9 bins, 2304 columns of 16 channels 141 -> 129 us; 128 x 32, 65536 columns
// of 20 channels, 24 kept, 4408 -> 4283); not shorter ones (128 x 16, 64 kept, 8 bins, 512 columns 37 us, 49 so).
template <int NT, int MZ, bool FULL, int PZC, bool STREAM>
__global__ __launch_bounds__(kThreads) void tz_fwd_fast_kernel(
    const float* __restrict__ x, float2* __restrict__ out, const float2* __restrict__ twz,
    long long planes, int Nz, int Lz, int nposz, int mt_rt, int ppb, int region_floats, int pzshift_rt, int inv_mt) {
  HIP_DYNAMIC_SHARED(float, smem)
  const int pzshift = PZC >= 0 ? PZC : pzshift_rt;
  const int mt = FULL ? NT / 2 + 1 : mt_rt;
  constexpr bool POW2 = (NT & (NT - 1)) == 0;  // else: an even length, rows unrotated, t stage as plain sums
  constexpr int QPR = POW2 ? NT / 4 : 1;       // quads per row
  constexpr int ROT = 16 / QPR > 0 ? 16 / QPR : 1;   // rows that share a rotation
  constexpr int H = NT / 2;
  const int Pz = 1 << pzshift;
  const int sT = tz_row_stride(Nz);            // row stride of T in float2
  float* S = smem;                             // [ppb * Nz] rows of QPR rotated quads
  float2* T = reinterpret_cast<float2*>(smem); // [ppb][mt][sT], same memory, later
  float2* TW = reinterpret_cast<float2*>(smem + region_floats);   // [Lz][Pz]
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;
  const int lane = tid & 63, wave = tid >> 6;
  const long long plane0 = xcd_contiguous_item(blockIdx.x, gridDim.x) * ppb;   // grid: a multiple of 8
  if (plane0 >= planes) return;
  const int np = (int)min((long long)ppb, planes - plane0);

  {
    const float4* src = reinterpret_cast<const float4*>(x + plane0 * Nz * NT);
    if constexpr (POW2) {
      const int tot4 = np * Nz * QPR;            // a multiple of 64 (checked on the host)
      for (int c0 = wave * 64; c0 < tot4; c0 += nthr) {
        const int p4 = c0 + lane;
        const int zl = p4 / QPR, sl = p4 - zl * QPR;
        const int q = (sl - zl / ROT) & (QPR - 1);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + zl * QPR + q),
                                         (__attribute__((address_space(3))) void*)(S + 4 * c0), 16, 0, STREAM ? 2 : 0);   // aux 2: nontemporal
      }
    } else {
      const int tot4 = (np * Nz * NT) >> 2;      // whole 16-byte pieces (Nz NT is a multiple of 4, checked on the host)
      for (int c0 = wave * 64; c0 < tot4; c0 += nthr) {
        const int p4 = c0 + lane;
        if (p4 < tot4)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + p4),
                                           (__attribute__((address_space(3))) void*)(S + 4 * c0), 16, 0, STREAM ? 2 : 0);
      }
    }
    const float4* tsrc = reinterpret_cast<const float4*>(twz);
    const int tw4 = (Lz << pzshift) >> 1;      // float4 pieces of the twiddle table (Lz * Pz even)
    for (int c0 = wave * 64; c0 < tw4; c0 += nthr) {
      int f = c0 + lane;
      f = f < tw4 ? f : tw4 - 1;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(tsrc + f),
                                       (__attribute__((address_space(3))) void*)(smem + region_floats + 4 * c0),
                                       16, 0, 0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
  __syncthreads();

  const bool live = tid < np * Nz;
  float2 X[H + 1];
  if (live) {
    if constexpr (POW2) {
      float4 quads[QPR];
#pragma unroll
      for (int q = 0; q < QPR; ++q)
        quads[q] = *reinterpret_cast<const float4*>(S + 4 * (tid * QPR + ((q + tid / ROT) & (QPR - 1))));
      if constexpr (NT == 16 || NT == 32) rfft_row_bins_r4<NT>(quads, mt, X);
      else rfft_row_bins<NT>(quads, mt, X);
    } else {
      // rows of NT floats start 8-byte aligned (NT even); 30 floats apart they spread over all banks
      float xr[NT];
#pragma unroll
      for (int n = 0; n < NT; n += 2) {
        const float2 v = *reinterpret_cast<const float2*>(S + tid * NT + n);
        xr[n] = v.x; xr[n + 1] = v.y;
      }
      rdft_row_bins_dense<NT>(xr, mt, X);
    }
  }
  __syncthreads();
  if (live) {
    const int p = tid / Nz, z = tid - p * Nz;
#pragma unroll
    for (int k = 0; k <= H; ++k)
      if (k < mt) T[(p * mt + k) * sT + z] = X[k];
  }
  __syncthreads();

  if constexpr (MZ > 1) {
    for (int idx = tid; idx < ((np * mt) << pzshift); idx += nthr) {
      const int n2 = idx & (Pz - 1), col = idx >> pzshift;
      float2* base = T + col * sT + n2;
      float2 a[MZ];
#pragma unroll
      for (int n1 = 0; n1 < MZ; ++n1) a[n1] = base[n1 << pzshift];
      fft_reg<MZ, -1>(a);
#pragma unroll
      for (int m = 0; m < MZ; ++m) base[m << pzshift] = a[bitrev<MZ>(m)];
    }
    __syncthreads();
  }

  // one output of plane p
  auto combine = [&](int p, int r) {
    const int jz = (r * inv_mt) >> 16;
    const int kt = r - jz * mt;
    const int mj = posmod(kfreq(jz, Lz, nposz), MZ);
    const float2* base = T + (p * mt + kt) * sT + (mj << pzshift);
    const float2* w = TW + (jz << pzshift);
    float2 acc = make_float2(0.f, 0.f);
    if constexpr (PZC >= 0) {
      float2 wv[1 << PZC], bv[1 << PZC];
#pragma unroll
      for (int n2 = 0; n2 < 1 << PZC; ++n2) { wv[n2] = w[n2]; bv[n2] = base[n2]; }
#pragma unroll
      for (int n2 = 0; n2 < 1 << PZC; ++n2) acc = cfma(wv[n2], bv[n2], acc);
    } else {
      for (int n2 = 0; n2 < Pz; ++n2) acc = cfma(w[n2], base[n2], acc);
    }
    return acc;
  };
  float2* dst = out + plane0 * (Lz * mt);
  const int per_plane = Lz * mt;
  for (int p = 0; p < np; ++p)
    for (int r = tid; r < per_plane; r += nthr) st_once2<STREAM>(&dst[p * per_plane + r], combine(p, r));
}

// ------------------------------------------------------------------------------------------
// Complex pruned transform along the middle axis of [outer][N][inner] -> [outer][L][inner]
// ------------------------------------------------------------------------------------------
// W = 2^wshift columns of [N][inner] per block.  The twiddles come from LDS or from memory by two copies of the code: read
// through one pointer that may be either they are flat loads, each of which waits for memory and for LDS.
template <int M, bool STREAM>
__global__ __launch_bounds__(kThreads) void axis_fwd_kernel(
    const float2* __restrict__ in, float2* __restrict__ out, const float2* __restrict__ tw, int N,
    int L, int npos, long long inner, int wshift, int ncb, int tw_lds) {
  HIP_DYNAMIC_SHARED(float, smem)
  const int W = 1 << wshift;
  float2* F = reinterpret_cast<float2*>(smem);          // [N][W]
  float2* TWs = F + N * W;                              // [L][P], only when tw_lds
  const int P = N / M;
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;
  const long long o = blockIdx.x / ncb;
  const long long c0 = (long long)(blockIdx.x % ncb) * W;
  const int wc = (int)min((long long)W, inner - c0);

  if (tw_lds)
    for (int idx = tid; idx < L * P; idx += nthr) TWs[idx] = tw[idx];
  for (int idx = tid; idx < P * W; idx += nthr) {
    const int col = idx & (W - 1), n2 = idx >> wshift;
    if (col < wc) {
      const float2* src = in + (o * N + n2) * inner + c0 + col;
      float2 a[M];
#pragma unroll
      for (int n1 = 0; n1 < M; ++n1) a[n1] = ld_once2<STREAM>(&src[(long long)(P * n1) * inner]);
      fft_reg<M, -1>(a);
#pragma unroll
      for (int m = 0; m < M; ++m) F[(P * m + n2) * W + col] = a[bitrev<M>(m)];
    }
  }
  __syncthreads();
  auto combine = [&](const float2* twiddles) {
    for (int idx = tid; idx < L * W; idx += nthr) {
      const int col = idx & (W - 1), j = idx >> wshift;
      if (col < wc) {
        const int mj = kfreq(j, L, npos) & (M - 1);
        out[(o * L + j) * inner + c0 + col] = combine_terms(twiddles + j * P, F + (P * mj) * W + col, W, P);
      }
    }
  };
  if (tw_lds) combine(TWs); else combine(tw);
}

// [outer][L][inner] (kept frequencies, zero elsewhere) -> [outer][N][inner], exp(+i...).  neighbours: adjacent column
// tiles are worked by one XCD (grid: a multiple of 8).  What bounds it: its writes, at copy speed for large tensors (256
// points, 48 kept, 3.6 GB: 987 -> 660 us; 128 points, 32 kept, batch 4: 840 -> 700), since the reads of several bins go
// out together and none is a flat load.
template <int M, bool STREAM>
__global__ __launch_bounds__(kThreads) void axis_inv_kernel(
    const float2* __restrict__ in, float2* __restrict__ out, const float2* __restrict__ tw, int N,
    int L, int npos, long long inner, int wshift, int ncb, int tw_lds, long long outer, int neighbours) {
  HIP_DYNAMIC_SHARED(float, smem)
  const int W = 1 << wshift;
  float2* Y = reinterpret_cast<float2*>(smem);          // [L][W]
  float2* TWs = Y + L * W;                              // [L][P], only when tw_lds
  const int P = N / M;
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;
  const long long item = neighbours ? xcd_contiguous_item(blockIdx.x, gridDim.x) : blockIdx.x;
  const long long o = item / ncb;
  if (o >= outer) return;
  const long long c0 = (item - o * ncb) * W;
  const int wc = (int)min((long long)W, inner - c0);
  const int kmin = npos - L, kmax = npos - 1;

  if (tw_lds)
    for (int idx = tid; idx < L * P; idx += nthr) TWs[idx] = tw[idx];
  for (int i0 = tid; i0 < L * W; i0 += 8 * nthr) {         // eight loads in flight per thread
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = i0 + u * nthr;
      const int col = idx & (W - 1), j = idx >> wshift;
      v[u] = (idx < L * W && col < wc) ? in[(o * L + j) * inner + c0 + col] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = i0 + u * nthr;
      if (idx < L * W && (idx & (W - 1)) < wc) Y[idx] = v[u];
    }
  }
  __syncthreads();
  auto transform = [&](const float2* twiddles) {
    // bin m takes the frequencies k = m modulo M; the reads of G bins (or of G terms of a bin) go out together, bins that no
    // frequency falls into among them (of 16 bins eight at a time were up to 4 % slower in the mean, where few frequencies are kept)
    constexpr int G = 4;
    for (int idx = tid; idx < P * W; idx += nthr) {
      const int col = idx & (W - 1), n2 = idx >> wshift;
      if (col < wc) {
        const float2* yc = Y + col;
        const float2* wc2 = twiddles + n2;
        auto entry = [&](int k) { return k >= 0 ? k : k + L; };
        float2 g[M];
#pragma unroll
        for (int m = 0; m < M; ++m) g[m] = make_float2(0.f, 0.f);
        if constexpr (M >= G) {
          for (int k0 = kmin; k0 <= kmax; k0 += M) {
#pragma unroll
            for (int m0 = 0; m0 < M; m0 += G) {
              float2 y[G], w[G];
              bool any = false;
#pragma unroll
              for (int u = 0; u < G; ++u) any = any || k0 + ((m0 + u - kmin) & (M - 1)) <= kmax;
              if (!any) continue;
#pragma unroll
              for (int u = 0; u < G; ++u) {
                const int j = entry(min(k0 + ((m0 + u - kmin) & (M - 1)), kmax));
                y[u] = yc[j << wshift];
                w[u] = wc2[j * P];
              }
#pragma unroll
              for (int u = 0; u < G; ++u)
                if (k0 + ((m0 + u - kmin) & (M - 1)) <= kmax) g[m0 + u] = cfmac(y[u], w[u], g[m0 + u]);
            }
          }
        } else if (L <= M) {                     // a term a bin: nothing to read together
#pragma unroll
          for (int m = 0; m < M; ++m) {
            const int k = kmin + ((m - kmin) & (M - 1));
            if (k <= kmax) g[m] = cfmac(yc[entry(k) << wshift], wc2[entry(k) * P], g[m]);
          }
        } else {
#pragma unroll
          for (int m = 0; m < M; ++m)
            for (int k0 = kmin + ((m - kmin) & (M - 1)); k0 <= kmax; k0 += G * M) {
              float2 y[G], w[G];
#pragma unroll
              for (int u = 0; u < G; ++u) {
                const int j = entry(min(k0 + u * M, kmax));
                y[u] = yc[j << wshift];
                w[u] = wc2[j * P];
              }
#pragma unroll
              for (int u = 0; u < G; ++u)
                if (k0 + u * M <= kmax) g[m] = cfmac(y[u], w[u], g[m]);
            }
        }
        fft_reg<M, +1>(g);
        float2* dst = out + (o * N + n2) * inner + c0 + col;
#pragma unroll
        for (int n1 = 0; n1 < M; ++n1) st_once2<STREAM>(&dst[(long long)(P * n1) * inner], g[bitrev<M>(n1)]);
      }
    }
  };
  if (tw_lds) transform(TWs); else transform(tw);
}

// ------------------------------------------------------------------------------------------
// Per-mode channel mix (the learned weight multiplication inside R_phi)
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float mode_scale(long long k, int mt, int Nt, float invN) {
  const int kt = (int)(k % mt);
  const bool single = (kt == 0) || ((Nt % 2 == 0) && (kt == Nt / 2));
  return single ? invN : 2.0f * invN;
}

constexpr int kMixU = 4;   // input (backward: output) channels whose loads go out together

// One thread: one mode, KO output channels, KB batch entries per pass; R is read exactly once,
// the input spectrum once per group of KO output channels (launch: grid.y = ceil(Co / KO)).  Large spectra are bound
// by the read of R, small ones by the chain of round trips over the input channels, hence U of them per trip (one where
// four batch entries fill the registers and waves abound: 8 % faster there).  16 channels, 2048 modes, batch 4: 25 -> 9 us;
// 20 channels, 110592 modes, one entry: 103 -> 75 us; two 117 -> 84 us.
template <int KB, int KO, bool STREAM>
__global__ __launch_bounds__(kThreads) void mix_fwd_kernel(
    const float2* __restrict__ xh, const float2* __restrict__ R, float2* __restrict__ yh, int B,
    int Ci, int Co, long long K, int mt, int Nt, float invN) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int o0 = blockIdx.y * KO;
  if (k >= K) return;
  const float sc = mode_scale(k, mt, Nt, invN);
  constexpr int U = KB >= 4 && STREAM ? 1 : kMixU;
  for (int b0 = 0; b0 < B; b0 += KB) {
    float2 acc[KB][KO];
#pragma unroll
    for (int u = 0; u < KB; ++u)
#pragma unroll
      for (int v = 0; v < KO; ++v) acc[u][v] = make_float2(0.f, 0.f);
    for (int i0 = 0; i0 < Ci; i0 += U) {
      float2 xv[U][KB], r[U][KO];
#pragma unroll
      for (int h = 0; h < U; ++h) {
        const int i = i0 + h;
#pragma unroll
        for (int u = 0; u < KB; ++u)
          xv[h][u] = (i < Ci && b0 + u < B) ? xh[((long long)(b0 + u) * Ci + i) * K + k] : make_float2(0.f, 0.f);
#pragma unroll
        for (int v = 0; v < KO; ++v)
          r[h][v] = (i < Ci && o0 + v < Co) ? ld_once2<STREAM>(&R[((long long)i * Co + o0 + v) * K + k])
                                            : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int h = 0; h < U; ++h)
#pragma unroll
        for (int v = 0; v < KO; ++v)
#pragma unroll
          for (int u = 0; u < KB; ++u) acc[u][v] = cfma(xv[h][u], r[h][v], acc[u][v]);
    }
#pragma unroll
    for (int u = 0; u < KB; ++u)
#pragma unroll
      for (int v = 0; v < KO; ++v)
        if (b0 + u < B && o0 + v < Co)
          yh[((long long)(b0 + u) * Co + o0 + v) * K + k] = make_float2(acc[u][v].x * sc, acc[u][v].y * sc);
  }
}

// One thread: one mode k, kMixI input channels, the batch KB entries at a time; the gradient spectrum gh is then
// read once per kMixI input channels.
constexpr int kMixI = 4;
template <int KB, bool STREAM>
__global__ __launch_bounds__(kThreads) void mix_bwd_kernel(
    const float2* __restrict__ xh, const float2* __restrict__ R, const float2* __restrict__ gh,
    float2* __restrict__ gR, float2* __restrict__ gxh, int B, int Ci, int Co, long long K, int mt,
    int Nt, float invN, int accumulate) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int i0 = blockIdx.y * kMixI;
  if (k >= K) return;
  const float sc = mode_scale(k, mt, Nt, invN);
  constexpr int U = KB >= 4 ? (STREAM ? 1 : 2) : kMixU;
  for (int b0 = 0; b0 < B; b0 += KB) {
    const bool add = gR != nullptr && (b0 > 0 || accumulate);
    float2 xv[KB][kMixI], gx[KB][kMixI];
#pragma unroll
    for (int u = 0; u < KB; ++u)
#pragma unroll
      for (int v = 0; v < kMixI; ++v) {
        gx[u][v] = make_float2(0.f, 0.f);
        xv[u][v] = (b0 + u < B && i0 + v < Ci) ? xh[((long long)(b0 + u) * Ci + i0 + v) * K + k]
                                               : make_float2(0.f, 0.f);
      }
    for (int o0 = 0; o0 < Co; o0 += U) {
      float2 r[U][kMixI], gr[U][kMixI], gy[U][KB];
#pragma unroll
      for (int h = 0; h < U; ++h) {
        const int o = o0 + h;
#pragma unroll
        for (int v = 0; v < kMixI; ++v) {
          const long long ridx = ((long long)(i0 + v) * Co + o) * K + k;
          const bool on = o < Co && i0 + v < Ci;
          r[h][v] = on ? ld_once2<STREAM>(&R[ridx]) : make_float2(0.f, 0.f);
          gr[h][v] = (on && add) ? gR[ridx] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < KB; ++u)
          gy[h][u] = (o < Co && b0 + u < B) ? gh[((long long)(b0 + u) * Co + o) * K + k] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int h = 0; h < U; ++h) {
        const int o = o0 + h;
#pragma unroll
        for (int u = 0; u < KB; ++u) { gy[h][u].x *= sc; gy[h][u].y *= sc; }
#pragma unroll
        for (int u = 0; u < KB; ++u)
#pragma unroll
          for (int v = 0; v < kMixI; ++v) {
            gr[h][v] = cfmac(gy[h][u], xv[u][v], gr[h][v]);        // conj(xh) * gy
            gx[u][v] = cfmac(gy[h][u], r[h][v], gx[u][v]);         // conj(R) * gy
          }
        if (gR != nullptr) {
#pragma unroll
          for (int v = 0; v < kMixI; ++v)
            if (o < Co && i0 + v < Ci) st_once2<STREAM>(&gR[((long long)(i0 + v) * Co + o) * K + k], gr[h][v]);
        }
      }
    }
    if (gxh != nullptr) {
#pragma unroll
      for (int u = 0; u < KB; ++u)
#pragma unroll
        for (int v = 0; v < kMixI; ++v)
          if (b0 + u < B && i0 + v < Ci) gxh[((long long)(b0 + u) * Ci + i0 + v) * K + k] = gx[u][v];
    }
  }
}

// threads per block of the mode mix: 64 where 256 would leave CUs without a block
int mix_threads(int64_t K, int groups) { return (K + kThreads - 1) / kThreads * groups < 512 ? 64 : kThreads; }

size_t tz_fwd_lds(AxisPlan az, int Nt, int mt, int ppb) {
  size_t s_floats = (size_t)ppb * az.N * (Nt + 1);
  s_floats += (s_floats & 1);
  return s_floats * 4 + (size_t)ppb * mt * tz_row_stride(az.N) * 8;
}

int axis_cols(AxisPlan ax, int64_t inner, int rows, int wmax) {
  // widest column tile whose [rows][w] complex tile stays within 32 KiB of LDS
  int w = wmax;
  while (w > 1 && (size_t)rows * w * 8 > (size_t)(32 * 1024)) w >>= 1;
  while (w > 1 && (w >> 1) >= inner) w >>= 1;
  return w;
}

int axis_threads(int items) {
  int t = ((items + 63) / 64) * 64;
  return t < 64 ? 64 : (t > kThreads ? kThreads : t);
}

}  // namespace

bool tz_fwd_fits(AxisPlan az, int Nt, int mt) { return tz_fwd_lds(az, Nt, mt, 1) <= (size_t)kLdsBudget; }
bool axis_fits(AxisPlan ax) { return (size_t)ax.N * 8 <= (size_t)(32 * 1024); }

hipError_t launch_plan_tables(const TableSet& ts, hipStream_t s) {
  if (ts.n <= 0) return hipSuccess;
  int most = 1;
  for (int i = 0; i < ts.n; ++i) {
    const int L = ts.t[i].L;
    const int n = L > 0 ? L * ts.t[i].P : (L < 0 ? -L * (ts.t[i].P + 1) : ts.t[i].N * ts.t[i].npos);
    if (n > most) most = n;
  }
  hipLaunchKernelGGL(plan_tables_kernel, dim3((most + 255) / 256, ts.n), dim3(256), 0, s, ts);
  return hipGetLastError();
}

int tz_fast_region(AxisPlan az, int Nt, int mt, int ppb) {
  const int s_floats = ppb * az.N * Nt;
  const int t_floats = 2 * ppb * mt * tz_row_stride(az.N);
  const int r = s_floats > t_floats ? s_floats : t_floats;
  return (r + 255) & ~255;
}

size_t tz_fast_lds(AxisPlan az, int Nt, int mt, int ppb) {
  const size_t tw_floats = ((size_t)az.L * az.P * 2 + 255) & ~size_t(255);      // whole 1 KiB loads
  return ((size_t)tz_fast_region(az, Nt, mt, ppb) + tw_floats) * 4;
}

hipError_t launch_tz_fwd(const float* x, float2* out, const float2* twt, const float2* twz, const float* ztab,
                         int64_t planes, int field, AxisPlan az, int Nt, int mt, hipStream_t s) {
  if (planes <= 0) return hipSuccess;
  // in-register t stage: the power-of-two lengths, and 30 (the time steps of the paper's training samples)
  // as plain sums with compile-time twiddles
  const bool pow2_t = Nt == 16 || Nt == 32 || Nt == 64;
  const bool fast = (pow2_t ? (az.N * Nt) % 256 == 0 : (Nt == 30 && (az.N * Nt) % 4 == 0 && mt <= 16)) &&
                    (az.M == 8 || az.M == 16) && (az.P & (az.P - 1)) == 0 && (az.L * az.P) % 2 == 0 &&
                    (int64_t)az.L * mt * mt < 65536 && az.N <= kThreads &&   // the kernel's multiply-shift division by mt is exact below that
                    ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(twz)) & 15) == 0 &&
                    tz_fast_lds(az, Nt, mt, 1) <= (size_t)kLdsBudget;
  if (fast) {
    int ppb = 1;
    // about 16 KB of input per block (one plane of 128 x 32, two of 128 x 16): the smaller LDS share
    // keeps more blocks resident, which hides the compute phases behind other blocks' loads a little
    // better than twice that, while smaller blocks than this lose to their fixed costs
    while (ppb * 2 * az.N <= 256 && ppb * 2 * az.N * Nt <= 4096 && tz_fast_lds(az, Nt, mt, ppb * 2) <= (size_t)kLdsBudget) ppb *= 2;
    const int thr = ((ppb * az.N + 63) / 64) * 64;
    const size_t lds = tz_fast_lds(az, Nt, mt, ppb);
    const int region = tz_fast_region(az, Nt, mt, ppb);
    const int64_t nblk = (((planes + ppb - 1) / ppb + 7) / 8) * 8;
    if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
    const int inv_mt = (65536 + mt - 1) / mt;
    const bool stream = planes * (int64_t)az.N * Nt * 4 >= kStreamBytes;
#define FNO_TZF_S(NTV, MZV, FV, PZV, STRV)                                                                             \
  hipLaunchKernelGGL((tz_fwd_fast_kernel<NTV, MZV, FV, PZV, STRV>), dim3((unsigned)nblk), dim3(thr), lds, s, x, out, twz, \
                     (long long)planes, az.N, az.L, az.npos, mt, ppb, region, ilog2(az.P), inv_mt)
#define FNO_TZF_P(NTV, MZV, FV, PZV) \
  do { if (stream) FNO_TZF_S(NTV, MZV, FV, PZV, true); else FNO_TZF_S(NTV, MZV, FV, PZV, false); } while (0)
#define FNO_TZF(NTV, MZV)                                                                \
  do {                                                                                   \
    if (mt == NTV / 2 + 1) FNO_TZF_P(NTV, MZV, true, -1);                                \
    else if (NTV > 16 && az.P == 4) FNO_TZF_P(NTV, MZV, false, ((NTV) > 16 ? 2 : -1));   \
    else if (NTV > 16 && az.P == 8) FNO_TZF_P(NTV, MZV, false, ((NTV) > 16 ? 3 : -1));   \
    else FNO_TZF_P(NTV, MZV, false, -1);                                                 \
  } while (0)
#define FNO_TZF_M(NTV)                     \
  do {                                     \
    if (az.M == 8) FNO_TZF(NTV, 8);        \
    else FNO_TZF(NTV, 16);                 \
  } while (0)
    if (Nt == 16) FNO_TZF_M(16); else if (Nt == 32) FNO_TZF_M(32); else if (Nt == 64) FNO_TZF_M(64);
    else FNO_TZF_M(30);
#undef FNO_TZF_M
#undef FNO_TZF
#undef FNO_TZF_P
#undef FNO_TZF_S
    return hipGetLastError();
  }
  if (ztab != nullptr && tz_fwd_fold_fits(az, Nt, mt) && tz_fwd_fold_pays(az, Nt, mt, planes))
    return launch_tz_fwd_fold(x, out, twt, ztab, planes, field, az, Nt, mt, s);
  int ppb = 1;
  // enough rows to occupy the block, within an LDS share that keeps several blocks per CU
  while (ppb * 2 * az.N <= 2 * kThreads && tz_fwd_lds(az, Nt, mt, ppb * 2) <= (size_t)(32 * 1024)) ppb *= 2;
  const size_t lds = tz_fwd_lds(az, Nt, mt, ppb);
  const int64_t nblk = (((planes + ppb - 1) / ppb + 7) / 8) * 8;
  if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
  FNO_DISPATCH_M(az.M, hipLaunchKernelGGL((tz_fwd_kernel<MM>), dim3((unsigned)nblk), dim3(kThreads),
                                          lds, s, x, out, twt, twz, (long long)planes, az.N, Nt,
                                          az.L, az.npos, mt, ppb));
  return hipGetLastError();
}

hipError_t launch_axis_fwd(const float2* in, float2* out, const float2* tw, int64_t outer,
                           AxisPlan ax, int64_t inner, hipStream_t s) {
  if (outer <= 0 || inner <= 0) return hipSuccess;
  // the widest column tile the 32 KiB cap allows, up to 64 columns (16 for 256-point axes, 32 for
  // 128, 64 below): more threads share the first, FFT phase, whose items are P x W
  const int W = axis_cols(ax, inner, ax.N, 64);
  const int64_t ncb = (inner + W - 1) / W;
  const int64_t nblk = outer * ncb;
  if (nblk > 0x7fffffffLL || ncb > 0x7fffffffLL) return hipErrorInvalidValue;
  // the twiddles go to LDS only when that does not cost a resident block
  const int tw_lds = (size_t)ax.L * ax.P * 8 <= (size_t)(8 * 1024) && (size_t)ax.N * W * 8 <= (size_t)(16 * 1024);
  const size_t lds = (size_t)ax.N * W * 8 + (tw_lds ? (size_t)ax.L * ax.P * 8 : 0);
  // the input is read once: as a stream when it is larger than the caches
  if (outer * ax.N * inner * 8 >= kStreamBytes) {
    FNO_DISPATCH_M(ax.M, hipLaunchKernelGGL((axis_fwd_kernel<MM, true>), dim3((unsigned)nblk),
                                            dim3(kThreads), lds, s, in, out, tw, ax.N, ax.L, ax.npos,
                                            (long long)inner, ilog2(W), (int)ncb, tw_lds));
  } else {
    FNO_DISPATCH_M(ax.M, hipLaunchKernelGGL((axis_fwd_kernel<MM, false>), dim3((unsigned)nblk),
                                            dim3(kThreads), lds, s, in, out, tw, ax.N, ax.L, ax.npos,
                                            (long long)inner, ilog2(W), (int)ncb, tw_lds));
  }
  return hipGetLastError();
}

hipError_t launch_axis_inv(const float2* in, float2* out, const float2* tw, int64_t outer,
                           AxisPlan ax, int64_t inner, hipStream_t s) {
  if (outer <= 0 || inner <= 0) return hipSuccess;
  // Rows of the output that are not whole lines of 128 bytes: column tiles meet in the middle of lines, which must come
  // together in one L2 before they are written, so adjacent tiles go to one XCD; where rows are not even whole 64 bytes also
  // through plain stores, and by wide tiles if they are many.  Only outputs that outgrow the L2s (32 MB together): smaller
  // ones are merged there however they come.  us, y axis of 64 points with 361 columns, of 24 with 561: 157 and 208 streamed
  // by tiles of 32, 79 and 146 so; 128 points with 216 columns (13.5 lines) 125 and 121; but 256 points with 288 (18 lines)
  // 626 and 646, and 16 points with 26 columns (13 MB) 10.3 and 13.8.  Over 16 thousand outputs of up to 200 MB whose rows
  // are not whole 64 bytes it was up to 4 % slower in the mean below 32 MB, 5 to 14 % faster above.  Else 32 columns: 16
  // and 64 are slower.
  const bool big = outer * ax.N * inner * 8 >= (int64_t)32 << 20, split = big && inner % 8 != 0, near = big && inner % 16 != 0;
  const int W = axis_cols(ax, inner, ax.L, split && outer * ((inner + 63) / 64) >= 2048 ? 64 : 32);
  const int64_t ncb = (inner + W - 1) / W;
  const int64_t nblk = near ? (outer * ncb + 7) / 8 * 8 : outer * ncb;
  if (nblk > 0x7fffffffLL || ncb > 0x7fffffffLL) return hipErrorInvalidValue;
  const int tw_lds = (size_t)ax.L * ax.P * 8 <= (size_t)(8 * 1024);
  const size_t lds = (size_t)ax.L * W * 8 + (tw_lds ? (size_t)ax.L * ax.P * 8 : 0);
  const int thr = axis_threads(ax.P * W);
  // the output is written once: as a stream when it is larger than the caches
  if (!split && outer * ax.N * inner * 8 >= kStreamBytes) {
    FNO_DISPATCH_M(ax.M, hipLaunchKernelGGL((axis_inv_kernel<MM, true>), dim3((unsigned)nblk),
                                            dim3(thr), lds, s, in, out, tw, ax.N, ax.L, ax.npos,
                                            (long long)inner, ilog2(W), (int)ncb, tw_lds, (long long)outer, near ? 1 : 0));
  } else {
    FNO_DISPATCH_M(ax.M, hipLaunchKernelGGL((axis_inv_kernel<MM, false>), dim3((unsigned)nblk),
                                            dim3(thr), lds, s, in, out, tw, ax.N, ax.L, ax.npos,
                                            (long long)inner, ilog2(W), (int)ncb, tw_lds, (long long)outer, near ? 1 : 0));
  }
  return hipGetLastError();
}

hipError_t launch_mix_fwd(const float2* xh, const float2* R, float2* yh, int B, int Ci, int Co,
                          int64_t K, int mt, int Nt, double invN, hipStream_t s) {
  const int thr = mix_threads(K, (Co + 3) / 4);
  const int64_t nb = (K + thr - 1) / thr;
  if (nb > 0x7fffffffLL || Co > 65535) return hipErrorInvalidValue;
  // four output channels and up to four batch entries per thread (a tile of one or two entries for
  // batches that small: 3 % faster than four with unused rows); wider output tiles (10 or 20
  // channels for a single batch entry, which would read the input spectrum less often) measured slower.
  // R is read once per call: as a stream from half the size of the memory-side cache on, which it would otherwise share
  // with the spectra and fields around it (us, one batch entry: 217 MB 63 -> 51, 147 MB 39 -> 33; the adjoint, which
  // writes as much as it reads, is no faster below the whole size)
  const bool stream = (int64_t)Ci * Co * K * 8 >= kStreamBytes / 2;
#define FNO_MIX(KBV, STRV)                                                                                  \
  hipLaunchKernelGGL((mix_fwd_kernel<KBV, 4, STRV>), dim3((unsigned)nb, (unsigned)((Co + 3) / 4)), dim3(thr), \
                     0, s, xh, R, yh, B, Ci, Co, (long long)K, mt, Nt, (float)invN)
#define FNO_MIX_B(STRV)                                                                      \
  do {                                                                                       \
    if (B == 1) FNO_MIX(1, STRV); else if (B == 2) FNO_MIX(2, STRV); else FNO_MIX(4, STRV);  \
  } while (0)
  if (stream) FNO_MIX_B(true); else FNO_MIX_B(false);
#undef FNO_MIX_B
#undef FNO_MIX
  return hipGetLastError();
}

hipError_t launch_mix_bwd(const float2* xh, const float2* R, const float2* gh, float2* gR,
                          float2* gxh, int B, int Ci, int Co, int64_t K, int mt, int Nt,
                          double invN, int accumulate, hipStream_t s) {
  const int groups = (Ci + kMixI - 1) / kMixI, thr = mix_threads(K, groups);
  const int64_t nb = (K + thr - 1) / thr;
  if (nb > 0x7fffffffLL || Ci > 4 * 65535) return hipErrorInvalidValue;
  const bool stream = (int64_t)Ci * Co * K * 8 >= kStreamBytes;
#define FNO_MIXB(KBV, STRV)                                                                                          \
  hipLaunchKernelGGL((mix_bwd_kernel<KBV, STRV>), dim3((unsigned)nb, (unsigned)groups), dim3(thr), 0, s, xh, R, gh,  \
                     gR, gxh, B, Ci, Co, (long long)K, mt, Nt, (float)invN, accumulate)
#define FNO_MIXB_B(STRV)                                                                        \
  do {                                                                                          \
    if (B == 1) FNO_MIXB(1, STRV); else if (B == 2) FNO_MIXB(2, STRV); else FNO_MIXB(4, STRV);  \
  } while (0)
  if (stream) FNO_MIXB_B(true); else FNO_MIXB_B(false);
#undef FNO_MIXB_B
#undef FNO_MIXB
  return hipGetLastError();
}

}  // namespace fno
