// Small layers: the x stage there, the mode mix and the x stage back in one launch (S3, S4, S5 of F, R_phi and F^-1 in
// eq. (3) of arXiv 2204.01205, and their adjoints, eq. (7)).
//
// Three kernels of a few microseconds each spend most of that on getting started, and on chains of loads that a chip with
// few blocks on it does not hide.  A block here owns W adjacent columns (ky, kz, kt) of the pruned field [B C][N][inner]
// with all channels: forward transforms to LDS, the product with the weights of its modes, transforms back.  Its inputs are
// in LDS before the first output is written and blocks share no column, so the result may take the place of the input.
//
// The forward takes a batch entry per block (with different channel counts its result has no place for several: one entry
// only), the adjoint all entries, over which the weights' gradient is a sum.
//
// The sums over the axis are plain, folded only in the pairs k and -k (forward) and n and N - n (inverse), whose cosines
// are the same and whose sines differ in sign; terms, roots and sums are double, so that the only rounding is that of the
// result.  The mix has the operations and the order of mix_fwd_kernel and mix_bwd_kernel.
#include "fno_device.h"

namespace fno {

namespace {

constexpr int kXmixThreads = 512;
constexpr size_t kXmixLds = 80 * 1024;

struct XMix {
  int B, Ci, Co, N, L, npos, K1;       // K1: frequencies k >= 0 with k or -k kept
  int inner, wshift, mt, Nt;
  float invN;
};

__device__ __forceinline__ float xmix_scale(const XMix& f, int column) {
  const int kt = column % f.mt;
  return kt == 0 || 2 * kt == f.Nt ? f.invN : 2.0f * f.invN;
}

// roots[r] = (cos, sin)(2 pi r / N)
__device__ __forceinline__ void xmix_roots(const XMix& f, double2* roots) {
  for (int r = threadIdx.x; r < f.N; r += kXmixThreads) {
    double s, c;
    sincospi(2.0 * double(r) / double(f.N), &s, &c);
    roots[r] = make_double2(c, s);
  }
}

// Kept frequencies of C channels: in (at the block's first column) -> A [C][N][W] -> X [C][L][W], and to `save` [C][L][inner]
// where that is not null.  Ends with the block's threads apart: X is complete after the next barrier.
__device__ __forceinline__ void xmix_forward(const XMix& f, const float2* __restrict__ in, int C, int wc, const double2* roots,
                                             float2* A, float2* X, float2* __restrict__ save) {
  const int W = 1 << f.wshift, tid = threadIdx.x;
  for (int i0 = tid; i0 < C * f.N * W; i0 += 8 * kXmixThreads) {         // eight loads in flight per thread
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int idx = min(i0 + u * kXmixThreads, C * f.N * W - 1), col = idx & (W - 1);
      v[u] = in[(long long)(idx >> f.wshift) * f.inner + min(col, wc - 1)];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + u * kXmixThreads < C * f.N * W) A[i0 + u * kXmixThreads] = v[u];
  }
  __syncthreads();
  for (int idx = tid; idx < C * f.K1 * W; idx += kXmixThreads) {
    const int col = idx & (W - 1), q = idx >> f.wshift, c = q / f.K1, k = q - c * f.K1;
    const float2* a = A + ((c * f.N) << f.wshift) + col;
    double cx = 0.0, cy = 0.0, sx = 0.0, sy = 0.0;
    int r = 0;                                   // k n modulo N
#pragma unroll 4
    for (int n = 0; n < f.N; ++n) {
      const float2 v = a[n << f.wshift];
      const double2 w = roots[r];
      cx = fma(double(v.x), w.x, cx); cy = fma(double(v.y), w.x, cy);
      sx = fma(double(v.x), w.y, sx); sy = fma(double(v.y), w.y, sy);
      r += k;
      r -= r >= f.N ? f.N : 0;
    }
    auto put = [&](int j, float2 v) {
      X[((c * f.L + j) << f.wshift) + col] = v;
      if (save != nullptr && col < wc) save[(long long)(c * f.L + j) * f.inner + col] = v;
    };
    if (k < f.npos) put(k, make_float2(float(cx + sy), float(cy - sx)));
    if (k >= 1 && k <= f.L - f.npos) put(f.L - k, make_float2(float(cx - sy), float(cy + sx)));
  }
}

// Y [C][L][W] -> out [C][N][inner] at the block's first column
__device__ __forceinline__ void xmix_inverse(const XMix& f, const float2* Y, int C, int wc, const double2* roots,
                                             float2* __restrict__ out) {
  const int W = 1 << f.wshift, half = f.N / 2 + 1;
  for (int idx = threadIdx.x; idx < C * half * W; idx += kXmixThreads) {
    const int col = idx & (W - 1), q = idx >> f.wshift, c = q / half, n = q - c * half;
    const float2* y = Y + ((c * f.L) << f.wshift) + col;
    double ax = 0.0, ay = 0.0, bx = 0.0, by = 0.0;
    auto add = [&](int first, int count, int r) {          // r: k n modulo N of the first
#pragma unroll 4
      for (int j = 0; j < count; ++j) {
        const float2 v = y[(first + j) << f.wshift];
        const double2 w = roots[r];
        ax = fma(double(v.x), w.x, ax); ay = fma(double(v.y), w.x, ay);
        bx = fma(double(v.y), w.y, bx); by = fma(double(v.x), w.y, by);
        r += n;
        r -= r >= f.N ? f.N : 0;
      }
    };
    add(0, f.npos, 0);
    add(f.npos, f.L - f.npos, posmod(-(f.L - f.npos) * n, f.N));
    if (col >= wc) continue;
    out[(long long)(c * f.N + n) * f.inner + col] = make_float2(float(ax - bx), float(ay + by));
    if (n > 0 && 2 * n != f.N) out[(long long)(c * f.N + f.N - n) * f.inner + col] = make_float2(float(ax + bx), float(ay - by));
  }
}

// in, out [B C][N][inner]; xh (nullable) [B Ci][L][inner]; out null: the spectrum alone, R is not read then.  One batch entry
// per block.
__global__ __launch_bounds__(kXmixThreads) void xmix_fwd_kernel(const float2* in, const float2* __restrict__ R,
                                                                float2* __restrict__ xh, float2* out, XMix f) {
  HIP_DYNAMIC_SHARED(float4, smem4)
  const int W = 1 << f.wshift, tid = threadIdx.x, b = blockIdx.y;
  const int c0 = blockIdx.x * W, wc = min(W, f.inner - c0);
  double2* roots = reinterpret_cast<double2*>(smem4);
  float2* X = reinterpret_cast<float2*>(roots + f.N);      // [Ci][L][W]
  float2* A = X + ((f.Ci * f.L) << f.wshift);              // [Ci][N][W], then Y [Co][L][W]
  const int K = f.L * f.inner;
  xmix_roots(f, roots);
  xmix_forward(f, in + (long long)b * f.Ci * f.N * f.inner + c0, f.Ci, wc, roots, A, X,
               xh != nullptr ? xh + (long long)b * f.Ci * K + c0 : nullptr);
  if (out == nullptr) return;
  __syncthreads();
  float2* Y = A;
  for (int idx = tid; idx < f.Co * f.L * W; idx += kXmixThreads) {
    const int col = idx & (W - 1), q = idx >> f.wshift, o = q / f.L, j = q - o * f.L;
    const float2* r0 = R + ((long long)o * f.L + j) * f.inner + c0 + min(col, wc - 1);
    const float2* x0 = X + (j << f.wshift) + col;
    float2 acc = make_float2(0.f, 0.f);
    constexpr int U = 16;                        // weights in flight
    for (int i0 = 0; i0 < f.Ci; i0 += U) {
      float2 r[U];
#pragma unroll
      for (int h = 0; h < U; ++h) r[h] = r0[(long long)min(i0 + h, f.Ci - 1) * f.Co * K];
#pragma unroll
      for (int h = 0; h < U; ++h)
        if (i0 + h < f.Ci) acc = cfma(x0[((i0 + h) * f.L) << f.wshift], r[h], acc);
    }
    const float sc = xmix_scale(f, c0 + col);
    Y[((o * f.L + j) << f.wshift) + col] = make_float2(acc.x * sc, acc.y * sc);
  }
  __syncthreads();
  xmix_inverse(f, Y, f.Co, wc, roots, out + (long long)b * f.Co * f.N * f.inner + c0);
}

// gR[i][o] = sum_b conj(xh[b][i]) gy[b][o] (accumulate: added to what gR holds) and, transformed back, gx[b][i] = sum_o
// conj(R[i][o]) gy[b][o]; `in` holds the cotangent [B Co][N][inner], `out` takes [B Ci][N][inner].  gR (xh is not read
// then) and out may be null.
template <int KB>
__global__ __launch_bounds__(kXmixThreads) void xmix_bwd_kernel(const float2* in, const float2* __restrict__ R,
                                                                const float2* __restrict__ xh, float2* __restrict__ gR,
                                                                float2* out, XMix f, int accumulate) {
  HIP_DYNAMIC_SHARED(float4, smem4)
  const int W = 1 << f.wshift, tid = threadIdx.x;
  const int c0 = blockIdx.x * W, wc = min(W, f.inner - c0);
  double2* roots = reinterpret_cast<double2*>(smem4);
  float2* G = reinterpret_cast<float2*>(roots + f.N);      // [B][Co][L][W]
  float2* A = G + ((f.B * f.Co * f.L) << f.wshift);        // [Co][N][W], then gx [B][Ci][L][W]
  const int K = f.L * f.inner;
  xmix_roots(f, roots);
  for (int b = 0; b < f.B; ++b) {
    if (b > 0) __syncthreads();                  // A has been read
    xmix_forward(f, in + (long long)b * f.Co * f.N * f.inner + c0, f.Co, wc, roots, A,
                 G + ((b * f.Co * f.L) << f.wshift), nullptr);
  }
  __syncthreads();
  float2* GX = A;
  for (int idx = tid; idx < f.Ci * f.L * W; idx += kXmixThreads) {
    const int col = idx & (W - 1), q = idx >> f.wshift, i = q / f.L, j = q - i * f.L;
    const long long at = (long long)j * f.inner + c0 + min(col, wc - 1);
    const float sc = xmix_scale(f, c0 + col);
    float2 xv[KB], gx[KB];
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      gx[u] = make_float2(0.f, 0.f);
      xv[u] = gR != nullptr ? xh[((long long)min(u, f.B - 1) * f.Ci + i) * K + at] : make_float2(0.f, 0.f);
    }
    constexpr int U = 8;
    for (int o0 = 0; o0 < f.Co; o0 += U) {
      float2 r[U], old[U];
#pragma unroll
      for (int h = 0; h < U; ++h) {
        const long long ridx = ((long long)i * f.Co + min(o0 + h, f.Co - 1)) * K + at;
        r[h] = R[ridx];
        old[h] = accumulate ? gR[ridx] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int h = 0; h < U; ++h) {
        const int o = o0 + h;
        if (o >= f.Co) break;
        float2 gr = old[h];
#pragma unroll
        for (int u = 0; u < KB; ++u)
          if (u < f.B) {
            float2 gy = G[(((u * f.Co + o) * f.L + j) << f.wshift) + col];
            gy.x *= sc;
            gy.y *= sc;
            gr = cfmac(gy, xv[u], gr);
            gx[u] = cfmac(gy, r[h], gx[u]);
          }
        if (gR != nullptr && col < wc) gR[((long long)i * f.Co + o) * K + at] = gr;
      }
    }
#pragma unroll
    for (int u = 0; u < KB; ++u)
      if (u < f.B) GX[(((u * f.Ci + i) * f.L + j) << f.wshift) + col] = gx[u];
  }
  __syncthreads();
  if (out != nullptr) xmix_inverse(f, GX, f.B * f.Ci, wc, roots, out + c0);
}

// from: channels of the field that is transformed, to: of the result
size_t xmix_lds(int B, int from, int to, AxisPlan ax, int W) {
  const size_t a = (size_t)from * ax.N, y = (size_t)B * to * ax.L;
  return (size_t)ax.N * 16 + ((size_t)B * from * ax.L + (a > y ? a : y)) * W * 8;
}

bool xmix_geometry(int B, int from, int to, AxisPlan ax, int64_t inner, int* wshift) {
  for (int s = inner >= 1024 ? 3 : 2; s >= 2; --s) {
    *wshift = s;
    if (xmix_lds(B, from, to, ax, 1 << s) <= kXmixLds) return true;
  }
  return false;
}

}  // namespace

// Where one launch is faster than three: as long as the chip is far from full (values of the pruned field), a block's own
// work is no longer than the launches saved, and the weights, which every batch entry's blocks read in runs of one tile,
// are few.  The work per column: multiply-adds of the sums, over all entries in an adjoint, and products of the mix, which
// weigh three quarters of one.  us, three launches and one,
// forward and (in brackets) forward and adjoint: 8 -> 8 channels, 16 points, 8 kept, 192 columns 35.6, 28.6 (70, 56); 12 ->
// 12, 12 points, 2 kept, 240 columns 42, 35 (87, 70); batch 4, 16 -> 16, 9 points, 336 columns 58, 49 (123, 108); 8 -> 16,
// 34 points, 10 kept, 320 columns (4512 multiply-adds) 53, 52 (111, 103); 20 -> 10, 36 points, 8 kept, 16 columns (in the
// adjoint 5120) forward and adjoint 80, 73; 29 -> 29, 16 points, 7 kept, batch 4 (3683 and 5887 products) 74, 66; but
// batch 2, 32 -> 32, 20 points, 8 kept, 144 columns (6016 and 8192, in the adjoint 12032) 78, 82 (163, 176); 16 -> 16, 19
// points, 1296 columns (394 thousand values) 67, 66 (135, 134).  The mix alone, one entry: 32 -> 32, 12 points, 11 kept, 105
// columns (11264 products beside 4768 multiply-adds; 9.5 MB) 45, 57 (adjoint 54, 71); weights alone, batch 3: 24 -> 24, 6
// points, 5 kept, 845 columns (20 MB) 64, 85.  An adjoint's block works all entries in turn: batch 4, 2 -> 2 channels, 52
// points (208 of the field in a chain) 57, 65; about 96 in a chain are as fast either way.  Over 7500 random forwards and
// 8700 adjoints of 2 to 32 channels, 6 to 72 points and up to 8 thousand columns, 0.2 and 0.7 % are more than 3 % slower in
// one launch than in three, 2.2 and 3.1 % the other way (0.1, 0.3, 7.1 and 7.6 % with the sums bounded apart, at 5000).
//
// The forward's choice is the same for one to four entries of as many channels out as in, each of which has blocks of its
// own; else the result has no place for several entries.
bool xmix_fits(int B, int Ci, int Co, AxisPlan ax, int64_t inner, bool adjoint) {
  const int from = adjoint ? Co : Ci, to = adjoint ? Ci : Co, most = Ci > Co ? Ci : Co;
  const int64_t K1 = 1 + (ax.npos - 1 > ax.L - ax.npos ? ax.npos - 1 : ax.L - ax.npos);
  const int64_t sums = from * K1 * ax.N + to * (int64_t)(ax.N / 2 + 1) * ax.L, mix = (int64_t)Ci * Co * ax.L;
  if (B > 4 || 4 * (adjoint ? B : 1) * sums + 3 * mix > 33600) return false;
  if (inner > 150000 || most * ax.N * inner > 150000 || mix * inner > (adjoint ? 1500000 : 1000000)) return false;
  if (adjoint && (B * most * ax.N * inner > 300000 || (B > 1 && B * ax.N > 96))) return false;
  if (!adjoint && B > 1 && Ci != Co) return false;
  int s;
  return xmix_geometry(adjoint ? B : 1, from, to, ax, inner, &s);
}

namespace {
XMix xmix_args(int B, int Ci, int Co, int from, int to, AxisPlan ax, int64_t inner, int mt, int Nt, double invN) {
  XMix f{B, Ci, Co, ax.N, ax.L, ax.npos, 1 + (ax.npos - 1 > ax.L - ax.npos ? ax.npos - 1 : ax.L - ax.npos),
         (int)inner, 0, mt, Nt, (float)invN};
  xmix_geometry(B, from, to, ax, inner, &f.wshift);
  return f;
}
}  // namespace

hipError_t launch_xmix_fwd(const float2* in, const float2* R, float2* xh, float2* out, int B, int Ci, int Co, AxisPlan ax,
                           int64_t inner, int mt, int Nt, double invN, hipStream_t s) {
  const XMix f = xmix_args(1, Ci, Co, Ci, Co, ax, inner, mt, Nt, invN);
  const unsigned nblk = (unsigned)((inner + (1 << f.wshift) - 1) >> f.wshift);
  hipLaunchKernelGGL(xmix_fwd_kernel, dim3(nblk, B), dim3(kXmixThreads), xmix_lds(1, Ci, Co, ax, 1 << f.wshift), s, in, R,
                     xh, out, f);
  return hipGetLastError();
}

hipError_t launch_xmix_bwd(const float2* in, const float2* R, const float2* xh, float2* gR, float2* out, int B, int Ci, int Co,
                           AxisPlan ax, int64_t inner, int mt, int Nt, double invN, int accumulate, hipStream_t s) {
  accumulate = accumulate && gR != nullptr;
  const XMix f = xmix_args(B, Ci, Co, Co, Ci, ax, inner, mt, Nt, invN);
  const unsigned nblk = (unsigned)((inner + (1 << f.wshift) - 1) >> f.wshift);
  const size_t lds = xmix_lds(B, Co, Ci, ax, 1 << f.wshift);
#define FNO_XM(KBV) hipLaunchKernelGGL((xmix_bwd_kernel<KBV>), dim3(nblk), dim3(kXmixThreads), lds, s, in, R, xh, gR, out, f, accumulate)
  if (B == 1) FNO_XM(1); else if (B == 2) FNO_XM(2); else FNO_XM(4);
#undef FNO_XM
  return hipGetLastError();
}

}  // namespace fno
