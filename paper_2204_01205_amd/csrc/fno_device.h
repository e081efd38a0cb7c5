// Device helpers shared by the kernel translation units of libfno (gfx950, wave64).
#pragma once
#include "fno_kernels.h"
#include <cmath>
#include "fft_reg.h"

namespace fno {

namespace {

constexpr int kThreads = 256;
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int kfreq(int j, int L, int npos) { return j < npos ? j : j - L; }
__device__ __forceinline__ int posmod(int a, int m) { int r = a % m; return r < 0 ? r + m : r; }

__device__ __forceinline__ float gelu_f(float z) {
  return 0.5f * z * (1.0f + erff(z * 0.70710678118654752440f));
}
// GELU for the forward epilogues without branches or erff: with a = |z| and the upper tail T(a) = (1 - erf(a / sqrt 2)) / 2,
// z Phi(z) = max(z, 0) - a T(a), and log2 T(a) is so close to a parabola that a polynomial of degree 6, fitted so that
// the largest error of a T(a) on [0, 6] is smallest, is within 5.1e-8 of it there.  It falls to -108 at 13.7 and would turn
// up beyond: all but its last factor stop there, so that the whole goes on falling, by 7.8 a unit, and T is zero from 16.1
// on.  10 instructions, one of them the exponential; 12 and a reciprocal for the rational form of Abramowitz & Stegun 7.1.28
// that stood here.  Error against the float64 definition, evaluated in float32: at most 2.8e-7 absolute, 6.2e-8 of the norm
// for N(0, 1) (7.1.28: 7.1e-7 and 2.3e-7).  Minus infinity gives NaN, as infinity times zero does.
__device__ __forceinline__ float gelu_fast_f(float z) {
  const float a = __builtin_amdgcn_fmed3f(fabsf(z), 0.0f, 13.7f);
  float p = fmaf(a, 3.3092776e-05f, -7.6921936e-04f);
  p = fmaf(a, p, 8.0807153e-03f);
  p = fmaf(a, p, -5.3412102e-02f);
  p = fmaf(a, p, -4.5877096e-01f);
  p = fmaf(a, p, -1.1512017f);
  p = fmaf(fabsf(z), p, -9.9999309e-01f);
  const float t = __builtin_amdgcn_exp2f(p);            // v_exp_f32, 1 ulp
  // max(z, 0) on the bits, whose sign is z's: one instruction (a median of three with infinity, or fmaxf, first quiets a
  // signalling NaN, which is a second one).  |z| and not a: a NaN stays one
  const float pos = __builtin_bit_cast(float, max(__builtin_bit_cast(int, z), 0));
  return fmaf(-fabsf(z), t, pos);
}
__device__ __forceinline__ float gelu_prime_f(float z) {
  const float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752440f));
  const float pdf = 0.39894228040143267794f * expf(-0.5f * z * z);
  return fmaf(z, pdf, cdf);
}

// Loads and stores of data that a kernel touches once.  STREAM: with the nontemporal hint, so that
// a stream much larger than the caches does not displace what other kernels and blocks reuse.  The
// launchers set it for tensors above kStreamBytes; below that the whole working set can live in the
// 256 MB memory-side cache from one kernel to the next, and the hint would throw that away
// (measured: +16 % on a block forward whose tensors are 84 MB, -4..-5 % from 335 MB up).
constexpr long long kStreamBytes = 256ll << 20;
template <bool STREAM, class T>
__device__ __forceinline__ T ld_once(const T* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool STREAM, class T>
__device__ __forceinline__ void st_once(T* p, T v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <bool STREAM>
__device__ __forceinline__ float2 ld_once2(const float2* p) {
  const v2f v = ld_once<STREAM>(reinterpret_cast<const v2f*>(p));
  return make_float2(v[0], v[1]);
}
template <bool STREAM>
__device__ __forceinline__ void st_once2(float2* p, float2 v) {
  st_once<STREAM>(reinterpret_cast<v2f*>(p), v2f{v.x, v.y});
}

// W consecutive floats at a 4-byte aligned address (ld_once and st_once of a vector take its own alignment: a template
// argument drops a type's aligned attribute).  Three go as two and one, which the compiler joins to a 12-byte
// access where the target has one; a vector of three elements may be widened to 16 bytes, past the run.
template <int W> struct run_of;
template <> struct run_of<1> { typedef float type; };
template <> struct run_of<2> { typedef v2f type; };
template <> struct run_of<4> { typedef v4f type; };
template <int W, bool STREAM>
__device__ __forceinline__ void load_run(const void* p, float* v) {
  if constexpr (W == 3) {
    load_run<2, STREAM>(p, v);
    load_run<1, STREAM>(static_cast<const float*>(p) + 2, v + 2);
  } else {
    typedef typename run_of<W>::type vec;
    typedef vec unaligned __attribute__((aligned(4)));
    vec q;
    if constexpr (STREAM) q = __builtin_nontemporal_load(static_cast<const unaligned*>(p));
    else q = *static_cast<const unaligned*>(p);
    if constexpr (W == 1) v[0] = q;
    else {
#pragma unroll
      for (int c = 0; c < W; ++c) v[c] = q[c];
    }
  }
}
template <int W, bool STREAM>
__device__ __forceinline__ void store_run(void* p, const float* v) {
  if constexpr (W == 3) {
    store_run<2, STREAM>(p, v);
    store_run<1, STREAM>(static_cast<float*>(p) + 2, v + 2);
  } else {
    typedef typename run_of<W>::type vec;
    typedef vec unaligned __attribute__((aligned(4)));
    vec q;
    if constexpr (W == 1) q = v[0];
    else {
#pragma unroll
      for (int c = 0; c < W; ++c) q[c] = v[c];
    }
    if constexpr (STREAM) __builtin_nontemporal_store(q, static_cast<unaligned*>(p));
    else *static_cast<unaligned*>(p) = q;
  }
}

// Loads and stores at 32-bit offsets from a base in scalar registers (uniform, below 2 GiB).  Lanes whose offset lies past
// the end read zeros and store nothing, so that no access needs a branch and every way through a loop has as many: wait
// counts are the smallest over all ways.  (A pointer that goes through an asm statement loses its address space, and
// flat loads count as LDS accesses too.)
constexpr unsigned kNowhere = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// W consecutive floats per lane
template <int W, bool STREAM>
__device__ __forceinline__ void buffer_load(__amdgpu_buffer_rsrc_t r, unsigned at, float (&y)[W]) {
  constexpr int aux = STREAM ? 2 : 0;            // nontemporal
  if constexpr (W == 1) {
    y[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, at, 0, aux));
  } else {
    typedef unsigned vec __attribute__((ext_vector_type(W)));
    vec q;
    if constexpr (W == 2) q = __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, aux);
    if constexpr (W == 3) q = __builtin_amdgcn_raw_buffer_load_b96(r, at, 0, aux);
    if constexpr (W == 4) q = __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, aux);
#pragma unroll
    for (int v = 0; v < W; ++v) {
      const unsigned e = q[v];
      y[v] = __builtin_bit_cast(float, e);
    }
  }
}
template <int W, bool STREAM>
__device__ __forceinline__ void buffer_store(__amdgpu_buffer_rsrc_t r, unsigned at, const float (&y)[W]) {
  constexpr int aux = STREAM ? 2 : 0;
  if constexpr (W == 1) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, y[0]), r, at, 0, aux);
  } else {
    typedef unsigned vec __attribute__((ext_vector_type(W)));
    vec q;
#pragma unroll
    for (int v = 0; v < W; ++v) q[v] = __builtin_bit_cast(unsigned, y[v]);
    if constexpr (W == 2) __builtin_amdgcn_raw_buffer_store_b64(q, r, at, 0, aux);
    if constexpr (W == 3) __builtin_amdgcn_raw_buffer_store_b96(q, r, at, 0, aux);
    if constexpr (W == 4) __builtin_amdgcn_raw_buffer_store_b128(q, r, at, 0, aux);
  }
}

// the value of lane ^ 1: the other part of a complex number
__device__ __forceinline__ float swap_pair(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ double swap_pair(double v) {
  typedef int v2i __attribute__((ext_vector_type(2)));
  v2i b = __builtin_bit_cast(v2i, v);
  b[0] = __builtin_amdgcn_mov_dpp(b[0], 0xB1, 0xF, 0xF, true);
  b[1] = __builtin_amdgcn_mov_dpp(b[1], 0xB1, 0xF, 0xF, true);
  return __builtin_bit_cast(double, b);
}

// A float as the exact sum of three bf16 values.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float bf16_low(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_high(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }
__device__ __forceinline__ unsigned bf16_pair(float a, float b) {
  const v2f v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
// the three parts of a and b, side by side
__device__ __forceinline__ void bf16_split(float a, float b, unsigned (&part)[3]) {
  part[0] = bf16_pair(a, b);
  const float ra = a - bf16_low(part[0]), rb = b - bf16_high(part[0]);
  part[1] = bf16_pair(ra, rb);
  part[2] = bf16_pair(ra - bf16_low(part[1]), rb - bf16_high(part[1]));
}

// Thread blocks are dealt to the chip's eight XCDs round robin.  For a grid padded to a multiple of
// eight blocks this is the work item of block `bid` under which every XCD walks a contiguous eighth
// of the items, so that the memory it has in flight at one time spans an eighth of the pages
// (measured on the forward (t, z) kernel: 6 % faster, and less spread between allocations).  The
// caller drops items past the end.
__device__ __forceinline__ long long xcd_contiguous_item(unsigned bid, unsigned nblocks) {
  return (long long)(bid & 7) * (nblocks >> 3) + (bid >> 3);
}

inline int ilog2(int v) { int l = 0; while ((1 << l) < v) ++l; return l; }

#define FNO_DISPATCH_M(Mval, CALL)                \
  switch (Mval) {                                 \
    case 1: { constexpr int MM = 1; CALL; } break;   \
    case 2: { constexpr int MM = 2; CALL; } break;   \
    case 4: { constexpr int MM = 4; CALL; } break;   \
    case 8: { constexpr int MM = 8; CALL; } break;   \
    case 16: { constexpr int MM = 16; CALL; } break; \
    case 32: { constexpr int MM = 32; CALL; } break; \
    default: return hipErrorInvalidValue;         \
  }

}  // namespace

}  // namespace fno
