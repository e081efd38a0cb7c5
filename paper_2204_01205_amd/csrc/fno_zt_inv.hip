// Inverse (z, t) stage of the transform chain (F^-1 of eq. (3) of arXiv 2204.01205 along the last
// two axes, complex-to-real over t) fused with the pointwise part of the block update of eq. (2) /
// Sec. 2.4, sigma(W x + b + K x).  Five kernels cover it, each in a translation unit of its own: two that
// own a column with a 16-point z FFT (fno_zt_inv_col.hip for 32 points of t, fno_zt_inv_col16.hip for 16),
// the chained matrix products for any lengths (fno_zt_inv_fold.hip), tiles of a column with that FFT
// (fno_zt_inv_tile.hip) and the generic one (fno_zt_inv_generic.hip).  This file: the table blobs that the column
// and the per-tile kernels read and the choice between them.
#include "fno_zt_inv.h"

namespace fno {

namespace {

// Tables of the column and per-tile kernels, one blob per residue group g in the kernel's LDS
// layout: cos / -sin rows [2 mt][NT], W transposed and padded [Cu][CP], z twiddles [Q][Lz],
// bias padded [CP].
__global__ void zt_tables_kernel(float* __restrict__ blob, const float2* __restrict__ twt,
                                 const float2* __restrict__ twz, const float* __restrict__ W, int w_so,
                                 int w_si, const float* __restrict__ bias, int Co, int Cu, int CP, int mt,
                                 int NT, int Nt, int Lz, int Pz, int Q, int blob_floats) {
  const int g = blockIdx.x;
  float* dst = blob + (long long)g * blob_floats;
  const int n_cs = 2 * mt * NT, n_wt = (W != nullptr) ? Cu * CP : 0, n_tw = 2 * Q * Lz;
  for (int idx = threadIdx.x; idx < blob_floats; idx += blockDim.x) {
    float v = 0.f;
    if (idx < n_cs) {
      // rows padded from the axis length Nt to the tile width NT with zeros
      const int k = idx / NT, t = idx - k * NT;
      const float2 w = t < Nt ? twt[(k >> 1) * Nt + t] : make_float2(0.f, 0.f);
      v = (k & 1) ? w.y : w.x;
    } else if (idx < n_cs + n_wt) {
      const int e = idx - n_cs;
      const int i = e / CP, o = e - i * CP;
      v = o < Co ? W[o * w_so + i * w_si] : 0.f;
    } else if (idx < n_cs + n_wt + n_tw) {
      const int e = idx - n_cs - n_wt;
      const int c = e >> 1, q = c / Lz, j = c - q * Lz;
      const float2 w = twz[j * Pz + g * Q + q];
      v = (e & 1) ? w.y : w.x;
    } else if (idx < n_cs + n_wt + n_tw + CP) {
      const int o = idx - n_cs - n_wt - n_tw;
      v = (bias != nullptr && o < Co) ? bias[o] : 0.f;
    }
    dst[idx] = v;
  }
}

// Does [a, a + n) meet [b, b + n), n floats?
bool overlap(const float* a, const float* b, int64_t n) {
  const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
  return a != nullptr && b != nullptr && (p < q ? q - p : p - q) < (uintptr_t)n * 4;
}

}  // namespace

hipError_t launch_zt_tables(float* blob, int groups, const float2* twt, const float2* twz, const float* W,
                            int w_so, int w_si, const float* bias, int Co, int Cu, int CP, int mt, int NT,
                            int Nt, int Lz, int Pz, int Q, int blob_floats, hipStream_t s) {
  hipLaunchKernelGGL(zt_tables_kernel, dim3(groups), dim3(256), 0, s, blob, twt, twz, W, w_so, w_si, bias, Co,
                     Cu, CP, mt, NT, Nt, Lz, Pz, Q, blob_floats);
  return hipGetLastError();
}

bool zt_inv_fits(AxisPlan az, int Nt, int mt, int Co) {
  return Co <= kMaxCo && zt_inv_lds(az, Nt, mt, Co) <= (size_t)(68 * 1024);
}

bool zt_tile_fits(AxisPlan az, int Nt, int mt, int Co, int Cu) {
  const int ntt = mfma_tile_nt(Nt);
  return ntt > 0 && mfma_nw(az, ntt, mt, Co, Cu) > 0;
}

// Whether the folded kernel is the faster one where it fits, against the per-tile kernel (tile) or the generic one: with
// many columns nearly always; with few its blocks, which hold whole columns, do not fill the chip.  Measured as the time
// of this stage for z of 8 to 512 points, t of 8 to 48, an eighth to all of the z frequencies, a quarter and half of
// the t bins, 4 to 32 channels, with and without the linear term.  576 columns, 18.8 thousand shapes: with the folded
// kernel wherever it fits 16 % are more than a tenth slower than on the other kernel, with this rule 4 % (and 1 % more
// than a tenth slower than on the folded one).  4096 columns, 6.1 thousand shapes: 6 % and 2 % (0.5 %).
bool zt_inv_fold_pays(AxisPlan az, int Nt, int mt, int Co, int Cu, int64_t ncols, bool tile) {
  const bool block = Cu > 0, narrow = Co <= 20 || !block, few = ncols <= 768;
  const int cp = Co <= 8 ? 8 : (Co <= 20 ? 20 : 32);       // channels that the other kernels pad to
  const bool filled = Co <= 20 && 3 * Co > 2 * cp;
  if (!tile) {
    // Short z axes leave the folded kernel's tiles of 16 row pairs mostly empty, and more than 16 points of t split what
    // little there is.  us, folded against generic, 576 columns: 8 x 24 planes, 6 bins, 8 channels 14.8 and 9.9, 20
    // channels 26.3 and 13.9; 16 x 16, 20 channels, 17.9 and 14.8; 24 x 20, 8 channels with the linear term, 20.9 and
    // 16.6; but 16 x 16, 12 channels, 0.87 to 1.  The generic kernel needs an FFT of at least eight points (z of 9 under t of 40, block with 20
    // channels, 2 times slower than folded) and room for three blocks per CU.
    if (az.M < 8 || az.N > 32 || zt_inv_lds(az, Nt, mt, Co) > (size_t)(160 * 1024 / 3)) return true;
    if (!few) return !(az.N <= 12 && Nt > 16 && filled);
    if (az.N <= 12) return !(narrow && (Nt > 16 || 4 * Co >= 3 * cp));
    if (az.N <= 16 && Nt <= 16 && narrow && 10 * Co > 9 * cp) return false;
    return !(Nt > 16 && Co >= 6 && Co <= 8);
  }
  // The per-tile kernel has a 16-point FFT over z, where the folded products grow with the kept frequencies and bins, and
  // pads the channels to 8, 20 or 32.  us, folded against per tile, convolutions with 8 bins, 576 columns: 16 x 32, 20
  // channels, 31.2 and 19.0; 128 x 32, 32 kept per side, 8 channels, 57 and 40; 128 x 16, 64 per side, 8 channels 63 and
  // 48, 12 channels 82 and 98, 32 per side 45 and 57, 24 channels 68 and 176.  4096 columns, with the linear term: 16 x
  // 32, 8 channels, 8 and 16 bins 1.2 and 1.2 to 1; 128 x 20, 20 channels, 5 and 10 bins, 0.82 to 1.
  //
  // Where the folded spectrum is large, one column fills a block's LDS: its four waves outnumber the column's tasks, or
  // two such blocks are all that a CU holds.  4096 columns, per tile and folded, us: 64 x 16, 24 kept, 9 bins, 20 channels
  // with the linear term 214 and 317; 32 x 24, 32 kept, 9 bins, 20 channels 142 and 256; 64 x 16, 64 kept, 9 bins, 8
  // channels 75 and 164; 128 x 16, 128 kept, 9 bins, 6 channels 259 and 474; but (16 channels, padded to 20 per tile) 128
  // x 24, 64 kept, 9 bins, 1024 columns, 194 and 141.  Over 1418 shapes of 1024 and 4096 columns, z of 32 to 256, t of 12
  // to 32, 4 to 32 channels, 7 % were more than a tenth slower folded than per tile without this part, 2 % are with it
  // (and under 1 % more than a tenth slower than folded).
  if (!few) {
    if (filled && (mt > 12 || (block && az.N <= 32 && Nt >= 20 && mt > 4))) return false;
    const FoldInvLoad l = zt_inv_fold_load(az, Nt, mt, Co, Cu);
    const bool same_pad = Co <= 20 && (Co + 3) / 4 * 4 == cp;
    return !((l.waves < 8 && l.products > 60) || (l.waves <= 8 && same_pad && l.products > 92));
  }
  if (az.N <= 16) return !(Co <= 20 || (Nt > 16 && !block));
  if (Co > 20 || mt <= 3) return true;
  const int k1 = 1 + (az.npos - 1 > az.L - az.npos ? az.npos - 1 : az.L - az.npos);
  if (mt <= 6) return !(k1 > 58 || (block && filled && (Nt == 16 || Nt == 32)));
  return !(filled || (2 * mt + 2) / 4 * (2 * ((k1 + 3) / 4) + 8) > 111);      // matrix instructions of a tile
}

hipError_t launch_zt_inv(const float2* a, float* out, const float2* twt, const float2* twz, const float* ztab,
                         int B, int Co, int Nx, int Ny, AxisPlan az, int Nt, int mt, Epilogue ep,
                         float* tables, hipStream_t s) {
  const int64_t ncols = (int64_t)B * Nx * Ny;
  if (ncols <= 0) return hipSuccess;
  if (Co > kMaxCo) return hipErrorInvalidValue;
  EpiArgs e{ep.u, ep.Cu, ep.W, ep.w_so, ep.w_si, ep.bias, ep.zsave, ep.act};
  const int NxNy = Nx * Ny;
  const bool aligned = ((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(ep.u) |
                         reinterpret_cast<uintptr_t>(ep.zsave) | reinterpret_cast<uintptr_t>(a) |
                         reinterpret_cast<uintptr_t>(tables)) & 15) == 0;
  if (aligned && tables != nullptr) {
    bool taken = false;
    hipError_t err = launch_zt_inv_col(a, out, twt, twz, B, Co, NxNy, az, Nt, mt, e, tables, s, &taken);
    if (err != hipSuccess || taken) return err;
    err = launch_zt_inv_col16(a, out, twt, twz, B, Co, NxNy, az, Nt, mt, e, tables, s, &taken);
    if (err != hipSuccess || taken) return err;
  }
  // A block in place (out or the pre-activation over u): the folded kernel reads the u of a point again after it may
  // have been written, from the blocks of its other channel groups and from overlapping runs of t.  The other kernels
  // read every point before they write it, from one block.
  const int Cu = e.u != nullptr ? e.Cu : 0;
  const int64_t total = ncols * Co * (int64_t)az.N * Nt;
  const bool in_place = overlap(e.u, out, total) || overlap(e.u, e.zsave, total);
  const bool tile = aligned && tables != nullptr && zt_inv_tile_fits(az, Nt, mt, Co, Cu);
  if (!in_place && ztab != nullptr && zt_inv_fold_fits(az, Nt, mt, Co, Cu) &&
      zt_inv_fold_pays(az, Nt, mt, Co, Cu, ncols, tile))
    return launch_zt_inv_fold(a, out, twt, ztab, ncols, Co, NxNy, az, Nt, mt, e, s);
  if (tile) return launch_zt_inv_tile(a, out, twt, twz, B, Co, NxNy, az, Nt, mt, e, tables, s);
  return launch_zt_inv_generic(a, out, twt, twz, ncols, Co, NxNy, az, Nt, mt, e, s);
}

}  // namespace fno
