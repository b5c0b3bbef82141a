// fp32 3x3 convolutions (every layer packed in 32-channel chunks: more than 16 input channels, or
// 9..16 with whole 16-channel output tiles beyond 16) on the fp16 matrix pipe.
//
// The fp32 MFMA runs at 1/16 of the fp16 rate, and at 80 % of it the tiled fp32 kernels had nowhere
// to go.  A float splits into two halves x = h + l with h = fp16(x), l = fp16(x - h), which hold 22
// to 23 of its 24 bits, and x w = h_x h_w + h_x l_w + l_x h_w up to 2^-22 of the product: three
// v_mfma_f32_16x16x32_f16 with fp32 accumulation do the work of eight v_mfma_f32_16x16x4_f32, and
// the sum has a fifth of the roundings.  Range: the operands are scaled by powers of two, which is
// exact.
//  * Weights per output channel at packing time, its largest magnitude to [2^14, 2^15); the exponent
//    travels in the lowest bits of the l halves of the channel's first eight weights.
//  * Activations per block: before a chunk is staged, its largest finite magnitude over the block's
//    tile sets the scale (a running maximum over the chunks; the accumulators are rescaled when it
//    grows), but at most 2^26 times its typical magnitude (the mean exponent of a sample), so that an
//    outlier does not cost its neighbours their precision: what is larger than the scale allows
//    overflows and goes the way of infinities, below.  The staged l halves carry a factor 2^11,
//    undone in the h_w they meet, which keeps them out of the fp16 subnormals: an element is carried
//    to 2^-23 of itself or 2^-50 of the tile's largest (2^-24 of its typical) element.
//  * An output that comes out non-finite (an input that is infinite or NaN, an overflow) is summed
//    again in plain fp32 (rescue), so such values propagate as in an fp32 convolution.
// Error against FP64 (normwise; fp32 MFMA kernels in brackets): 128 -> 128 channels 3.7e-7 (4.3e-7),
// the U-Net's heads at 1920 x 1080 at most 1.6e-6 (1.7e-6).
//
// Tiling as k_conv_lds: blocks of 4 waves stacked vertically, TN rows x 16 px each, all sharing TM
// m-tiles; the chunk's input tile with its halo in LDS as two planes (64-byte pixels, 16-byte
// groups swizzled on bits 1-2 of the pixel index).  Taps in order, dx outer: the next tap's B
// operands are read during the current one's MFMAs.  The weight operands (A) come straight from
// global memory (the four waves read the same fragments from L1) and each m-tile's are reloaded in
// place after its last use, 36 MFMAs ahead of the next, so no barrier and no LDS space goes to them.
// One order of sums for every entry point: 32-channel chunks, taps dx outer and dy inner, the three
// products, then the bias; the block's tile decides the scale, so launches of equal sizes agree bit
// for bit.
// What bounds it: for 32-channel blocks the vector memory path (address unit 80 % busy, mostly with
// A) and 1000 vector instructions per wave and chunk beside 216 MFMAs; for 64-channel blocks the
// MFMAs (54 % of the rate at the 2.0 GHz the card holds).  1920 x 1080, before (fp32 MFMA) and now:
// 16 -> 32 162 -> 181 us, 32 -> 32 317 -> 190 us, 64 -> 64 (540 x 960) 322 -> 120 us, 128 -> 128
// (270 x 480) 298 -> 103 us, 384 -> 128 841 -> 284 us, 96 -> 32 899 -> 367 us; the U-Net 5.59 -> 2.36 ms.
// Not kept: persistent blocks (fetching the next tile during the current one: registers spill),
// weights of all three tap rows live at once (spills), 8 channels per staging load.
#include <algorithm>

#include "conv_common.h"

using namespace aps;

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kOutlier = 26;
constexpr uint32_t kOut = 0xffffff00u;  // a byte offset past the end of any row_load range

// 16 bytes at byte offset off of a range (uniform base), `skip` floats further on; zeros past its end
__device__ inline f32x4 row_load(const float* base, uint32_t bytes, uint32_t off, int skip) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + skip), 0, bytes - 4 * skip, 0x00020000);
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

__device__ inline f32x4 mmah(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// 2^e, -126 <= e <= 127
__device__ inline float pow2(int e) { return __builtin_bit_cast(float, (uint32_t)(e + 127) << 23); }

// The same value, but not known to be loop-invariant: what is computed from it is not hoisted out of
// the chunk loop, where it would hold registers
__device__ inline int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Exponent that scales a largest magnitude m (0, or finite) to [2^14, 2^15)
__device__ inline int scale_exp(float m) {
  const int e = 14 - ((int)((__builtin_bit_cast(uint32_t, m) >> 23) & 0xff) - 127);
  return m == 0.f ? 0 : e > 126 ? 126 : e;
}

// Input channel ci of pixel (iy, ix) after the input transform, in the order of stage8
template <int MODE>
__device__ inline float conv_input(const ConvArgs& a, int n, int iy, int ix, int ci) {
  const float* x = static_cast<const float*>(a.x);
  const float* x2 = static_cast<const float*>(a.x2);
  if (iy < 0 || iy >= a.H || ix < 0 || ix >= a.W) return 0.f;
  if constexpr (MODE == APS_CONV_POOL2) {
    const size_t rs = 2 * (size_t)a.W * a.Cx;
    const float* p = x + (((size_t)n * 2 * a.H + 2 * iy) * 2 * a.W + 2 * ix) * a.Cx + ci;
    return ((p[0] + p[a.Cx]) + (p[rs] + p[rs + a.Cx])) * 0.25f;
  } else if constexpr (MODE == APS_CONV_UP2_CAT) {
    return ci < a.Cx ? x[(((size_t)n * (a.H / 2) + iy / 2) * (a.W / 2) + ix / 2) * a.Cx + ci]
                     : x2[(((size_t)n * a.H + iy) * a.W + ix) * a.C2 + (ci - a.Cx)];
  } else {
    const size_t o = (((size_t)n * a.H + iy) * a.W + ix) * a.Cx + ci;
    if constexpr (MODE == kModeReluMask) return x2[o] > 0.f ? x[o] : 0.f;
    return x[o];
  }
}

// Fragment f (in units of 512 halves) of channel tile ct, tap t, chunk c, half p (0: h, 1: l)
__device__ inline uint32_t wfrag(int ct, int t, int c, int p, int nchunk) {
  return (uint32_t)(((ct * 9 + t) * nchunk + c) * 2 + p) * 512u;
}

// Scale exponent of output channel 16 ct + k: e + 128 in the lowest bits of the l halves of weights
// (tap 0, input channels 0..7), bit exp_bit(b) in channel b
__device__ inline int exp_bit(int b) { return (b >> 1) + 4 * (b & 1); }
__device__ inline int weight_exp(const uint16_t* wp, int ct, int k, int nchunk) {
  const u32x4 v = *reinterpret_cast<const u32x4*>(wp + wfrag(ct, 0, 0, 1, nchunk) + k * 8);
  const uint32_t t = (v[0] & 0x10001) | (v[1] & 0x10001) << 1 | (v[2] & 0x10001) << 2 | (v[3] & 0x10001) << 3;
  const int e = (t & 15) | (t >> 12 & 0xf0);
  return e ? e - 128 : 0;  // no bits: the channel's weights are all zero
}

// One output channel of one pixel in plain fp32
template <int MODE>
__device__ inline float rescue(const ConvArgs& a, const uint16_t* wp, int n, int row, int col, int co) {
  const int Cin = a.cvalid, ct = co >> 4, k = co & 15;
  const float sw = pow2(-weight_exp(wp, ct, k, a.nchunk));
  float s = 0.f;
  for (int c = 0; c < a.nchunk; ++c)
    for (int d = 0; d < 9; ++d) {
      const int t = (d % 3) * 3 + d / 3;  // taps dx outer, dy inner
      for (int g = 0; g < 4; ++g)
        for (int e = 0; e < 8; ++e) {
          const int ci = c * 32 + g * 8 + e;
          if (ci >= Cin) continue;
          const uint32_t o = wfrag(ct, t, c, 0, a.nchunk) + (g * 16 + k) * 8 + e;
          const float w = ((float)__builtin_bit_cast(_Float16, wp[o]) + (float)__builtin_bit_cast(_Float16, wp[o + 512])) * sw;
          s += w * conv_input<MODE>(a, n, row + t / 3 - 1, col + t % 3 - 1, ci);
        }
    }
  return s;
}

// The value of lane l ^ 1 (DPP quad_perm [1,0,3,2]).  By value on purpose: a bit cast applied
// directly to a vector-element subscript was compiled as a read of element 0.
__device__ inline float lane_xor1(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}

// ReLU, store, and with a.pool the 2x2 mean in the order of the POOL2 input transform
template <int TM, int TN>
__device__ inline void epilogue_f32(const ConvArgs& a, f32x4 (&acc)[TM][TN], int row0, int tx0,
                                    int cob, int n, int lane) {
  float* y = static_cast<float*>(a.y);
  float* yp = static_cast<float*>(a.pool);
  const int col = tx0 + (lane & 15);
#pragma unroll
  for (int j0 = 0; j0 < TN; j0 += 2) {
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const int co = (cob * TM + m) * 16 + 4 * (lane >> 4);
      if (co >= a.Cout) continue;
      f32x4 h[2];
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int j = j0 + jj, row = row0 + j;
        f32x4 v = acc[m][j];
        if (a.relu) {
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = fmaxf(v[q], 0.f);
        }
        h[jj] = v;
        if (row < a.H && col < a.W) {
          const float vv[4] = {v[0], v[1], v[2], v[3]};
          store_out<float>(y + (((size_t)n * a.H + row) * a.W + col) * a.ldy, a.ldy, co, a.Cout, vv);
        }
      }
      if (yp) {
        f32x4 nb[2];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int q = 0; q < 4; ++q) nb[jj][q] = lane_xor1(h[jj][q]);
        const int row = row0 + j0;
        if ((lane & 1) == 0 && row < a.H && col < a.W)
          *reinterpret_cast<f32x4*>(yp + (((size_t)n * (a.H / 2) + row / 2) * (a.W / 2) + col / 2) * a.Cout + co) =
              ((h[0] + nb[0]) + (h[1] + nb[1])) * 0.25f;
      }
    }
  }
}

// PF: the next chunk's loads are in flight during the MFMAs (two blocks per CU).  Without it three
// 32-channel blocks fit, which is worth more to them (96 -> 32 channels at 1080p: 387 us with, 347 us
// without; 192 -> 64 at 540 x 960: 284 and 295 us).  A single chunk has no next one (64-channel
// blocks held to three per CU spill: 32 -> 64 at 540 x 960 97 us against 84 us).
template <int MODE, int TM, int TN, int HEAD, bool PF>
__global__ __launch_bounds__(256, PF || TM == 4 ? 2 : 3) void k_conv_split(ConvArgs a) {
  constexpr int ROWS = 4 * TN, SH = ROWS + 2, SW = 18, NPX = SH * SW;
  constexpr int NXT = (NPX * 8 + 255) / 256;  // (pixel, 4 channels) items per thread and chunk
  constexpr int PL = NPX * 32;          // halves per plane
  constexpr int XS_HEAD = HEAD ? 2 * head_lds_elems<float, float, TM, HEAD>() : 0;
  __shared__ __attribute__((aligned(16))) uint16_t Xs[2 * PL > XS_HEAD ? 2 * PL : XS_HEAD];
  __shared__ float red[4];
  __shared__ uint32_t rede[4];

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const TileId tid_ = xcd_tile(blockIdx.x, a.ntiles, a.nco);
  if (tid_.tile >= a.ntiles) return;
  const int tx0 = (tid_.tile % a.ntx) * 16, ty0 = (tid_.tile / a.ntx) * ROWS;
  const int cob = tid_.cob, n = blockIdx.z;
  const float* x = static_cast<const float*>(a.x);
  const float* x2 = static_cast<const float*>(a.x2);
  const uint16_t* wp = static_cast<const uint16_t*>(a.wp);
  const int Cin = a.Cx + a.C2;
  // This thread stages channels [g4, g4 + 4) of tile pixels tid / 8 + 32 k: a wave's load reads 8
  // pixels' whole 128-byte chunks (with 8 channels per thread and 16 pixels per load the same bytes
  // cost the address unit twice the cycles, which bounded the 32-channel layers).
  const int g4 = (tid & 7) * 4, pl = tid >> 3;
  // Byte offsets at chunk 0 from the tile's first input row; past the end (reads as zeros) where
  // the pixel is outside the image.
  const int yb = std::max(ty0 - 1, 0), rows = std::min(ty0 + ROWS + 1, a.H) - yb;
  uint32_t xo[NXT];  // into x, or once the chunks have passed its channels into the skip tensor
  auto offsets = [&](bool skip) {
    int r = opaque(pl) / SW, col = pl - r * SW;
#pragma unroll
    for (int k = 0; k < NXT; ++k) {
      const int iy = ty0 - 1 + r, ix = tx0 - 1 + col;
      const bool in = pl + 32 * k < NPX && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
      uint32_t o;
      if (MODE == APS_CONV_UP2_CAT && skip) o = (uint32_t)(((iy - yb) * a.W + ix) * a.C2 + g4);
      else if (MODE == APS_CONV_UP2_CAT) o = (uint32_t)(((iy / 2 - yb / 2) * (a.W / 2) + ix / 2) * a.Cx + g4);
      else if (MODE == APS_CONV_POOL2) o = (uint32_t)((2 * (iy - yb) * 2 * a.W + 2 * ix) * a.Cx + g4);
      else o = (uint32_t)(((iy - yb) * a.W + ix) * a.Cx + g4);
      xo[k] = in ? o * 4 : kOut;
      col += 32 - SW;  // the next item is 32 pixels on
      ++r;
      if (col >= SW) {
        col -= SW;
        ++r;
      }
    }
  };
  offsets(false);
  const size_t row0 = (size_t)n * a.H + yb;
  const float* xb = MODE == APS_CONV_POOL2 ? x + row0 * 4 * a.W * a.Cx
                    : MODE == APS_CONV_UP2_CAT ? x + ((size_t)n * (a.H / 2) + yb / 2) * (a.W / 2) * a.Cx
                                               : x + row0 * a.W * a.Cx;
  const uint32_t xbytes = MODE == APS_CONV_POOL2 ? (uint32_t)rows * 4 * a.W * a.Cx * 4
                          : MODE == APS_CONV_UP2_CAT ? (uint32_t)((yb + rows + 1) / 2 - yb / 2) * (a.W / 2) * a.Cx * 4
                                                     : (uint32_t)rows * a.W * a.Cx * 4;
  const float* sb = x2 + row0 * a.W * (MODE == APS_CONV_UP2_CAT ? a.C2 : a.Cx);
  const uint32_t sbytes = (uint32_t)rows * a.W * (MODE == APS_CONV_UP2_CAT ? a.C2 : a.Cx) * 4;

  // Global loads of the next chunk, unconditional: no branch join makes the compiler wait for them
  // before the current chunk's MFMAs (the pooled and masked transforms are evaluated here).
  f32x4 px[NXT];
  auto fetch = [&](int c) {
    const int cb = c * 32, ch = cb + g4;
    if (MODE == APS_CONV_UP2_CAT && cb >= a.Cx && cb < a.Cx + 32) offsets(true);  // the first such chunk
    // element by element: input rows whose bytes do not fit 32-bit offsets, and a chunk that spans
    // both tensors of the concat
    if (a.big || (MODE == APS_CONV_UP2_CAT && cb < a.Cx && cb + 32 > a.Cx)) {
#pragma unroll
      for (int k = 0; k < NXT; ++k) {
        __builtin_amdgcn_sched_barrier(0);  // one item's addresses live at a time
        const int p = opaque(pl) + 32 * k, r = p / SW, iy = ty0 - 1 + r, ix = tx0 - 1 + p - r * SW;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          px[k][q] = p < NPX && ch + q < Cin ? conv_input<MODE>(a, n, iy, ix, ch + q) : 0.f;
      }
      return;
    }
    const bool first = MODE != APS_CONV_UP2_CAT || cb < a.Cx;  // uniform
    const float* src = first ? xb : sb;
    const uint32_t nb = first ? xbytes : sbytes;
#pragma unroll
    for (int k = 0; k < NXT; ++k) {
      if constexpr (MODE == APS_CONV_UP2_CAT) {
        px[k] = row_load(src, nb, ch < Cin ? xo[k] : kOut, first ? cb : cb - a.Cx);
      } else {
        const uint32_t o = ch < Cin ? xo[k] : kOut;
        if constexpr (MODE == APS_CONV_DIRECT) {
          px[k] = row_load(xb, xbytes, o, cb);
        } else if constexpr (MODE == kModeReluMask) {
          const f32x4 gr = row_load(xb, xbytes, o, cb), yv = row_load(sb, sbytes, o, cb);
#pragma unroll
          for (int q = 0; q < 4; ++q) px[k][q] = yv[q] > 0.f ? gr[q] : 0.f;
        } else {
          const uint32_t dc = 4 * a.Cx, rs = 8 * a.W * a.Cx;
          auto at = [&](uint32_t d) { return row_load(xb, xbytes, o == kOut ? kOut : o + d, cb); };
          px[k] = ((at(0) + at(dc)) + (at(rs) + at(rs + dc))) * 0.25f;
        }
      }
    }
  };

  const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
  f16x8 A[TM][2];  // [m-tile][h, l] of the current tap
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(wp), 0, 0xffffffffu, 0x00020000);
  auto load_a = [&](int m, int dy, int dx, int c) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
      A[m][p] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(
          wr, lane * 16, wfrag(cob * TM + m, dy * 3 + dx, c, p, a.nchunk) * 2, 0));
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int m = 0; m < TM; ++m)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[m][j] = zero4;
  int erun = 0;  // largest biased exponent that has set the scale in this block
  int ex = 0;    // the activations' scale exponent

  if (PF) fetch(0);
#pragma unroll
  for (int m = 0; m < TM; ++m) load_a(m, 0, 0, 0);
  for (int c = 0; c < a.nchunk; ++c) {
    if (!PF) fetch(c);
    // the chunk's largest finite magnitude over the block (the barrier also ends the previous
    // chunk's reads of Xs)
    if (c * 32 + 32 > a.cvalid) {  // channels past the layer's inputs (padded rows)
#pragma unroll
      for (int k = 0; k < NXT; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (c * 32 + g4 + q >= a.cvalid) px[k][q] = 0.f;
    }
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < NXT; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) mx = fmaxf(mx, __builtin_fabsf(px[k][q]));
    if (__any(mx == __builtin_inff())) {  // an infinite input: the scale follows the finite ones
      mx = 0.f;
#pragma unroll
      for (int k = 0; k < NXT; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float v = __builtin_fabsf(px[k][q]);
          mx = v < __builtin_inff() && v > mx ? v : mx;
        }
    }
    // mean exponent of a sample of the finite non-zero elements: sum and count in one word
    uint32_t es = 0;
#pragma unroll
    for (int k = 0; k < NXT; k += 4) {
      const uint32_t e = __builtin_bit_cast(uint32_t, px[k][k >> 2 & 3]) >> 23 & 0xff;
      es += e != 0 && e != 255 ? e + 0x10000u : 0u;
    }
    mx = wave_max(mx);
    es = (uint32_t)wave_isum((int)es);
    if (lane == 0) {
      red[wave] = mx;
      rede[wave] = es;
    }
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    const int em = __builtin_amdgcn_readfirstlane((int)(__builtin_bit_cast(uint32_t, mx) >> 23 & 0xff));
    const uint32_t s01 = rede[0], s23 = rede[1], s45 = rede[2], s67 = rede[3];
    const uint32_t cnt = __builtin_amdgcn_readfirstlane((s01 >> 16) + (s23 >> 16) + (s45 >> 16) + (s67 >> 16));
    const uint32_t sum = __builtin_amdgcn_readfirstlane((s01 & 0xffff) + (s23 & 0xffff) + (s45 & 0xffff) + (s67 & 0xffff));
    // an element over 2^kOutlier of the typical one does not set the scale: it overflows, and the
    // outputs it reaches are summed in fp32
    const int ec = cnt ? std::min(em, (int)(sum / cnt) + kOutlier) : em;
    if (em != 0 && ec > erun) {
      const int en = std::min(14 + 127 - ec, 126);
      if (erun > 0 && en != ex) {
        const float f = pow2(std::max(en - ex, -126));
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[m][j] *= f;
      }
      erun = ec;
      ex = en;
    }
    const float sx = pow2(ex);
#pragma unroll
    for (int k = 0; k < NXT; ++k) {
      const int p = pl + 32 * k;
      f16x4 hv, lv;
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        const float v0 = px[k][e], v1 = px[k][e + 1];
        const f16x2 h2 = __builtin_convertvector(f32x2{v0 * sx, v1 * sx}, f16x2);
        // v sx - h is exact; times 2^11 it has the range of h, not the subnormals below it
        const f16x2 l2 = __builtin_convertvector(f32x2{__builtin_fmaf(v0, sx, -(float)h2[0]) * 2048.f,
                                                       __builtin_fmaf(v1, sx, -(float)h2[1]) * 2048.f}, f16x2);
        hv[e] = h2[0];
        hv[e + 1] = h2[1];
        lv[e] = l2[0];
        lv[e + 1] = l2[1];
      }
      if (p < NPX) {
        uint16_t* d = Xs + p * 32 + (((g4 >> 3) ^ (pl >> 1 & 3)) << 3) + (g4 & 4);  // (p >> 1) % 4 = (pl >> 1) % 4
        *reinterpret_cast<f16x4*>(d) = hv;
        *reinterpret_cast<f16x4*>(d + PL) = lv;
      }
    }
    __syncthreads();
    const bool more = c + 1 < a.nchunk;
    if (PF && more) fetch(c + 1);
    if constexpr (MODE == APS_CONV_POOL2 || MODE == kModeReluMask) __builtin_amdgcn_sched_barrier(0);
    f16x8 B[2][TN][2];
    auto load_b = [&](int t, f16x8 (&v)[TN][2]) {
      const int dx = t / 3, dy = t % 3, col = (lane & 15) + dx;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wave * TN + dy + j;  // pixel row SW + col, (pixel >> 1) % 4 = (row + col / 2) % 4
        const uint16_t* bp = Xs + (row * SW + col) * 32 + (((lane >> 4) ^ ((row + (col >> 1)) & 3)) << 3);
#pragma unroll
        for (int p = 0; p < 2; ++p) v[j][p] = *reinterpret_cast<const f16x8*>(bp + p * PL);
      }
    };
    load_b(0, B[0]);
#pragma unroll
    for (int t = 0; t < 9; ++t) {  // taps dx outer, dy inner
      __builtin_amdgcn_sched_barrier(0);  // one tap's operands (and the next one's) live at a time
      if (t < 8) load_b(t + 1, B[(t + 1) & 1]);
      auto& b = B[t & 1];
#pragma unroll
      for (int m = 0; m < TM; ++m) {
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = mmah(A[m][1], b[j][0], acc[m][j]);
        const f16x8 hs = A[m][0] * (_Float16)0x1p-11f;  // the staged l halves carry 2^11
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = mmah(hs, b[j][1], acc[m][j]);
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = mmah(A[m][0], b[j][0], acc[m][j]);
        // the m-tile's operands for the next tap
        if (t < 8) load_a(m, (t + 1) % 3, (t + 1) / 3, c);
        else if (more) load_a(m, 0, 0, c + 1);
      }
    }
  }

  // back to the layer's scale (exact), the bias, and plain fp32 where a sum is not finite
  float nf = 0.f;  // NaN if any sum is not finite
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int ct = cob * TM + m, co0 = ct * 16 + 4 * (lane >> 4);
    if (ct * 16 >= a.Cout) continue;
    int se[4];
    float bv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      se[q] = -ex - weight_exp(wp, ct, 4 * (lane >> 4) + q, a.nchunk);
      bv[q] = a.bias && co0 + q < a.Cout ? a.bias[co0 + q] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        nf = __builtin_fmaf(acc[m][j][q], 0.f, nf);
        acc[m][j][q] = __builtin_ldexpf(acc[m][j][q], se[q]) + bv[q];
      }
  }
  if (__any(nf != 0.f)) {
    const int col = tx0 + (lane & 15);
    for (int i = 0; i < TM * TN * 4; ++i) {  // one copy of the loop, the accumulator by selection
      const int m = i / (TN * 4), j = (i / 4) % TN, q = i & 3;
      const int row = ty0 + wave * TN + j, co = (cob * TM + m) * 16 + 4 * (lane >> 4) + q;
      float v = 0.f;
#pragma unroll
      for (int k = 0; k < TM * TN * 4; ++k)
        if (k == i) v = acc[k / (TN * 4)][(k / 4) % TN][k & 3];
      if (__builtin_fabsf(v) < __builtin_inff() || row >= a.H || col >= a.W || co >= a.Cout) continue;
      v = rescue<MODE>(a, wp, n, row, col, co) + (a.bias ? a.bias[co] : 0.f);
#pragma unroll
      for (int k = 0; k < TM * TN * 4; ++k)
        if (k == i) acc[k / (TN * 4)][(k / 4) % TN][k & 3] = v;
    }
  }
  if constexpr (HEAD) {
    __syncthreads();  // the head's re-layout reuses Xs
    conv_epilogue<float, float, TM, TN, HEAD, true>(a, acc, ty0 + wave * TN, tx0, cob, n, lane, wave,
                                                    reinterpret_cast<float*>(Xs));
  } else {
    epilogue_f32<TM, TN>(a, acc, ty0 + wave * TN, tx0, cob, n, lane);
  }
}

template <int MODE, int HEAD>
void launch_m(const ConvArgs& a, hipStream_t st) {
  ConvArgs b = a;
  b.ntx = (a.W + 15) / 16;
  b.nchunk = (a.Cx + a.C2 + 31) / 32;
  if (!b.cvalid) b.cvalid = a.Cx + a.C2;
  const int irows = std::min(a.H, 18);  // input rows of a tile
  b.big = (size_t)irows * (MODE == APS_CONV_POOL2 ? 4 : 1) * a.W * std::max(a.Cx, a.C2) * 4 >= 0xffff0000ull;
  // 8-row blocks (TN = 2) for small problems
  const bool wide = a.Cout > 32, tn2 = (size_t)a.N * a.H * a.W < 64 * 64 * 8;
  const int rows = tn2 ? 8 : 16;
  b.ntiles = b.ntx * ((a.H + rows - 1) / rows);
  b.nco = wide ? (a.Cout + 63) / 64 : 1;
  dim3 grid(xcd_grid(b.ntiles, b.nco), 1, a.N);
  const bool pf = b.nchunk > 1;
  if (!wide) {
    if (tn2) k_conv_split<MODE, 2, 2, HEAD, false><<<grid, 256, 0, st>>>(b);
    else k_conv_split<MODE, 2, 4, HEAD, false><<<grid, 256, 0, st>>>(b);
  } else if (tn2) {
    if (pf) k_conv_split<MODE, 4, 2, HEAD, true><<<grid, 256, 0, st>>>(b);
    else k_conv_split<MODE, 4, 2, HEAD, false><<<grid, 256, 0, st>>>(b);
  } else {
    if (pf) k_conv_split<MODE, 4, 4, HEAD, true><<<grid, 256, 0, st>>>(b);
    else k_conv_split<MODE, 4, 4, HEAD, false><<<grid, 256, 0, st>>>(b);
  }
}

// Packing: one block per output channel of the padded channel tiles (the layout of wfrag).
__global__ __launch_bounds__(256) void k_pack_split(const float* __restrict__ w, int Cout, int Cin, int nchunk,
                                                   uint16_t* __restrict__ out, int transpose) {
  __shared__ float red[4];
  const int co = blockIdx.x, lane = threadIdx.x, ct = co >> 4, k = co & 15;
  auto get = [&](int t, int ci) {
    if (co >= Cout || ci >= Cin) return 0.f;
    return transpose ? w[((size_t)ci * 9 + (8 - t)) * Cout + co] : w[((size_t)co * 9 + t) * Cin + ci];
  };
  const int total = 9 * nchunk * 32;
  float mx = 0.f;
  for (int i = lane; i < total; i += 256) {
    const float v = __builtin_fabsf(get(i / (nchunk * 32), i % (nchunk * 32)));
    mx = v < __builtin_inff() && v > mx ? v : mx;
  }
  mx = wave_max(mx);
  if ((lane & 63) == 0) red[lane >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const int e = scale_exp(mx), bits = mx == 0.f ? 0 : e + 128;
  const float s = pow2(e);
  for (int i = lane; i < total; i += 256) {
    const int t = i / (nchunk * 32), ci = i % (nchunk * 32);
    const float v = get(t, ci) * s;
    const _Float16 h = (_Float16)v;
    // infinities and NaN stay in h alone
    const _Float16 l = __builtin_fabsf(v) < __builtin_inff() ? (_Float16)(v - (float)h) : (_Float16)0.f;
    uint16_t lb = __builtin_bit_cast(uint16_t, l);
    if (t == 0 && ci < 8) lb = (uint16_t)((lb & ~1u) | ((bits >> exp_bit(ci)) & 1));
    const uint32_t o = wfrag(ct, t, ci >> 5, 0, nchunk) + ((ci >> 3 & 3) * 16 + k) * 8 + (ci & 7);
    out[o] = __builtin_bit_cast(uint16_t, h);
    out[o + 512] = lb;
  }
}

}  // namespace

namespace aps {

void pack_split(const float* w, int Cout, int Cin, void* packed, int transpose, hipStream_t st) {
  const int tiles = (Cout + 16 * kMaxTM - 1) / (16 * kMaxTM) * kMaxTM;
  k_pack_split<<<tiles * 16, 256, 0, st>>>(w, Cout, Cin, (Cin + 31) / 32, static_cast<uint16_t*>(packed), transpose);
}

void conv_split(const ConvArgs& a, hipStream_t st) {
  if (a.hw) {
    // heads of up to 64 logits keep the four-m-tile epilogue (fewer registers); 65..80 take five
#define APS_SPLIT(MODE)                          \
  if (a.hK > 64) launch_m<MODE, 5>(a, st);       \
  else launch_m<MODE, 4>(a, st);
    if (a.mode == APS_CONV_POOL2) { APS_SPLIT(APS_CONV_POOL2) }
    else if (a.mode == APS_CONV_UP2_CAT) { APS_SPLIT(APS_CONV_UP2_CAT) }
    else { APS_SPLIT(APS_CONV_DIRECT) }
#undef APS_SPLIT
    return;
  }
  if (a.mode == APS_CONV_POOL2) launch_m<APS_CONV_POOL2, 0>(a, st);
  else if (a.mode == APS_CONV_UP2_CAT) launch_m<APS_CONV_UP2_CAT, 0>(a, st);
  else if (a.mode == kModeReluMask) launch_m<kModeReluMask, 0>(a, st);
  else launch_m<APS_CONV_DIRECT, 0>(a, st);
}

}  // namespace aps
