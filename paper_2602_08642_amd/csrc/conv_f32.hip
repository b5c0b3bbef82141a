// fp32 3x3 convolutions (every layer packed in 32-channel chunks: more than 16 input channels, or
// 9..16 with whole 16-channel output tiles beyond 16) on the fp16 matrix pipe.
//
// The fp32 MFMA runs at 1/16 of the fp16 rate, and at 80 % of it the tiled fp32 kernels had nowhere
// to go.  A float splits into two halves x = h + l with h = fp16(x), l = fp16(x - h), which hold 23 of
// its 24 bits, and x w = h_x h_w + h_x l_w + l_x h_w up to 2^-22 of the product: three
// v_mfma_f32_16x16x32_f16 with fp32 accumulation do the work of eight v_mfma_f32_16x16x4_f32, and
// the sum has a fifth of the roundings.  Range: the operands are scaled by powers of two, which is
// exact, and both l halves carry a factor 2^11, which keeps their last places on fp16's grid (2^-24): an
// operand's bits are there down to 2^-26 of the largest (kTop, kLow).  The cross products, 2^11 too
// large, are summed apart and added once per chunk.
//  * Weights per output channel at packing time, the largest to [2^14, 2^15); the exponents are in a
//    table behind the weights.  A channel whose weights are further apart than 2^26, or not finite, puts
//    its block of 32 or 64 channels on plain fp32 products (below).
//  * Activations per block: before a chunk is staged, the largest and the smallest magnitude of the
//    block's tile set the scale (kept from chunk to chunk where it holds both; the accumulators are
//    rescaled where it changes).  A tile that is further apart than 2^26 takes several passes over the
//    chunk, each with the elements of its range and zeros for the others, so every element is carried to
//    2^-23 of itself whatever its neighbours are.  An infinity, or scales further apart than 2^72 (kSpan),
//    put the block on plain fp32 products; NaN needs nothing.
//  * Plain products: the weights as they are, in the order of k_conv_f32 (equal bits).
// Time by the input (32 -> 32 at 1920 x 1080, 128 -> 128 at 480 x 270): ordinary tiles 179 and 102 us;
// half of the elements at 2^-30 or 2^-60 of the others, two passes, 290 and 182; plain products in every
// block 450 and 340.  (A scale for the typical element, with the outputs that meet a larger one summed
// again one by one, took 37 and 36 ms for half of the elements 2^30 apart.)
// What the halves leave out: the last of 24 bits where l rounds, and l_x l_w, up to 2^-22 of a product.
// Error against FP64 (normwise; fp32 MFMA kernels in brackets): 128 -> 128 channels 2.4e-7 (4.2e-7),
// the U-Net's heads at 1920 x 1080 7.9e-7 (1.5e-6).
//
// Tiling as k_conv_lds: blocks of 4 waves stacked vertically, TN rows x 16 px each, all sharing TM
// m-tiles; the chunk's input tile with its halo in LDS as two planes (64-byte pixels, 16-byte
// groups swizzled on bits 1-2 of the pixel index).  Two m-tiles at a time go through the taps, dx
// outer (so that the cross products of two suffice): each B operand is read again in place for the
// next tap after its last use.  The weight operands (A) come straight from global memory (the four
// waves read the same fragments from L1), a tap ahead, so no barrier and no LDS space goes to them.
// One order of sums for every entry point and size: 32-channel chunks, taps dx outer and dy inner, then
// the bias.  Powers of two change no bits, so the tile an output lies in matters only where it takes
// several passes over a chunk or plain products.
// What bounds it: for 32-channel blocks one chunk's latency (load, range, staging, MFMAs in turn, with
// three blocks per CU) and 1000 vector instructions per wave and chunk beside 216 MFMAs; for 64-channel
// blocks the MFMAs.  1920 x 1080, before (fp32 MFMA) and now:
// 16 -> 32 162 -> 156 us, 32 -> 32 317 -> 176 us, 64 -> 64 (960 x 540) 322 -> 125 us, 128 -> 128
// (480 x 270) 298 -> 105 us, 384 -> 128 841 -> 303 us, 96 -> 32 899 -> 363 us; the U-Net 5.59 -> 2.37 ms.
// Not kept: persistent blocks (fetching the next tile during the current one: registers spill),
// weights of all three tap rows live at once (spills), 8 channels per staging load.
#include <algorithm>

#include "conv_common.h"

using namespace aps;

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

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

// A value of exponent field f scaled by 2^e lies in the halves' range if f + e is at most kTop (h below
// 2^15) and, for all of its bits, at least kLow (its last place at 2^-35, that of l); subnormals
// count as f = 1.
constexpr int kTop = 141, kLow = 115;
// Scales of a block this far apart: the accumulators (sums up to 2^44 at the least scale, last places
// from 2^-47 at the greatest) stay finite and above the fp32 subnormals when they change scale.
constexpr int kSpan = 72;
constexpr int kPlain = 0x7fffffff;  // in the exponent table: not a channel for the halves
__device__ inline int exp_field(float v) { return std::max((int)(__builtin_bit_cast(uint32_t, v) >> 23 & 0xff), 1); }

// Input channels [ci, ci + 4) of pixel (iy, ix) after the input transform, in the order of stage8 (channel
// counts are multiples of 4); zeros outside the image and from channel `past` on
template <int MODE>
__device__ inline f32x4 conv_input4(const ConvArgs& a, int n, int iy, int ix, int ci, int past) {
  const float* x = static_cast<const float*>(a.x);
  const float* x2 = static_cast<const float*>(a.x2);
  f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
  if (iy < 0 || iy >= a.H || ix < 0 || ix >= a.W || ci >= past) return v;
  auto get = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  if constexpr (MODE == APS_CONV_POOL2) {
    const size_t rs = 2 * (size_t)a.W * a.Cx;
    const float* p = x + (((size_t)n * 2 * a.H + 2 * iy) * 2 * a.W + 2 * ix) * a.Cx + ci;
    v = ((get(p) + get(p + a.Cx)) + (get(p + rs) + get(p + rs + a.Cx))) * 0.25f;
  } else if constexpr (MODE == APS_CONV_UP2_CAT) {
    v = get(ci < a.Cx ? x + (((size_t)n * (a.H / 2) + iy / 2) * (a.W / 2) + ix / 2) * a.Cx + ci
                      : x2 + (((size_t)n * a.H + iy) * a.W + ix) * a.C2 + (ci - a.Cx));
  } else {
    const size_t o = (((size_t)n * a.H + iy) * a.W + ix) * a.Cx + ci;
    v = get(x + o);
    if constexpr (MODE == kModeReluMask) {
      const f32x4 y = get(x2 + o);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = y[q] > 0.f ? v[q] : 0.f;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (ci + q >= past) v[q] = 0.f;
  return v;
}

// A wave's values reduced, in lane 63 (rows of 16 lanes by shifts, then across the rows)
template <int CTRL, typename F>
__device__ inline uint32_t dpp_step(uint32_t v, F f) {
  return f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false));
}
template <typename F>
__device__ inline uint32_t wave_reduce(uint32_t v, F f) {
  v = dpp_step<0x111>(v, f);  // row_shr:1, 2, 4, 8
  v = dpp_step<0x112>(v, f);
  v = dpp_step<0x114>(v, f);
  v = dpp_step<0x118>(v, f);
  v = dpp_step<0x142>(v, f);  // row_bcast:15
  return dpp_step<0x143>(v, f);  // row_bcast:31
}

// Fragment f (in units of 512 halves) of channel tile ct, tap t, chunk c, half p (0: h, 1: l)
__device__ inline uint32_t wfrag(int ct, int t, int c, int p, int nchunk) {
  return (uint32_t)(((ct * 9 + t) * nchunk + c) * 2 + p) * 512u;
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

template <int MODE, int TM, int TN, int HEAD>
__global__ __launch_bounds__(256, TM == 4 ? 2 : 3) void k_conv_split(ConvArgs a) {
  constexpr int ROWS = 4 * TN, SH = ROWS + 2, SW = 18, NPX = SH * SW;
  constexpr int NXT = (NPX * 8 + 255) / 256;  // (pixel, 4 channels) items per thread and chunk
  constexpr int PL = NPX * 32;          // halves per plane
  constexpr int XS_HEAD = HEAD ? 2 * head_lds_elems<float, float, TM, HEAD>() : 0;
  __shared__ __attribute__((aligned(16))) uint16_t Xs[2 * PL > XS_HEAD ? 2 * PL : XS_HEAD];
  __shared__ uint32_t red[2][4];

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const TileId tid_ = xcd_tile(blockIdx.x, a.ntiles, a.nco);
  if (tid_.tile >= a.ntiles) return;
  const int tx0 = (tid_.tile % a.ntx) * 16, ty0 = (tid_.tile / a.ntx) * ROWS;
  const int cob = tid_.cob, n = blockIdx.z;
  const float* x = static_cast<const float*>(a.x);
  const float* x2 = static_cast<const float*>(a.x2);
  const int Cin = a.Cx + a.C2;
  // This thread stages channels [g4, g4 + 4) of tile pixels tid / 8 + 32 k: a wave's load reads 8
  // pixels' whole 128-byte chunks (with 8 channels per thread and 16 pixels per load the same bytes
  // cost the address unit twice the cycles).
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
  const size_t row0 = (size_t)n * a.H + yb;
  const float* xb = MODE == APS_CONV_POOL2 ? x + row0 * 4 * a.W * a.Cx
                    : MODE == APS_CONV_UP2_CAT ? x + ((size_t)n * (a.H / 2) + yb / 2) * (a.W / 2) * a.Cx
                                               : x + row0 * a.W * a.Cx;
  const uint32_t xbytes = MODE == APS_CONV_POOL2 ? (uint32_t)rows * 4 * a.W * a.Cx * 4
                          : MODE == APS_CONV_UP2_CAT ? (uint32_t)((yb + rows + 1) / 2 - yb / 2) * (a.W / 2) * a.Cx * 4
                                                     : (uint32_t)rows * a.W * a.Cx * 4;
  const float* sb = x2 + row0 * a.W * (MODE == APS_CONV_UP2_CAT ? a.C2 : a.Cx);
  const uint32_t sbytes = (uint32_t)rows * a.W * (MODE == APS_CONV_UP2_CAT ? a.C2 : a.Cx) * 4;

  // Global loads of a chunk (the pooled and masked transforms are evaluated here).  Not fetched ahead
  // during the MFMAs: 44 registers that cost the 32-channel blocks one of three blocks per CU and make
  // the 64-channel blocks spill (64 -> 64 at 540 x 960 127 us, 149 with it), for two blocks overlap.
  f32x4 px[NXT];
  auto fetch = [&](int c) {
    const int cb = c * 32, ch = cb + g4;
    if (cb == 0 || (MODE == APS_CONV_UP2_CAT && cb >= a.Cx && cb < a.Cx + 32)) offsets(cb >= a.Cx);
    // input rows whose bytes do not fit 32-bit offsets, and a chunk that spans both tensors of the concat
    if (a.big || (MODE == APS_CONV_UP2_CAT && cb < a.Cx && cb + 32 > a.Cx)) {
#pragma unroll
      for (int k = 0; k < NXT; ++k) {
        __builtin_amdgcn_sched_barrier(0);  // one item's addresses live at a time
        const int p = opaque(pl) + 32 * k, r = p / SW;
        px[k] = conv_input4<MODE>(a, n, ty0 - 1 + r, tx0 - 1 + p - r * SW, ch, p < NPX ? a.cvalid : 0);
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
  const F32Pack pk = f32_pack(a.Cout, a.cvalid);
  const float* wf = static_cast<const float*>(a.wp);
  // the block's scale exponents, channel 16 cob TM + lane; in plain fp32 if one channel has none
  const int nch = (a.Cout + 15) / 16 * 16, ch0 = cob * TM * 16;
  const int we = lane < TM * 16 && ch0 + lane < nch ? reinterpret_cast<const int*>(wf + pk.table)[ch0 + lane] : 0;
  // Tiles past the last output channel read zeros.  Two m-tiles of a tap at a time (load_a: step s is
  // tap s % 9 of the m-tiles 2 (s / 9) + [0, 2)).
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wf), 0, (uint32_t)(pk.plain * 4), 0x00020000);
  constexpr int S = TM / 2 * 9;
  f16x8 A[2][2][2];  // [step parity][m-tile][h, l]
  auto load_a = [&](int s, int c, f16x8 (&v)[2][2]) {
    const int t = s % 9, dx = t / 3, dy = t % 3;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p)
        v[q][p] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(
            wr, lane * 16, wfrag(cob * TM + s / 9 * 2 + q, dy * 3 + dx, c, p, a.nchunk) * 2, 0));
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int m = 0; m < TM; ++m)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[m][j] = zero4;
  int ex = 0, exlo = 1000, exhi = -1000;  // the activations' scale exponent, the least and greatest so far
  float lim = 0.f;  // not 0: only the chunk's elements below it are left to do

  load_a(0, 0, A[0]);
  bool plain = __any(we == kPlain);
  for (int c = 0; c < a.nchunk && !plain;) {
    fetch(c);
    if (c * 32 + 32 > a.cvalid) {  // channels past the layer's inputs (padded rows)
#pragma unroll
      for (int k = 0; k < NXT; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (c * 32 + g4 + q >= a.cvalid) px[k][q] = 0.f;
    }
    if (lim != 0.f) {
#pragma unroll
      for (int k = 0; k < NXT; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) px[k][q] = __builtin_fabsf(px[k][q]) < lim ? px[k][q] : 0.f;
    }
    // the largest and the smallest non-zero magnitude over the block (NaN: in neither; the barrier
    // also ends the previous chunk's reads of Xs)
    float mx = 0.f;
    uint32_t mw = ~0u;  // twice the smallest's bits, less 1: zeros come out largest
#pragma unroll
    for (int k = 0; k < NXT; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = px[k][q];  // by value: see lane_xor1
        mx = fmaxf(mx, __builtin_fabsf(v));
        mw = std::min(mw, (__builtin_bit_cast(uint32_t, v) << 1) - 1);
      }
    const uint32_t mb = wave_reduce(__builtin_bit_cast(uint32_t, mx), [](uint32_t x, uint32_t y) { return std::max(x, y); });
    mw = wave_reduce(mw, [](uint32_t x, uint32_t y) { return std::min(x, y); });
    if (lane == 63) {
      red[0][wave] = mb;
      red[1][wave] = mw;
    }
    __syncthreads();
    const uint32_t most = __builtin_amdgcn_readfirstlane(std::max(std::max(red[0][0], red[0][1]), std::max(red[0][2], red[0][3])));
    const uint32_t least = __builtin_amdgcn_readfirstlane(std::min(std::min(red[1][0], red[1][1]), std::min(red[1][2], red[1][3])));
    bool part = false;  // elements remain for another pass over the chunk
    if (most) {
      const int fh = std::max((int)(most >> 23), 1), fl = std::max((int)((least + 1) >> 24), 1);  // exponent fields
      if (exhi < exlo || fh + ex > kTop || fl + ex < kLow) {
        // in the middle of what holds them all, so that few chunks move it; else for the largest
        const int hi = kTop - fh, lo = kLow - fl, en = std::min(lo <= hi ? (lo + hi) >> 1 : hi, 126), d = en - ex;
        const bool fresh = exhi < exlo;
        exlo = std::min(exlo, en);
        exhi = std::max(exhi, en);
        if (fh == 255 || exhi - exlo > kSpan) {
          plain = true;
          break;
        }
        ex = en;
        if (!fresh && d != 0) {
          const float f = pow2(d);
#pragma unroll
          for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[m][j] *= f;
        }
      }
      part = fl + ex < kLow;
    }
    lim = part ? pow2(kLow - 127 - ex) : 0.f;
    if (part) {
#pragma unroll
      for (int k = 0; k < NXT; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) px[k][q] = __builtin_fabsf(px[k][q]) < lim ? 0.f : px[k][q];
    }
    const int cn = part ? c : c + 1;
    const float sx = pow2(ex);
#pragma unroll
    for (int k = 0; k < NXT; ++k) {
      const int p = pl + 32 * k;
      f16x4 hv, lv;
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        const float v0 = px[k][e], v1 = px[k][e + 1];
        const f16x2 h2 = __builtin_convertvector(f32x2{v0 * sx, v1 * sx}, f16x2);
        // v sx - h is exact; times 2^11 its last place is on fp16's grid
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
    f16x8 B[TN][2];
    uint32_t bo[4];  // of a tap column: offsets for rows r % 4, recomputed (held over the chunks they spill)
    auto load_b = [&](int t, int j) {
      const int dx = t / 3, dy = t % 3;
      if (dy == 0 && j == 0) {
        const int l = opaque(lane), col = (l & 15) + dx;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          bo[r] = (wave * TN * SW + col) * 32 + (((l >> 4) ^ ((wave * TN + r + (col >> 1)) & 3)) << 3);
      }
      const uint16_t* bp = Xs + bo[(dy + j) & 3] + (dy + j) * SW * 32;
#pragma unroll
      for (int p = 0; p < 2; ++p) B[j][p] = *reinterpret_cast<const f16x8*>(bp + p * PL);
    };
#pragma unroll
    for (int j = 0; j < TN; ++j) load_b(0, j);
#pragma unroll
    for (int g = 0; g < TM / 2; ++g) {
      f32x4 cr[2][TN];  // the cross products, 2^11 too large
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < TN; ++j) cr[q][j] = zero4;
#pragma unroll
      for (int t = 0; t < 9; ++t) {  // taps dx outer, dy inner
        const int s = g * 9 + t;
        __builtin_amdgcn_sched_barrier(0);  // one step's operands (and the next one's weights) live at a time
        if (s + 1 < S) load_a(s + 1, c, A[(s + 1) & 1]);
        const auto& w = A[s & 1];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
          for (int q = 0; q < 2; ++q) cr[q][j] = mmah(w[q][1], B[j][0], cr[q][j]);
#pragma unroll
          for (int q = 0; q < 2; ++q) acc[2 * g + q][j] = mmah(w[q][0], B[j][0], acc[2 * g + q][j]);
#pragma unroll
          for (int q = 0; q < 2; ++q) cr[q][j] = mmah(w[q][0], B[j][1], cr[q][j]);
          if (s + 1 < S) load_b((s + 1) % 9, j);  // in place
        }
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[2 * g + q][j] += cr[q][j] * 0x1p-11f;
    }
    c = cn;
    if (c < a.nchunk) load_a(0, c, A[0]);
  }

  if (!plain) {
    // back to the layer's scale (exact) and the bias
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const int co0 = (cob * TM + m) * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int se = -ex - __shfl(we, m * 16 + 4 * (lane >> 4) + q, 64);
        const float bv = a.bias && co0 + q < a.Cout ? a.bias[co0 + q] : 0.f;
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j][q] = __builtin_ldexpf(acc[m][j][q], se) + bv;
      }
    }
  } else {
    // k_conv_f32's sums: the bias, 16-channel chunks, taps dx outer and dy inner, plain fp32 products
    const int tid = opaque(threadIdx.x), lane = tid & 63, pl = tid >> 3, g4 = (tid & 7) * 4;
    float* Xf = reinterpret_cast<float*>(Xs);  // 32 channels a pixel, their 16-byte groups permuted
    const __amdgpu_buffer_rsrc_t pr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wf) + pk.plain, 0, (uint32_t)((pk.table - pk.plain) * 4), 0x00020000);
    const int n16 = (a.cvalid + 15) / 16;
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const int co0 = (cob * TM + m) * 16 + 4 * (lane >> 4);
      f32x4 b0 = zero4;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (a.bias && co0 + q < a.Cout) b0[q] = a.bias[co0 + q];
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[m][j] = b0;
    }
    for (int c = 0; c < a.nchunk; ++c) {
      __syncthreads();
#pragma unroll 1
      for (int p = pl; p < NPX; p += 32) {
        const int r = p / SW;
        *reinterpret_cast<f32x4*>(Xf + p * 32 + (((g4 >> 2) ^ (p & 7)) << 2)) =
            conv_input4<MODE>(a, n, ty0 - 1 + r, tx0 - 1 + p - r * SW, c * 32 + g4, a.cvalid);
      }
      __syncthreads();
      for (int c16 = 2 * c; c16 < std::min(2 * c + 2, n16); ++c16)
#pragma unroll 1
        for (int t = 0; t < 9; ++t) {
          const int dx = t / 3, dy = t % 3;
          f32x4 W[TM];
#pragma unroll
          for (int m = 0; m < TM; ++m)
            W[m] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                pr, lane * 16, (uint32_t)((((cob * TM + m) * 9 + dy * 3 + dx) * n16 + c16) * 1024), 0));
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int p = (wave * TN + dy + j) * SW + (lane & 15) + dx;
            const f32x4 b = *reinterpret_cast<const f32x4*>(Xf + p * 32 + ((((c16 & 1) * 4 + (lane >> 4)) ^ (p & 7)) << 2));
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m][j] = mma4(W[m], b, acc[m][j]);
          }
        }
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
  if (!wide) {
    if (tn2) k_conv_split<MODE, 2, 2, HEAD><<<grid, 256, 0, st>>>(b);
    else k_conv_split<MODE, 2, 4, HEAD><<<grid, 256, 0, st>>>(b);
  } else {
    if (tn2) k_conv_split<MODE, 4, 2, HEAD><<<grid, 256, 0, st>>>(b);
    else k_conv_split<MODE, 4, 4, HEAD><<<grid, 256, 0, st>>>(b);
  }
}

// Packing: one block per output channel of the 16-channel tiles (the layouts of wfrag and f32_pack).
// The plain part: [channel tile][tap][16-channel chunk][lane][4], lane l output channel l % 16 and
// input channels 4 (l / 16) + [0, 4).
__global__ __launch_bounds__(256) void k_pack_split(const float* __restrict__ w, int Cout, int Cin, int nchunk,
                                                   float* __restrict__ packed, int transpose) {
  __shared__ float red[2][4];
  const int co = blockIdx.x, lane = threadIdx.x, ct = co >> 4, k = co & 15;
  auto get = [&](int t, int ci) {
    if (co >= Cout || ci >= Cin) return 0.f;
    return transpose ? w[((size_t)ci * 9 + (8 - t)) * Cout + co] : w[((size_t)co * 9 + t) * Cin + ci];
  };
  const int total = 9 * nchunk * 32;
  const float inf = __builtin_inff();
  // the largest and the smallest magnitude that is not zero; the largest infinite if one is not finite
  float mx = 0.f, mn = inf;
  for (int i = lane; i < total; i += 256) {
    const float v = __builtin_fabsf(get(i / (nchunk * 32), i % (nchunk * 32)));
    mx = fmaxf(mx, v < inf ? v : inf);
    mn = fminf(mn, v == 0.f ? inf : v);
  }
  mx = wave_max(mx);
  mn = -wave_max(-mn);
  if ((lane & 63) == 0) {
    red[0][lane >> 6] = mx;
    red[1][lane >> 6] = mn;
  }
  __syncthreads();
  mx = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
  mn = fminf(fminf(red[1][0], red[1][1]), fminf(red[1][2], red[1][3]));
  int e = 0;
  if (mx > 0.f) e = std::min(kTop - exp_field(mx), 126);
  const bool plain = mx == inf || (mx > 0.f && exp_field(mn) + e < kLow);
  const float s = plain ? 0.f : pow2(e);
  const F32Pack pk = f32_pack(Cout, Cin);
  const int n16 = (Cin + 15) / 16;
  uint16_t* out = reinterpret_cast<uint16_t*>(packed);
  for (int i = lane; i < total; i += 256) {
    const int t = i / (nchunk * 32), ci = i % (nchunk * 32);
    const float x = get(t, ci), v = plain ? 0.f : x * s;
    const _Float16 h = (_Float16)v, l = (_Float16)((v - (float)h) * 2048.f);
    const uint32_t o = wfrag(ct, t, ci >> 5, 0, nchunk) + ((ci >> 3 & 3) * 16 + k) * 8 + (ci & 7);
    out[o] = __builtin_bit_cast(uint16_t, h);
    out[o + 512] = __builtin_bit_cast(uint16_t, l);
    if (ci < 16 * n16)
      packed[pk.plain + ((size_t)(ct * 9 + t) * n16 + (ci >> 4)) * 256 + ((ci >> 2 & 3) * 16 + k) * 4 + (ci & 3)] = x;
  }
  if (lane == 0) reinterpret_cast<int*>(packed + pk.table)[co] = plain ? kPlain : e;
}

}  // namespace

namespace aps {

void pack_split(const float* w, int Cout, int Cin, void* packed, int transpose, hipStream_t st) {
  k_pack_split<<<(Cout + 15) / 16 * 16, 256, 0, st>>>(w, Cout, Cin, (Cin + 31) / 32, static_cast<float*>(packed), transpose);
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
