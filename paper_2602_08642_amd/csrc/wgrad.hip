// bf16 weight and bias gradients of a convolution (k = 1 or 3) as a per-wave row sweep:
//   dW[co][tap][ci] = sum_px dY[px][co] X[px + d_tap][ci],   db[co] = sum_px dY[px][co]
// MFMA: M = 16 output channels, N = 16 input channels, K = 32 consecutive pixels of a row.  The
// pixels are the contraction index and the channels are contiguous in memory (NHWC), so the
// operands need a transpose: the rows are staged in LDS as they are ([pixel][32 channels]) and
// read with ds_read_b64_tr_b16, which hands each lane four pixels of one channel.
// A wave owns a 32 x 32 channel tile (all taps: 9 x 4 accumulators) and a band of 32 columns x R
// rows, and walks down the band without block barriers: one X row per step (34 pixels, each of
// its three column shifts read once) against the dY rows above, at and below it, which stay in
// registers as operands, so every X and dY row is staged once per band and a step is 8 operand
// fragments for 36 MFMAs.  The next step's global loads are in flight during the MFMAs.  The
// bias gradient is one more MFMA per dY fragment against ones, in the tiles of the first input
// channel block only.  The four waves of a block (four bands) add their tiles in LDS in a fixed
// order and write one partial per block; k_wgrad_sweep_reduce adds the partials in a fixed order.
// What bounds it: a step is about 450 instructions for 36 MFMAs, and its operand reads wait on the
// LDS between them (over the concat layers of a training step MFMA busy 17 %, LDS 21 %), so two waves
// per SIMD run as fast as one each: the launches of the two-block rule below.  For one channel tile the reads of X, dY
// and the mask (52 MB at 32 -> 32, 4 x 256 x 256) set 10 us of it.  The element-wise staging into
// channel-major LDS rows that this replaces took, with its separate bias and split reductions,
// 95 us at 32 -> 32 and 4 x 256 x 256 (64 + 7 + 10 + 4 us, gaps included); the two kernels here
// take 20 us; at (64 up + 32 skip) -> 32 227 -> 32 us.  Deeper register prefetch (2 to 4 rows) and
// 16 x 32 tiles at twice the waves changed nothing or were slower.
#include <algorithm>

#include "aps_common.h"
#include "mfma_frag.h"

using namespace aps;

namespace {

constexpr int kPS = 48;     // elements per staged pixel: 96 bytes, so that the four pixels x 32
                            // bytes a 16-lane group reads fall on distinct banks
constexpr int kCols = 32;   // columns per band = K of one MFMA
constexpr long kWgBlocks = 512;  // two blocks of four waves per CU
// Rounds of blocks whose partial sums the workspace holds; with more images than that a wave walks several
// bands (384 -> 128 channels, 64 images of 256 x 256: 228 MB without, 4096 of 16 x 16: 1.8 GB).
constexpr long kWgRounds = 4;

struct Args {
  const uint16_t *x, *x2, *dy, *ym;
  int N, H, W, Cx, C2, ldy, Cout;
  int R, nseg_c, nseg_r, nunit, ncit, ntile, splits;
  float* part;
};

typedef short trv __attribute__((ext_vector_type(4)));

// operand fragment from staged pixels p0 .. p0 + 31 and channels c0 .. c0 + 15: lane l gets channel
// c0 + l % 16 of pixels p0 + 8 (l / 16) + 0..7
__device__ inline Frag<uint16_t> read_tr(const uint16_t* row, int p0, int c0, int lane) {
  const int i = lane & 15;
  const uint16_t* p = row + (p0 + 8 * (lane >> 4) + (i >> 2)) * kPS + c0 + 4 * (i & 3);
  auto lds = [](const uint16_t* q) {
    return (__attribute__((address_space(3))) trv*)const_cast<uint16_t*>(q);
  };
  const trv a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds(p));
  const trv b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds(p + 4 * kPS));
  Frag<uint16_t> f;
  f.v = __builtin_bit_cast(u16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  return f;
}

__device__ inline void lds_sync() {  // orders this wave's LDS accesses across its lanes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v where the bf16 y > 0 (positive, finite or +inf: bits 1 .. 0x7f80), else 0
__device__ inline u16x8 relu_mask(u16x8 v, u16x8 y) {
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const u16x8 c = __builtin_elementwise_min(y - (uint16_t)1, (u16x8)(uint16_t)0x7f80) - (uint16_t)0x7f80;
  return v & __builtin_bit_cast(u16x8, __builtin_bit_cast(s16x8, c) >> (short)15);
}

// 16 bytes at byte offset off of a row of `bytes` bytes (uniform base); zeros where off is past it
__device__ inline u16x8 row_load(const uint16_t* base, uint32_t bytes, uint32_t off) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, bytes, 0x00020000);
  return __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// VEC: dY (and mask) rows of whole aligned 16-byte pieces; else they are read element by element.
// MANY: more bands than waves (with the loop over bands, the others lose 1 to 2 %).
template <int KS, int MODE, bool VEC, bool MANY>
__global__ __launch_bounds__(256, 2) void k_wgrad_sweep(Args a) {
  constexpr int KK = KS * KS, R1 = KS / 2, XW = kCols + 2 * R1;
  constexpr int NF = KK * 4 + 2;                    // fragments of a wave's tile, bias included
  constexpr int NX = (XW * 4 + 63) / 64;            // 16-byte X loads per lane and row
  constexpr int ROWS = (XW + kCols) * kPS;          // staged elements per wave
  constexpr int RED = 2 * NF * 64 * 8;              // two waves' tiles, in 2-byte elements
  __shared__ __attribute__((aligned(16))) uint16_t lds[4 * ROWS > RED ? 4 * ROWS : RED];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // Blocks go round-robin over the 8 XCDs, each with its own L2: an XCD takes a contiguous range of
  // (split, tile) with the tiles of a pixel split side by side, so the rows they share are read
  // from memory once.
  const int idx = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (idx >= a.splits * a.ntile) return;
  const int split = idx / a.ntile, tile = idx % a.ntile;
  const int cot = tile / a.ncit, cit = tile % a.ncit;
  const int H = a.H, W = a.W, Cin = a.Cx + a.C2;
  uint16_t* Xs = lds + wave * ROWS;
  uint16_t* Ys = Xs + XW * kPS;

  f32x4 acc[KK][2][2], bacc[2];
#pragma unroll
  for (int t = 0; t < KK; ++t)
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[t][m][s] = f32x4{0.f, 0.f, 0.f, 0.f};
  bacc[0] = bacc[1] = f32x4{0.f, 0.f, 0.f, 0.f};

  // whole waves; the block meets again at the barriers below
  for (int unit = split * 4 + wave; unit < a.nunit; unit += a.splits * 4) {
    const int n = unit / (a.nseg_c * a.nseg_r), u = unit % (a.nseg_c * a.nseg_r);
    const int x0 = (u % a.nseg_c) * kCols, y0 = (u / a.nseg_c) * a.R, y1 = min(y0 + a.R, H);
    const u16x8 zero = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
    // this lane's 16-byte pieces: X piece k = pixel (lane + 64 k) / 4, channels 8 (lane % 4) + [0,8)
    // of the input tile; dY piece k the same of the output tile
    const int g8 = 8 * (lane & 3), ci = cit * 32 + g8, co = cot * 32 + g8;
    // byte offsets from the band's first column (a row's may not fit 32 bits); past the end where the
    // piece is outside the image or the tensor
    constexpr uint32_t kOut = 0xfffffff0u;
    const int xb = max(x0 - R1, 0), nx = min(x0 + kCols + R1, W) - xb, ny = min(kCols, W - x0);
    const int ncx = (xb + nx + 1) / 2 - xb / 2;  // coarse columns (UP2_CAT)
    uint32_t xo[NX], so[NX], yo[2], mo[2];
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int p = (lane >> 2) + 16 * k, ix = x0 - R1 + p;
      const bool in = p < XW && ix >= 0 && ix < W && ci < Cin;
      if constexpr (MODE == APS_CONV_UP2_CAT) {
        xo[k] = in && ci < a.Cx ? (uint32_t)((ix / 2 - xb / 2) * a.Cx + ci) * 2 : kOut;
        so[k] = in && ci >= a.Cx ? (uint32_t)((ix - xb) * a.C2 + ci - a.Cx) * 2 : kOut;
      } else {
        xo[k] = in ? (uint32_t)((MODE == APS_CONV_POOL2 ? 2 : 1) * (ix - xb) * a.Cx + ci) * 2 : kOut;
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int px = (lane >> 2) + 16 * k;
      // channels of [Cout, ldy) may come along: they only reach rows of dW that are not written
      yo[k] = px < ny && co < a.ldy ? (uint32_t)(px * a.ldy + co) * 2 : kOut;
      mo[k] = px < ny && co < a.Cout ? (uint32_t)(px * a.Cout + co) * 2 : kOut;
    }
    // the band's first row of the image, and the elements from one of its rows to the next
    const size_t img = (size_t)n * H * W;
    const size_t xs = MODE == APS_CONV_POOL2 ? 4 * (size_t)W * a.Cx : MODE == APS_CONV_UP2_CAT ? (size_t)(W / 2) * a.Cx : (size_t)W * a.Cx;
    const uint16_t* xp = MODE == APS_CONV_POOL2 ? a.x + (4 * img + 2 * xb) * a.Cx
                         : MODE == APS_CONV_UP2_CAT ? a.x + (img / 4 + xb / 2) * a.Cx : a.x + (img + xb) * a.Cx;
    const uint16_t* x2p = a.x2 + (img + xb) * a.C2;
    const uint16_t* yp = a.dy + (img + x0) * a.ldy;
    const uint16_t* mp = a.ym ? a.ym + (img + x0) * a.Cout : yp;
    u16x8 xr[NX], yr[2], mr[2];
    auto load_x = [&](int iy) {
      const bool in = iy >= 0 && iy < H;
      if constexpr (MODE == APS_CONV_POOL2) {
        // 2x2 mean in the order and rounding of the forward's input transform
        const size_t rs = xs / 2;
        const uint16_t* q = xp + (in ? iy : 0) * xs;
        const uint32_t nb = in ? (uint32_t)(4 * nx) * a.Cx : 0u, dc = (uint32_t)a.Cx * 2;
#pragma unroll
        for (int k = 0; k < NX; ++k) {
          // an offset past the end stays past it: kOut + dc does not wrap for the lanes in use
          const uint32_t o1 = xo[k] == kOut ? kOut : xo[k] + dc;
          const u16x8 q0 = row_load(q, nb, xo[k]), q1 = row_load(q, nb, o1);
          const u16x8 q2 = row_load(q + rs, nb, xo[k]), q3 = row_load(q + rs, nb, o1);
          float r[8];
#pragma unroll
          for (int e = 0; e < 8; ++e)
            r[e] = ((bf2f(q0[e]) + bf2f(q1[e])) + (bf2f(q2[e]) + bf2f(q3[e]))) * 0.25f;
          const u16x4 lo = f2bf4(r[0], r[1], r[2], r[3]), hi = f2bf4(r[4], r[5], r[6], r[7]);
          xr[k] = u16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
      } else if constexpr (MODE == APS_CONV_UP2_CAT) {
        const int r = in ? iy : 0;
        const uint16_t* q = xp + (r / 2) * xs;
        const uint16_t* q2 = x2p + r * ((size_t)W * a.C2);
        const uint32_t nb = in ? (uint32_t)(2 * ncx) * a.Cx : 0u, nb2 = in ? (uint32_t)(2 * nx) * a.C2 : 0u;
        const bool has_x = cit * 32 < a.Cx, has_2 = cit * 32 + 32 > a.Cx;  // a tile may span both
#pragma unroll
        for (int k = 0; k < NX; ++k) {
          if (has_x && has_2) xr[k] = row_load(q, nb, xo[k]) | row_load(q2, nb2, so[k]);
          else if (has_x) xr[k] = row_load(q, nb, xo[k]);
          else xr[k] = row_load(q2, nb2, so[k]);
        }
      } else {
        const uint16_t* q = xp + (in ? iy : 0) * xs;
        const uint32_t nb = in ? (uint32_t)(2 * nx) * a.Cx : 0u;
#pragma unroll
        for (int k = 0; k < NX; ++k) xr[k] = row_load(q, nb, xo[k]);
      }
    };
    auto load_y = [&](int py) {  // y0 <= py < y1 <= H
      const uint16_t* q = yp + py * ((size_t)W * a.ldy);
      // without a mask an empty row (zeros): the load stays unconditional, so no wait is placed here
      const uint16_t* m = a.ym ? mp + py * ((size_t)W * a.Cout) : q;
      const uint32_t mb = a.ym ? (uint32_t)(2 * ny) * a.Cout : 0u;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if constexpr (VEC) {
          yr[k] = row_load(q, (uint32_t)(2 * ny) * a.ldy, yo[k]);
          mr[k] = row_load(m, mb, mo[k]);
        } else {
          const int px = (lane >> 2) + 16 * k;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const bool ok = px < ny && co + e < a.Cout;
            yr[k][e] = ok ? q[(size_t)px * a.ldy + co + e] : (uint16_t)0;
            if (a.ym) mr[k][e] = ok ? m[(size_t)px * a.Cout + co + e] : (uint16_t)0;
          }
        }
      }
    };
    Frag<uint16_t> A[3][2];  // dY rows r - 1, r, r + 1 of the current X row r
#pragma unroll
    for (int k = 0; k < 3; ++k) A[k][0].v = A[k][1].v = zero;
    Frag<uint16_t> ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones.v[e] = 0x3f80;

    // X row r needs dY rows r - R1 .. r + R1; row r + R1 is staged with it
    load_x(y0 - R1);
    load_y(y0);
    for (int r = y0 - R1; r < y1 + R1; ++r) {
      const int yn = r + R1;
      lds_sync();  // the previous step's reads are behind
#pragma unroll
      for (int k = 0; k < NX; ++k) {
        const int p = (lane >> 2) + 16 * k;
        if (p < XW) *reinterpret_cast<u16x8*>(Xs + p * kPS + g8) = xr[k];
      }
      if (yn < y1) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
          *reinterpret_cast<u16x8*>(Ys + ((lane >> 2) + 16 * k) * kPS + g8) =
              a.ym ? relu_mask(yr[k], mr[k]) : yr[k];
      }
      if (r + 1 < y1 + R1) load_x(r + 1);
      if (yn + 1 < y1) load_y(yn + 1);
      lds_sync();
      if constexpr (KS == 3) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          A[0][m] = A[1][m];
          A[1][m] = A[2][m];
        }
      }
      if (yn < y1) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          A[2][m] = read_tr(Ys, 0, 16 * m, lane);
          if (cit == 0) bacc[m] = mma(A[2][m], ones, bacc[m]);
        }
      }
      if (r < 0 || r >= H) continue;
#pragma unroll
      for (int dx = 0; dx < KS; ++dx) {
        Frag<uint16_t> B[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) B[s] = read_tr(Xs, dx, 16 * s, lane);
        // dY row r + R1 - ky meets X row r in tap row ky
#pragma unroll
        for (int ky = 0; ky < KS; ++ky) {
          const int q = r + R1 - ky;
          if (q < y0 || q >= y1) continue;
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int s = 0; s < 2; ++s)
              acc[ky * KS + dx][m][s] = mma(A[2 - ky][m], B[s], acc[ky * KS + dx][m][s]);
        }
      }
    }
    if (!MANY) break;
  }
  // add the four waves' tiles, (0 + 2) + (1 + 3), and write the block's partial: fragment f of
  // the tile as 64 consecutive float4
  f32x4* red = reinterpret_cast<f32x4*>(lds);
  auto each = [&](auto fn) {
#pragma unroll
    for (int t = 0; t < KK; ++t)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int s = 0; s < 2; ++s) fn((t * 2 + m) * 2 + s, acc[t][m][s]);
    fn(KK * 4, bacc[0]);
    fn(KK * 4 + 1, bacc[1]);
  };
  __syncthreads();
  if (wave >= 2) each([&](int f, f32x4& v) { red[((wave - 2) * NF + f) * 64 + lane] = v; });
  __syncthreads();
  if (wave < 2) each([&](int f, f32x4& v) { v += red[(wave * NF + f) * 64 + lane]; });
  __syncthreads();
  if (wave == 1) each([&](int f, f32x4& v) { red[f * 64 + lane] = v; });
  __syncthreads();
  if (wave == 0) {
    f32x4* out = reinterpret_cast<f32x4*>(a.part) + ((size_t)split * a.ntile + tile) * NF * 64;
    each([&](int f, f32x4& v) { out[f * 64 + lane] = v + red[f * 64 + lane]; });
  }
}

// 16 consecutive float4 of a tile per block: split lane r = t / 16 (16 lanes) adds the partials
// r, r + 16, ... in order into two accumulators, then the lanes are added in lane order.
__global__ __launch_bounds__(256) void k_wgrad_sweep_reduce(const f32x4* __restrict__ part, int splits,
                                                            int ntile, int ncit, int KK, int Cout,
                                                            int Cin, float* __restrict__ dw,
                                                            float* __restrict__ db) {
  __shared__ f32x4 red[16][16];
  const int t = threadIdx.x, e = t & 15, r = t >> 4;
  const int NF = KK * 4 + 2, tile = blockIdx.y, idx = blockIdx.x * 16 + e;
  const int f = idx >> 6, lane = idx & 63;
  const int cot = tile / ncit, cit = tile % ncit;
  if (f >= KK * 4 && (cit != 0 || !db)) return;  // whole blocks: 64 % 16 == 0
  const size_t stride = (size_t)ntile * NF * 64;
  const f32x4* p = part + (size_t)tile * NF * 64 + idx;
  f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0;
  int k = r;
#pragma unroll 2
  for (; k + 16 < splits; k += 32) {
    s0 += p[(size_t)k * stride];
    s1 += p[(size_t)(k + 16) * stride];
  }
  if (k < splits) s0 += p[(size_t)k * stride];
  red[r][e] = s0 + s1;
  __syncthreads();
  if (r != 0) return;
  f32x4 v = red[0][e];
#pragma unroll
  for (int q = 1; q < 16; ++q) v += red[q][e];
  if (f < KK * 4) {
    const int tap = f >> 2, m = (f >> 1) & 1, s = f & 1;
    const int ci = cit * 32 + s * 16 + (lane & 15), co0 = cot * 32 + m * 16 + 4 * (lane >> 4);
    if (ci < Cin)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (co0 + q < Cout) dw[((size_t)(co0 + q) * KK + tap) * Cin + ci] = v[q];
  } else if ((lane & 15) == 0) {  // every column of the ones product holds the same sum
    const int co0 = cot * 32 + (f - KK * 4) * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (co0 + q < Cout) db[co0 + q] = v[q];
  }
}

struct Plan {
  int ncot, ncit, R, nseg_c, nseg_r, nunit, splits;
  size_t bytes;
};

// Band height.  Two blocks fit a CU, and a launch of a few blocks more than that takes another
// round (64+32 -> 32 channels at 4 x 256 x 256: 528 blocks 39 us, 480 blocks 27 us), so the rows
// are cut into as many bands as stay within kWgBlocks.  Short bands cost halo rows and partial
// sums: at least 4 rows, and 8 where one channel tile covers the layer, whose halo rows come from
// memory and not from an L2 (32 -> 32 at 4 x 256 x 256: 4 rows 22.8 us, 8 rows 20.2 us; 32 -> 64 at
// 4 x 128 x 128, two tiles: 20.5 and 24.8 us).
Plan plan(int N, int H, int W, int Cin, int Cout, int KS) {
  Plan p{};
  p.ncot = (Cout + 31) / 32;
  p.ncit = (Cin + 31) / 32;
  p.nseg_c = (W + kCols - 1) / kCols;
  const long tiles = (long)p.ncot * p.ncit;
  const long bands = std::max(1L, std::max(1L, kWgBlocks / tiles) * 4 / ((long)N * p.nseg_c));
  const long R = std::min<long>(H, std::max<long>(tiles == 1 ? 8 : 4, (H + bands - 1) / bands));
  p.R = (int)R;
  p.nseg_r = (int)((H + R - 1) / R);
  p.nunit = N * p.nseg_c * p.nseg_r;
  const long most = 4 * std::max(1L, kWgRounds * kWgBlocks / tiles);  // waves per channel tile
  const long per = (p.nunit + most - 1) / most;  // bands per wave, as many for each as can be
  p.splits = (int)((p.nunit + 4 * per - 1) / (4 * per));
  p.bytes = (size_t)p.splits * tiles * (KS * KS * 4 + 2) * 64 * sizeof(f32x4);
  return p;
}

}  // namespace

namespace aps {

size_t wgrad_sweep_workspace(int N, int H, int W, int Cin, int Cout, int KS) {
  return plan(N, H, W, Cin, Cout, KS).bytes;
}

void wgrad_sweep(const void* x, const void* x2, int mode, int N, int H, int W, int Cx, int C2,
                 const void* dy, const void* ymask, int ldy, int Cout, int KS, float* dw, float* db,
                 void* ws, hipStream_t st) {
  const Plan p = plan(N, H, W, Cx + C2, Cout, KS);
  Args a{};
  a.x = static_cast<const uint16_t*>(x);
  a.x2 = static_cast<const uint16_t*>(x2);
  a.dy = static_cast<const uint16_t*>(dy);
  a.ym = static_cast<const uint16_t*>(ymask);
  a.N = N;
  a.H = H;
  a.W = W;
  a.Cx = Cx;
  a.C2 = C2;
  a.ldy = ldy;
  a.Cout = Cout;
  a.R = p.R;
  a.nseg_c = p.nseg_c;
  a.nseg_r = p.nseg_r;
  a.nunit = p.nunit;
  a.ncit = p.ncit;
  // 16-byte gradient rows (and mask rows): else element by element
  const bool vec = ldy % 8 == 0 && (reinterpret_cast<uintptr_t>(dy) & 15) == 0 &&
                   (!ymask || (Cout % 8 == 0 && (reinterpret_cast<uintptr_t>(ymask) & 15) == 0));
  a.part = static_cast<float*>(ws);
  a.ntile = p.ncot * p.ncit;
  a.splits = p.splits;
  const int grid = (p.splits * a.ntile + 7) / 8 * 8;
  const bool many = p.nunit > 4 * p.splits;
#define APS_WG(KS, MODE)                                                   \
  if (many) {                                                              \
    if (vec) k_wgrad_sweep<KS, MODE, true, true><<<grid, 256, 0, st>>>(a); \
    else k_wgrad_sweep<KS, MODE, false, true><<<grid, 256, 0, st>>>(a);    \
  } else {                                                                 \
    if (vec) k_wgrad_sweep<KS, MODE, true, false><<<grid, 256, 0, st>>>(a);\
    else k_wgrad_sweep<KS, MODE, false, false><<<grid, 256, 0, st>>>(a);   \
  }
#define APS_WG_M(KS)                                                       \
  if (mode == APS_CONV_POOL2) { APS_WG(KS, APS_CONV_POOL2) }               \
  else if (mode == APS_CONV_UP2_CAT) { APS_WG(KS, APS_CONV_UP2_CAT) }      \
  else { APS_WG(KS, APS_CONV_DIRECT) }
  if (KS == 3) { APS_WG_M(3) }
  else { APS_WG_M(1) }
#undef APS_WG_M
#undef APS_WG
  const int NF = KS * KS * 4 + 2;
  k_wgrad_sweep_reduce<<<dim3(NF * 4, p.ncot * p.ncit), 256, 0, st>>>(
      reinterpret_cast<const f32x4*>(ws), p.splits, p.ncot * p.ncit, p.ncit, KS * KS, Cout, Cx + C2, dw, db);
}

}  // namespace aps
