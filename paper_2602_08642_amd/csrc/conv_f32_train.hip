// fp32 3x3 convolutions of training layers with a ReLU, on v_mfma_f32_16x16x4_f32.  The sign of such a
// layer's sums decides which gradients pass, and sums within their rounding of zero come out with
// either sign: a forward pass summed in another order or precision (k_conv_split) gives gradients
// further from these by far more than either one's rounding (128 -> 256 channels at 260 x 278: 5e-4
// of their norm).  So the training forward pass keeps plain fp32 products in one order (bias, 16-channel
// chunks, dx outer, dy inner).  The other passes of the fp32 3x3 layers in 32-channel chunks (inference,
// data gradients, training layers without a ReLU) run in k_conv_split, at about 2.5 times the rate.
#include <algorithm>
#include <type_traits>

#include "conv_common.h"

using namespace aps;

namespace {

constexpr uint32_t kNoPixel = 0xffffffffu;

// Tile, row reuse and register prefetch of k_conv_lds: chunks of 16 input channels (4 per lane and
// fragment, 4 MFMAs per fragment pair), pixel stride 20 floats in LDS (conflict-free for the 16 lanes
// of a B fragment).  Bound by the fp32 MFMA rate (77 % of it over a U-Net).
template <int MODE, int TM, int TN>
__global__ __launch_bounds__(256, 2) void k_conv_f32(ConvArgs a) {
  constexpr int KC = 16, ROWS = 4 * TN, SH = ROWS + 2, SW = 18, PS = 20;
  constexpr int NXV = SH * SW * 4, NXT = (NXV + 255) / 256;  // input 16-B vectors per chunk
  constexpr int NAV = TM * 9 * 64, NAT = (NAV + 255) / 256;  // weight 16-B vectors per chunk
  __shared__ __attribute__((aligned(16))) float Xs[SH * SW * PS];
  __shared__ __attribute__((aligned(16))) float As[NAV * 4];

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const TileId tid_ = xcd_tile(blockIdx.x, a.ntiles, a.nco);
  if (tid_.tile >= a.ntiles) return;
  const int tx0 = (tid_.tile % a.ntx) * 16, ty0 = (tid_.tile / a.ntx) * ROWS;
  const int cob = tid_.cob, n = blockIdx.z;
  const float* x = static_cast<const float*>(a.x);
  const float* x2 = static_cast<const float*>(a.x2);
  const float* wp = static_cast<const float*>(a.wp);
  float* y = static_cast<float*>(a.y);
  const int Cin = a.Cx + a.C2;
  // This thread stages channel group g (4 channels) of tile pixel 16 w + l % 16 + 64 k, g = l / 16
  // (lane l of wave w; bank-conflict-free writes; offsets in floats).
  const int g4 = ((tid >> 4) & 3) * 4;
  const int pl = (tid >> 6) * 16 + (tid & 15);
  uint32_t xo[NXT], so[MODE == APS_CONV_UP2_CAT ? NXT : 1];
#pragma unroll
  for (int k = 0; k < NXT; ++k) {
    const int p = pl + 64 * k, r = p / SW, col = p - r * SW;
    const int iy = ty0 - 1 + r, ix = tx0 - 1 + col;
    const bool in = p < SH * SW && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
    uint32_t o = kNoPixel;
    if (in) {
      if constexpr (MODE == APS_CONV_POOL2)
        o = (uint32_t)((((size_t)n * 2 * a.H + 2 * iy) * (2 * a.W) + 2 * ix) * a.Cx + g4);
      else if constexpr (MODE == APS_CONV_UP2_CAT)
        o = (uint32_t)((((size_t)n * (a.H / 2) + iy / 2) * (a.W / 2) + ix / 2) * a.Cx + g4);
      else
        o = (uint32_t)((((size_t)n * a.H + iy) * a.W + ix) * a.Cx + g4);
    }
    xo[k] = o;
    if constexpr (MODE == APS_CONV_UP2_CAT)
      so[k] = in ? (uint32_t)((((size_t)n * a.H + iy) * a.W + ix) * a.C2 + g4) : kNoPixel;
  }
  const int wlast = (a.Cout + 15) / 16 * 9 - 1;  // weight rows (channel tile, tap) past it repeat it

  f32x4 px[NXT], pa[NAT];  // clang vector types: HIP's struct vectors are not promoted here
  uint32_t okbits = 0;
  const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
  auto fetch = [&](int c) {
    const int cb = c * KC;
    const bool in_ch = cb + g4 < Cin;
    okbits = 0;
#pragma unroll
    for (int k = 0; k < NXT; ++k) {
      const bool ok = xo[k] != kNoPixel && in_ch;
      okbits |= (uint32_t)ok << k;
      if constexpr (MODE == APS_CONV_DIRECT) {
        px[k] = *reinterpret_cast<const f32x4*>(x + (ok ? xo[k] + cb : 0u));
      } else if constexpr (MODE == APS_CONV_UP2_CAT) {
        const float* src = cb + g4 < a.Cx ? x + (xo[k] + cb) : x2 + (so[k] + (cb - a.Cx));
        px[k] = *reinterpret_cast<const f32x4*>(ok ? src : x);
      } else {
        f32x4 v = zero4;
        if (ok) {
          const uint32_t rs = (uint32_t)(2 * a.W * a.Cx);
          const uint32_t o = xo[k] + cb;
          const f32x4 q0 = *reinterpret_cast<const f32x4*>(x + o);
          const f32x4 q1 = *reinterpret_cast<const f32x4*>(x + (o + a.Cx));
          const f32x4 q2 = *reinterpret_cast<const f32x4*>(x + (o + rs));
          const f32x4 q3 = *reinterpret_cast<const f32x4*>(x + (o + rs + a.Cx));
          v = ((q0 + q1) + (q2 + q3)) * 0.25f;
        }
        px[k] = v;
      }
    }
#pragma unroll
    for (int k = 0; k < NAT; ++k)
      pa[k] = *reinterpret_cast<const f32x4*>(wp + (size_t)(std::min(cob * TM * 9 + wave + 4 * k, wlast) * a.nchunk + c) * 256 + lane * 4);
  };
  auto put = [&]() {
#pragma unroll
    for (int k = 0; k < NXT; ++k) {
      const int p = pl + 64 * k;
      if (p < SH * SW) *reinterpret_cast<f32x4*>(Xs + p * PS + g4) = (okbits >> k) & 1u ? px[k] : zero4;
    }
#pragma unroll
    for (int k = 0; k < NAT; ++k) {
      const int v = tid + 256 * k;
      if (v < NAV) *reinterpret_cast<f32x4*>(As + v * 4) = pa[k];
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    f32x4 b0 = f32x4{0.f, 0.f, 0.f, 0.f};
    const int co0 = (cob * TM + m) * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (a.bias && co0 + q < a.Cout) b0[q] = a.bias[co0 + q];
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[m][j] = b0;
  }

  fetch(0);
  put();
  __syncthreads();
  for (int c = 0; c < a.nchunk; ++c) {
    const bool more = c + 1 < a.nchunk;
    if (more) fetch(c + 1);
    if constexpr (MODE == APS_CONV_POOL2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      __builtin_amdgcn_sched_barrier(0);
      f32x4 A[3][TM];
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int m = 0; m < TM; ++m) A[dy][m] = *reinterpret_cast<const f32x4*>(As + ((m * 9 + dy * 3 + dx) * 64 + lane) * 4);
#pragma unroll
      for (int ir = 0; ir < TN + 2; ++ir) {
        const f32x4 B = *reinterpret_cast<const f32x4*>(Xs + ((wave * TN + ir) * SW + (lane & 15) + dx) * PS + (lane >> 4) * 4);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          const int j = ir - dy;
          if (j >= 0 && j < TN) {
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m][j] = mma4(A[dy][m], B, acc[m][j]);
          }
        }
      }
    }
    if (more) {
      __syncthreads();
      put();
      __syncthreads();
    }
  }
  const int col = tx0 + (lane & 15);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int row = ty0 + wave * TN + j;
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const int co = (cob * TM + m) * 16 + 4 * (lane >> 4);
      if (co >= a.Cout || row >= a.H || col >= a.W) continue;
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = a.relu ? fmaxf(acc[m][j][q], 0.f) : acc[m][j][q];
      store_out<float>(y + (((size_t)n * a.H + row) * a.W + col) * a.ldy, a.ldy, co, a.Cout, v);
    }
  }
}

// Row sweep of the layers with 16 -> 32, 32 -> 32 and 32 -> 64 channels (direct input), of which the tiled
// kernel computes two chunks at most for one staged tile.  A wave walks a band of 32 columns down R rows
// without block barriers: the weights (9 taps x CH chunks of 16 channels for MS m-tiles: both with 16
// input channels; with 32 one per wave, its neighbour waves taking the others, so that two waves fit a
// SIMD) stay in registers, and each input row is read from HBM once per band into a ring of three LDS
// rows, each held as CH planes of [36 px][20 floats] (the tiled kernel's pixel pitch, so the 16 lanes of a
// B read hit distinct banks).  The sums have the tiled kernel's order, and its bits.  Ring row i + 3 is
// staged into the slot of row i after this step's reads of it (one wave's LDS operations complete in
// program order).  Tiled and swept: 16 -> 32 at 1920 x 1080 198 and 163 us, 32 -> 32 344 and 307, 32 -> 64
// at 960 x 540 166 and 158; at 4 x 256 x 256 29 and 27, 55 and 45, 86 and 83.
constexpr int kSwCols = 32;  // output columns per band (two 16-pixel n-tiles)
constexpr int kSwPix = 36;   // staged input positions per row
constexpr int kCsfPS = 20;       // floats per staged pixel of a 16-channel plane

template <int CH, int MS>
__global__ __launch_bounds__(256) void k_conv_sweep_f32(ConvArgs a, int R, int nseg, int nunit) {
  constexpr int PL = kSwPix * kCsfPS;           // floats of one plane of a ring row
  constexpr int XR = CH * PL, XN = 3 * XR;      // ring of three rows
  constexpr int NU = 34 * CH * 4;               // 16-byte units of an input row (34 pixels)
  constexpr int NLD = (NU + 63) / 64;
  constexpr int D = 2;                          // input rows in flight in registers
  __shared__ __attribute__((aligned(16))) float lds[4][XN];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int unit = blockIdx.x * 4 + wave, n = blockIdx.y;
  if (unit >= nunit) return;  // the whole wave; nothing below synchronises waves
  const int H = a.H, W = a.W, Cx = a.Cx;
  // MS = 1: the Cout / 16 m-tiles of a band segment go to neighbouring waves
  const int nm = a.Cout >> 4;
  const int mt0 = MS == 2 ? 0 : unit % nm, bs = MS == 2 ? unit : unit / nm;
  const int x0 = (bs / nseg) * kSwCols, y0 = (bs % nseg) * R;
  float* X = lds[wave];
  for (int e = lane * 4; e < XN; e += 256) *reinterpret_cast<f32x4*>(X + e) = f32x4{0.f, 0.f, 0.f, 0.f};

  // weights (16-channel chunk packing): fragment (m, tap, chunk c), lane l = output channel
  // 16 m + l % 16, input channels 16 c + 4 (l / 16) + [0, 4)
  const float* wp = static_cast<const float*>(a.wp);
  f32x4 w[MS][9][CH];
#pragma unroll
  for (int m = 0; m < MS; ++m)
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int c = 0; c < CH; ++c)
        w[m][t][c] = *reinterpret_cast<const f32x4*>(wp + ((size_t)(((mt0 + m) * 9 + t) * CH + c) * 64 + lane) * 4);
  f32x4 bias[MS];
#pragma unroll
  for (int m = 0; m < MS; ++m) bias[m] = *reinterpret_cast<const f32x4*>(a.bias + 16 * (mt0 + m) + 4 * (lane >> 4));
  int bo[2][3];  // B read offsets within a plane: pixel 16 s + l % 16 + dx, channels 4 (l / 16)
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) bo[s][dx] = (16 * s + (lane & 15) + dx) * kCsfPS + 4 * (lane >> 4);

  // input rows: unit u = lane + 64 k is pixel u / (4 CH) (column x0 - 1 + u / (4 CH)), chunk
  // (u % (4 CH)) / 4, channels 4 (u % 4) .. + 3 of it
  const uint32_t img_bytes = (uint32_t)((size_t)H * W * Cx * sizeof(float));
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(static_cast<const float*>(a.x) + (size_t)n * H * W * Cx), 0, img_bytes, 0x00020000);
  auto load_row = [&](int iy, f32x4 (&v)[NLD]) {
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int u = lane + 64 * k, px = u / (4 * CH), xc = x0 - 1 + px;
      const bool in = u < NU && iy >= 0 && iy < H && xc >= 0 && xc < W;
      const uint32_t off = in ? (uint32_t)((((size_t)iy * W + xc) * Cx + 4 * (u % (4 * CH))) * sizeof(float)) : img_bytes;
      v[k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
    }
  };
  auto store_row = [&](float* dst, const f32x4 (&v)[NLD]) {
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int u = lane + 64 * k, px = u / (4 * CH), wv = u % (4 * CH);
      if (u < NU) *reinterpret_cast<f32x4*>(dst + (wv >> 2) * PL + px * kCsfPS + 4 * (wv & 3)) = v[k];
    }
  };
  float* y = static_cast<float*>(a.y);
  const int ylast = min(y0 + R, H) - 1;
  auto emit = [&](const f32x4 (&acc)[2][MS], int o) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int col = x0 + 16 * s + (lane & 15);
#pragma unroll
      for (int m = 0; m < MS; ++m) {
        const int co = 16 * (mt0 + m) + 4 * (lane >> 4);
        f32x4 v = acc[s][m];
        if (a.relu) {
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = fmaxf(v[q], 0.f);
        }
        if (col < W) *reinterpret_cast<f32x4*>(y + (((size_t)n * H + o) * W + col) * a.ldy + co) = v;
      }
    }
  };

  // ring row k (input row y0 - 1 + k) sits in slot k % 3; rows 0..2 are staged up front and rows
  // 3, 4 wait in registers gx[k % 2]
  {
    f32x4 v[NLD];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      load_row(y0 - 1 + k, v);
      store_row(X + k * XR, v);
    }
  }
  f32x4 gx[D][NLD];
#pragma unroll
  for (int k = 3; k < 3 + D; ++k) load_row(y0 - 1 + k, gx[k % D]);

  int s0 = 0;  // slot of ring row i
  auto step = [&](auto ph, int i) {
    constexpr int G = (decltype(ph)::value + 3) % D;  // == (i + 3) % D
    const int s1 = s0 == 2 ? 0 : s0 + 1, s2 = s1 == 2 ? 0 : s1 + 1;
    const float* rows[3] = {X + s0 * XR, X + s1 * XR, X + s2 * XR};
    wave_lds_sync();
    f32x4 acc[2][MS];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int m = 0; m < MS; ++m) acc[s][m] = bias[m];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        __builtin_amdgcn_sched_barrier(0);  // one tap column's operands live at a time
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const f32x4 b = *reinterpret_cast<const f32x4*>(rows[dy] + c * PL + bo[s][dx]);
#pragma unroll
            for (int m = 0; m < MS; ++m) acc[s][m] = mma4(w[m][3 * dy + dx][c], b, acc[s][m]);
          }
      }
    wave_lds_sync();
    const int o = y0 + i;
    if (o <= ylast) emit(acc, o);
    store_row(X + s0 * XR, gx[G]);  // ring row i + 3 into the slot of row i
    load_row(y0 + 2 + i + D, gx[G]);
    s0 = s1;
  };
  for (int i = 0; i < R; i += 4) {  // R % 4 == 0 (host)
    step(std::integral_constant<int, 0>{}, i);
    step(std::integral_constant<int, 1>{}, i + 1);
    step(std::integral_constant<int, 2>{}, i + 2);
    step(std::integral_constant<int, 3>{}, i + 3);
  }
}

// false: the tiled kernel.  At least half of the resident waves with segments of 8 rows: with fewer a wave's
// first rows are most of its time (16 -> 32 at 128 x 128, 64 segments: 25 us, tiled 6; at 3 x 200 x 311,
// 750: 27.4 and 26.8; at 4 x 256 x 256, 1024: 27.2 and 29.7).
bool launch_sweep(const ConvArgs& a, hipStream_t st) {
  if (a.mode != APS_CONV_DIRECT || a.C2 != 0 || a.ldy != a.Cout ||
      !((a.Cout == 32 && (a.Cx == 16 || a.Cx == 32)) || (a.Cout == 64 && a.Cx == 32)))
    return false;
  if ((size_t)a.H * a.W * a.Cx * 4 >= (1ull << 31) || a.N > 65535) return false;
  const long nband = (a.W + kSwCols - 1) / kSwCols;
  const int wps = a.Cx == 32 ? a.Cout / 16 : 1;  // waves per band segment
  if (a.N * nband * wps * ((a.H + 7) / 8) < 2 * kSweepGroups) return false;
  // four steps per loop iteration; two halo rows and about ten steps' time before the first output
  const SweepPlan plan = sweep_plan(a.N, a.H, nband * wps, 4, 12);
  const long nunit = nband * plan.nseg * wps;
  if (nunit > (1L << 30) / 4) return false;
  ConvArgs b = a;
  b.wp = static_cast<const float*>(a.wp) + f32_pack(a.Cout, a.Cx).plain;
  const dim3 g((unsigned)((nunit + 3) / 4), a.N);
  if (a.Cx == 32) k_conv_sweep_f32<2, 1><<<g, 256, 0, st>>>(b, (int)plan.R, (int)plan.nseg, (int)nunit);
  else k_conv_sweep_f32<1, 2><<<g, 256, 0, st>>>(b, (int)plan.R, (int)plan.nseg, (int)nunit);
  return true;
}

template <int MODE>
void launch(const ConvArgs& a, hipStream_t st) {
  ConvArgs b = a;
  b.ntx = (a.W + 15) / 16;
  b.nchunk = (a.Cx + a.C2 + 15) / 16;
  b.wp = static_cast<const float*>(a.wp) + f32_pack(a.Cout, a.Cx + a.C2).plain;
  // 8-row blocks (TN = 2) for small problems, and for POOL2 with TM = 4, whose 16-row variant
  // does not fit in 256 VGPRs
  const bool wide = a.Cout > 32;
  const bool tn2 = (size_t)a.N * a.H * a.W < 64 * 64 * 8 || (wide && MODE == APS_CONV_POOL2);
  const int rows = tn2 ? 8 : 16;
  b.ntiles = b.ntx * ((a.H + rows - 1) / rows);
  b.nco = wide ? (a.Cout + 63) / 64 : 1;
  dim3 grid(xcd_grid(b.ntiles, b.nco), 1, a.N);
  if (!wide) {
    if (tn2) k_conv_f32<MODE, 2, 2><<<grid, 256, 0, st>>>(b);
    else k_conv_f32<MODE, 2, 4><<<grid, 256, 0, st>>>(b);
  } else if (tn2) {
    k_conv_f32<MODE, 4, 2><<<grid, 256, 0, st>>>(b);
  } else if constexpr (MODE != APS_CONV_POOL2) {
    k_conv_f32<MODE, 4, 4><<<grid, 256, 0, st>>>(b);
  }
}

}  // namespace

namespace aps {

void conv_f32(const ConvArgs& a, hipStream_t st) {
  if (launch_sweep(a, st)) return;
  if (a.mode == APS_CONV_POOL2) launch<APS_CONV_POOL2>(a, st);
  else if (a.mode == APS_CONV_UP2_CAT) launch<APS_CONV_UP2_CAT>(a, st);
  else launch<APS_CONV_DIRECT>(a, st);
}

}  // namespace aps
