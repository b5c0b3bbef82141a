// fp32 3x3 convolutions of training layers with a ReLU, on v_mfma_f32_16x16x4_f32.  The sign of such a
// layer's sums decides which gradients pass, and sums within their rounding of zero come out with
// either sign: a forward pass summed in another order or precision (k_conv_split) gives gradients
// further from these by far more than either one's rounding (128 -> 256 channels at 260 x 278: 5e-4
// of their norm).  So the training forward pass keeps plain fp32 products in one order (bias, 16-channel
// chunks, dx outer, dy inner).  The other passes of the fp32 3x3 layers in 32-channel chunks (inference,
// data gradients, training layers without a ReLU) run in k_conv_split, at about 2.5 times the rate.
#include <algorithm>

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
  if (a.mode == APS_CONV_POOL2) launch<APS_CONV_POOL2>(a, st);
  else if (a.mode == APS_CONV_UP2_CAT) launch<APS_CONV_UP2_CAT>(a, st);
  else launch<APS_CONV_DIRECT>(a, st);
}

}  // namespace aps
