// Backward of the gathering pyramidal filter (App. A), hand-written for gfx950.
//
// Forward per output pixel q of level l:  y_q = sum_k w_qk v_qk,  w_q = softmax(z_q) over the
// joint [kd | ku | kt] block (eqs. app-softmax-mid/full), v_qk the gathered value of tap k.
//   dLoss/dz_qk  = w_qk (<g_q, v_qk> - <g_q, y_q>)           (softmax Jacobian)
//   dLoss/dv_qk  = w_qk g_q, routed back to the pixel tap k read:
//     kd taps -> L^l            (eq. app-gather, edge-clamped)
//     ku taps -> Lhat^{l+1}     (eq. app-upsample), which is the output of level l+1
//     kt taps -> W(prev)        (eq. app-recon-full) and through the bilinear warp to prev.
// The coarser reconstructed levels are recomputed with the forward kernel, not stored; the
// pass then runs fine-to-coarse, level l handing dLoss/dLhat^{l+1} to level l+1.
// The transposes are gathers over the pixels that read each input pixel (deterministic), the taps
// that the edge clamped folded into the edge's own tap where the weights are written;
// only the warp's bilinear splat into prev uses atomics.
#include "filter_common.h"

using namespace aps;
using namespace aps::flt;

namespace {

struct BwdArgs {
  LevelArgs f;          // forward inputs of the level (f.out unused)
  const float4* gout;   // dLoss/dLhat^l [N, H, W]
  void* glogits;        // [N, H, W, gstride] in the gradient dtype
  int gstride;
  int gvec;             // gradient rows are whole aligned 16-byte pieces
  float* wbuf;          // [NK][N, H, W] normalised weights for the transposes, a plane per tap
  size_t plane;         // N H W
};

__device__ inline void gstore(float* p, float v) { *p = v; }
__device__ inline void gstore(uint16_t* p, float v) { *p = f2bf(v); }
__device__ inline void gstore16(float* p, const float* v) {
  *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
}
__device__ inline void gstore16(uint16_t* p, const float* v) {
  const u16x4 lo = f2bf4(v[0], v[1], v[2], v[3]), hi = f2bf4(v[4], v[5], v[6], v[7]);
  *reinterpret_cast<u16x8*>(p) = u16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

// dLoss/dz of one level and the weights the transposes need.  Bound by memory: the logit row, the
// gradient row and a float per tap and pixel.  The weights go out as one plane per tap, so that a
// wave's stores (and the transposes' reads of a shifted row) are whole lines, and the gradient row
// as 16-byte pieces; with [pixel][tap] weights and 2-byte gradient stores, each store instruction
// touched 64 lines.  4 x 256 x 256, 43 taps, bf16: 82 -> 24 us.

// With c, the weight `from` joins `to`
__device__ inline void fold_move(float& to, float& from, bool c) {
  to += c ? from : 0.f;
  from = c ? 0.f : from;
}

// K x K taps of pixel (x, y): taps clamped to the edge join the edge's tap, outermost first
template <int K>
__device__ inline void fold(float* w, int x, int y, int W, int H) {
  constexpr int R = K / 2;
#pragma unroll
  for (int d = R; d > 0; --d) {
    const bool l = x - d < 0, r = x + d > W - 1;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      fold_move(w[i * K + R - d + 1], w[i * K + R - d], l);
      fold_move(w[i * K + R + d - 1], w[i * K + R + d], r);
    }
  }
#pragma unroll
  for (int d = R; d > 0; --d) {
    const bool t = y - d < 0, b = y + d > H - 1;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      fold_move(w[(R - d + 1) * K + i], w[(R - d) * K + i], t);
      fold_move(w[(R + d - 1) * K + i], w[(R + d) * K + i], b);
    }
  }
}

template <int KD, int KU, int KT, bool HU, bool HT, typename LT, typename GT>
__global__ __launch_bounds__(256) void k_level_bwd(BwdArgs b) {
  const LevelArgs& a = b.f;
  using G = Geo<KD, KU, KT, HU, HT>;
  constexpr int NK = G::NK;
  constexpr int VW = LogitVec<LT>::kW;
  constexpr int NKP = (NK + VW - 1) / VW * VW;
  __shared__ float4 Ls[G::LS];
  __shared__ float4 Cs[G::CS];
  __shared__ float4 Ts[G::PS];

  const int H = a.H, W = a.W;
  const int tid = threadIdx.x, tx = tid % TW, ty = tid / TW;
  const int x0 = blockIdx.x * TW, y0 = blockIdx.y * TH, n = blockIdx.z;
  const int x = x0 + tx, y = y0 + ty;
  const bool in = x < W && y < H;
  const size_t pix = ((size_t)n * H + y) * W + x;

  float z[NKP];
  if (in) LogitVec<LT>::template load<NKP>(static_cast<const LT*>(a.logits) + pix * a.kstride, z);
  stage_tiles<G>(a, Ls, Cs, Ts, x0, y0, n, HU, HT);
  __syncthreads();
  if (!in) return;

  float m = z[0];
#pragma unroll
  for (int k = 1; k < NK; ++k) m = fmaxf(m, z[k]);
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    z[k] = softmax_exp(z[k] - m);
    sum += z[k];
  }
  const float inv = 1.f / sum;
#pragma unroll
  for (int k = 0; k < NK; ++k) z[k] *= inv;
  // d_k = <g, v_k>; taps of a block that is not part of this output (the standalone reproject and
  // upsample terms) stay 0 and take only their share of the normalisation, -w_k <g, y>
  const float4 g = b.gout[pix];
  constexpr int VG = 16 / sizeof(GT), NKG = (NK + VG - 1) / VG * VG;
  float d[NKG];
#pragma unroll
  for (int k = 0; k < NKG; ++k) d[k] = 0.f;
  float gy = 0.f;  // <g, y> = sum_k w_k d_k
  for_each_tap<KD, KU, KT, HU, HT>(a, Ls, Cs, Ts, tx, ty, x, y, x0, y0, [&](int k, float4 v) {
    d[k] = g.x * v.x + g.y * v.y + g.z * v.z;
    gy += z[k] * d[k];
  });
#pragma unroll
  for (int k = 0; k < NK; ++k) d[k] = z[k] * (d[k] - gy);
  GT* gl = static_cast<GT*>(b.glogits) + pix * b.gstride;
  if (b.gvec) {
#pragma unroll
    for (int k = 0; k < NKG; k += VG) gstore16(gl + k, d + k);
    const float zero[VG] = {};
    for (int k = NKG; k < b.gstride; k += VG) gstore16(gl + k, zero);
  } else {
#pragma unroll
    for (int k = 0; k < NK; ++k) gstore(gl + k, d[k]);
    for (int k = NK; k < b.gstride; ++k) gstore(gl + k, 0.f);
  }
  // a tap whose read was clamped to the edge joins the tap that reads the edge pixel, so that the
  // transposes see unclamped taps only
  constexpr int RM = KD > KT ? KD / 2 : KT / 2, RB = RM > 2 ? RM : 2;
  if (x0 < RB || y0 < RB || x0 + TW + RB > W || y0 + TH + RB > H) {
    fold<KD>(z, x, y, W, H);
    if constexpr (HU && KU == 3) fold<3>(z + G::ND, x / 2, y / 2, W / 2, H / 2);
    if constexpr (HU && KU == 2) {  // tap 1 of the last pixel of a row or column reads past it
      float* u = z + G::ND;
      fold_move(u[0], u[1], x == W - 1);
      fold_move(u[2], u[3], x == W - 1);
      fold_move(u[0], u[2], y == H - 1);
      fold_move(u[1], u[3], y == H - 1);
    }
    if constexpr (HT) fold<KT>(z + G::ND + G::NU, x, y, W, H);
  }
  float* wb = b.wbuf + pix;
#pragma unroll
  for (int k = 0; k < NK; ++k) wb[k * b.plane] = z[k];
}

// Sum over the K x K same-resolution taps that read pixel (x, y): tap d of pixel (x, y) - d (the
// clamped taps are folded, k_level_bwd).  G: the block's gradient tile with a halo of RG pixels,
// zeros outside the image.
template <int K, int RG>
__device__ __forceinline__ float4 same_T(const float* __restrict__ w, size_t plane, const float4* G, int H, int W, int n, int x, int y, int tx, int ty) {
  constexpr int R = K / 2, GW = TW + 2 * RG;
  float ax = 0.f, ay = 0.f, az = 0.f;
  const float* wp = w + ((size_t)n * H + y) * W + x;
#pragma unroll 1
  for (int dy = -R; dy <= R; ++dy)
#pragma unroll
    for (int dx = -R; dx <= R; ++dx) {
      const bool in = (unsigned)(y - dy) < (unsigned)H && (unsigned)(x - dx) < (unsigned)W;
      const float wq = in ? wp[((dy + R) * K + (dx + R)) * plane - (ptrdiff_t)(dy * W + dx)] : 0.f;
      const float4 gq = G[(ty + RG - dy) * GW + (tx + RG - dx)];
      ax += wq * gq.x;
      ay += wq * gq.y;
      az += wq * gq.z;
    }
  return make_float4(ax, ay, az, 0.f);
}

// Transposes at one resolution: kd taps -> out (KD > 0), and kt taps -> dLoss/dW(prev), whose
// bilinear warp's transpose is splatted into grad_prev (KT > 0; float atomics, order not fixed).
// The splats of a block land close together: they are added up in an LDS box around the block's
// middle pixel's target first and flushed with one atomic per touched value (12 global atomics per
// pixel, strided by 16 bytes over a wave, and the transposes' own uncoalesced reads took 77 + 80 us
// at 4 x 256 x 256; now 29 us for both); targets outside the box go straight to memory.
constexpr int kBoxW = 48, kBoxH = 20;
template <int KD, int KT>
__global__ __launch_bounds__(256) void k_gatherT(const float* __restrict__ wd, const float* __restrict__ wt,
                                                 size_t plane, const float4* __restrict__ g, int H, int W,
                                                 float4* __restrict__ out, const float2* __restrict__ mv,
                                                 float* __restrict__ grad_prev) {
  constexpr int RG = (KD > KT ? KD : KT) / 2, GW = TW + 2 * RG, GH = TH + 2 * RG;
  __shared__ float4 G[GH * GW];
  __shared__ float box[KT ? kBoxH * kBoxW * 3 : 1];
  __shared__ int org[2];
  const int tid = threadIdx.x, tx = tid % TW, ty = tid / TW;
  const int x0 = blockIdx.x * TW, y0 = blockIdx.y * TH, n = blockIdx.z, x = x0 + tx, y = y0 + ty;
  const size_t img = (size_t)n * H * W;
  for (int k = tid; k < GH * GW; k += 256) {
    const int yy = y0 - RG + k / GW, xx = x0 - RG + k % GW;
    G[k] = yy >= 0 && yy < H && xx >= 0 && xx < W ? g[img + (size_t)yy * W + xx] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const bool in = x < W && y < H;
  WarpTaps t{};
  if constexpr (KT > 0) {
    for (int k = tid; k < kBoxH * kBoxW * 3; k += 256) box[k] = 0.f;
    if (in) t = warp_taps(mv[img + (size_t)y * W + x], H, W, x, y);
    if (x == min(x0 + TW / 2, W - 1) && y == min(y0 + TH / 2, H - 1)) {
      org[0] = t.xa - tx - (kBoxW - TW) / 2;
      org[1] = t.ya - ty - (kBoxH - TH) / 2;
    }
  }
  __syncthreads();
  if constexpr (KD > 0) {
    if (in) out[img + (size_t)y * W + x] = same_T<KD, RG>(wd, plane, G, H, W, n, x, y, tx, ty);
  }
  if constexpr (KT > 0) {
    float* P = grad_prev + img * 4;
    const int bx = org[0], by = org[1];
    if (in) {
      const float4 gw = same_T<KT, RG>(wt, plane, G, H, W, n, x, y, tx, ty);
      const int xs[4] = {t.xa, t.xb, t.xa, t.xb}, ys[4] = {t.ya, t.ya, t.yb, t.yb};
      const float ws[4] = {t.gy * t.gx, t.gy * t.fx, t.fy * t.gx, t.fy * t.fx};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (ws[k] == 0.f) continue;
        const int cx = xs[k] - bx, cy = ys[k] - by;
        const float v[3] = {ws[k] * gw.x, ws[k] * gw.y, ws[k] * gw.z};
        if ((unsigned)cx < (unsigned)kBoxW && (unsigned)cy < (unsigned)kBoxH) {
          float* d = box + (cy * kBoxW + cx) * 3;
#pragma unroll
          for (int c = 0; c < 3; ++c) atomicAdd(d + c, v[c]);
        } else {
          float* d = P + ((size_t)ys[k] * W + xs[k]) * 4;
#pragma unroll
          for (int c = 0; c < 3; ++c) atomicAdd(d + c, v[c]);
        }
      }
    }
    __syncthreads();
    for (int k = tid; k < kBoxH * kBoxW * 3; k += 256) {
      const float v = box[k];
      if (v == 0.f) continue;  // untouched (or nothing to add); touched entries lie inside the image
      const int p = k / 3;
      atomicAdd(P + ((size_t)(by + p / kBoxW) * W + bx + p % kBoxW) * 4 + k % 3, v);
    }
  }
}

// dLoss/dLhat^{l+1}[P] = sum over fine q and ku taps reading P of w[tap][q] * g[q].  Along an axis
// (clamped taps folded) tap t reads P from the two fine pixels q with q / 2 + t - 1 = P (KU = 3), or
// from 2 P - t and 2 P + 1 - t (KU = 2).
template <int KU>
__global__ __launch_bounds__(256) void k_gatherT_up(const float* __restrict__ w, size_t plane,
                                                    const float4* __restrict__ g, int N,
                                                    int Hf, int Wf, float4* __restrict__ outc) {
  const int Hc = Hf / 2, Wc = Wf / 2;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)N * Hc * Wc) return;
  const int X = (int)(i % Wc), Y = (int)((i / Wc) % Hc), n = (int)(i / ((size_t)Wc * Hc));
  float ax = 0.f, ay = 0.f, az = 0.f;
#pragma unroll
  for (int ty = 0; ty < KU; ++ty)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int qy = KU == 2 ? 2 * Y + a - ty : 2 * (Y - ty + 1) + a;
#pragma unroll
      for (int tx = 0; tx < KU; ++tx)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int qx = KU == 2 ? 2 * X + b - tx : 2 * (X - tx + 1) + b;
          const bool ok = (unsigned)qy < (unsigned)Hf && (unsigned)qx < (unsigned)Wf;
          const size_t q = ((size_t)n * Hf + qy) * Wf + qx;
          const float wq = ok ? w[(ty * KU + tx) * plane + q] : 0.f;
          const float4 gq = ok ? g[q] : make_float4(0.f, 0.f, 0.f, 0.f);
          ax += wq * gq.x;
          ay += wq * gq.y;
          az += wq * gq.z;
        }
    }
  outc[i] = make_float4(ax, ay, az, 0.f);
}

template <int KD, int KU, int KT, typename LT, typename GT>
int launch_bwd_t(const BwdArgs& b, bool hu, bool ht, int N, hipStream_t st) {
  dim3 grid((b.f.W + TW - 1) / TW, (b.f.H + TH - 1) / TH, N);
  if (hu && ht) k_level_bwd<KD, KU, KT, true, true, LT, GT><<<grid, 256, 0, st>>>(b);
  else if (hu) k_level_bwd<KD, KU, KT, true, false, LT, GT><<<grid, 256, 0, st>>>(b);
  else if (ht) k_level_bwd<KD, KU, KT, false, true, LT, GT><<<grid, 256, 0, st>>>(b);
  else k_level_bwd<KD, KU, KT, false, false, LT, GT><<<grid, 256, 0, st>>>(b);
  APS_LAUNCH_CHECK();
  return APS_OK;
}

template <int KD, int KU, int KT>
int launch_bwd_k(const BwdArgs& b, int ldt, int gdt, bool hu, bool ht, int N, hipStream_t st) {
  if (ldt == APS_F32 && gdt == APS_F32) return launch_bwd_t<KD, KU, KT, float, float>(b, hu, ht, N, st);
  if (ldt == APS_BF16 && gdt == APS_BF16)
    return launch_bwd_t<KD, KU, KT, uint16_t, uint16_t>(b, hu, ht, N, st);
  if (ldt == APS_BF16 && gdt == APS_F32)
    return launch_bwd_t<KD, KU, KT, uint16_t, float>(b, hu, ht, N, st);
  return APS_ERR_UNSUPPORTED;
}

int launch_bwd(BwdArgs& b, int ldt, int gdt, int KD, int KU, int KT, bool hu, bool ht, int N,
               hipStream_t st) {
  b.plane = (size_t)N * b.f.H * b.f.W;
  b.gvec = b.gstride % (gdt == APS_BF16 ? 8 : 4) == 0 && (reinterpret_cast<uintptr_t>(b.glogits) & 15) == 0;
  if (KD == 5 && KU == 3 && KT == 3) return launch_bwd_k<5, 3, 3>(b, ldt, gdt, hu, ht, N, st);
  if (KD == 7 && KU == 3 && KT == 3) return launch_bwd_k<7, 3, 3>(b, ldt, gdt, hu, ht, N, st);
  if (KD == 5 && KU == 2 && KT == 5) return launch_bwd_k<5, 2, 5>(b, ldt, gdt, hu, ht, N, st);
  if (KD == 3 && KU == 3 && KT == 3) return launch_bwd_k<3, 3, 3>(b, ldt, gdt, hu, ht, N, st);
  return APS_ERR_UNSUPPORTED;
}

// kd transpose into out (KD > 0) and kt transpose into gprev (KT > 0) of one level
int launch_gatherT(int KD, int KT, const float* wbuf, int kt0, size_t plane, const float4* g, int N,
                   int H, int W, float4* out, const float2* mv, float* gprev, hipStream_t st) {
  const dim3 grid((W + TW - 1) / TW, (H + TH - 1) / TH, N);
  const float* wt = wbuf + (size_t)kt0 * plane;
#define APS_GT(D, T)                                                                              \
  if (KD == D && KT == T) {                                                                       \
    k_gatherT<D, T><<<grid, 256, 0, st>>>(wbuf, wt, plane, g, H, W, out, mv, gprev);              \
    APS_LAUNCH_CHECK();                                                                           \
    return APS_OK;                                                                                \
  }
  APS_GT(3, 0) APS_GT(5, 0) APS_GT(7, 0) APS_GT(3, 3) APS_GT(5, 3) APS_GT(7, 3) APS_GT(5, 5) APS_GT(0, 3) APS_GT(0, 5)
#undef APS_GT
  return APS_ERR_UNSUPPORTED;
}

int launch_up_T(int KU, const float* w, size_t plane, const float4* g, int N, int Hf, int Wf,
                float4* outc, hipStream_t st) {
  const size_t n = (size_t)N * (Hf / 2) * (Wf / 2);
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (KU == 3) k_gatherT_up<3><<<blocks, 256, 0, st>>>(w, plane, g, N, Hf, Wf, outc);
  else if (KU == 2) k_gatherT_up<2><<<blocks, 256, 0, st>>>(w, plane, g, N, Hf, Wf, outc);
  else return APS_ERR_UNSUPPORTED;
  APS_LAUNCH_CHECK();
  return APS_OK;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

extern "C" {

size_t aps_denoise_pyramid_bwd_workspace_size(int N, int H, int W, int levels, int KD, int KU,
                                              int KT, int temporal) {
  size_t b = 256;
  for (int l = 1; l < levels; ++l) b += 2 * align256((size_t)N * (H >> l) * (W >> l) * sizeof(float4));
  const int nk0 = level_k(0, levels, KD, KU, KT, temporal != 0);
  b += align256((size_t)N * H * W * nk0 * sizeof(float));
  return b;
}

int aps_denoise_pyramid_bwd(const float* const* L, const void* const* logits, int logit_dtype,
                            const int* kstride, int levels, int KD, int KU, int KT,
                            const float* prev, const float* mv, int N, int H, int W,
                            const float* grad_out, void* const* grad_logits, int grad_dtype,
                            const int* gstride, float* const* grad_L, float* grad_prev, void* ws,
                            size_t ws_bytes, void* stream) {
  if (levels < 1 || levels > APS_MAX_LEVELS) return APS_ERR_UNSUPPORTED;
  if (N < 0 || H < 0 || W < 0) return APS_ERR_SHAPE;
  const int div = 1 << (levels - 1);
  if (H % div || W % div) return APS_ERR_SHAPE;
  if ((size_t)N * H * W == 0) return APS_OK;
  if (!L || !logits || !kstride || !grad_out || !grad_logits || !gstride || !grad_L)
    return APS_ERR_NULL;
  if (prev && !mv) return APS_ERR_NULL;
  if (grad_dtype != APS_F32 && grad_dtype != APS_BF16) return APS_ERR_UNSUPPORTED;
  const bool temporal = prev != nullptr;
  for (int l = 0; l < levels; ++l) {
    if (!L[l] || !logits[l] || !grad_logits[l] || !grad_L[l]) return APS_ERR_NULL;
    const int K = level_k(l, levels, KD, KU, KT, temporal);
    if (!kstride_ok(kstride[l], K, logit_dtype) || gstride[l] < K) return APS_ERR_SHAPE;
  }
  if (!ws || ws_bytes < aps_denoise_pyramid_bwd_workspace_size(N, H, W, levels, KD, KU, KT, temporal))
    return APS_ERR_WORKSPACE;
  char* wp = static_cast<char*>(ws);
  float4* rec[APS_MAX_LEVELS] = {};
  float4* gC[APS_MAX_LEVELS] = {};
  for (int l = 1; l < levels; ++l) {
    const size_t bytes = align256((size_t)N * (H >> l) * (W >> l) * sizeof(float4));
    rec[l] = reinterpret_cast<float4*>(wp);
    wp += bytes;
    gC[l] = reinterpret_cast<float4*>(wp);
    wp += bytes;
  }
  float* wbuf = reinterpret_cast<float*>(wp);
  hipStream_t st = as_stream(stream);

  // 1. recompute Lhat^{L-1} .. Lhat^1 (coarse to fine) with the forward kernel
  for (int l = levels - 1; l >= 1; --l) {
    LevelArgs a{};
    a.L = reinterpret_cast<const float4*>(L[l]);
    a.logits = logits[l];
    a.kstride = kstride[l];
    a.coarse = l < levels - 1 ? rec[l + 1] : nullptr;
    a.out = rec[l];
    a.H = H >> l;
    a.W = W >> l;
    a.eval_g = 1;
    a.eval_u = l < levels - 1;
    const int r = launch_level(a, logit_dtype, KD, KU, KT, l < levels - 1, false, N, st);
    if (r != APS_OK) return r;
  }
  // 2. fine to coarse
  for (int l = 0; l < levels; ++l) {
    const bool hu = l < levels - 1, ht = l == 0 && temporal;
    const int Hl = H >> l, Wl = W >> l;
    BwdArgs b{};
    b.f.L = reinterpret_cast<const float4*>(L[l]);
    b.f.logits = logits[l];
    b.f.kstride = kstride[l];
    b.f.coarse = hu ? rec[l + 1] : nullptr;
    b.f.prev = reinterpret_cast<const float4*>(prev);
    b.f.mv = reinterpret_cast<const float2*>(mv);
    b.f.H = Hl;
    b.f.W = Wl;
    b.f.eval_g = 1;
    b.f.eval_u = hu;
    b.f.eval_t = ht;
    b.gout = l == 0 ? reinterpret_cast<const float4*>(grad_out) : gC[l];
    b.glogits = grad_logits[l];
    b.gstride = gstride[l];
    b.wbuf = wbuf;
    int r = launch_bwd(b, logit_dtype, grad_dtype, KD, KU, KT, hu, ht, N, st);
    if (r != APS_OK) return r;
    r = launch_gatherT(KD, ht && grad_prev ? KT : 0, wbuf, KD * KD + (hu ? KU * KU : 0), b.plane, b.gout, N,
                       Hl, Wl, reinterpret_cast<float4*>(grad_L[l]), b.f.mv, grad_prev, st);
    if (r != APS_OK) return r;
    if (hu) {
      r = launch_up_T(KU, wbuf + (size_t)KD * KD * b.plane, b.plane, b.gout, N, Hl, Wl, gC[l + 1], st);
      if (r != APS_OK) return r;
    }
  }
  return APS_OK;
}

// ---- standalone terms: reproject (kt block) and upsample (ku block) ------------------------

size_t aps_reproject_bwd_workspace_size(int N, int H, int W, int KD, int KU, int KT,
                                        int has_upsample) {
  const int nk = KD * KD + (has_upsample ? KU * KU : 0) + KT * KT;
  return align256((size_t)N * H * W * nk * sizeof(float)) + 256;
}

int aps_reproject_bwd(const float* prev, const float* mv, const void* logits0, int logit_dtype,
                      int kstride, int KD, int KU, int KT, int has_upsample, int N, int H, int W,
                      const float* grad_accum, void* grad_logits0, int grad_dtype, int gstride,
                      float* grad_prev, void* ws, size_t ws_bytes, void* stream) {
  if (N < 0 || H < 0 || W < 0) return APS_ERR_SHAPE;
  if (has_upsample && (H % 2 || W % 2)) return APS_ERR_SHAPE;
  if ((size_t)N * H * W == 0) return APS_OK;
  if (!prev || !mv || !logits0 || !grad_accum || !grad_logits0) return APS_ERR_NULL;
  if (grad_dtype != APS_F32 && grad_dtype != APS_BF16) return APS_ERR_UNSUPPORTED;
  const int nk = KD * KD + (has_upsample ? KU * KU : 0) + KT * KT;
  if (!kstride_ok(kstride, nk, logit_dtype) || gstride < nk) return APS_ERR_SHAPE;
  if (!ws || ws_bytes < aps_reproject_bwd_workspace_size(N, H, W, KD, KU, KT, has_upsample))
    return APS_ERR_WORKSPACE;
  hipStream_t st = as_stream(stream);
  BwdArgs b{};
  b.f.logits = logits0;
  b.f.kstride = kstride;
  b.f.prev = reinterpret_cast<const float4*>(prev);
  b.f.mv = reinterpret_cast<const float2*>(mv);
  b.f.H = H;
  b.f.W = W;
  b.f.eval_t = 1;
  b.gout = reinterpret_cast<const float4*>(grad_accum);
  b.glogits = grad_logits0;
  b.gstride = gstride;
  b.wbuf = static_cast<float*>(ws);
  int r = launch_bwd(b, logit_dtype, grad_dtype, KD, KU, KT, has_upsample != 0, true, N, st);
  if (r != APS_OK) return r;
  if (grad_prev)
    r = launch_gatherT(0, KT, b.wbuf, KD * KD + (has_upsample ? KU * KU : 0), b.plane, b.gout, N, H, W,
                       nullptr, b.f.mv, grad_prev, st);
  return r;
}

size_t aps_upsample_bwd_workspace_size(int N, int H, int W, int KD, int KU, int KT,
                                       int has_temporal) {
  const int nk = KD * KD + KU * KU + (has_temporal ? KT * KT : 0);
  return align256((size_t)N * H * W * nk * sizeof(float)) + 256;
}

int aps_upsample_bwd(const float* coarse, const void* logits, int logit_dtype, int kstride, int KD,
                     int KU, int KT, int has_temporal, int N, int H, int W,
                     const float* grad_accum, void* grad_logits, int grad_dtype, int gstride,
                     float* grad_coarse, void* ws, size_t ws_bytes, void* stream) {
  if (N < 0 || H < 0 || W < 0 || H % 2 || W % 2) return APS_ERR_SHAPE;
  if ((size_t)N * H * W == 0) return APS_OK;
  if (!coarse || !logits || !grad_accum || !grad_logits || !grad_coarse) return APS_ERR_NULL;
  if (grad_dtype != APS_F32 && grad_dtype != APS_BF16) return APS_ERR_UNSUPPORTED;
  const int nk = KD * KD + KU * KU + (has_temporal ? KT * KT : 0);
  if (!kstride_ok(kstride, nk, logit_dtype) || gstride < nk) return APS_ERR_SHAPE;
  if (!ws || ws_bytes < aps_upsample_bwd_workspace_size(N, H, W, KD, KU, KT, has_temporal))
    return APS_ERR_WORKSPACE;
  hipStream_t st = as_stream(stream);
  BwdArgs b{};
  b.f.logits = logits;
  b.f.kstride = kstride;
  b.f.coarse = reinterpret_cast<const float4*>(coarse);
  b.f.H = H;
  b.f.W = W;
  b.f.eval_u = 1;
  b.gout = reinterpret_cast<const float4*>(grad_accum);
  b.glogits = grad_logits;
  b.gstride = gstride;
  b.wbuf = static_cast<float*>(ws);
  const int r = launch_bwd(b, logit_dtype, grad_dtype, KD, KU, KT, true, has_temporal != 0, N, st);
  if (r != APS_OK) return r;
  return launch_up_T(KU, b.wbuf + (size_t)KD * KD * b.plane, b.plane, b.gout, N, H, W,
                     reinterpret_cast<float4*>(grad_coarse), st);
}

}  // extern "C"
