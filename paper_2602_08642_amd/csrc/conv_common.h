// Shared by the convolution kernels (conv.hip: bf16 and the small layers; conv_f32.hip: the fp32
// 3x3 layers): arguments, block order, staging of transformed inputs, epilogues.
#pragma once
#include "aps_common.h"
#include "mfma_frag.h"

namespace aps {

constexpr int kChunk = 32;
constexpr int kMaxTM = 4;
constexpr int kModeReluMask = 3;  // internal staging mode of the data-gradient convolution

struct ConvArgs {
  const void* x;
  const void* x2;
  int N, H, W;   // output (= conv input after the transform) size
  int Cx, C2, mode;
  const void* wp;
  const float* bias;
  int Cout, nchunk, ntx;
  void* y;
  int ldy, relu;
  // optional 1x1 head fused into the epilogue (see k_conv); store_main = also write y
  const void* hw;
  const float* hb;
  int hK;
  void* hy;
  int hldy, store_main;
  // optional side output of three head channels [hside_off, hside_off + 3) as [N,H,W,4] (the
  // fourth entry 0), written from the staged logit rows (conv_epilogue)
  void* hside;
  int hside_off;
  // optional 2x2 average pool of the (bf16-rounded) output, [N, H/2, W/2, Cout] (k_conv_lds)
  void* pool;
  int ntiles, nco;  // pixel tiles per image, output-channel blocks (block order: xcd_tile)
  int cvalid;       // fp32 3x3: input channels at and past this one are zeros (0: none)
  int big;          // fp32 3x3: a tile's input rows exceed 32-bit byte offsets
};

// Blocks are dispatched round-robin over the 8 XCDs (block id % 8), each with its own L2.  XCD x
// takes the contiguous tile range [x T8, (x+1) T8) and, per tile, all channel blocks back to back,
// so the halo rows shared by neighbouring tiles and the input tile shared by a tile's channel
// blocks are re-read from that XCD's L2 rather than from HBM.  grid.x = 8 T8 nco; blocks past the
// last tile exit.
struct TileId {
  int tile, cob;
};
__device__ inline TileId xcd_tile(int id, int ntiles, int nco) {
  const int t8 = (ntiles + 7) / 8, xcd = id & 7, k = id >> 3;
  return TileId{xcd * t8 + k / nco, k % nco};
}
inline int xcd_grid(int ntiles, int nco) { return 8 * ((ntiles + 7) / 8) * nco; }

// Orders this wave's LDS accesses across lanes: a compiler barrier for memory operations (the
// LDS itself completes one wave's operations in program order).  Plain signal fences are not
// enough where the two sides use different vector types, which type-based alias analysis may
// then take as disjoint.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- 8-element vectors of the storage type ---------------------------------------------
struct V8f {
  float v[8];
};

__device__ inline V8f load8(const float* p) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  return V8f{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
__device__ inline V8f load8(const uint16_t* p) {
  const u16x8 h = *reinterpret_cast<const u16x8*>(p);
  V8f r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r.v[e] = bf2f(h[e]);
  return r;
}
__device__ inline void store8(float* p, const V8f& r) {
  *reinterpret_cast<float4*>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(r.v[4], r.v[5], r.v[6], r.v[7]);
}
__device__ inline void store8(uint16_t* p, const V8f& r) {
  u16x8 h;
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = f2bf(r.v[e]);
  *reinterpret_cast<u16x8*>(p) = h;
}
// Stage channels [ci, ci+8) of input pixel (iy, ix) into LDS.
template <typename T>
__device__ inline void stage8(const ConvArgs& a, int n, int iy, int ix, int ci, T* dst) {
  const int Cin = a.Cx + a.C2;
  if (iy < 0 || iy >= a.H || ix < 0 || ix >= a.W || ci >= Cin) {
    zero8(dst);
    return;
  }
  const T* x = static_cast<const T*>(a.x);
  if ((a.mode == APS_CONV_DIRECT || a.mode == kModeReluMask) && ci + 8 > a.Cx) {
    // channel tail of a row whose stride is not a multiple of 8 (padded logit gradients)
    const size_t o = (((size_t)n * a.H + iy) * a.W + ix) * a.Cx + ci;
    const T* y = static_cast<const T*>(a.x2);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool ok = ci + e < a.Cx && (a.mode == APS_CONV_DIRECT || Ld<T>::get(y, o + e) > 0.f);
      dst[e] = ok ? x[o + e] : T(0);
    }
  } else if (a.mode == APS_CONV_DIRECT) {
    copy8(dst, x + (((size_t)n * a.H + iy) * a.W + ix) * a.Cx + ci);
  } else if (a.mode == kModeReluMask) {
    // x = dLoss/dy, x2 = y (post-ReLU output, same layout): stage dy where y > 0, else 0
    const size_t o = (((size_t)n * a.H + iy) * a.W + ix) * a.Cx + ci;
    const V8f g = load8(x + o), y = load8(static_cast<const T*>(a.x2) + o);
    V8f r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r.v[e] = y.v[e] > 0.f ? g.v[e] : 0.f;
    store8(dst, r);
  } else if (a.mode == APS_CONV_POOL2) {
    const int W2 = 2 * a.W;
    const T* p = x + (((size_t)n * 2 * a.H + 2 * iy) * W2 + 2 * ix) * a.Cx + ci;
    const V8f q0 = load8(p), q1 = load8(p + a.Cx), q2 = load8(p + (size_t)W2 * a.Cx),
              q3 = load8(p + (size_t)W2 * a.Cx + a.Cx);
    V8f r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r.v[e] = ((q0.v[e] + q1.v[e]) + (q2.v[e] + q3.v[e])) * 0.25f;
    store8(dst, r);
  } else {  // APS_CONV_UP2_CAT
    if (ci < a.Cx) {
      const int Hh = a.H / 2, Wh = a.W / 2;
      copy8(dst, x + (((size_t)n * Hh + iy / 2) * Wh + ix / 2) * a.Cx + ci);
    } else {
      const T* x2 = static_cast<const T*>(a.x2);
      copy8(dst, x2 + (((size_t)n * a.H + iy) * a.W + ix) * a.C2 + (ci - a.Cx));
    }
  }
}

template <typename TO>
__device__ inline void store_out(TO* p, int ldy, int co0, int Cout, const float* v);
template <>
__device__ inline void store_out<float>(float* p, int ldy, int co0, int Cout, const float* v) {
  if ((ldy & 3) == 0 && co0 + 4 <= ldy) {
    *reinterpret_cast<float4*>(p + co0) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (co0 + q < Cout) p[co0 + q] = v[q];
  }
}
template <>
__device__ inline void store_out<uint16_t>(uint16_t* p, int ldy, int co0, int Cout, const float* v) {
  if ((ldy & 3) == 0 && co0 + 4 <= ldy) {
    *reinterpret_cast<u16x4*>(p + co0) = f2bf4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (co0 + q < Cout) p[co0 + q] = f2bf(v[q]);
  }
}

// s_waitcnt immediate (gfx9 encoding) that waits for all vector memory operations only:
// vmcnt = 0, expcnt = 7 and lgkmcnt = 15 (no wait on those).
constexpr int kWaitVm0 = 0x0F70;

// LDS the fused head's epilogue needs, in elements of the tile type T: per wave a [16 px][16 TM
// ch] re-layout region (row pitch 16 TM + 8 or + 4), then per wave a [16 px][<= 16 HM ch] staging
// region for the head outputs (type TO).  The kernels size their input tile at least this large.
// HM = head m-tiles (4: up to 64 logits, 5: up to 80); 0 = no fused head.
template <typename T, typename TO, int TM, int HM>
constexpr int head_lds_elems() {
  return 4 * 16 * (TM * 16 + (sizeof(T) == 2 ? 8 : 4)) + 4 * 16 * 16 * HM * (int)(sizeof(TO) / sizeof(T));
}

// Epilogue shared by the convolution kernels: bias, optional ReLU, store; with HEAD, the fused
// 1x1 head.  acc[m][j] holds output rows row0 + j, channels 16 (cob TM + m) + 4 (lane / 16) + q,
// pixel column tx0 + lane % 16.  Xs is the block's LDS tile, reused by the head's re-layout.
template <typename T, typename TO, int TM, int TN, int HEAD, bool BIAS_IN_ACC = false>
__device__ inline void conv_epilogue(const ConvArgs& a, f32x4 (&acc)[TM][TN], int row0, int tx0,
                                     int cob, int n, int lane, int wave, T* Xs) {
  TO* y = static_cast<TO*>(a.y);
  const int col = tx0 + (lane & 15);
  float bv[TM][4];  // this lane's bias values, loaded once
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int co0 = (cob * TM + m) * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      bv[m][q] = !BIAS_IN_ACC && co0 + q < a.Cout && a.bias ? a.bias[co0 + q] : 0.f;
  }
  if constexpr (!HEAD) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int row = row0 + j;
      if (row >= a.H || col >= a.W) continue;
      TO* py = y + (((size_t)n * a.H + row) * a.W + col) * a.ldy;
#pragma unroll
      for (int m = 0; m < TM; ++m) {
        const int co0 = (cob * TM + m) * 16 + 4 * (lane >> 4);
        if (co0 >= a.Cout) continue;
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float t = acc[m][j][q] + bv[m][q];
          v[q] = a.relu ? fmaxf(t, 0.f) : t;
        }
        store_out<TO>(py, a.ldy, co0, a.Cout, v);
      }
    }
  } else {
    // Fused 1x1 head on this layer's output (all Cout = 16 TM channels are in this block):
    // each wave re-lays its row-j tile [16 px][16 TM ch] out through its own LDS region as MFMA
    // B fragments and multiplies it by the packed head weights (held in registers), the same
    // operands in the same order as the stand-alone 1x1 convolution of the stored tile.  The
    // regions are per wave, so after the caller's barrier only wave-local ordering is needed.
    // Head outputs go out through a second per-wave region: the row's [npx][hldy] run of
    // logits is contiguous in memory, so the wave writes it with 16-byte vector stores to
    // consecutive addresses (channels in [hK, hldy) as zeros) instead of one 8- or 16-byte piece
    // per lane and 16-channel group at the pixel stride, which measured about twice as slow.
    constexpr int CC = TM * 16, YP = CC + (sizeof(T) == 2 ? 8 : 4), HM = HEAD;
    T* Ys = Xs + wave * 16 * YP;
    TO* Os = reinterpret_cast<TO*>(Xs + 4 * 16 * YP) + wave * 16 * 16 * HM;
    const bool staged = a.hldy <= 16 * HM && (a.hldy * (int)sizeof(TO)) % 16 == 0 &&
                        (reinterpret_cast<uintptr_t>(a.hy) & 15) == 0;
    const int npx = a.W - tx0 < 16 ? a.W - tx0 : 16;
    const T* hw = static_cast<const T*>(a.hw);
    TO* hy = static_cast<TO*>(a.hy);
    Frag<T> hwf[HM][TM / 2];
#pragma unroll
    for (int mh = 0; mh < HM; ++mh)
#pragma unroll
      for (int cc = 0; cc < TM / 2; ++cc)
        if (mh * 16 < a.hK) frag_load(hwf[mh][cc], hw + ((((size_t)mh * (TM / 2)) + cc) * 64 + lane) * 8);
    // head biases: unconditional loads (index clamped to a valid entry), then one wait for them
    // and the head weights here.  Left to the compiler, the wait for a value loaded under a
    // branch is placed at each use inside the later (branching) store code, and as vmcnt also
    // counts stores, every one of those waits would drain all stores issued before it.
    float hb[HM][4];
#pragma unroll
    for (int mh = 0; mh < HM; ++mh)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = mh * 16 + 4 * (lane >> 4) + q;
        const float v = a.hb[k < a.hK ? k : 0];
        hb[mh][q] = k < a.hK ? v : 0.f;
      }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int row = row0 + j;
      const bool inpx = row < a.H && col < a.W;
#pragma unroll
      for (int m = 0; m < TM; ++m) {
        const int co0 = m * 16 + 4 * (lane >> 4);
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float t = acc[m][j][q] + bv[m][q];
          v[q] = a.relu ? fmaxf(t, 0.f) : t;
        }
        if constexpr (sizeof(T) == 2)
          *reinterpret_cast<u16x4*>(Ys + (lane & 15) * YP + co0) = f2bf4(v[0], v[1], v[2], v[3]);
        else
          *reinterpret_cast<float4*>(Ys + (lane & 15) * YP + co0) = make_float4(v[0], v[1], v[2], v[3]);
        if (a.store_main && inpx)
          store_out<TO>(y + (((size_t)n * a.H + row) * a.W + col) * a.ldy, a.ldy, co0, a.Cout, v);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      Frag<T> bf[TM / 2];
#pragma unroll
      for (int cc = 0; cc < TM / 2; ++cc) frag_load(bf[cc], Ys + (lane & 15) * YP + 32 * cc + 8 * (lane >> 4));
      if (staged) {
#pragma unroll
        for (int mh = 0; mh < HM; ++mh) {
          const int k0 = mh * 16 + 4 * (lane >> 4);
          if (mh * 16 >= a.hldy) break;
          f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
          if (mh * 16 < a.hK) {
#pragma unroll
            for (int cc = 0; cc < TM / 2; ++cc) h = mma(hwf[mh][cc], bf[cc], h);
          }
          float o[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) o[q] = k0 + q < a.hK ? h[q] + hb[mh][q] : 0.f;
          if (k0 < a.hldy) {
            if constexpr (sizeof(TO) == 2)
              *reinterpret_cast<u16x4*>(Os + (lane & 15) * a.hldy + k0) = f2bf4(o[0], o[1], o[2], o[3]);
            else
              *reinterpret_cast<f32x4*>(Os + (lane & 15) * a.hldy + k0) = f32x4{o[0], o[1], o[2], o[3]};
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (row < a.H) {
          const int nvec = npx * a.hldy * (int)sizeof(TO) / 16;
          uint4* dst = reinterpret_cast<uint4*>(hy + (((size_t)n * a.H + row) * a.W + tx0) * a.hldy);
          const uint4* src = reinterpret_cast<const uint4*>(Os);
          // nontemporal: the logits are read back only by the filter, after the other heads
          for (int v = lane; v < nvec; v += 64)
            __builtin_nontemporal_store(reinterpret_cast<const u32x4*>(src)[v], reinterpret_cast<u32x4*>(dst) + v);
          if (a.hside && lane < npx) {
            const TO* op = Os + lane * a.hldy + a.hside_off;
            TO* sp = static_cast<TO*>(a.hside) + (((size_t)n * a.H + row) * a.W + tx0 + lane) * 4;
            if constexpr (sizeof(TO) == 2)
              *reinterpret_cast<u16x4*>(sp) = u16x4{op[0], op[1], op[2], (uint16_t)0};
            else
              *reinterpret_cast<f32x4*>(sp) = f32x4{op[0], op[1], op[2], 0.f};
          }
        }
      } else {
#pragma unroll
        for (int mh = 0; mh < HM; ++mh) {
          if (mh * 16 >= a.hK) break;
          f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int cc = 0; cc < TM / 2; ++cc) h = mma(hwf[mh][cc], bf[cc], h);
          const int k0 = mh * 16 + 4 * (lane >> 4);
          if (inpx && k0 < a.hK) {
            float o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = h[q] + hb[mh][q];
            store_out<TO>(hy + (((size_t)n * a.H + row) * a.W + col) * a.hldy, a.hldy, k0, a.hK, o);
          }
        }
      }
      // the next row's re-layout overwrites Ys
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

// v_mfma_f32_16x16x4_f32, four steps: channels 4 g + [0, 4) of lane group g
__device__ inline f32x4 mma4(f32x4 a, f32x4 b, f32x4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], c, 0, 0, 0);
}

// Packed weights of an fp32 3x3 layer in 32-channel chunks, in floats: the fp16 halves, the weights as
// they are in 16-channel chunks (k_pack_split's plain part), and a scale exponent per output channel.
// All three are exact in 16-channel output tiles.
struct F32Pack {
  size_t plain, table, total;
};
__host__ __device__ inline F32Pack f32_pack(int Cout, int Cin) {
  const size_t ct = (size_t)(Cout + 15) / 16, split = ct * 9 * ((Cin + 31) / 32) * 512;
  const size_t plain = ct * 9 * ((Cin + 15) / 16) * 256;
  return F32Pack{split, split + plain, split + plain + ct * 16};
}

// fp32 3x3 layers in 32-channel chunks (conv_f32.hip); sizes checked by the entry points
// (fp32_offsets_fit).  hw set: with the fused 1x1 head.
void pack_split(const float* w, int Cout, int Cin, void* packed, int transpose, hipStream_t st);
void conv_split(const ConvArgs& a, hipStream_t st);
// the same layers forward in training with a ReLU (conv_f32_train.hip)
void conv_f32(const ConvArgs& a, hipStream_t st);

}  // namespace aps
