// What the conv GEMM kernels share: tile geometry, the destination and gather arithmetic, the
// epilogue, raw buffer descriptors and the transposed weight stage.
#pragma once

#include <type_traits>

#include "kernels.h"

namespace numbat {

namespace {

constexpr int GK = 32;          // reduction elements per pipeline step
constexpr int GROW = GK + 8;    // bf16 per LDS row (80 bytes: conflict-free 16-byte fragment reads)

template <int V>
using Ic = std::integral_constant<int, V>;

// f(Ic<I>{}), ..., f(Ic<N - 1>{})
template <int I, int N, typename F>
__device__ __forceinline__ void static_for_ic(F&& f) {
  if constexpr (I < N) {
    f(Ic<I>{});
    static_for_ic<I + 1, N>(f);
  }
}

// NW waves in rows of WN: each owns TM x TN blocks of 32 x 32
template <int TM, int TN, int NW = 4, int WN = 1>
struct GemmShape {
  static constexpr int WTM = TM * 32, WTN = TN * 32;  // rows and columns per wave
  static constexpr int WM = NW / WN;
  static constexpr int BM = WM * WTM, BN = WN * WTN;
  static constexpr int BV = (BN + 63) / 64;    // B vectors per thread per step
  static constexpr int B_BYTES = 2 * BN * GROW * 2;
  static constexpr int STAGE_LD = WTN + 4;                  // fp32 per staged row
  static constexpr int STAGE_BYTES = NW * 8 * STAGE_LD * 4;  // 8 rows per wave
  static constexpr int SMEM = B_BYTES > STAGE_BYTES ? B_BYTES : STAGE_BYTES;
};

__device__ __forceinline__ void grid_pos(uint32_t m, const GemmPhase& P, uint32_t& img, uint32_t& gi, uint32_t& gj) {
  img = fdiv(m, P.div_ghw);
  const uint32_t rem = m - img * (uint32_t)(P.gh * P.gw);
  gi = fdiv(rem, P.div_gw);
  gj = rem - gi * (uint32_t)P.gw;
}

// logical tile of this block.  With the XCD-aware order: n tile fastest, then m tile,
// then phase, so the blocks sharing rows of the gathered operand (and halo rows of
// neighbouring tiles) share an XCD; otherwise the launch order (m tile fastest).
struct TileId {
  int mt, nt, ph;
};
__device__ __forceinline__ TileId tile_id(bool remap) {
  if (!remap) return TileId{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z};
  const uint32_t gx = gridDim.x, gy = gridDim.y;  // m tiles, n tiles
  const uint32_t lg = xcd_remap(blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z), gx * gy * gridDim.z);
  return TileId{(int)((lg / gy) % gx), (int)(lg % gy), (int)(lg / (gx * gy))};
}

// The per-phase geometry a block needs, read from the kernel arguments once at entry
// (the phase is chosen by the block index, so every field access would otherwise be a
// dependent scalar load)
struct Geo {
  int m, gh, gw;
  FastDiv div_gw, div_ghw;
  int doff_h, doff_w;
  int tw, th, dh0, dw0, tsh, tsw;
};
__device__ __forceinline__ Geo load_geo(const GemmPhase& P) {
  Geo g;
  g.m = P.m;
  g.gh = P.gh;
  g.gw = P.gw;
  g.div_gw = P.div_gw;
  g.div_ghw = P.div_ghw;
  g.doff_h = P.doff_h;
  g.doff_w = P.doff_w;
  g.tw = P.tw;
  g.th = P.th;
  g.dh0 = P.dh0;
  g.dw0 = P.dw0;
  g.tsh = P.tsh;
  g.tsw = P.tsw;
  return g;
}
__device__ __forceinline__ void geo_pos(uint32_t m, const Geo& G, uint32_t& img, uint32_t& gi, uint32_t& gj) {
  img = fdiv(m, G.div_ghw);
  const uint32_t rem = m - img * (uint32_t)(G.gh * G.gw);
  gi = fdiv(rem, G.div_gw);
  gj = rem - gi * (uint32_t)G.gw;
}

// destination element offset of GEMM row m (-1 past the phase's rows)
__device__ __forceinline__ int64_t dst_offset(const ConvGemmArgs& a, const Geo& G, int m) {
  if (m >= G.m) return -1;
  uint32_t img, gi, gj;
  geo_pos((uint32_t)m, G, img, gi, gj);
  return (((int64_t)img * a.hd + (int)gi * a.dstep_h + G.doff_h) * a.wd + (int)gj * a.dstep_w + G.doff_w) *
         a.dst_pix;
}

// Byte offset (from the tile's gather base, without the halo) of GEMM row m's anchor
// pixel, and the bitmask of its taps that fall inside the image.  The taps form a grid
// (rows of tw taps with constant steps), so the mask is the outer product of the grid
// rows that stay inside the image height and the grid columns inside its width.
__device__ __forceinline__ void row_gather(const ConvGemmArgs& a, const Geo& G, int m, uint32_t img0,
                                           uint32_t& vrow, uint32_t& vmask) {
  vrow = 0;
  vmask = 0;
  if (m >= G.m) return;
  uint32_t img, gi, gj;
  geo_pos((uint32_t)m, G, img, gi, gj);
  const int ih0 = (int)gi * a.gstride_h, iw0 = (int)gj * a.gstride_w;
  vrow = (uint32_t)((((int64_t)(img - img0) * a.hs + ih0) * a.ws + iw0) * (a.src_pix * 2));
  // (kernel sides are at most 5: fixed-trip, branch-free loops)
  uint32_t cols = 0;
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const int iw = iw0 + G.dw0 + j * G.tsw;
    cols |= (j < G.tw && (unsigned)iw < (unsigned)a.ws ? 1u : 0u) << j;
  }
  uint32_t mk = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int ih = ih0 + G.dh0 + i * G.tsh;
    mk |= (i < G.th && (unsigned)ih < (unsigned)a.hs ? cols : 0u) << (i * G.tw);
  }
  vmask = mk;  // bits >= taps stay clear, so a walk past the last tap reads zeros
}

// Shared epilogue: per-channel (mean, M2) partials of the tile's rows (phase 0, when
// requested) and the bf16 output, staged through LDS as fp32 and written as 16-byte
// vectors of 8 channels.  Accumulator register r of a lane sits on wave row
// 8*(r/4) + 4*(lane/32) + (r%4) of its 32-row block, column lane%32 of its 32-column block.
// sum of the NW waves' partials of column c, in a fixed pairwise order
template <int NW>
__device__ __forceinline__ float wave_sum(const float* r, int ld, int c) {
  const float s4 = (r[c] + r[ld + c]) + (r[2 * ld + c] + r[3 * ld + c]);
  if constexpr (NW == 4) return s4;
  else return s4 + ((r[4 * ld + c] + r[5 * ld + c]) + (r[6 * ld + c] + r[7 * ld + c]));
}

// `active` false: a wave that holds no accumulators of its own (the second half of a
// block whose halves split the reduction) and only takes the block's barriers.  `wave_id`: the
// rows the wave holds, where they are not those of its place in the block.
template <int TM, int TN, int NW = 4, int WN = 1>
__device__ __forceinline__ void gemm_epilogue(const ConvGemmArgs& a, const GemmPhase& P, const TileId& T,
                                              f32x16 (&acc)[TM][TN], int m0, int n0, unsigned char* smem,
                                              const int64_t* s_dst, float (*s_red)[TN * 32 * WN], float* s_mean,
                                              bool active = true, int wave_id = -1) {
  using S = GemmShape<TM, TN, NW, WN>;
  static_assert(S::WM == 4 || S::WM == 8, "4 or 8 rows of waves");
  constexpr int BM = S::BM, BN = S::BN, WTM = S::WTM;
  const int tid = threadIdx.x, lane = tid & 63, wave_in = wave_id >= 0 ? wave_id : tid >> 6;
  const int wave = wave_in / WN, wc = (wave_in % WN) * S::WTN;  // the wave's rows, its first column
  const int l32 = lane & 31, half = lane >> 5;
  float* stage = reinterpret_cast<float*>(smem);
  __syncthreads();  // the main loop's last LDS reads are done before staging reuses LDS
  // ---- per-channel (mean, M2) of this tile's rows from the fp32 accumulators (phase 0)
  if (a.stats_part != nullptr && T.ph == 0) {
    const int left = P.m - m0;
    const int count = left < BM ? left : BM;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[i][j][r];
      s += __shfl_xor(s, 32);
      if (lane < 32 && active) s_red[wave][wc + j * 32 + lane] = s;
    }
    __syncthreads();
    if (tid < BN) s_mean[tid] = wave_sum<S::WM>(&s_red[0][0], BN, tid) / (float)count;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const float mu = s_mean[wc + j * 32 + l32];
      float q = 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = wave * WTM + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
          const float d = acc[i][j][r] - mu;
          q += (row < count) ? d * d : 0.f;
        }
      q += __shfl_xor(q, 32);
      if (lane < 32 && active) s_red[wave][wc + j * 32 + lane] = q;
    }
    __syncthreads();
    if (tid < BN && n0 + tid < a.nout) {
      const float q = wave_sum<S::WM>(&s_red[0][0], BN, tid);
      a.stats_part[(int64_t)T.mt * a.nout + n0 + tid] = make_float2(s_mean[tid], q);
    }
  }

  // ---- inference epilogue constants: per column a scale and a shift (bias: 1, bias[n];
  // eval-mode BN: gamma rstd, beta - mean gamma rstd), in s_red rows 0 and 1 (the
  // statistics, which share that space, are never asked for with them)
  const int post = a.post;
  if (post != kPostNone) {
    __syncthreads();
    if (tid < BN) {
      const int col = n0 + tid;
      float sc = 1.f, sh = 0.f;
      if (col < a.nout) {
        if (post == kPostBias) {
          sh = a.post_bias[col];
        } else {
          sc = a.post_gamma[col] * (1.0f / sqrtf(a.post_var[col] + a.post_eps));
          sh = a.post_beta[col] - a.post_mean[col] * sc;
        }
      }
      s_red[0][tid] = sc;
      s_red[1][tid] = sh;
    }
    __syncthreads();
  }
  auto post_op = [&](float (&f)[8], int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float z = __builtin_fmaf(f[e], s_red[0][wc + c0 + e], s_red[1][wc + c0 + e]);
      f[e] = post == kPostBnSilu ? z * sigmoidf_fast(z) : z;
    }
  };

  // ---- output
  if (!active) return;  // (no block barrier follows)
  if ((a.nout & 7) == 0) {
    // stage 8 rows per wave in LDS as fp32 (register group g = r/4 of every 32-row block),
    // then write 16-byte vectors of 8 channels
    float* st = stage + wave_in * 8 * S::STAGE_LD;
    constexpr int VPR = S::WTN / 8;  // vectors per staged row
    // (the staging rows are private to the wave, and one wave's LDS accesses complete in
    // issue order, so the rounds need no barrier)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) st[(4 * half + e) * S::STAGE_LD + j * 32 + l32] = acc[i][j][4 * g + e];
        __builtin_amdgcn_wave_barrier();
        for (int v = lane; v < 8 * VPR; v += 64) {
          const int r = v / VPR, c8 = v - r * VPR;
          const int col = n0 + wc + c8 * 8;
          const int64_t d = s_dst[wave * WTM + i * 32 + 8 * g + r];
          if (col < a.nout && d >= 0) {
            const float4 lo = *reinterpret_cast<const float4*>(&st[r * S::STAGE_LD + c8 * 8]);
            const float4 hi = *reinterpret_cast<const float4*>(&st[r * S::STAGE_LD + c8 * 8 + 4]);
            float f[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            uint4* p = reinterpret_cast<uint4*>(a.dst + d + col);
            if (post != kPostNone) post_op(f, c8 * 8);
            if (a.accumulate) {
              float o[8];
              unpack8(*p, o);
#pragma unroll
              for (int e = 0; e < 8; ++e) f[e] += o[e];
            }
            // (non-temporal: the tile is written once and read by a later kernel; measured
            // 3-12% faster across the conv layers than a default store)
            const uint4 v = pack8(f);
            __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(p));
          }
        }
      }
  } else {
    // channel counts that are not a multiple of 8: scalar stores straight from the accumulators
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t d = s_dst[wave * WTM + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)];
        if (d < 0) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = n0 + wc + j * 32 + l32;
          if (col < a.nout) {
            float v = acc[i][j][r];
            if (post != kPostNone) {
              v = __builtin_fmaf(v, s_red[0][wc + j * 32 + l32], s_red[1][wc + j * 32 + l32]);
              if (post == kPostBnSilu) v = v * sigmoidf_fast(v);
            }
            if (a.accumulate) v += bf2f(a.dst[d + col]);
            a.dst[d + col] = (bf16_t)f2bf(v);
          }
        }
      }
  }
}

constexpr uint32_t kOob = 0x80000000u;  // a buffer offset past every range below
constexpr int kRecords = 0x7ffffff0;    // buffer range (bytes); in-range offsets stay below kOob - 2^24

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base) {
  // raw buffer, stride 0, range kRecords; word 3 = 0x00020000 (32-bit data format, the
  // setting for linear loads on this architecture)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, kRecords, 0x00020000);
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef short v4s_t __attribute__((ext_vector_type(4)));
typedef unsigned v2u_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v4s_t lds_v4s_t;

// Transposed B stage ([BK reduction rows][BN columns], rows of 2*BN bytes): 16-byte chunk
// c of row r sits in slot c ^ bt_swizzle(r).  A transposing read (ds_read_b64_tr_b16)
// of a 16-lane group covers 4 consecutive rows x 32 bytes; the swizzle puts those 4
// segments in distinct quarters of the 256-byte bank window (rows of 192 or 64 bytes
// already do).
template <int BN>
__device__ __forceinline__ int bt_swizzle(int r) {
  return (BN == 64 || BN == 192) ? 4 * ((r >> 1) & 1) : BN == 128 ? 4 * (r & 3) : 0;
}

}  // namespace

}  // namespace numbat
