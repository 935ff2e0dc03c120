// 3x3 stride-1 padding-1 convolutions on gfx950 MFMA from an input halo staged in LDS: the
// forward and the data gradient of ConvGemmArgs, optionally with the previous layer's BN + SiLU
// (or this layer's backward) applied to the staged halo.
#include <cstdlib>

#include "conv_tile.h"

namespace numbat {

namespace {

// ---------------------------------------------------------------------------
// 3x3, stride-1, padding-1 convolutions (the forward and, with the weights read in place
// and flipped, the data gradient): the input halo of a tile is staged in LDS once per
// 32-channel chunk and all nine taps are read out of it.  A tile is BM consecutive output
// pixels (linear over image, row, column); the source pixels its taps reach are the
// contiguous linear range [m0 - W - 1, m0 + BM + W + 1), because tap (r, s) of output
// pixel m reads source pixel m + (r - 1) W + (s - 1) whenever that pixel is inside the
// image (taps that leave the image read zeros instead: each lane keeps the LDS address of
// every tap of its rows, pointing at a zero row for the taps outside the image).  Per
// chunk the tile loads about BM + 2W pixels instead of 9 BM, so the loads are mostly the
// weights.
//
// Pipeline: one step is KT taps (1, or a whole tap row of 3) of one chunk, 32 reduction
// elements per tap: the weights of those taps (BN rows of 64 bytes per tap, or for the
// data gradient 32 rows of BN columns read with transposing LDS reads) in one of SB
// stages (prefetch distance SB - 1 steps), and the chunk's halo, two deep: the next
// chunk's halo is issued at the first step of the current one.  The waits are exact: at
// step s the loads issued after the weights of s are the later steps' weights, plus the
// next halo on the steps right after a chunk's first.  Every step issues the same loads;
// past the end of K they read zeros.  Halo buffers and weight stages are distinct LDS
// objects selected at compile time (two chunks per loop trip), so the compiler can tell an
// in-flight load's target from the buffer being read.
template <int TM, int TN, int HI, int KT, int SB, bool BT, int TC, int KP>
struct HaloShape {
  using G = GemmShape<TM, TN, 4>;
  static constexpr int NW = 4;
  static constexpr int SPC = 9 / KT;                   // steps per chunk
  static constexpr int HPAD = HI * NW * 16;            // halo pixels per buffer (16 per load instruction)
  static constexpr int HBYTES = (HPAD + 1) * 64;       // + one zero row read by out-of-image taps
  // buffer 0 stages the epilogue (of 4 KP waves on two-block tiles) and the halves' exchange
  static constexpr int STG = KP == 2 && TM == 2 ? 2 * G::STAGE_BYTES : G::STAGE_BYTES;
  static constexpr int XCH = KP == 2 ? 4 * 64 * 64 * TM : 0;
  static constexpr int H0MIN = STG > XCH ? STG : XCH;
  static constexpr int H0BYTES = HBYTES >= H0MIN ? HBYTES : H0MIN;
  static constexpr int TBYTES = G::BN * 64;            // the weights of one tap: BN x 32 elements
  static constexpr int BI = KT * G::BN / 16;           // weight load instructions per step (all waves)
  static constexpr int BI_MIN = BI / NW, BI_MAX = (BI + NW - 1) / NW;
  static_assert(KT == 1 || KT == 3, "one tap or one tap row per step");
  static_assert((2 * SPC) % SB == 0, "stage of a step known at compile time over two chunks");
  static_assert(SB >= 2 && SB <= 3 && SB - 1 <= SPC, "prefetch within one chunk");
  // two-dimensional tiles (TC > 0): TR x TC output pixels of one image, whose padded halo of
  // (TR + 2) x (TC + 2) pixels fits the buffer
  static constexpr int TR = TC > 0 ? G::BM / TC : 0;
  static_assert(TC == 0 || (G::BM % TC == 0 && (TR + 2) * (TC + 2) <= HPAD), "2D tile and its halo");
};

// Waves per SIMD the register allocation is held to.  The prologues on two-dimensional tiles of
// two reduction halves need the two blocks per CU that their LDS allows; left to itself the
// compiler took 129 registers for the forward (128 fit twice) and 269 for the backward (256 fit
// twice): 16 x 160 x 160 x 48, forward 81.1 us with one block per CU and 57.2 with two, backward
// 96.0 and 68.6 (on the four-wave kernel with one accumulator set: 62.0 and 67.1).
constexpr int halo_min_waves(int tc, int pro, int kv, int kp) {
  return tc > 0 && pro != kProNone && kp == 2 ? 2 * kv : 1;
}

// KV = 2: eight waves in two halves of four; half 0 issues every load, half k multiplies
// reduction slice k (16 channels) of every tap, and the halves add their sums through LDS
// before the epilogue (twice the waves per SIMD to cover a step's latencies, same LDS).  On
// tiles of two 32-row blocks per wave (TM = 2) the halves exchange one block each, so all eight
// waves take part in the epilogue.
//
// TL: problems whose last chunk holds at most 16 channels skip that chunk's second slice (a
// uniform branch per tap, which the other problems' kernels do without).
//
// PRO (kProFwd, kProBwd): an element-wise prologue on each 32-channel chunk of the staged
// halo, once per element, before any tap reads it; its per-channel constants sit in dynamic
// LDS (2 or 4 floats per source channel, sized at launch), and the loading lanes (of a
// forward's two halves, both on linear tiles) transform their chunks between their load wait
// and the barrier.  kProBwd (the data gradient, four waves): the halo holds g, each lane also loads y for its own halo chunks (into
// registers, a chunk ahead), and dy = BN + SiLU backward (g, y) replaces g in place; dy of
// the tile's own pixels is also stored (first column tile only).
template <int TM, int TN, int HI, int KT, int SB, bool BT, int TC, int PRO, int KV, int KP, bool TL>
__global__ __launch_bounds__(256 * KV, halo_min_waves(TC, PRO, KV, KP)) void convhalo_kernel(ConvGemmArgs a) {
  using G = GemmShape<TM, TN, 4>;
  using Sh = HaloShape<TM, TN, HI, KT, SB, BT, TC, KP>;
  constexpr bool XROWS = KV == 2 && TM == 2;  // the halves share out the rows of the epilogue
  // On linear tiles both halves transform the forward prologue's halo, at a barrier more per
  // chunk (16 x 40 x 40 x 192, 256-row tiles: 35.6 -> 30.7 us, 16 x 20 x 20 x 288, 128-row ones: 30.7 ->
  // 27.9); two-dimensional tiles overlap half 0's transform with their CU's other block (32 x
  // 160 x 160, 32 -> 64: 76.4 us with both halves, 73.2 with half 0).
  constexpr bool PSHARE = PRO == kProFwd && KV == 2 && TC == 0;
  constexpr int TR = Sh::TR;
  constexpr int BM = G::BM, BN = G::BN, WTM = G::WTM, NW = 4, SPC = Sh::SPC, D = SB - 1;
  constexpr int BI = Sh::BI, BI_MIN = Sh::BI_MIN, BI_MAX = Sh::BI_MAX, TBYTES = Sh::TBYTES;
  // memory operations a chunk's first step issues besides the weights: the next halo, and
  // with the backward prologue also the chunk's dy stores and the next chunk's y loads
  constexpr int XB = PRO == kProBwd ? 3 * HI : HI;
  static_assert((D - 1) * BI_MIN + XB <= 60, "load counter range");

  __shared__ __attribute__((aligned(16))) unsigned char sH0[Sh::H0BYTES];
  __shared__ __attribute__((aligned(16))) unsigned char sH1[Sh::HBYTES];
  __shared__ __attribute__((aligned(16))) unsigned char sB0[KT * TBYTES];
  __shared__ __attribute__((aligned(16))) unsigned char sB1[KT * TBYTES];
  __shared__ __attribute__((aligned(16))) unsigned char sB2[SB > 2 ? KT * TBYTES : 16];
  __shared__ int64_t s_dst[BM];
  __shared__ float s_red[XROWS ? 8 : NW][BN];
  __shared__ float s_mean[BN];
  // prologue constants, [2 or 4][cs]: forward scale, shift; backward a, b, c, d (bn_bwd_fold)
  extern __shared__ __attribute__((aligned(16))) float s_pro[];
  static_assert(PRO != kProFwd || !BT, "the BN + SiLU prologue is a forward's");
  static_assert(PRO != kProBwd || (BT && KV == 1), "the BN + SiLU backward prologue: a data gradient, four waves");
  static_assert(KV == 1 || KV == 2, "one or two reduction halves");
  auto hbuf = [&](auto hc) __attribute__((always_inline)) -> unsigned char* {
    if constexpr (decltype(hc)::value == 0) return sH0;
    else return sH1;
  };
  auto bstage = [&](auto bc) __attribute__((always_inline)) -> unsigned char* {
    constexpr int b = decltype(bc)::value;
    if constexpr (b == 0) return sB0;
    else if constexpr (b == 1) return sB1;
    else return sB2;
  };

  const TileId T{(int)blockIdx.x, (int)blockIdx.y, 0};
  const GemmPhase& P = a.ph[0];
  const Geo Ge = load_geo(P);
  const int m0 = T.mt * BM;
  const int n0 = T.nt * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = KV == 2 ? (wv & 3) : wv;  // the wave's rows (and load slots)
  const int kh = KV == 2 ? (wv >> 2) : 0;     // its reduction half
  const int l32 = lane & 31, half = lane >> 5;
  const int W = a.ws, H = a.hs, cs = a.cs, nout = a.nout;
  const int64_t pix2 = a.src_pix * 2;
  const int64_t npix = (int64_t)a.nimg * H * W;
  // a two-dimensional tile: image img2, output rows h0 .. h0 + TR, columns w0 .. w0 + TC
  // (the host checks that TR divides H and TC divides W, so every tile is whole)
  int img2 = 0, h0 = 0, w0 = 0;
  if constexpr (TC > 0) {
    const int ncol = W / TC, nrow = H / TR;
    img2 = T.mt / (nrow * ncol);
    const int rem = T.mt - img2 * nrow * ncol;
    const int tr = rem / ncol;
    h0 = tr * TR;
    w0 = (rem - tr * ncol) * TC;
  }

  // zero rows read by out-of-image taps (never a load target)
  if (tid < 4) {
    *reinterpret_cast<u32x4*>(sH0 + Sh::HPAD * 64 + tid * 16) = u32x4{0u, 0u, 0u, 0u};
    *reinterpret_cast<u32x4*>(sH1 + Sh::HPAD * 64 + tid * 16) = u32x4{0u, 0u, 0u, 0u};
  }
  // prologue: the BN constants of every source channel (published by the barrier below,
  // before any halo is transformed)
  if constexpr (PRO == kProFwd) {
    for (int ch = tid; ch < cs; ch += NW * 64 * KV)
      bn_fold(a.pro_gamma[ch], a.pro_beta[ch], a.pro_mean[ch], a.pro_var[ch], a.pro_eps, s_pro[ch], s_pro[cs + ch]);
    __syncthreads();
  } else if constexpr (PRO == kProBwd) {
    for (int ch = tid; ch < cs; ch += NW * 64 * KV)
      bn_bwd_fold(a.pro_gamma[ch], a.pro_beta[ch], a.pro_mean[ch], a.pro_rstd[ch], a.pro_dgamma[ch],
                  a.pro_dbeta[ch], a.pro_m, s_pro[ch], s_pro[cs + ch], s_pro[2 * cs + ch], s_pro[3 * cs + ch]);
    __syncthreads();
  }

  // ---- halo loads: instruction q of this wave fills pixels (q*NW + wave)*16 .. +16; the
  // lane's slot is lane % 4 of pixel lane / 4, holding chunk slot ^ ((pixel >> 2) & 3).
  // Linear tiles: halo pixel j is source pixel m0 - W - 1 + j.  Two-dimensional tiles:
  // halo pixel j is (row j / (TC + 2), column j % (TC + 2)) of the padded window whose
  // corner is (h0 - 1, w0 - 1); its pixels outside the image load zeros (the padding).
  const int64_t hbase_px =
      TC > 0 ? ((int64_t)img2 * H + h0 - 1) * W + w0 - 1 : (int64_t)m0 - W - 1;
  const __amdgpu_buffer_rsrc_t rsA = buffer_rsrc(a.src + hbase_px * a.src_pix);
  uint32_t hoff[HI];
  // channel of the lane's chunk within a 32-channel chunk, the same for every instruction
  const int hc8 = 8 * ((lane & 3) ^ ((lane >> 4) & 3));
#pragma unroll
  for (int q = 0; q < HI; ++q) {
    const int j = (q * NW + wave) * 16 + (lane >> 2);
    if constexpr (TC > 0) {
      const int hr = j / (TC + 2), hcol = j - hr * (TC + 2);
      const bool ok = j < (TR + 2) * (TC + 2) && (unsigned)(h0 - 1 + hr) < (unsigned)H &&
                      (unsigned)(w0 - 1 + hcol) < (unsigned)W;
      hoff[q] = ok ? (uint32_t)(((int64_t)hr * W + hcol) * pix2 + hc8 * 2) : kOob;
    } else {
      const int64_t src_px = hbase_px + j;
      const bool ok = src_px >= 0 && src_px < npix && j < BM + 2 * W + 2;
      hoff[q] = ok ? (uint32_t)(j * pix2 + hc8 * 2) : kOob;
    }
  }
  // backward prologue: byte offset of the lane's chunk of halo instruction q in y and dy (one
  // pixel stride; relative to the tensor's halo base pixel; valid where hoff[q] is),
  // and whether its pixel is one of the tile's own output pixels (the halo's interior)
  auto chunk_off = [&](int q) __attribute__((always_inline)) -> uint32_t {
    const int j = (q * NW + wave) * 16 + (lane >> 2);
    if constexpr (TC > 0) {
      const int hr = j / (TC + 2), hcol = j - hr * (TC + 2);
      return (uint32_t)(((int64_t)hr * W + hcol) * a.pro_y_pix * 2 + hc8 * 2);
    } else {
      return (uint32_t)(j * a.pro_y_pix * 2 + hc8 * 2);
    }
  };
  auto interior = [&](int q) __attribute__((always_inline)) -> bool {
    const int j = (q * NW + wave) * 16 + (lane >> 2);
    if constexpr (TC > 0) {
      const int hr = j / (TC + 2), hcol = j - hr * (TC + 2);
      return hr >= 1 && hr <= TR && hcol >= 1 && hcol <= TC;
    } else {
      return j >= W + 1 && j < W + 1 + BM;
    }
  };
  const __amdgpu_buffer_rsrc_t rsY = buffer_rsrc(PRO == kProBwd ? a.pro_y + hbase_px * a.pro_y_pix : a.src);
  const __amdgpu_buffer_rsrc_t rsD = buffer_rsrc(PRO == kProBwd ? a.pro_dy + hbase_px * a.pro_y_pix : a.dst);
  u32x4 yv[PRO == kProBwd ? HI : 1];  // y of the lane's chunks of the next chunk to transform

  // ---- weight loads: instruction u of a step covers 1 KiB of tap u / (BI / KT)'s stage
  const __amdgpu_buffer_rsrc_t rsB = buffer_rsrc(P.wt);
  constexpr int BPT = BN / 16;  // load instructions per tap
  uint32_t boff[BI_MAX];
  int bch[BI_MAX];  // non-transposed: channel of the lane's chunk; transposed: o row of the stage
  int btap[BI_MAX];  // tap of the step (0 .. KT-1) the instruction loads
#pragma unroll
  for (int j = 0; j < BI_MAX; ++j) {
    const int u = j * NW + wave;     // instruction index within the step
    const int tp = u / BPT, v = u % BPT;
    btap[j] = tp;
    if constexpr (!BT) {
      // stage row = output channel n0 + row, 64 bytes = 32 channels of one tap
      const int row = v * 16 + (lane >> 2), o = n0 + row;
      const int lc = (lane & 3) ^ ((row >> 2) & 3);
      const bool ok = u < BI && o < nout;
      boff[j] = ok ? (uint32_t)(((int64_t)o * 9 * cs + tp * cs + lc * 8) * 2) : kOob;
      bch[j] = ok ? lc * 8 : (1 << 20);
    } else {
      // stage row = reduction channel o (of the 32-channel chunk), 2*BN bytes = output
      // channels n0 .. n0 + BN of one (flipped) tap
      const int byte = v * 1024 + lane * 16;
      const int row = byte / (2 * BN), slot = (byte % (2 * BN)) / 16;
      const int ch = slot ^ bt_swizzle<BN>(row);
      const bool ok = u < BI && n0 + ch * 8 < nout;
      boff[j] = ok ? (uint32_t)(((int64_t)row * 9 * nout + n0 + ch * 8) * 2) : kOob;
      bch[j] = ok ? row : (1 << 20);
    }
  }
  const int nchunk = (cs + 31) / 32;
  const int nsteps = SPC * nchunk;

  auto issue_halo = [&](auto hc, int c) __attribute__((always_inline)) {
    if (KV == 2 && kh != 0) return;
    unsigned char* Hb = hbuf(hc);
    const int cb = 32 * c;
#pragma unroll
    for (int q = 0; q < HI; ++q) {
      const uint32_t v = cb + hc8 < cs ? hoff[q] : kOob;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void_t*)(Hb + (q * NW + wave) * 1024), 16, v,
                                               (uint32_t)(cb * 2), 0, 0);
    }
  };
  // weights of step s (chunk s / SPC, taps KT * (s % SPC) ..) into stage bc
  auto issue_b = [&](auto bc, int s) __attribute__((always_inline)) {
    if (KV == 2 && kh != 0) return;
    unsigned char* Bb = bstage(bc);
    const int c = s / SPC, t0 = KT * (s - SPC * c), cb = 32 * c;
    const bool live = s < nsteps;
    uint32_t so;
    if constexpr (!BT) so = (uint32_t)((t0 * cs + cb) * 2);
    else so = (uint32_t)(((int64_t)cb * 9 + 8 - t0) * nout * 2);  // the flipped tap 8 - t
#pragma unroll
    for (int j = 0; j < BI_MAX; ++j) {
      if (j * NW + wave < BI) {  // wave-uniform
        const uint32_t v = (live && cb + bch[j] < cs) ? boff[j] : kOob;
        // (transposed: tap t0 + btap is 8 - t0 - btap, btap rows of weights lower)
        const uint32_t sv = BT ? so - (uint32_t)(btap[j] * nout * 2) : so;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_void_t*)(Bb + (j * NW + wave) * 1024), 16, v, sv, 0, 0);
      }
    }
  };

  // ---- this lane's A rows: the LDS address of every tap of its rows (linear tiles: the
  // zero row for taps outside the image; two-dimensional tiles: the padded window holds
  // those zeros itself)
  uint32_t aaddr[TM][9];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int prow = wave * WTM + i * 32 + l32;
    if constexpr (TC > 0) {
      const int ir = prow / TC, ic = prow - ir * TC;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const int p = (ir + r) * (TC + 2) + ic + s;
          aaddr[i][3 * r + s] = (uint32_t)(p * 64 + (((half) ^ ((p >> 2) & 3)) << 4));
        }
      continue;
    }
    const int m = m0 + prow;
    uint32_t mask = 0;
    if (m < Ge.m) {
      uint32_t img, oh, ow;
      geo_pos((uint32_t)m, Ge, img, oh, ow);
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const bool in = (unsigned)((int)oh + r - 1) < (unsigned)H && (unsigned)((int)ow + s - 1) < (unsigned)W;
          mask |= (in ? 1u : 0u) << (3 * r + s);
        }
    }
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const int p = prow + r * W + s;
        const uint32_t ad = (uint32_t)(p * 64 + (((half) ^ ((p >> 2) & 3)) << 4));
        const uint32_t zr = (uint32_t)(Sh::HPAD * 64 + half * 16);
        aaddr[i][3 * r + s] = ((mask >> (3 * r + s)) & 1u) ? ad : zr;
      }
  }
  // transposed B reads (see convdma_kernel): lane l = 16 g + 4 e + q reads 4 columns of
  // rows 8 (g / 2) + e and that + 4 of each 16-row slice
  uint32_t btoff[BT ? TN : 1];
  if constexpr (BT) {
    const int g = lane >> 4, e = (lane & 15) >> 2, q = lane & 3;
    const int r0 = 8 * (g >> 1) + e;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = 4 * j + 2 * (g & 1) + (q >> 1);
      btoff[j] = (uint32_t)(r0 * 2 * BN + (c ^ bt_swizzle<BN>(r0)) * 16 + (q & 1) * 8);
    }
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // the backward prologue on a tile whose plain kernel has two reduction halves: the second
  // 16-channel slice of every step goes to accumulators of its own, added last, so the sums
  // (and dx) equal the plain kernel's bit for bit
  constexpr bool SPLIT = PRO == kProBwd && KP == 2;
  f32x16 acc2[SPLIT ? TM : 1][SPLIT ? TN : 1];
  if constexpr (SPLIT) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc2[i][j][r] = 0.f;
  }

  // multiply one tap (t, within the step's stage at tap slot tk) from halo buffer hc
  // (half_chunk: a last chunk of at most 16 channels, whose second slice would multiply zeros)
  auto compute_tap = [&](const unsigned char* Hb, const unsigned char* Bb, auto tc, auto khc, bool half_chunk)
                         __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value, KH = decltype(khc)::value;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (KV == 2 && ks != KH) continue;  // (compile-time after unrolling)
      if (TL && ks == 1 && half_chunk) continue;
      u32x4 af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const u32x4*>(Hb + (aaddr[i][t] ^ (uint32_t)(32 * ks)));
      if constexpr (!BT) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int row = j * 32 + l32;
          bf[j] = *reinterpret_cast<const u32x4*>(Bb + row * 64 + ((((2 * ks + half) ^ ((row >> 2) & 3))) << 4));
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const unsigned char* pb = Bb + btoff[j] + ks * 16 * 2 * BN;
          const v4s_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)pb);
          const v4s_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)(pb + 4 * 2 * BN));
          const v2u_t lo = __builtin_bit_cast(v2u_t, r0), hi = __builtin_bit_cast(v2u_t, r1);
          bf[j][0] = lo.x;
          bf[j][1] = lo.y;
          bf[j][2] = hi.x;
          bf[j][3] = hi.y;
        }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (SPLIT) {
            if (ks == 0) acc[i][j] = mfma32x32x16(af[i], bf[j], acc[i][j]);
            else acc2[SPLIT ? i : 0][SPLIT ? j : 0] = mfma32x32x16(af[i], bf[j], acc2[SPLIT ? i : 0][SPLIT ? j : 0]);
          } else {
            acc[i][j] = mfma32x32x16(af[i], bf[j], acc[i][j]);
          }
        }
    }
  };
  // wait for this wave's loads of the step (N later loads stay in flight), then every wave's
  auto sync = [&](auto nc) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(decltype(nc)::value) : "memory");
  };
  // backward prologue: y of this lane's chunks of chunk c, into registers (zeros past the
  // channels and outside the image)
  auto issue_y = [&](int c) __attribute__((always_inline)) {
    if constexpr (PRO == kProBwd) {
      const int cb = 32 * c;
#pragma unroll
      for (int q = 0; q < HI; ++q) {
        const uint32_t v = (hoff[q] != kOob && cb + hc8 < cs) ? chunk_off(q) : kOob;
        yv[q] = __builtin_amdgcn_raw_buffer_load_b128(rsY, v, (uint32_t)(cb * 2), 0);
      }
    }
  };
  // backward prologue: the chunks of chunk c's halo that halo wave `wave` loaded (landed
  // and visible) become dy in place, from g there and y in yv.  A lane's chunks are the same
  // 8 channels for every halo instruction (slot (lane & 3) ^ ((lane >> 4) & 3)); they are
  // done in two passes of 4 channels, each with its 16 constants in registers (the
  // accumulators stay live, so the working set is kept small), the second pass storing the
  // whole chunk.  One dy store per halo instruction, issued by every wave whatever its
  // lanes hold (out of range where the chunk is not the tile's own pixel, or in another
  // column tile's block), so the wave's count of memory operations is fixed.
  auto transform_bwd = [&](auto hc, int c) __attribute__((always_inline)) {
    unsigned char* Hb = hbuf(hc);
    const int cb = 32 * c;
    const int ch = cb + hc8 < cs ? cb + hc8 : 0;
#pragma unroll
    for (int ps = 0; ps < 2; ++ps) {
      float ka[4], kb[4], kc[4], kd[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ka[e] = s_pro[ch + 4 * ps + e];
        kb[e] = s_pro[cs + ch + 4 * ps + e];
        kc[e] = s_pro[2 * cs + ch + 4 * ps + e];
        kd[e] = s_pro[3 * cs + ch + 4 * ps + e];
      }
#pragma unroll
      for (int q = 0; q < HI; ++q) {
        const bool live = hoff[q] != kOob && cb + hc8 < cs;
        unsigned char* p = Hb + (q * NW + wave) * 1024 + lane * 16;
        // pass 0: the first 4 channels; pass 1: the last 4, with the first 4 as pass 0 left them
        u32x4 v;
        if (ps == 0) {
          const uint2 h = *reinterpret_cast<const uint2*>(p);
          v = u32x4{h.x, h.y, 0u, 0u};
        } else {
          v = *reinterpret_cast<const u32x4*>(p);
        }
        const uint32_t g0 = v[2 * ps], g1 = v[2 * ps + 1];
        const uint32_t y0 = yv[q][2 * ps], y1 = yv[q][2 * ps + 1];
        const float o0 = bn_silu_bwd_apply(bf2f(g0 & 0xffffu), bf2f(y0 & 0xffffu), ka[0], kb[0], kc[0], kd[0]);
        const float o1 = bn_silu_bwd_apply(bf2f(g0 >> 16), bf2f(y0 >> 16), ka[1], kb[1], kc[1], kd[1]);
        const float o2 = bn_silu_bwd_apply(bf2f(g1 & 0xffffu), bf2f(y1 & 0xffffu), ka[2], kb[2], kc[2], kd[2]);
        const float o3 = bn_silu_bwd_apply(bf2f(g1 >> 16), bf2f(y1 >> 16), ka[3], kb[3], kc[3], kd[3]);
        const uint2 oh = make_uint2(pack2(o0, o1), pack2(o2, o3));
        if (live) *reinterpret_cast<uint2*>(p + 8 * ps) = oh;
        if (ps == 1) {
          const uint32_t so = (live && T.nt == 0 && interior(q)) ? chunk_off(q) : kOob;
          __builtin_amdgcn_raw_buffer_store_b128(u32x4{v[0], v[1], oh.x, oh.y}, rsD, so, (uint32_t)(cb * 2), 0);
          // wait states before anything rewrites the store's data registers: with the
          // scheduling barrier right after it, the compiler issued a VALU write to the first
          // data register on the next cycle, and about one 16-byte store in 20000 then wrote
          // that register's new value (measured; none with this pause)
          asm volatile("s_nop 4");
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // prologue: this lane's 16-byte chunks of chunk c's halo (landed: the wait before
  // this covers them) become the previous layer's activations, SiLU(BN(y)), in place;
  // chunks that loaded zeros (padding, past the image or the channels) stay zero
  auto transform = [&](auto hc, int c) __attribute__((always_inline)) {
    if constexpr (PRO != kProFwd) return;
    unsigned char* Hb = hbuf(hc);
    const int cb = 32 * c;
#pragma unroll
    for (int q = 0; q < HI; ++q) {
      if (KV == 2 && (PSHARE ? (q & 1) != kh : kh != 0)) continue;  // (uniform)
      if (hoff[q] != kOob && cb + hc8 < cs) {
        u32x4* p = reinterpret_cast<u32x4*>(Hb + (q * NW + wave) * 1024 + lane * 16);
        const u32x4 v = *p;
        float f[8];
        unpack8(uint4{v[0], v[1], v[2], v[3]}, f);
        const int ch = cb + hc8;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = bn_silu_apply(f[e], s_pro[ch + e], s_pro[cs + ch + e]);
        const uint4 o = pack8(f);
        *p = u32x4{o.x, o.y, o.z, o.w};
      }
    }
  };
  // step k (0 .. SPC-1) of a chunk c of parity h (halo buffer h): wait, issue the next
  // halo (k = 0) and the weights D steps ahead, multiply the step's KT taps
  auto step = [&](auto hc, auto kc, int c, auto khc) __attribute__((always_inline)) {
    constexpr int h = decltype(hc)::value, k = decltype(kc)::value;
    constexpr int sl = h * SPC + k;  // step index within the two-chunk trip
    constexpr int waitn = (D - 1) * BI_MIN + ((k >= 1 && k <= D - 1) ? XB : 0);
    if constexpr (PRO == kProFwd && k == 0) {
      // the chunk's halo has landed for this wave: transform this lane's part, then publish
      // (they are half 0's loads: it publishes them before both halves transform)
      if constexpr (PSHARE) sync(Ic<waitn>{});
      else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(waitn) : "memory");
      transform(hc, c);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else if constexpr (PRO == kProBwd && k == 0) {
      // as the forward's (the wait also covers this chunk's y, loaded before its halo), then
      // this wave's y loads of the next chunk
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(waitn) : "memory");
      transform_bwd(hc, c);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      issue_y(c + 1);
    } else {
      sync(Ic<waitn>{});
    }
    if constexpr (k == 0) issue_halo(Ic<1 - h>{}, c + 1);
    issue_b(Ic<(sl + D) % SB>{}, SPC * c + k + D);
    const unsigned char* Hb = hbuf(hc);
    const unsigned char* Bb = bstage(Ic<sl % SB>{});
    const bool half_chunk = TL && 32 * c + 16 >= cs;  // (uniform)
#pragma unroll
    for (int tt = 0; tt < KT; ++tt) {
      // (compile-time tap index: KT * k + tt)
      if constexpr (KT == 1) compute_tap(Hb, Bb, Ic<k>{}, khc, half_chunk);
      else {
        if (tt == 0) compute_tap(Hb, Bb, Ic<3 * k + 0>{}, khc, half_chunk);
        if (tt == 1) compute_tap(Hb, Bb + TBYTES, Ic<3 * k + 1>{}, khc, half_chunk);
        if (tt == 2) compute_tap(Hb, Bb + 2 * TBYTES, Ic<3 * k + 2>{}, khc, half_chunk);
      }
    }
  };
  auto chunk = [&](auto hc, int c, auto khc) __attribute__((always_inline)) {
    step(hc, Ic<0>{}, c, khc);
    step(hc, Ic<1>{}, c, khc);
    step(hc, Ic<2>{}, c, khc);
    if constexpr (SPC == 9) {
      step(hc, Ic<3>{}, c, khc);
      step(hc, Ic<4>{}, c, khc);
      step(hc, Ic<5>{}, c, khc);
      step(hc, Ic<6>{}, c, khc);
      step(hc, Ic<7>{}, c, khc);
      step(hc, Ic<8>{}, c, khc);
    }
  };

  issue_y(0);  // (before the halo, as at every chunk's first step)
  issue_halo(Ic<0>{}, 0);
  issue_b(Ic<0>{}, 0);
  if constexpr (D >= 2) issue_b(Ic<1>{}, 1);
  // destination offsets of the tile's rows (the epilogue's), under the first loads
  for (int r = tid; r < BM; r += NW * 64) {
    const int m = TC > 0 ? (img2 * H + h0 + r / (TC > 0 ? TC : 1)) * W + w0 + r % (TC > 0 ? TC : 1) : m0 + r;
    s_dst[r] = dst_offset(a, Ge, m);
  }
  // the main loop, one copy per reduction half (a compile-time slice choice)
  auto main_loop = [&](auto khc) __attribute__((always_inline)) {
    int c = 0;
    for (; c + 2 <= nchunk; c += 2) {
      chunk(Ic<0>{}, c, khc);
      chunk(Ic<1>{}, c + 1, khc);
    }
    if (c < nchunk) chunk(Ic<0>{}, c, khc);
  };
  if (KV == 1 || kh == 0) main_loop(Ic<0>{});
  else main_loop(Ic<1>{});
  // the loads issued past the last step land before the halo buffer becomes staging space
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  if constexpr (XROWS) {
    // two 32-row blocks per wave: half h keeps block h and hands the other one over, a 32 x 32
    // block of each of the eight waves at a time through halo buffer 0 (32 KiB); the epilogue
    // then runs on eight waves of 32 rows, 2 wave + h
    f32x4* xb = reinterpret_cast<f32x4*>(sH0);
    f32x16 own[1][TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      f32x16 give;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        give[r] = kh == 0 ? acc[TM - 1][j][r] : acc[0][j][r];
        own[0][j][r] = kh == 0 ? acc[0][j][r] : acc[TM - 1][j][r];
      }
      if (j > 0) __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q)
        xb[((kh * 4 + wave) * 4 + q) * 64 + lane] = f32x4{give[4 * q], give[4 * q + 1], give[4 * q + 2], give[4 * q + 3]};
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = xb[(((1 - kh) * 4 + wave) * 4 + q) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) own[0][j][4 * q + e] += v[e];
      }
    }
    gemm_epilogue<1, TN, 8>(a, P, T, own, m0, n0, sH0, s_dst, s_red, s_mean, true, 2 * wave + kh);
    return;
  } else if constexpr (KV == 2) {
    // half 1 hands its sums to half 0, one 32 x 32 block of each wave at a time through
    // halo buffer 0 (16 KiB: 4 waves x 64 lanes x 16 floats); the sum is half 0 + half 1
    f32x4* xb = reinterpret_cast<f32x4*>(sH0);
    static_assert(Sh::H0BYTES >= 4 * 64 * 64, "exchange space");
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (kh == 1) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x4 v;
            v[0] = acc[i][j][4 * q];
            v[1] = acc[i][j][4 * q + 1];
            v[2] = acc[i][j][4 * q + 2];
            v[3] = acc[i][j][4 * q + 3];
            xb[(wave * 4 + q) * 64 + lane] = v;
          }
        }
        __syncthreads();
        if (kh == 0) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = xb[(wave * 4 + q) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
          }
        }
        __syncthreads();
      }
  }
  if constexpr (SPLIT) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += acc2[SPLIT ? i : 0][SPLIT ? j : 0][r];
  }
  if constexpr (!XROWS) gemm_epilogue<TM, TN, NW>(a, P, T, acc, m0, n0, sH0, s_dst, s_red, s_mean, kh == 0);
}

// halo kernel instantiations: (32-row tiles per wave, 32-column tiles, halo load
// instructions per wave, taps per step, weight stages, tile columns); a linear BM-row tile
// (tile columns 0) of a W-wide image needs BM + 2 W + 2 halo pixels, a two-dimensional
// TR x TC tile (TC tile columns) (TR + 2) x (TC + 2), 16 per instruction
struct HInst {
  int tm, tn, hi, kt, sb, tc, kv;  // kv: reduction halves (of four waves each)
};
constexpr HInst kH[] = {
    {1, 3, 4, 3, 2, 0, 2},   // 0: 128 x 96, W <= 63, a tap row per step, two weight stages
    {2, 3, 7, 1, 3, 0, 1},   // 1: 256 x 96, W <= 95, one tap per step, three weight stages
    {1, 2, 4, 3, 2, 0, 2},   // 2: 128 x 64, W <= 63
    {2, 2, 7, 1, 3, 0, 1},   // 3: 256 x 64, W <= 95
    {2, 3, 6, 1, 3, 32, 1},  // 4: 256 x 96 on 8 x 32 output pixels (a 10 x 34 halo), one tap per step
    {2, 2, 6, 1, 3, 32, 1},  // 5: 256 x 64 on 8 x 32
    {1, 3, 5, 3, 2, 0, 2},   // 6: 128 x 96, W <= 95, a tap row per step (small grids)
    {1, 2, 5, 3, 2, 0, 2},   // 7: 128 x 64, W <= 95
    {2, 3, 6, 3, 3, 0, 2},   // 8: 256 x 96, W <= 63, eight waves, a tap row per step, three stages
    {2, 3, 7, 3, 2, 0, 2},   // 9: 256 x 96, W <= 95, eight waves, a tap row per step
    {2, 2, 6, 1, 3, 32, 2},  // 10: 256 x 64 on 8 x 32, eight waves
};
constexpr int kNumH = sizeof(kH) / sizeof(kH[0]);
// a linear 256-row tile of eight waves
constexpr bool linear256(const HInst& c) { return c.tm == 2 && c.kv == 2 && c.tc == 0; }

template <int I>
hipError_t launch_h(const ConvGemmArgs& a, hipStream_t s) {
  if constexpr (I < kNumH) {
    constexpr HInst c = kH[I];
    using G = GemmShape<c.tm, c.tn, 4>;
    dim3 grid((unsigned)((a.ph[0].m + G::BM - 1) / G::BM), (unsigned)((a.nout + G::BN - 1) / G::BN), 1);
    // the backward prologue keeps four waves: its y registers and transform do not fit the
    // eight-wave form's 128 registers per lane
    const dim3 block(256 * c.kv);
    // the prologue's per-channel constants (dynamic LDS, sized to the channels so that the
    // blocks per CU stay those of the plain kernel wherever the channels allow)
    const size_t fwd_smem = (size_t)2 * a.cs * sizeof(float), bwd_smem = (size_t)4 * a.cs * sizeof(float);
    const bool tl = (a.cs & 31) != 0 && (a.cs & 31) <= 16;
    if (a.bt && a.pro_kind == kProBwd) {
      if constexpr (linear256(c)) return hipErrorInvalidValue;  // (convhalo_pick gives it 128-row tiles)
      else
        NUMBAT_LAUNCH((convhalo_kernel<c.tm, c.tn, c.hi, c.kt, c.sb, true, c.tc, kProBwd, 1, c.kv, false>), grid,
                      dim3(256), bwd_smem, s, a);
    } else if (a.pro_kind == kProFwd)
      NUMBAT_LAUNCH((convhalo_kernel<c.tm, c.tn, c.hi, c.kt, c.sb, false, c.tc, kProFwd, c.kv, c.kv, false>), grid, block,
                    fwd_smem, s, a);
    else if (a.bt && tl)
      NUMBAT_LAUNCH((convhalo_kernel<c.tm, c.tn, c.hi, c.kt, c.sb, true, c.tc, kProNone, c.kv, c.kv, true>), grid, block,
                    0, s, a);
    else if (a.bt)
      NUMBAT_LAUNCH((convhalo_kernel<c.tm, c.tn, c.hi, c.kt, c.sb, true, c.tc, kProNone, c.kv, c.kv, false>), grid, block,
                    0, s, a);
    else if (tl)
      NUMBAT_LAUNCH((convhalo_kernel<c.tm, c.tn, c.hi, c.kt, c.sb, false, c.tc, kProNone, c.kv, c.kv, true>), grid, block,
                    0, s, a);
    else
      NUMBAT_LAUNCH((convhalo_kernel<c.tm, c.tn, c.hi, c.kt, c.sb, false, c.tc, kProNone, c.kv, c.kv, false>), grid, block,
                    0, s, a);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <int I>
hipError_t launch_h_id(int id, const ConvGemmArgs& a, hipStream_t s) {
  if constexpr (I >= kNumH) return hipErrorInvalidValue;
  else return id == I ? launch_h<I>(a, s) : launch_h_id<I + 1>(id, a, s);
}

}  // namespace

// 3x3, stride 1, padding 1, 8-multiple source channels, one phase
bool convhalo_shape(const ConvGemmArgs& a) {
  const GemmPhase& P = a.ph[0];
  if (a.nphase != 1 || a.cs % 8 != 0 || P.taps != 9 || a.gstride_h != 1 || a.gstride_w != 1 ||
      a.dstep_h != 1 || a.dstep_w != 1 || P.gh != a.hs || P.gw != a.ws || a.hd != a.hs || a.wd != a.ws)
    return false;
  if (!a.bt)
    for (int r = 0; r < 3; ++r)
      for (int q = 0; q < 3; ++q)
        if (P.off[r * 3 + q] != (int32_t)((uint32_t)(uint16_t)(int16_t)(r - 1) | ((uint32_t)(q - 1) << 16)))
          return false;
  // weight offsets of one step are 32-bit
  return (int64_t)a.nout * 9 * a.cs * 2 < (int64_t)kRecords;
}

// the halo pixels a tile needs: a linear BM-row tile (tc 0) of a w-wide image, or a
// two-dimensional (BM / tc) x tc one
static int halo_pixels(int bm, int tc, int w) { return tc > 0 ? (bm / tc + 2) * (tc + 2) : bm + 2 * w + 2; }

// Whether eight-wave tiles are well filled in whole rounds of 256 and have more than one chunk to
// walk (18 x 232 x 13, 32 -> 176 columns: 20.4 us, 17.0 on 128-row tiles, whose blocks overlap)
static bool linear256_fills(int64_t tiles256, int cs) {
  const int64_t rounds = (tiles256 + 255) / 256;
  return cs > 32 && (double)tiles256 / (double)(256 * rounds) >= (rounds > 1 ? 0.75 : 0.66);
}
// 96 or 64 columns per tile (3 or 2): 96 for their multiples (of a forward from 256 tiles up: 9 x 23 x
// 23, 176 -> 192 16.8 us, 14.0 on 64 columns); other counts take the one with less work per CU (its
// most tiles times their columns) unless eight-wave tiles of 96 fill their rounds.  Data gradients,
// us, 64 against 96 columns: 14 x 14, 136 <- 64 6.7 : 8.4, 22 x 29 x 29, 152 <- 80 11.4 : 13.5, 4 x 53 x 53,
// 560 <- 64 15.7 : 18.0; forward 14 x 28 x 28, 128 -> 272 17.5 : 20.2; 16 x 80 x 80, 192 -> 80 52.0 : 39.9.
static int halo_columns(int64_t m, int nout, int cs, int w, bool bt) {
  const int64_t c96 = (nout + 95) / 96, c64 = (nout + 63) / 64;
  if (c96 * 96 > c64 * 64) return 2;
  const int64_t t256 = (m + 255) / 256, rows = w > 63 ? t256 : (m + 127) / 128;
  if (nout % 96 == 0 && (bt || w > 63 || rows * c96 >= 256)) return 3;
  if (w <= 63 && linear256_fills(t256 * c96, cs)) return 3;
  if (w > 63 && w <= 95 && t256 * c96 >= 100 && t256 * c96 <= 256) return 3;
  return (rows * c64 + 255) / 256 * 64 < (rows * c96 + 255) / 256 * 96 ? 2 : 3;
}

// Halo kernel tile, from a sweep of the instantiations over the detector's 3x3 stride-1
// layers at batch 16 (each layer alone): 96 or 64 columns (halo_columns);
// images up to 63 pixels wide on 128-row tiles with a whole tap row (three taps) per
// step and two weight stages (40 x 40, 192 channels: forward 33.6 -> 29.6 us, data
// gradient 29.4 -> 24.0), up to 95 wide on 256-row tiles with one tap per step and three
// stages (80 x 80, 96 channels: 35.4 -> 28.3 and 28.9 -> 22.6 us); wider images on
// two-dimensional tiles of 8 x 32 output pixels with one tap per step and three stages,
// when 32 divides the width and 8 the height (160 x 160, 48 channels: forward 54.5 -> 51.1,
// data gradient 44.2 -> 39.3 us against the direct-to-LDS kernel; a linear tile of a
// 160-wide image needs 2.5 image rows of halo and measured 30-80% slower, 4 x 32 tiles
// with a tap row per step 10-20% slower, and 8 x 16 tiles on the 80-wide layers 13-18%
// slower than their linear 256-row tiles).  Fewer than 160 256-row tiles leave CUs idle:
// images of 64 to 95 columns then take 128-row tiles.  Forward grids of fewer than 256 tiles
// keep the direct-to-LDS kernel on two-dimensional tiles, where 64 tiles or more walk a long
// reduction (16 images of 20 x 20, 576 -> 192: 31.0 against 35.3 us; 288 -> 288: the layer's
// training pass 96.2 against 101.7 us) and on 64 to 95 columns up to 32 channels, to 64 below
// 160 tiles (2 x 76 x 76, 48 -> 288 10.1 against 12.1 us); elsewhere the halo kernel is as fast or
// faster (4 images of 26 x 26 x 128: 8.2 us against 11.5, 8 of 40 x 40 x 192: 15.0 and 20.0).
// Returns variant kVariantGeneric when the halo
// kernel is not used.
//
// Linear 256 x 96 tiles of eight waves (one block per CU): a wave's 64 x 96 share needs 5 LDS
// fragments per 6 products where 32 x 96 needs 8, and the CU loads the weights once instead of
// once per 128-row block, so they are faster wherever whole rounds of 256 tiles are well
// filled.  Forward / data gradient, us, against 128-row tiles (W <= 63) or four waves (W <=
// 95): 16 x 40 x 40 x 192 (200 tiles) 25.3 -> 22.7 / 23.1 -> 21.1, 14 images (175) 21.7 -> 19.3 /
// 19.9 -> 17.7, 32 images (400) 43.2 -> 38.8 / 40.5 -> 36.4, 16 x 40 x 40 x 384 (400) 74.7 -> 66.3 /
// 70.6 -> 64.9; 8 images (100) 17.1 -> 19.5, 16 x 52 x 52, 96 -> 192 columns (338) 22.1 -> 23.7.  80
// x 80 x 96: 4 images (100) 18.9 -> 13.9, 10 (250) 17.2 -> 15.4, 16 (400) 23.2 -> 27.1.
// Two-dimensional 64-column tiles take eight waves (on one block per CU) from 800 tiles up: 16 x
// 160 x 160 x 48 42.1 -> 38.5 / 36.7 -> 33.1, 8 x 160 x 160, 32 -> 64 18.8 -> 18.0; 4 x 160 x 160 x 64
// (400) 14.5 -> 15.6.
// pro_bwd: the tile of the backward prologue, whose sums have the plain kernel's order on
// 128-row tiles too.
TileCfg convhalo_pick(int64_t m, int nout, int cs, int h, int w, bool bt, bool any_grid, bool pro_bwd) {
  const int tn = halo_columns(m, nout, cs, w, bt);
  const int64_t cols = (nout + 32 * tn - 1) / (32 * tn), tiles256 = (m + 255) / 256 * cols;
  HInst want{2, tn, 0, 1, 3, 0, 1};
  if (w > 95) {
    want.tc = 32;
    if (tn == 2 && tiles256 >= 800) want.kv = 2;
  } else if (w > 63) {
    if (tn == 3 && tiles256 >= 100 && tiles256 <= 256) want = pro_bwd ? HInst{1, 3, 0, 3, 2, 0, 2} : HInst{2, 3, 0, 3, 2, 0, 2};
    else if (tiles256 < 160) want = HInst{1, tn, 0, 3, 2, 0, 2};
  } else {
    want = tn == 3 && linear256_fills(tiles256, cs) && !pro_bwd ? HInst{2, 3, 0, 3, 3, 0, 2} : HInst{1, tn, 0, 3, 2, 0, 2};
  }
  const TileCfg none{0, 0, -1, kVariantGeneric};
  const int bm = 128 * want.tm;
  if (want.tc > 0 && (w % want.tc != 0 || bm % want.tc != 0 || h % (bm / want.tc) != 0)) return none;
  const int64_t tiles = ((m + bm - 1) / bm) * cols;
  // (of 256-row tiles half as many cover the grid that 256 of 128 rows do)
  const int64_t full = linear256(want) ? 128 : 256;
  // (one chunk of at most 24 channels: the gather of taps is as cheap as the halo.  16 x 219 x 24,
  // 16 -> 8: 14.5 us, 11.2 on the direct-to-LDS kernel, 10 x 159 x 11, 16 -> 336 17.2 and 14.7; 8
  // channels, which that kernel does not take, past two blocks per CU: 18 x 54 x 54, 8 -> 112 17.5 us,
  // 15.3 on the register-staged kernel, but 23 x 73 x 73, 8 -> 16 12.6 and 14.7)
  if (!bt && !any_grid && w <= 95 && cs < 32 && (cs > 8 || tiles > 512)) return none;
  if (!bt && !any_grid && tiles < full && (want.tc > 0 || (cs >= 256 && tiles >= full / 4))) return none;
  if (!bt && !any_grid && w > 63 && cs <= 64 && tiles256 < (cs <= 32 ? 256 : 160)) return none;
  int best = -1;
  for (int i = 0; i < kNumH; ++i) {
    const HInst& c = kH[i];
    if (c.tm != want.tm || c.tn != tn || c.kt != want.kt || c.sb != want.sb || c.tc != want.tc || c.kv != want.kv) continue;
    if (c.hi * 64 < halo_pixels(bm, want.tc, w)) continue;
    if (best < 0 || c.hi < kH[best].hi) best = i;
  }
  if (best < 0) return none;
  return TileCfg{128 * kH[best].tm, 32 * kH[best].tn, best, kVariantHalo};
}

int64_t convhalo_last_pixel(const TileCfg& t, int w) {
  const int tc = kH[t.id].tc;
  return tc > 0 ? (int64_t)(t.bm / tc + 1) * w + tc + 1 : (int64_t)t.bm + 2 * (int64_t)w + 1;
}

hipError_t convhalo_launch(const ConvGemmArgs& a, const TileCfg& t, hipStream_t s, int cls) {
  if (t.variant != kVariantHalo || t.id < 0 || t.id >= kNumH || !convhalo_shape(a)) return hipErrorInvalidValue;
  if (a.pro_kind == kProFwd && (a.bt || a.cs > kProMaxC || a.pro_mean == nullptr)) return hipErrorInvalidValue;
  if (a.pro_kind == kProBwd && (!a.bt || a.cs > kProMaxC || a.pro_y == nullptr || a.pro_dy == nullptr))
    return hipErrorInvalidValue;
  if (a.pro_kind != kProNone && a.pro_kind != kProFwd && a.pro_kind != kProBwd) return hipErrorInvalidValue;
  const HInst& c = kH[t.id];
  if (c.hi * 64 < halo_pixels(t.bm, c.tc, a.ws)) return hipErrorInvalidValue;
  // a two-dimensional tile must divide the image (every tile whole)
  if (c.tc > 0 && (a.ws % c.tc != 0 || a.hs % (t.bm / c.tc) != 0)) return hipErrorInvalidValue;
  trace_begin(cls);
  const hipError_t e = launch_h_id<0>(t.id, a, s);
  trace_end(cls);
  return e;
}

}  // namespace numbat
