// Implicit-GEMM convolution on gfx950 MFMA (bf16 in, fp32 accumulate).
//
// Computes the GEMM family described with ConvGemmArgs: the forward convolution (one
// phase) and all stride phases of a data gradient (one launch, blockIdx.z = phase).
// Kernels:
//  * convdma_kernel, for source channel counts that are multiples of 8 and at least 16 (every
//    layer of the detector but the image input): both operands reach LDS through loads that
//    write LDS directly, in 2 to 4 stages, with 4 or 8 waves split along M or, on tiles of up
//    to 256 x 192 outputs, eight waves in four rows of two;
//  * convgemm_kernel, for any other channel count that is a multiple of 8 (and tiles
//    whose address span exceeds 31 bits): each wave loads its own MFMA A fragments (16
//    contiguous bytes per lane) from global memory into a register ring several steps
//    deep; only the weight tile B, shared by the four waves, goes through LDS;
//  * convstem_kernel, the RGB image layer's forward (3 channels, 3x3, stride 2): a patch's
//    input pixels staged once in LDS;
//  * convnarrow_kernel, forward only, for other inputs of fewer than 8 channels: the
//    reduction (tap, channel) is packed densely and gathered element by element.  Every row keeps a
//    pointer to its source pixel and a bitmask of the taps that land inside the image;
//    padding lanes read a zero constant, so every step issues the same loads and waits
//    are counted exactly.
// (3x3 stride-1 layers have a kernel of their own in conv_halo.hip, small grids with long
// reductions in conv_split.hip.)  All use 32x32x16 MFMAs (the full-rate bf16 form on gfx950)
// and share one epilogue: optional per-tile batch-statistics partials, then fp32 results staged
// through LDS and written as 16-byte vectors of 8 channels (bf16, rounded once, after the
// optional accumulate, and the inference post-op where asked).
#include <cstdlib>

#include "conv_tile.h"

namespace numbat {

namespace {

// Sixteen zero bytes in the code object.  Gather lanes that fall on zero padding (or
// past the end of K or N) load from here instead of being predicated off, so every
// step issues the same number of loads and the compiler can wait for exactly the ring
// slot it needs instead of for every outstanding load.
// (Not const: a const object would live in the constant address space, and a select
// between it and a global pointer would degrade every gather load to a flat load.)
__device__ __attribute__((aligned(16))) u32x4 kZero16 = {0u, 0u, 0u, 0u};

// Four waves split the tile's rows; each wave owns TM*32 rows and all BN columns and
// multiplies with 32x32x16 MFMAs.  A (the gathered operand) is never shared between
// waves, and an MFMA lane's A fragment -- 8 consecutive channels of one pixel at one
// tap -- is 16 contiguous bytes in NHWC, so every wave loads its A fragments straight
// from global memory into a register ring.  Only B (the weights, shared by the four
// waves) is staged through LDS.  One pipeline step covers GK = 32 reduction elements,
// i.e. two MFMA k-slices.
template <int TM, int TN, int D>
__global__ __launch_bounds__(256) void convgemm_kernel(ConvGemmArgs a) {
  using S = GemmShape<TM, TN>;
  constexpr int BM = S::BM, BN = S::BN, BV = S::BV, WTM = S::WTM;
  static_assert(D >= 1 && D <= 4, "prefetch depth 1..4");

  __shared__ __attribute__((aligned(16))) unsigned char smem[S::SMEM];
  __shared__ int32_t s_toff[kMaxTaps];
  __shared__ int64_t s_dst[BM];
  __shared__ float s_red[4][BN];
  __shared__ float s_mean[BN];
  typedef bf16_t BTile[BN][GROW];
  BTile* Bs = reinterpret_cast<BTile*>(smem);

  const TileId T = tile_id(a.remap != 0);
  const GemmPhase& P = a.ph[T.ph];
  const int m0 = T.mt * BM;
  if (m0 >= P.m) return;  // this phase has fewer tiles; uniform exit before any barrier
  const int n0 = T.nt * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;  // MFMA row / column, k group

  if (tid < P.taps) {
    const int off = P.off[tid];
    const int dh = (int)(int16_t)(off & 0xffff), dw = off >> 16;
    s_toff[tid] = (dh * a.ws + dw) * (int)a.src_pix;
  }
  for (int r = tid; r < BM; r += 256) {
    const int m = m0 + r;
    int64_t d = -1;
    if (m < P.m) {
      uint32_t img, gi, gj;
      grid_pos((uint32_t)m, P, img, gi, gj);
      d = (((int64_t)img * a.hd + (int)gi * a.dstep_h + P.doff_h) * a.wd + (int)gj * a.dstep_w + P.doff_w) *
          a.dst_pix;
    }
    s_dst[r] = d;
  }

  // A: this lane's rows (one per 32-row block of the wave) and the taps inside the image
  const bf16_t* rowp[TM];
  uint32_t rmask[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wave * WTM + i * 32 + l32;
    rowp[i] = a.src;
    rmask[i] = 0;
    if (m < P.m) {
      uint32_t img, gi, gj;
      grid_pos((uint32_t)m, P, img, gi, gj);
      const int ih0 = (int)gi * a.gstride_h, iw0 = (int)gj * a.gstride_w;
      rowp[i] = a.src + ((int64_t)img * a.hs * a.ws + (int64_t)ih0 * a.ws + iw0) * a.src_pix;
      uint32_t mk = 0;
      for (int t = 0; t < P.taps; ++t) {
        const int off = P.off[t];
        const int ih = ih0 + (int)(int16_t)(off & 0xffff), iw = iw0 + (off >> 16);
        if ((unsigned)ih < (unsigned)a.hs && (unsigned)iw < (unsigned)a.ws) mk |= 1u << t;
      }
      rmask[i] = mk;
    }
  }
  // B: cooperative rows of the weight tile
  const int cv = tid & 3, rb = tid >> 2;
  const bf16_t* bptr[BV];
  bool bok[BV];
#pragma unroll
  for (int j = 0; j < BV; ++j) {
    const int row = rb + 64 * j;
    const int o = n0 + row;
    bok[j] = row < BN && o < a.nout;
    bptr[j] = P.wt + (int64_t)(bok[j] ? o : 0) * P.ktot + cv * 8;
  }
  // reduction position of this lane's next A fragment: k = slice * 16 + half * 8
  int tapA = (half * 8) / a.cs;
  int cA = half * 8 - tapA * a.cs;
  const int nk = (P.ktot + GK - 1) / GK;
  __syncthreads();

  const bf16_t* zp = reinterpret_cast<const bf16_t*>(&kZero16);
  // ring slot: TM rows x 2 k-slices of A fragments, BV vectors of B
  u32x4 ra[D][2 * TM], rbv[D][BV];
  auto advance = [&]() __attribute__((always_inline)) {
    cA += 16;
    if (a.cs >= 16) {
      if (cA >= a.cs) {
        cA -= a.cs;
        ++tapA;
      }
    } else {
      while (cA >= a.cs) {
        cA -= a.cs;
        ++tapA;
      }
    }
  };
  auto load_a = [&](u32x4 (&xa)[2 * TM]) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bool tok = tapA < P.taps;
      const int toff = s_toff[tok ? tapA : 0] + cA;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const bool ok = tok && ((rmask[i] >> tapA) & 1u);
        xa[ks * TM + i] = *reinterpret_cast<const u32x4*>(ok ? rowp[i] + toff : zp);
      }
      advance();
    }
  };
  auto load_b = [&](int kt, u32x4 (&xb)[BV]) __attribute__((always_inline)) {
    const int kb = kt * GK + cv * 8;
#pragma unroll
    for (int j = 0; j < BV; ++j) {
      const bool ok = bok[j] && kb < P.ktot;
      xb[j] = *reinterpret_cast<const u32x4*>(ok ? bptr[j] + kt * GK : zp);
    }
  };
  auto store_b = [&](int buf, const u32x4 (&xb)[BV]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < BV; ++j)
      if (rb + 64 * j < BN) *reinterpret_cast<u32x4*>(&Bs[buf][rb + 64 * j][cv * 8]) = xb[j];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto compute = [&](int buf, const u32x4 (&xa)[2 * TM]) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      u32x4 bfr[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bfr[j] = *reinterpret_cast<const u32x4*>(&Bs[buf][j * 32 + l32][ks * 16 + half * 8]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(xa[ks * TM + i], bfr[j], acc[i][j]);
    }
  };

  // step kt (ring slot u = kt mod D): stage B(kt+1) in LDS, fetch B(kt+1+D), multiply
  // A(kt) with B(kt), then fetch A(kt+D) into the slot just consumed.
  auto step = [&](auto uc, int kt) __attribute__((always_inline)) {
    constexpr int u = decltype(uc)::value;
    constexpr int nxt = (u + 1) % D;
    store_b((kt + 1) & 1, rbv[nxt]);
    load_b(kt + 1 + D, rbv[nxt]);
    compute(kt & 1, ra[u]);
    load_a(ra[u]);
    __syncthreads();
  };
  auto prologue = [&](auto dc) __attribute__((always_inline)) {
    constexpr int d = decltype(dc)::value;
    load_a(ra[d]);
    load_b(d, rbv[d]);
  };

  // Loads past the end of K read zeros, so every load is issued unconditionally.
  if (nk > 0) {
    prologue(Ic<0>{});
    if constexpr (D > 1) prologue(Ic<1>{});
    if constexpr (D > 2) prologue(Ic<2>{});
    if constexpr (D > 3) prologue(Ic<3>{});
    store_b(0, rbv[0]);
    load_b(D, rbv[0]);
    __syncthreads();
  }
  for (int kb = 0; kb < nk; kb += D) {
    step(Ic<0>{}, kb);
    if constexpr (D > 1) {
      if (kb + 1 < nk) step(Ic<1 % D>{}, kb + 1);
    }
    if constexpr (D > 2) {
      if (kb + 2 < nk) step(Ic<2 % D>{}, kb + 2);
    }
    if constexpr (D > 3) {
      if (kb + 3 < nk) step(Ic<3 % D>{}, kb + 3);
    }
  }

  gemm_epilogue<TM, TN>(a, P, T, acc, m0, n0, smem, s_dst, s_red, s_mean);
}

// ---------------------------------------------------------------------------
// Fast path for source channel counts that are multiples of 8 and at least 16 (every layer
// of the detector except the 3-channel image).
//
// Both operands are staged through LDS and the gathered operand is loaded coalesced: a
// thread always loads the same 16-byte chunk (8 channels) of the step's reduction
// elements, and the threads with the same row cover the row's contiguous bytes, so one
// wave instruction reads whole rows -- 8 or 16 of them.  (Gathering MFMA fragments
// straight from global memory reads 32 rows per instruction; the L1 path's cost grows
// with the rows, not the bytes, an instruction touches, and that design stalled on it.)
//
// Loads are raw buffer loads.  The gather base sits halo_px pixels before the first
// image of the tile, so every in-image address is a non-negative 32-bit offset: row
// offset (fixed for the whole reduction) + the thread's tap-and-channel offset.  A tap
// outside the image swaps the offset for one past the buffer's range, which the hardware
// answers with zeros; so does a weight row past nout or a reduction index past ktot.
// Each thread walks its own reduction position (tap, channel) with adds and selects:
// 8-multiple channel counts never split a chunk between taps, and with 32 or more channels a
// step of up to 64 elements (with 16 or more, of 32) crosses at most two tap boundaries.
// ---------------------------------------------------------------------------
// Direct-to-LDS variant of the staged fast path.  The loads of both operands write LDS
// themselves (buffer_load ... lds: lane i of a wave instruction deposits its 16 bytes
// at the instruction's LDS base + 16*i), so a pipeline step costs no VGPR staging and no
// LDS store instructions, and the prefetch depth lives in LDS stages instead of a
// register ring.  A stage holds BK reduction elements (64 or 32) of every row, in
// unpadded rows of 2*BK bytes; a wave instruction fills 1 KiB of consecutive rows.
// Bank conflicts on the 16-byte fragment reads (16 lanes, 16 rows, one 256-byte bank
// window) are avoided by storing 16-byte chunk k of row r in slot k ^ ((r / W) % C),
// with W rows per bank window and C chunks per row: rows sharing a window differ in
// their byte offset, rows of different windows in their slot.  A load lane picks the
// chunk its fixed LDS slot needs, so the swizzle costs nothing per step.
//
// Stage s of each operand is its own LDS object, so the compiler can tell the stages
// apart when it counts the loads an LDS read must wait for; every step issues the same
// loads (past the end of K they read zeros), and a step begins with a wait for its own
// loads (the later stages stay in flight) and a barrier, after which the stage it frees
// is refilled before its multiply.
template <int TM, int TN, int S, int BK, int NW, int WN, bool BT>
struct DmaShape {
  using G = GemmShape<TM, TN, NW, WN>;
  static constexpr int ROWB = 2 * BK;               // bytes per LDS row
  static constexpr int CPR = BK / 8;                // 16-byte chunks per row
  static constexpr int RPI = 1024 / ROWB;           // rows per wave load instruction
  static constexpr int WIN = 256 / ROWB;            // rows per 256-byte bank window
  static constexpr int AI = G::BM / RPI / NW;       // A load instructions per wave per step
  // B load instructions per step (all waves): BN rows of BK elements, or (transposed B)
  // BK rows of BN elements
  static constexpr int BI = BT ? BK * G::BN * 2 / 1024 : (G::BN + RPI - 1) / RPI;
  static constexpr int BI_MIN = BI / NW;                 // ... issued by every wave
  static constexpr int BI_MAX = (BI + NW - 1) / NW;      // ... issued by the first waves
  static constexpr int A_ELEMS = G::BM * BK, B_ELEMS = BI * 512;
  // stage 0 of A doubles as the epilogue's staging area
  static constexpr int A0_ELEMS = 2 * A_ELEMS >= G::STAGE_BYTES ? A_ELEMS : G::STAGE_BYTES / 2;
  // loads still in flight when a step's own are done (every wave issues at least
  // AI + BI_MIN loads per step; a wave that issues more waits a little longer)
  static constexpr int PENDING = (S - 2) * (AI + BI_MIN);
  static_assert(G::BM % (NW * RPI) == 0, "A rows per step split evenly over the waves");
};

template <int TM, int TN, int S, int BK, int NW, int WN, bool BT>
__global__ __launch_bounds__(NW * 64) void convdma_kernel(ConvGemmArgs a) {
  using G = GemmShape<TM, TN, NW, WN>;
  using Sh = DmaShape<TM, TN, S, BK, NW, WN, BT>;
  constexpr int BM = G::BM, BN = G::BN, WTM = G::WTM;
  constexpr int AI = Sh::AI, BI = Sh::BI, BI_MAX = Sh::BI_MAX, RPI = Sh::RPI, CPR = Sh::CPR, WIN = Sh::WIN;
  static_assert(S >= 2 && S <= 4, "2..4 LDS stages");
  static_assert(BK == 32 || BK == 64, "stage depth");
  static_assert(Sh::PENDING <= 63, "load counter range");
  static_assert(NW == 4 || NW == 8, "4 or 8 waves");

  __shared__ __attribute__((aligned(16))) bf16_t sA0[Sh::A0_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sA1[Sh::A_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sA2[Sh::A_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sA3[Sh::A_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sB0[Sh::B_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sB1[Sh::B_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sB2[Sh::B_ELEMS];
  __shared__ __attribute__((aligned(16))) bf16_t sB3[Sh::B_ELEMS];
  __shared__ int64_t s_dst[BM];
  __shared__ float s_red[G::WM][BN];
  __shared__ float s_mean[BN];
  auto stage_a = [&](auto sc) __attribute__((always_inline)) -> bf16_t* {
    constexpr int s = decltype(sc)::value;
    if constexpr (s == 0) return sA0;
    else if constexpr (s == 1) return sA1;
    else if constexpr (s == 2) return sA2;
    else return sA3;
  };
  auto stage_b = [&](auto sc) __attribute__((always_inline)) -> bf16_t* {
    constexpr int s = decltype(sc)::value;
    if constexpr (s == 0) return sB0;
    else if constexpr (s == 1) return sB1;
    else if constexpr (s == 2) return sB2;
    else return sB3;
  };

  // (launch order: the XCD-aware order measured no faster for these GEMMs; a constant
  // keeps the block's first loads from waiting on a kernel argument)
  const TileId T = tile_id(false);
  const GemmPhase& P = a.ph[T.ph];
  const Geo Ge = load_geo(P);
  {
    // every kernel argument the prologue needs, loaded at once and completed before the
    // early-exit test (otherwise the compiler splits them into dependent rounds after it)
    const bf16_t* src = a.src;
    const bf16_t* wt = P.wt;
    const int64_t spx = a.src_pix;
    const int hs = a.hs, ws = a.ws, cs = a.cs, nout = a.nout, halo = a.halo_px, gsh = a.gstride_h,
              gsw = a.gstride_w, kt = P.ktot, tw = P.tw, t0 = P.toff0, cst = P.cstep, rst = P.rstep;
    asm volatile("" ::"s"(src), "s"(wt), "s"(spx), "s"(hs), "s"(ws), "s"(cs), "s"(nout), "s"(halo), "s"(gsh),
                 "s"(gsw), "s"(kt), "s"(tw), "s"(t0), "s"(cst), "s"(rst), "s"(Ge.m), "s"(Ge.gh), "s"(Ge.gw),
                 "s"(Ge.th), "s"(Ge.dh0), "s"(Ge.dw0), "s"(Ge.tsh), "s"(Ge.tsw), "s"(Ge.div_gw.mul),
                 "s"(Ge.div_gw.shift), "s"(Ge.div_ghw.mul), "s"(Ge.div_ghw.shift));
  }
  const int m0 = T.mt * BM;
  if (m0 >= Ge.m) return;  // this phase has fewer tiles; uniform exit before any barrier
  const int n0 = T.nt * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  // Load instruction q of this wave fills rows (NW*q + wave)*RPI .. +RPI; the lane's LDS
  // slot is lane % CPR of row lane / CPR in it, which holds chunk slot ^ ((row / WIN) % CPR)
  // (the same for every q)
  const int lrow = lane / CPR;
  const int kc = (lane % CPR) ^ (((wave * RPI + lrow) / WIN) % CPR);

  const uint32_t img0 = fdiv((uint32_t)m0, Ge.div_ghw);
  const __amdgpu_buffer_rsrc_t rsA =
      buffer_rsrc(a.src + ((int64_t)img0 * a.hs * a.ws - a.halo_px) * a.src_pix);
  uint32_t vrow[AI], vmask[AI];  // the rows this thread loads
#pragma unroll
  for (int q = 0; q < AI; ++q) row_gather(a, Ge, m0 + (NW * q + wave) * RPI + lrow, img0, vrow[q], vmask[q]);
  const __amdgpu_buffer_rsrc_t rsB = buffer_rsrc(P.wt);
  const int p_tw = P.tw, p_ktot = P.ktot, p_taps = P.taps, cs = a.cs;
  const uint32_t p_cstep = (uint32_t)P.cstep, p_rstep = (uint32_t)P.rstep;
  uint32_t voffb[BI_MAX];
  // transposed B (OHWI weights read in place): instruction j of this lane covers stage row
  // brw[j] (reduction index kb + brw[j] = (tap, o)), 16-byte column chunk bch[j]; the
  // walk keeps o, the tap's grid column and the byte offset of (o, tap) per instruction
  int bo[BT ? BI_MAX : 1], btap[BT ? BI_MAX : 1], btc[BT ? BI_MAX : 1];
  const uint32_t w_ostep = (uint32_t)P.wostep, w_cstep = (uint32_t)P.wcstep, w_rstep = (uint32_t)P.wrstep;
  if constexpr (!BT) {
#pragma unroll
    for (int j = 0; j < BI_MAX; ++j) {
      const int row = (NW * j + wave) * RPI + lrow, o = n0 + row;
      voffb[j] = (row < BN && o < a.nout) ? (uint32_t)(((int64_t)o * p_ktot + kc * 8) * 2) : kOob;
    }
  } else {
#pragma unroll
    for (int j = 0; j < BI_MAX; ++j) {
      const int byte = (NW * j + wave) * 1024 + lane * 16;
      const int row = byte / (2 * BN), slot = (byte % (2 * BN)) / 16;
      const int chunk = slot ^ bt_swizzle<BN>(row);
      const bool colok = n0 + chunk * 8 < a.nout;
      // reduction index row = tap * cs + o (row < BK <= 2 * cs: at most two wraps)
      int o = row, tp = 0, tc = 0;
      uint32_t off = (uint32_t)P.wtoff0 + (uint32_t)((n0 + chunk * 8) * 2);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const bool wrap = o >= cs;
        o = wrap ? o - cs : o;
        tp += wrap ? 1 : 0;
        tc += wrap ? 1 : 0;
        const bool rw = tc == p_tw;
        tc = rw ? 0 : tc;
        off += wrap ? (rw ? w_rstep : w_cstep) : 0u;
      }
      bo[j] = o;
      btap[j] = colok ? tp : 31;  // a chunk past nout never loads
      btc[j] = tc;
      voffb[j] = off;
    }
  }
  int ch = kc * 8, tap = 0, tcol = 0;
  uint32_t toff = (uint32_t)P.toff0;
  auto wrap_taps = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const bool wrap = ch >= cs;
      ch = wrap ? ch - cs : ch;
      tap += wrap ? 1 : 0;
      tcol += wrap ? 1 : 0;
      const bool rw = tcol == p_tw;
      tcol = rw ? 0 : tcol;
      toff += wrap ? (rw ? p_rstep : p_cstep) : 0u;
    }
  };
  wrap_taps();
  const int nk = (p_ktot + BK - 1) / BK;

  // issue the loads of step kt into stage s; the A walk advances by one step
  auto issue = [&](auto sc, int kt) __attribute__((always_inline)) {
    bf16_t* A = stage_a(sc);
    bf16_t* B = stage_b(sc);
    const uint32_t lo = toff + 2u * (uint32_t)ch;
    const int tq = tap < 31 ? tap : 31;  // past the last tap: bit 31 is clear
#pragma unroll
    for (int q = 0; q < AI; ++q) {
      const uint32_t t = (uint32_t)__builtin_amdgcn_sbfe((int)vmask[q], tq, 1);
      const uint32_t vo = (t & (vrow[q] + lo)) | (~t & kOob);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void_t*)(A + (NW * q + wave) * RPI * BK), 16, vo, 0, 0, 0);
    }
    if constexpr (!BT) {
      const int kb = kt * BK;
      const bool kin = kb + kc * 8 < p_ktot;
#pragma unroll
      for (int j = 0; j < BI_MAX; ++j) {
        if (NW * j + wave < BI) {  // wave-uniform
          // (the select stays out of the builtin's argument list: written inline, the host
          // pass drops the kernel's launch stub)
          const uint32_t vb = kin ? voffb[j] : kOob;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_void_t*)(B + (NW * j + wave) * 512), 16, vb,
                                                   (uint32_t)kb * 2, 0, 0);
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < BI_MAX; ++j) {
        if (NW * j + wave < BI) {  // wave-uniform
          const uint32_t vb = btap[j] < p_taps ? voffb[j] + (uint32_t)bo[j] * w_ostep : kOob;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_void_t*)(B + (NW * j + wave) * 512), 16, vb, 0, 0, 0);
          // next step: o advances by BK, wrapping into later taps
          int o = bo[j] + BK, tp = btap[j], tc = btc[j];
          uint32_t off = voffb[j];
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            const bool wrap = o >= cs;
            o = wrap ? o - cs : o;
            tp += wrap ? 1 : 0;
            tc += wrap ? 1 : 0;
            const bool rw = tc == p_tw;
            tc = rw ? 0 : tc;
            off += wrap ? (rw ? w_rstep : w_cstep) : 0u;
          }
          bo[j] = o;
          btap[j] = tp;
          btc[j] = tc;
          voffb[j] = off;
        }
      }
    }
    ch += BK;
    wrap_taps();
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment byte offsets: row (wave rows + l32) of A, l32 of B; k-slice ks sits in chunk
  // 2*ks + half, stored in slot (2*ks + half) ^ ((l32 / WIN) % CPR)
  const int sw = (l32 / WIN) % CPR;
  const int wm = wave / WN, wn = wave % WN;  // the wave's place in the tile
  const uint32_t arow = (uint32_t)(wm * WTM + l32) * (BK * 2), brow = (uint32_t)(wn * G::WTN + l32) * (BK * 2);
  uint32_t koff[BK / 16];
#pragma unroll
  for (int ks = 0; ks < BK / 16; ++ks) koff[ks] = (uint32_t)(((2 * ks + half) ^ sw) * 16);
  // transposed B: lane l = 16 g + 4 e + q reads 4 columns (8 bytes) of rows 8 (g / 2) + e
  // and that + 4 of the 16-row slice, columns 32 j + 16 (g % 2) + 4 q ..; the read hands
  // each lane 4 consecutive rows of one column, two reads make its fragment
  uint32_t btoff[BT ? TN : 1];
  if constexpr (BT) {
    const int g = lane >> 4, e = (lane & 15) >> 2, q = lane & 3;
    const int r0 = 8 * (g >> 1) + e;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = 4 * (wn * TN + j) + 2 * (g & 1) + (q >> 1);
      btoff[j] = (uint32_t)(r0 * 2 * BN + (c ^ bt_swizzle<BN>(r0)) * 16 + (q & 1) * 8);
    }
  }
  auto compute = [&](auto sc) __attribute__((always_inline)) {
    const unsigned char* A = reinterpret_cast<const unsigned char*>(stage_a(sc));
    const unsigned char* B = reinterpret_cast<const unsigned char*>(stage_b(sc));
    u32x4 af[2][TM], bf[2][TN];
    auto rd = [&](int ks, u32x4 (&xa)[TM], u32x4 (&xb)[TN]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i) xa[i] = *reinterpret_cast<const u32x4*>(A + arow + i * 32 * BK * 2 + koff[ks]);
      if constexpr (!BT) {
#pragma unroll
        for (int j = 0; j < TN; ++j) xb[j] = *reinterpret_cast<const u32x4*>(B + brow + j * 32 * BK * 2 + koff[ks]);
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const unsigned char* pb = B + btoff[j] + ks * 16 * 2 * BN;
          const v4s_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)pb);
          const v4s_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)(pb + 4 * 2 * BN));
          const v2u_t lo = __builtin_bit_cast(v2u_t, r0), hi = __builtin_bit_cast(v2u_t, r1);
          xb[j][0] = lo.x;
          xb[j][1] = lo.y;
          xb[j][2] = hi.x;
          xb[j][3] = hi.y;
        }
      }
    };
    rd(0, af[0], bf[0]);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      if (ks + 1 < BK / 16) rd(ks + 1, af[(ks + 1) & 1], bf[(ks + 1) & 1]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(af[ks & 1][i], bf[ks & 1][j], acc[i][j]);
    }
  };
  // this wave's loads of the current step are done (the later stages' stay in flight),
  // then every wave's: the stage is complete in LDS and the stage read last step is free
  auto sync = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(Sh::PENDING) : "memory");
  };
  // step kt reads stage u = kt mod S and refills stage (kt - 1) mod S with step kt + S - 1
  auto step = [&](auto uc, int kt) __attribute__((always_inline)) {
    constexpr int u = decltype(uc)::value;
    sync();
    issue(Ic<(u + S - 1) % S>{}, kt + S - 1);
    compute(uc);
  };
  if (nk > 0) static_for_ic<0, S - 1>([&](auto ic) { issue(ic, decltype(ic)::value); });
  // destination offsets of the tile's rows, needed only by the epilogue: computed while
  // the first stages load (the first step's barrier publishes them)
  for (int r = tid; r < BM; r += NW * 64) s_dst[r] = dst_offset(a, Ge, m0 + r);
  int kb = 0;
  for (; kb + S <= nk; kb += S) static_for_ic<0, S>([&](auto ic) { step(ic, kb + decltype(ic)::value); });
  static_for_ic<0, S - 1>([&](auto ic) {
    if (kb + decltype(ic)::value < nk) step(ic, kb + decltype(ic)::value);
  });
  // the loads issued past the last step land in LDS before stage 0 becomes staging space
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  gemm_epilogue<TM, TN, NW, WN>(a, P, T, acc, m0, n0, reinterpret_cast<unsigned char*>(sA0), s_dst, s_red, s_mean);
}

// ---------------------------------------------------------------------------
// Forward convolution of a narrow input (fewer than 8 channels: the RGB image).  The
// reduction k = (tap, channel) is packed densely (K = taps * ci, e.g. 27, padded to a
// multiple of 16), so an MFMA A fragment -- 8 consecutive k of one output pixel -- is
// gathered element by element: a per-k table in LDS holds each k's offset from the
// pixel's anchor and its tap, and a tap outside the image reads a zero.  The weights
// (OHWI is already [o][k]) sit in LDS for the whole block.  One pass over K, then the
// shared epilogue (statistics partials, 16-byte output vectors).
template <int TM, int TN>
struct NarrowShape {
  using G = GemmShape<TM, TN>;
  static constexpr int KMAX = ((kMaxTaps * 7 + 15) / 16) * 16;  // 176
  static constexpr int BROW = KMAX + 8;                           // bf16 per weight row (odd multiple of 16 bytes)
  static constexpr int B_BYTES = G::BN * BROW * 2;
  static constexpr int SM = B_BYTES > G::STAGE_BYTES ? B_BYTES : G::STAGE_BYTES;
};

template <int TM, int TN>
__global__ __launch_bounds__(256) void convnarrow_kernel(ConvGemmArgs a) {
  using G = GemmShape<TM, TN>;
  using Sh = NarrowShape<TM, TN>;
  constexpr int BM = G::BM, BN = G::BN, WTM = G::WTM, BROW = Sh::BROW;
  __shared__ __attribute__((aligned(16))) unsigned char smem[Sh::SM];
  __shared__ int32_t s_koff[Sh::KMAX];  // element offset of k from the pixel's anchor
  __shared__ int32_t s_ktap[Sh::KMAX];  // tap of k (31 past K: bit 31 of a tap mask is clear)
  __shared__ int64_t s_dst[BM];
  __shared__ float s_red[4][BN];
  __shared__ float s_mean[BN];
  bf16_t* Bs = reinterpret_cast<bf16_t*>(smem);

  const TileId T{(int)blockIdx.x, (int)blockIdx.y, 0};
  const GemmPhase& P = a.ph[0];
  const int m0 = T.mt * BM, n0 = T.nt * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int ktot = P.ktot, nks = (ktot + 15) / 16, kp = nks * 16;

  for (int k = tid; k < kp; k += 256) {
    int off = 0, tap = 31;
    if (k < ktot) {
      tap = k / a.cs;
      const int c = k - tap * a.cs;
      const int o = P.off[tap];
      off = (int)(((int16_t)(o & 0xffff) * a.ws + (o >> 16)) * a.src_pix) + c;
    }
    s_koff[k] = off;
    s_ktap[k] = tap;
  }
  for (int e = tid; e < BN * kp; e += 256) {
    const int r = e / kp, k = e - r * kp, o = n0 + r;
    Bs[r * BROW + k] = (o < a.nout && k < ktot) ? P.wt[(int64_t)o * ktot + k] : (bf16_t)0;
  }
  for (int r = tid; r < BM; r += 256) {
    const int m = m0 + r;
    int64_t d = -1;
    if (m < P.m) {
      uint32_t img, gi, gj;
      grid_pos((uint32_t)m, P, img, gi, gj);
      d = (((int64_t)img * a.hd + (int)gi * a.dstep_h + P.doff_h) * a.wd + (int)gj * a.dstep_w + P.doff_w) *
          a.dst_pix;
    }
    s_dst[r] = d;
  }
  // this lane's rows: anchor element (the tap (0, 0) pixel before padding) and the taps
  // inside the image
  const bf16_t* rowp[TM];
  uint32_t rmask[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wave * WTM + i * 32 + l32;
    rowp[i] = a.src;
    rmask[i] = 0;
    if (m < P.m) {
      uint32_t img, gi, gj;
      grid_pos((uint32_t)m, P, img, gi, gj);
      const int ih0 = (int)gi * a.gstride_h, iw0 = (int)gj * a.gstride_w;
      rowp[i] = a.src + ((int64_t)img * a.hs * a.ws + (int64_t)ih0 * a.ws + iw0) * a.src_pix;
      uint32_t mk = 0;
      for (int t = 0; t < P.taps; ++t) {
        const int off = P.off[t];
        const int ih = ih0 + (int)(int16_t)(off & 0xffff), iw = iw0 + (off >> 16);
        if ((unsigned)ih < (unsigned)a.hs && (unsigned)iw < (unsigned)a.ws) mk |= 1u << t;
      }
      rmask[i] = mk;
    }
  }
  __syncthreads();

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const bf16_t* zp = reinterpret_cast<const bf16_t*>(&kZero16);
  for (int ks = 0; ks < nks; ++ks) {
    const int kb = ks * 16 + half * 8;
    int koff[8];
    uint32_t ktap[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      koff[e] = s_koff[kb + e];
      ktap[e] = (uint32_t)s_ktap[kb + e];
    }
    u32x4 af[TM], bf[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      uint32_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool ok = (rmask[i] >> ktap[e]) & 1u;
        h[e] = (uint32_t)*(ok ? rowp[i] + koff[e] : zp);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) af[i][q] = h[2 * q] | (h[2 * q + 1] << 16);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[j] = *reinterpret_cast<const u32x4*>(&Bs[(j * 32 + l32) * BROW + kb]);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(af[i], bf[j], acc[i][j]);
  }
  gemm_epilogue<TM, TN>(a, P, T, acc, m0, n0, smem, s_dst, s_red, s_mean);
}

// ---------------------------------------------------------------------------
// Forward convolution of the RGB image layer (3 channels, 3x3, stride 2, padding 1;
// output rows a multiple of 4 and columns of 64): a block computes a 4 x 64 patch of
// output pixels.  The 9 x 129 input pixels it reads are loaded once into LDS, each
// padded to 4 channels (8 bytes, the fourth zero), and the reduction is ordered as
// k = 16 r + 4 s + c (tap row r, tap column s, channel c; zero weights at c = 3 and
// past s = 2), so the 8 consecutive k of an MFMA fragment are 16 aligned bytes of one
// input row (s = 0, 1), or 8 bytes (s = 2) and four zeros.  Wave w owns output row w of
// the patch.  The weights, as [o][k], stay in LDS; then the shared epilogue.
constexpr int kStemCols = 129, kStemPitch = 130;  // input pixels per patch row, LDS pitch (pixels)
constexpr int kStemKp = 56;                       // bf16 per weight row (48 + 8)

__global__ __launch_bounds__(256) void convstem_kernel(ConvGemmArgs a) {
  using G = GemmShape<2, 2>;
  constexpr int BN = G::BN;
  constexpr int PATCH = 9 * kStemPitch * 8;  // bytes
  constexpr int SM = PATCH > G::STAGE_BYTES ? PATCH : G::STAGE_BYTES;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SM];
  __shared__ __attribute__((aligned(16))) bf16_t s_w[BN * kStemKp];
  __shared__ int64_t s_dst[256];
  __shared__ float s_red[4][BN];
  __shared__ float s_mean[BN];
  const GemmPhase& P = a.ph[0];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  // tile: blockIdx.x = patch column, blockIdx.y = patch row, blockIdx.z = image
  const int oj0 = blockIdx.x * 64, oi0 = blockIdx.y * 4, img = blockIdx.z;
  const int ntc = P.gw >> 6, ntr = P.gh >> 2;
  const TileId T{(int)((img * ntr + blockIdx.y) * ntc + blockIdx.x), 0, 0};
  const int m0 = T.mt * 256;

  // input patch: rows 2 oi0 - 1 + pr, columns 2 oj0 - 1 + pc; all loads first
  constexpr int kPix = 9 * kStemCols, kRounds = (kPix + 255) / 256;
  uint32_t lo[kRounds], hi[kRounds];
#pragma unroll
  for (int u = 0; u < kRounds; ++u) {
    const int e = tid + 256 * u;
    const int pr = e / kStemCols, pc = e - pr * kStemCols;
    const int ih = 2 * oi0 - 1 + pr, iw = 2 * oj0 - 1 + pc;
    lo[u] = hi[u] = 0u;
    if (e < kPix && (unsigned)ih < (unsigned)a.hs && (unsigned)iw < (unsigned)a.ws) {
      const bf16_t* px = a.src + (((int64_t)img * a.hs + ih) * a.ws + iw) * a.src_pix;
      lo[u] = (uint32_t)px[0] | ((uint32_t)px[1] << 16);
      hi[u] = (uint32_t)px[2];
    }
  }
  // weights [o][k = 16 r + 4 s + c] from OHWI [o][r][s][c]: zeros first, then the
  // tensor read contiguously (2-byte elements, loads issued before the stores)
  for (int e = tid; e < BN * kStemKp / 2; e += 256) reinterpret_cast<uint32_t*>(s_w)[e] = 0u;
  constexpr int kWRounds = 64 * 27 / 256 + 1;
  bf16_t wv[kWRounds];
  const int nwt = a.nout * 27;
#pragma unroll
  for (int u = 0; u < kWRounds; ++u) {
    const int e = tid + 256 * u;
    wv[u] = e < nwt ? P.wt[e] : (bf16_t)0;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kWRounds; ++u) {
    const int e = tid + 256 * u;
    if (e < nwt) {
      const int o = e / 27, k = e - o * 27;
      const int r = k / 9, sc = k - r * 9, s = sc / 3, c = sc - s * 3;
      s_w[o * kStemKp + r * 16 + s * 4 + c] = wv[u];
    }
  }
  for (int r = tid; r < 256; r += 256) {
    const int oi = oi0 + (r >> 6), oj = oj0 + (r & 63);
    s_dst[r] = (((int64_t)img * a.hd + oi) * a.wd + oj) * a.dst_pix;
  }
#pragma unroll
  for (int u = 0; u < kRounds; ++u) {
    const int e = tid + 256 * u;
    if (e < kPix) {
      const int pr = e / kStemCols, pc = e - pr * kStemCols;
      *reinterpret_cast<uint2*>(smem + (pr * kStemPitch + pc) * 8) = make_uint2(lo[u], hi[u]);
    }
  }
  __syncthreads();

  // A fragment of output pixel (row wave, column 32 i + l32), tap row ks: input patch row
  // 2 wave + ks, columns 2 oj + half * 2 (16 bytes: s = 0, 1) or + 2 (8 bytes: s = 2)
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 3; ++ks) {
    u32x4 af[2], bf[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned char* px = smem + ((2 * wave + ks) * kStemPitch + 2 * (32 * i + l32)) * 8;
      if (half == 0) {
        af[i] = *reinterpret_cast<const u32x4*>(px);
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(px + 16);
        af[i] = u32x4{v.x, v.y, 0u, 0u};
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) bf[j] = *reinterpret_cast<const u32x4*>(&s_w[(j * 32 + l32) * kStemKp + ks * 16 + half * 8]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma32x32x16(af[i], bf[j], acc[i][j]);
  }
  gemm_epilogue<2, 2>(a, P, T, acc, m0, 0, smem, s_dst, s_red, s_mean);
}

template <int TN>
hipError_t launch_narrow(const ConvGemmArgs& a, hipStream_t s) {
  using G = GemmShape<2, TN>;
  dim3 grid((unsigned)((a.ph[0].m + G::BM - 1) / G::BM), (unsigned)((a.nout + G::BN - 1) / G::BN), 1);
  NUMBAT_LAUNCH((convnarrow_kernel<2, TN>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

struct GInst {
  int tm, tn, d;  // 32-row tiles per wave (4 waves along M), 32-col tiles, prefetch depth (generic kernel)
};
constexpr GInst kG[] = {
    {2, 4, 2},  // 0: 256 x 128
    {2, 3, 3},  // 1: 256 x 96
    {2, 2, 4},  // 2: 256 x 64
    {2, 1, 4},  // 3: 256 x 32
    {1, 4, 3},  // 4: 128 x 128
    {1, 3, 4},  // 5: 128 x 96
    {1, 2, 4},  // 6: 128 x 64
    {1, 1, 4},  // 7: 128 x 32
};


template <int TM, int TN, int S, int BK, int NW, int WN = 1>
void launch_dma(const ConvGemmArgs& a, int mmax, hipStream_t s) {
  using Sh = GemmShape<TM, TN, NW, WN>;
  dim3 grid((unsigned)((mmax + Sh::BM - 1) / Sh::BM), (unsigned)((a.nout + Sh::BN - 1) / Sh::BN), (unsigned)a.nphase);
  if (a.bt)
    NUMBAT_LAUNCH((convdma_kernel<TM, TN, S, BK, NW, WN, true>), grid, dim3(NW * 64), 0, s, a);
  else
    NUMBAT_LAUNCH((convdma_kernel<TM, TN, S, BK, NW, WN, false>), grid, dim3(NW * 64), 0, s, a);
}

template <int I>
hipError_t launch_g(const ConvGemmArgs& a, int variant, hipStream_t s) {
  constexpr GInst c = kG[I];
  using Sh = GemmShape<c.tm, c.tn>;
  int mmax = 0;
  for (int p = 0; p < a.nphase; ++p) mmax = a.ph[p].m > mmax ? a.ph[p].m : mmax;
  if (variant == kVariantDma3)
    launch_dma<c.tm, c.tn, 3, 64, 4>(a, mmax, s);
  else if (variant == kVariantDma2)
    launch_dma<c.tm, c.tn, 2, 64, 4>(a, mmax, s);
  else if (variant == kVariantDma32)
    launch_dma<c.tm, c.tn, 3, 32, 4>(a, mmax, s);
  else if (variant == kVariantDma3W8 && c.tn <= 4)
    launch_dma<1, c.tn <= 4 ? c.tn : 4, 3, 64, 8>(a, mmax, s);
  else {
    dim3 grid((unsigned)((mmax + Sh::BM - 1) / Sh::BM), (unsigned)((a.nout + Sh::BN - 1) / Sh::BN),
              (unsigned)a.nphase);
    NUMBAT_LAUNCH((convgemm_kernel<c.tm, c.tn, c.d>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

int tap_dh(int32_t off) { return (int)(int16_t)(off & 0xffff); }
int tap_dw(int32_t off) { return off >> 16; }

// Source channels the direct-to-LDS kernel takes: multiples of 8 (a lane's 16-byte chunk never
// splits a tap) of which a step crosses at most two taps (at least 16 channels for 32-deep
// steps, 32 for 64-deep ones).
bool dma_channels(int cs, int variant) { return cs % 8 == 0 && cs >= (variant == kVariantDma32 ? 16 : 32); }

// Fills in the tap walk of the fast path (tw, toff0, cstep, rstep, halo_px) and reports
// whether the fast path applies: the kernel's channel counts, taps forming a grid with
// unit steps, and every gathered byte of a tile within 32-bit buffer offsets.
bool prepare_fast(ConvGemmArgs& a, const TileCfg& t) {
  return dma_channels(a.cs, t.variant) && convgemm_taps(a, t.bm);
}

}  // namespace

bool convgemm_taps(ConvGemmArgs& a, int bm) {
  const int64_t pix2 = a.src_pix * 2;
  int halo = 0;
  for (int p = 0; p < a.nphase; ++p) {
    const GemmPhase& P = a.ph[p];
    for (int t = 0; t < P.taps; ++t) {
      const int lin = tap_dh(P.off[t]) * a.ws + tap_dw(P.off[t]);
      halo = -lin > halo ? -lin : halo;
    }
  }
  a.halo_px = halo;
  int64_t worst = 0;
  for (int p = 0; p < a.nphase; ++p) {
    GemmPhase& P = a.ph[p];
    int tw = 1;
    while (tw < P.taps && tap_dh(P.off[tw]) == tap_dh(P.off[0])) ++tw;
    if (P.taps % tw != 0) return false;
    const int sw = tw > 1 ? tap_dw(P.off[1]) - tap_dw(P.off[0]) : 0;
    const int sh = P.taps > tw ? tap_dh(P.off[tw]) - tap_dh(P.off[0]) : 0;
    int64_t maxlin = 0;
    for (int t = 0; t < P.taps; ++t) {
      const int i = t / tw, j = t % tw;
      if (tap_dh(P.off[t]) != tap_dh(P.off[0]) + i * sh || tap_dw(P.off[t]) != tap_dw(P.off[0]) + j * sw) return false;
      const int64_t lin = (int64_t)tap_dh(P.off[t]) * a.ws + tap_dw(P.off[t]) + halo;
      maxlin = lin > maxlin ? lin : maxlin;
    }
    if ((int64_t)a.nout * P.ktot * 2 >= (int64_t)kRecords) return false;  // weight offsets are 32-bit too
    P.tw = tw;
    P.th = P.taps / tw;
    P.dh0 = tap_dh(P.off[0]);
    P.dw0 = tap_dw(P.off[0]);
    P.tsh = sh;
    P.tsw = sw;
    P.toff0 = (int32_t)(((int64_t)tap_dh(P.off[0]) * a.ws + tap_dw(P.off[0]) + halo) * pix2);
    P.cstep = (int32_t)((int64_t)sw * pix2);
    P.rstep = (int32_t)(((int64_t)sh * a.ws - (int64_t)(tw - 1) * sw) * pix2);
    // a tile's rows span at most bm / (gh*gw) + 2 images
    const int64_t imgs = bm / ((int64_t)P.gh * P.gw) + 2;
    const int64_t span = (imgs * a.hs * a.ws + halo + maxlin) * pix2 + (int64_t)a.cs * 2 + 16;
    worst = span > worst ? span : worst;
  }
  return worst < (int64_t)kOob - (1 << 24);
}

// Eight-wave tiles whose waves stand in four rows of two: a wave's share of a 256 x 192 tile is
// 64 x 96 (5 LDS fragments per 6 products), and a CU loads 448 rows per 49152 products where 128
// x 64 tiles load 192 per 8192.  Latency still bounds it (the matrix cores are busy a quarter of
// the time: 35% of the waves' cycles wait for loads, 34% at the barrier or to issue), but less: 160 x
// 160 stride 2, 96 -> 192 19 -> 25% busy.  One block per CU, so the grid has to fill whole rounds
// of 256 blocks: the tile is taken where the GEMM's own area is at least a share `eff` of the
// rounds' area and nout fills its columns to 10%.  Measured, us, against the rule below it:
//  forward (eff 0.6, reductions of 256 or more, past two rounds of 512): 16 x 40 x 40, 960 -> 384
//   (0.78) 33.7 -> 29.0, 80 x 80, 576 -> 192 (0.78) 63.4 -> 48.2, 160 x 160 stride 2, 96 -> 192 (0.78) 64.5 -> 55.9; 12 x 52 x 52 x
//   256 on 256 x 128 (0.99) 17.8 -> 12.1, 100 x 100 stride 2, 64 -> 128 (0.61) 19.6 -> 14.0; 40 x 40 x 320
//   (0.65, a sixth of the columns idle) 15.1 -> 16.4.  Short reductions are bound by memory, and
//   one block per CU overlaps its output with nothing: training passes of 80 x 80 x 192 148.8
//   -> 150.8, 32 images of 80 x 80 x 128 170.2 -> 175.3; past two
//   rounds below 512: 5 x 229 x 229, 400 -> 352 174 -> 196
//  data gradient (eff 0.8, at most two rounds; the weights' transposing reads cost more): 40 x
//   40, 960 <- 384 (0.98) 35.6 -> 33.1, 52 x 52 x 256 (0.99) 14.5 -> 10.7; 40 x 40, 768 <- 384 (0.78) 28.8 ->
//   30.2; six rounds, 4 x 125 x 144, 624 <- 272, the training pass 283.9 -> 287.4
//  128 x 128 tiles, for one round of at least 140 (data gradient 225) blocks: 20 x 20, 1152 -> 576
//   (250) 18.6 -> 14.9, 40 x 40 stride 2, 384 -> 576 (250) 37.7 -> 33.7, 26 x 26, 512 -> 256 (170) 12.5 -> 9.8; 8
//   x 26 x 26 (86) 9.4 -> 10.0.
enum { kWide256x192 = 0, kWide256x128 = 1, kWide128x128 = 4 };  // (generic tiles of as many rows have these ids)
TileCfg wide_pick(int64_t m, int nout, int ktot, bool bt) {
  TileCfg best{0, 0, -1, kVariantGeneric};
  double best_eff = bt ? 0.8 : 0.6;
  constexpr int kT[2][3] = {{256, 192, kWide256x192}, {256, 128, kWide256x128}};
  for (const auto& t : kT) {
    const int64_t cols = (nout + t[1] - 1) / t[1], tiles = (m + t[0] - 1) / t[0] * cols, rounds = (tiles + 255) / 256;
    if (cols * t[1] * 10 > (int64_t)nout * 11 || (bt ? rounds > 2 : ktot < (rounds > 2 ? 512 : 256))) continue;
    const double eff = (double)m * nout / ((double)rounds * 256 * t[0] * t[1]);
    if (eff >= best_eff) {
      best_eff = eff;
      best = TileCfg{t[0], t[1], t[2], kVariantWide};
    }
  }
  if (best.variant == kVariantWide) return best;
  const int64_t cols = (nout + 127) / 128, tiles = (m + 127) / 128 * cols;
  if (tiles <= 256 && tiles >= (bt ? 225 : 140) && cols * 1280 <= (int64_t)nout * 12 && m <= 16384)
    return TileCfg{128, 128, kWide128x128, kVariantWide};
  return best;
}

// Tile and kernel choice, fitted to timings of every (kernel, tile, stages) choice over
// the forward and data-gradient GEMMs of the detector's layers at batch 16, weighted by
// how often each shape occurs (within 1% of the per-layer best in total):
//  * forward (K-major weights): N tile the least padding among 128, 96 and 64 columns
//    (ties to the wider; 64 when fewer than 400 blocks of 128 rows); more than 32768
//    rows, three stages of 32 reduction elements (three blocks per CU for 128-row tiles),
//    256-row tiles when the reduction is 768 or longer, 64 columns when it is shorter
//    than 512 and 64 divides N; 8193..32768 rows, two stages of 64 (two blocks per CU) on
//    128 x 96 tiles when 96 divides N <= 192, else 128 x 64; up to 8192 rows, reductions
//    of 3000 or more into N >= 256: three stages of 64 on 128 x 96 (else x 128) tiles
//    when one block per CU covers the grid; otherwise 128 x 64 tiles, two stages of 64
//    when the grid exceeds 256 blocks, else three;
//  * data gradient (weights read in place through transposing LDS reads, which favour
//    64-column tiles): more than 32768 rows as the forward, with 64 columns on 128-row
//    tiles; 8193..32768 rows, eight waves on 256 x 96 (or x 64) tiles with three stages
//    of 64 when the reduction is 1000 or longer and one such block per CU covers the
//    grid, else 128 x 64 with three stages of 32; up to 8192 rows, 128 x 64 with two
//    stages of 64 when the grid holds 300 blocks or more, else three;
//  * generic kernel (fewer than 16 channels, or beyond 31-bit offsets): 256-row tiles unless that leaves
//    fewer than 512 blocks.
TileCfg convgemm_pick(int64_t m_max, int nout, int cs, int ktot, int nphase, bool bt, bool generic) {
  const int bns[4] = {128, 96, 64, 32};
  const int ncand = nout <= 32 ? 4 : 3;
  int bn = 128;
  int64_t waste = INT64_MAX;
  for (int i = 0; i < ncand; ++i) {
    const int64_t w = ((nout + bns[i] - 1) / bns[i]) * bns[i] - nout;
    if (w < waste) {
      waste = w;
      bn = bns[i];
    }
  }
  const bool fast = !generic && dma_channels(cs, kVariantDma32);
  // Channel counts that are no multiple of 16 or below 32, which the 64 columns below were not
  // fitted on, keep the least padding where 64 columns pad over a fifth more: 16 x 219 x 219
  // stride 2, 88 <- 24 122 us, and 87 on 96 columns; 2 x 149 x 149, 824 -> 88 262 and 150.
  const bool unfitted = cs % 16 != 0 || cs < 32;
  const bool narrower64 = unfitted && (int64_t)(nout + 63) / 64 * 64 * 5 > (int64_t)((nout + bn - 1) / bn) * bn * 6;
  if (fast && cs >= 32 && nphase == 1) {
    const TileCfg t = wide_pick(m_max, nout, ktot, bt);
    if (t.variant == kVariantWide) return t;
  }
  int bm, variant;
  if (fast && !bt) {
    const int64_t mt = (m_max + 127) / 128;
    const int64_t blocks128 = mt * ((nout + bn - 1) / bn);
    if (blocks128 < 400 && bn > 64 && !narrower64) bn = 64;
    bm = 128;
    if (m_max > 32768) {
      variant = kVariantDma32;
      bm = ktot >= 768 ? 256 : 128;
      if (ktot < 512 && nout % 64 == 0) bn = 64;
    } else if (m_max > 8192) {
      variant = kVariantDma2;
      bn = (nout % 96 == 0 && nout <= 192) ? 96 : 64;
    } else if (ktot >= 3000 && nout >= 256) {
      // long reductions: one 128 x 96 (or x 128) block per CU with three 64-deep stages,
      // when the grid fits one round
      variant = kVariantDma3;
      bn = (nout % 96 == 0 && mt * (nout / 96) <= 256) ? 96 : mt * ((nout + 127) / 128) <= 256 ? 128 : 64;
    } else {
      bn = 64;
      variant = mt * ((nout + 63) / 64) > 256 ? kVariantDma2 : kVariantDma3;
    }
  } else if (fast) {
    // (so do they on short reductions into many rows that are no whole 64-byte lines, where the
    // output is the work and neighbouring tiles share its lines: 14 x 65 x 239, 216 <- 40 73.2 us ->
    // 45.2, 26 x 86 x 86 stride 2, 600 <- 16 168 -> 118, 16 x 143 x 143 stride 2, 104 <- 40 55.5 -> 39.7; whole
    // lines 4 x 151 x 132 stride 2, 896 <- 16 36.0 on 64 columns, 46.2 on 128)
    const bool least = narrower64 || (unfitted && nout % 32 != 0 && ktot <= 256 && m_max > (nphase > 1 ? 8192 : 32768));
    const int bn64 = bn < 64 || least ? bn : 64;
    bm = 128;
    if (m_max > 32768) {
      variant = kVariantDma32;
      if (ktot >= 768) bm = 256;
      else bn = bn64;
    } else if (m_max > 8192) {
      const int bn8 = nout % 96 == 0 ? 96 : bn64;
      const int64_t blocks8 = ((m_max + 255) / 256) * ((nout + bn8 - 1) / bn8) * nphase;
      if (ktot >= 1000 && blocks8 <= 256) {
        variant = kVariantDma3W8;
        bm = 256;
        bn = bn8;
      } else {
        variant = kVariantDma32;
        bn = bn64;
      }
    } else {
      bn = bn64;
      const int64_t blocks = ((m_max + 127) / 128) * ((nout + bn - 1) / bn) * nphase;
      variant = blocks >= 300 ? kVariantDma2 : kVariantDma3;
    }
  } else {
    const int64_t blocks256 = ((m_max + 255) / 256) * ((nout + bn - 1) / bn);
    bm = blocks256 < 512 && !generic ? 128 : 256;
    variant = kVariantGeneric;
  }
  // fewer than 32 channels: a 64-deep step would cross more than two taps
  if (fast && !dma_channels(cs, variant)) {
    variant = kVariantDma32;
    bm = 128;
  }
  int id = (bm == 128 ? 4 : 0) + (bn == 128 ? 0 : bn == 96 ? 1 : bn == 64 ? 2 : 3);
  return TileCfg{bm, bn, id, variant};
}

// narrow input (ci < 8): 256-row tiles, 32 or 64 columns
TileCfg narrow_pick(int nout) { return TileCfg{256, nout <= 32 ? 32 : 64, -1, kVariantGeneric}; }

// the RGB image layer's shape: 3 channels, 3x3 taps at offsets -1..1, stride 2, at most
// 64 output channels, output rows a multiple of 4 and columns of 64, 256-row tiles
bool stem_shape(const ConvGemmArgs& a, const TileCfg& t) {
  const GemmPhase& P = a.ph[0];
  if (a.nphase != 1 || a.cs != 3 || P.taps != 9 || a.gstride_h != 2 || a.gstride_w != 2 || a.nout > 64 ||
      t.bm != 256 || P.gh % 4 != 0 || P.gw % 64 != 0 || a.nimg > 65535 || P.gh / 4 > 65535)
    return false;
  for (int r = 0; r < 3; ++r)
    for (int q = 0; q < 3; ++q)
      if (P.off[r * 3 + q] != (int32_t)((uint32_t)(uint16_t)(int16_t)(r - 1) | ((uint32_t)(q - 1) << 16))) return false;
  return true;
}

hipError_t convnarrow_launch(const ConvGemmArgs& a, const TileCfg& t, hipStream_t s) {
  if (a.nphase != 1 || a.ph[0].ktot > NarrowShape<2, 2>::KMAX || a.ph[0].taps > kMaxTaps)
    return hipErrorInvalidValue;
  if (stem_shape(a, t)) {
    trace_begin(KC_CONV_FWD);
    dim3 grid((unsigned)(a.ph[0].gw / 64), (unsigned)(a.ph[0].gh / 4), (unsigned)a.nimg);
    NUMBAT_LAUNCH(convstem_kernel, grid, dim3(256), 0, s, a);
    trace_end(KC_CONV_FWD);
    return hipGetLastError();
  }
  trace_begin(KC_CONV_FWD);
  const hipError_t e = t.bn == 32 ? launch_narrow<1>(a, s) : launch_narrow<2>(a, s);
  trace_end(KC_CONV_FWD);
  return e;
}

bool convgemm_direct(ConvGemmArgs a, const TileCfg& t) {
  if (t.variant == kVariantSplit) return a.cs % 8 == 0 && convgemm_taps(a, t.bm);
  return t.variant != kVariantGeneric && prepare_fast(a, t);
}

hipError_t convgemm_launch(ConvGemmArgs a, const TileCfg& t, hipStream_t s, int cls) {
  if (t.variant == kVariantSplit) return convsplit_launch(a, t, s, cls);
  // a problem the fast paths cannot take runs the generic kernel on the same tile
  const int variant = (t.variant != kVariantGeneric && prepare_fast(a, t)) ? t.variant : kVariantGeneric;
  if (a.bt && variant == kVariantGeneric) return hipErrorInvalidValue;  // needs K-major B
  a.remap = 0;
#ifdef NUMBAT_TUNING
  if (const char* e = getenv("NUMBAT_REMAP_CONV")) a.remap = atoi(e);
#endif
  if (variant == kVariantWide) {
    int mmax = 0;
    for (int p = 0; p < a.nphase; ++p) mmax = a.ph[p].m > mmax ? a.ph[p].m : mmax;
    trace_begin(cls);
    if (t.id == kWide256x192) launch_dma<2, 3, 4, 32, 8, 2>(a, mmax, s);
    else if (t.id == kWide256x128) launch_dma<2, 2, 4, 32, 8, 2>(a, mmax, s);
    else launch_dma<1, 2, 3, 64, 8, 2>(a, mmax, s);
    trace_end(cls);
    return hipGetLastError();
  }
  trace_begin(cls);
  hipError_t e;
  switch (t.id) {
    case 0: e = launch_g<0>(a, variant, s); break;
    case 1: e = launch_g<1>(a, variant, s); break;
    case 2: e = launch_g<2>(a, variant, s); break;
    case 3: e = launch_g<3>(a, variant, s); break;
    case 4: e = launch_g<4>(a, variant, s); break;
    case 5: e = launch_g<5>(a, variant, s); break;
    case 6: e = launch_g<6>(a, variant, s); break;
    default: e = launch_g<7>(a, variant, s); break;
  }
  trace_end(cls);
  return e;
}

}  // namespace numbat
