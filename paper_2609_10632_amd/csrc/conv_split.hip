// Implicit-GEMM convolution for problems with few output tiles (one image, deep layers with
// small maps, small batches) on gfx950 MFMA: the waves of a block split the reduction.
//
// The GEMM family of ConvGemmArgs (forward, data-gradient phases) on tiles of 32 or 64 rows.
// Such problems have long reductions and few tiles: on 128-row tiles a 20 x 20 x 576 image
// fills 12-36 of the 256 CUs and each of those walks 81 steps behind a block barrier.  Here
// every wave of a block owns the whole tile over its own share of the 64-deep reduction
// steps (wave w takes steps w, w + NW, ...): it loads both operands of a step into LDS
// stages of its own (buffer_load ... lds), waits for nothing but those loads and multiplies,
// so the main loop has no barrier; the waves' sums meet once, through LDS, in a fixed order.
// What bounds it: the load path into LDS, about 55 bytes per clock and CU when a wave
// instruction covers 8 rows of 128 bytes, which is why a step is 64 elements deep.
//
// Channel counts are any multiple of 8 (a lane's 16-byte chunk never splits a tap): each lane
// derives the tap and channel of its chunk from the reduction index by an exact division.
#include <cstdlib>

#include "conv_tile.h"

namespace numbat {

namespace {

constexpr int kBK = 64;  // reduction elements per step

// TM x TN blocks of 32 x 32 per tile, NW waves, two stages per wave
template <int TM, int TN, int NW>
struct SplitShape {
  static constexpr int BM = 32 * TM, BN = 32 * TN, NT = 64 * NW;
  static constexpr int ABYTES = BM * 2 * kBK, BBYTES = BN * 2 * kBK;
  static constexpr int STG = ABYTES + BBYTES;   // one wave's stage
  static constexpr int LPS = STG / 1024;        // load instructions per wave and step
  static constexpr int LD = BN + 4;             // fp32 per row of a wave's sums in LDS
  static constexpr int RED = NW * BM * LD * 4;  // the waves' sums (in stage 0's space)
  static constexpr int S0 = NW * STG > RED ? NW * STG : RED;
  static constexpr int VEC = BM * BN / 8;       // output vectors of the tile
  static constexpr int VPT = (VEC + NT - 1) / NT;
  static constexpr int NG = NT / BN;            // row groups of the column statistics
  static_assert(S0 + NW * STG + 8 * BM + 4 * (NG + 1) * BN <= 160 * 1024, "LDS");
  static_assert(NT >= BN, "a thread per column");
};

template <int TM, int TN, int NW, bool BT>
__global__ __launch_bounds__(64 * NW) void convsplit_kernel(ConvGemmArgs a, FastDiv dcs) {
  using Sh = SplitShape<TM, TN, NW>;
  constexpr int BM = Sh::BM, BN = Sh::BN, NT = Sh::NT, LPS = Sh::LPS, LD = Sh::LD, NG = Sh::NG;
  constexpr int AI = BM / 8, BI = BN / 8;  // load instructions per step: rows of 128 bytes, 8 each

  __shared__ __attribute__((aligned(16))) unsigned char sS0[Sh::S0];
  __shared__ __attribute__((aligned(16))) unsigned char sS1[NW * Sh::STG];
  __shared__ int64_t s_dst[BM];
  __shared__ float s_col[NG][BN];
  __shared__ float s_mean[BN];

  // logical tile: with a.remap the m tile is fastest and each XCD takes a contiguous range,
  // so the tiles that share weight columns share an L2; otherwise the launch order
  const uint32_t gx = gridDim.x, gy = gridDim.y;
  uint32_t lg = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  if (a.remap) lg = xcd_remap(lg, gx * gy * gridDim.z);
  const int mt = (int)(lg % gx), nt = (int)((lg / gx) % gy), phase = (int)(lg / (gx * gy));
  const GemmPhase& P = a.ph[phase];
  const Geo Ge = load_geo(P);
  const int m0 = mt * BM, n0 = nt * BN;
  if (m0 >= P.m) return;  // this phase has fewer tiles; uniform exit before any barrier
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int cs = a.cs, ktot = P.ktot, taps = P.taps, nout = a.nout;

  // ---- A: instruction q of a stage fills rows 8 q + lane / 8; the lane's slot lane % 8 holds
  // 16-byte chunk slot ^ ((row / 2) % 8) of the row's 64 reduction elements
  const int lrow = lane >> 3;
  const int kc0 = (lane & 7) ^ (lrow >> 1);  // even q; odd q: kc0 ^ 4
  const uint32_t img0 = fdiv((uint32_t)m0, P.div_ghw);
  const __amdgpu_buffer_rsrc_t rsA = buffer_rsrc(a.src + ((int64_t)img0 * a.hs * a.ws - a.halo_px) * a.src_pix);
  const __amdgpu_buffer_rsrc_t rsB = buffer_rsrc(P.wt);
  uint32_t vrow[AI], vmask[AI];
  const int tw = P.tw;
#pragma unroll
  for (int q = 0; q < AI; ++q) row_gather(a, Ge, m0 + 8 * q + lrow, img0, vrow[q], vmask[q]);
  for (int r = tid; r < BM; r += NT) s_dst[r] = dst_offset(a, Ge, m0 + r);
  // a tap's grid row is (tap * tinv) >> 16 (exact for tap < 32), its byte offsets from there
  const uint32_t tinv = (65536u + (uint32_t)tw - 1) / (uint32_t)tw;
  const uint32_t acol = (uint32_t)P.cstep, arow = (uint32_t)(P.rstep + (tw - 1) * P.cstep), a0 = (uint32_t)P.toff0;
  const uint32_t wcol = (uint32_t)P.wcstep, wrow = (uint32_t)(P.wrstep + (tw - 1) * P.wcstep), w0 = (uint32_t)P.wtoff0;
  const uint32_t wostep = (uint32_t)P.wostep;

  // ---- B: K-major rows (one output channel, 64 elements), laid out as A's; or, transposed,
  // rows of one reduction element and BN columns
  uint32_t boff[BI];
  int brow[BT ? BI : 1];
#pragma unroll
  for (int j = 0; j < BI; ++j) {
    if constexpr (!BT) {
      const int o = n0 + 8 * j + lrow;
      boff[j] = o < nout ? (uint32_t)((int64_t)o * ktot * 2) : kOob;
    } else {
      const int byte = j * 1024 + lane * 16;
      const int row = byte / (2 * BN), slot = (byte % (2 * BN)) / 16;
      const int ch = slot ^ bt_swizzle<BN>(row);
      brow[j] = row;
      boff[j] = n0 + ch * 8 < nout ? (uint32_t)((n0 + ch * 8) * 2) : kOob;
    }
  }

  auto stage = [&](auto sc) __attribute__((always_inline)) -> unsigned char* {
    return (decltype(sc)::value == 0 ? sS0 : sS1) + wave * Sh::STG;
  };
  // loads of step kt (past the reduction's end they read zeros)
  auto issue = [&](auto sc, int kt) __attribute__((always_inline)) {
    unsigned char* A = stage(sc);
    unsigned char* B = A + Sh::ABYTES;
    const int kb = kt * kBK;
    uint32_t lo[2], kk[2];
    int tp[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t k = (uint32_t)(kb + 8 * (e ? kc0 ^ 4 : kc0));
      const uint32_t t = fdiv(k, dcs);
      const uint32_t r = (t * tinv) >> 16;
      lo[e] = a0 + r * arow + (t - r * (uint32_t)tw) * acol + 2u * (k - t * (uint32_t)cs);
      tp[e] = t < 31u ? (int)t : 31;  // past the last tap: bit 31 is clear
      kk[e] = k;
    }
#pragma unroll
    for (int q = 0; q < AI; ++q) {
      const uint32_t t = (uint32_t)__builtin_amdgcn_sbfe((int)vmask[q], tp[q & 1], 1);
      const uint32_t vo = (t & (vrow[q] + lo[q & 1])) | (~t & kOob);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void_t*)(A + q * 1024), 16, vo, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      uint32_t vb;
      if constexpr (!BT) {
        vb = (kk[j & 1] < (uint32_t)ktot && boff[j] != kOob) ? boff[j] + 2u * kk[j & 1] : kOob;
      } else {
        const uint32_t k = (uint32_t)(kb + brow[j]);
        const uint32_t t = fdiv(k, dcs);
        const uint32_t r = (t * tinv) >> 16;
        const uint32_t wo = w0 + r * wrow + (t - r * (uint32_t)tw) * wcol + (k - t * (uint32_t)cs) * wostep;
        vb = (t < (uint32_t)taps && boff[j] != kOob) ? boff[j] + wo : kOob;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_void_t*)(B + j * 1024), 16, vb, 0, 0, 0);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment offsets: row l32 (+ 32 i), chunk 2 ks + half in slot chunk ^ ((row / 2) % 8)
  const uint32_t frow = (uint32_t)l32 * 128u;
  const int fsw = (l32 >> 1) & 7;
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
  // this wave's loads of the step are done (the next step's stay in flight); read its
  // fragments, then refill the stage while multiplying
  auto step = [&](auto sc, int kt) __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS) : "memory");
    const unsigned char* A = stage(sc);
    const unsigned char* B = A + Sh::ABYTES;
    u32x4 af[4][TM], bf[4][TN];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const uint32_t ko = frow + (uint32_t)(((2 * ks + half) ^ fsw) * 16);
#pragma unroll
      for (int i = 0; i < TM; ++i) af[ks][i] = *reinterpret_cast<const u32x4*>(A + i * 32 * 128 + ko);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (!BT) {
          bf[ks][j] = *reinterpret_cast<const u32x4*>(B + j * 32 * 128 + ko);
        } else {
          const unsigned char* pb = B + btoff[j] + ks * 16 * 2 * BN;
          const v4s_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)pb);
          const v4s_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)(pb + 4 * 2 * BN));
          const v2u_t lo = __builtin_bit_cast(v2u_t, r0), hi = __builtin_bit_cast(v2u_t, r1);
          bf[ks][j] = u32x4{lo.x, lo.y, hi.x, hi.y};
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the stage is read: refill it
    __builtin_amdgcn_sched_barrier(0);
    issue(sc, kt + 2 * NW);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(af[ks][i], bf[ks][j], acc[i][j]);
  };
  const int nk = (ktot + kBK - 1) / kBK;
  issue(Ic<0>{}, wave);
  issue(Ic<1>{}, wave + NW);
  for (int kt = wave; kt < nk; kt += 2 * NW) {
    step(Ic<0>{}, kt);
    if (kt + NW < nk) step(Ic<1>{}, kt + NW);
  }
  // the loads issued past the last step land before the stages become the waves' sums
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // ---- the waves' sums: [wave][row][LD], added in a fixed pairwise order
  float* red = reinterpret_cast<float*>(sS0);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        red[(wave * BM + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * LD + j * 32 + l32] = acc[i][j][r];
  __syncthreads();
  constexpr int VPR = BN / 8;
  float f[Sh::VPT][8];
#pragma unroll
  for (int u = 0; u < Sh::VPT; ++u) {
    const int v = tid + u * NT;
    if (v < Sh::VEC) {
      const int row = v / VPR, c8 = (v - row * VPR) * 8;
      float s[NW][8];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float* p = red + (w * BM + row) * LD + c8;
        const float4 lo = *reinterpret_cast<const float4*>(p), hi = *reinterpret_cast<const float4*>(p + 4);
        s[w][0] = lo.x, s[w][1] = lo.y, s[w][2] = lo.z, s[w][3] = lo.w;
        s[w][4] = hi.x, s[w][5] = hi.y, s[w][6] = hi.z, s[w][7] = hi.w;
      }
#pragma unroll
      for (int h = 1; h < NW; h *= 2)
#pragma unroll
        for (int w = 0; w < NW; w += 2 * h)
#pragma unroll
          for (int e = 0; e < 8; ++e) s[w][e] += s[w + h][e];
#pragma unroll
      for (int e = 0; e < 8; ++e) f[u][e] = s[0][e];
    }
  }

  // ---- per-channel (mean, M2) of the tile's rows (phase 0, when requested)
  if (a.stats_part != nullptr && phase == 0) {
    // (each thread overwrites elements of wave 0's sums that only it has read)
#pragma unroll
    for (int u = 0; u < Sh::VPT; ++u) {
      const int v = tid + u * NT;
      if (v < Sh::VEC) {
        const int row = v / VPR, c8 = (v - row * VPR) * 8;
        float* p = red + row * LD + c8;
        *reinterpret_cast<float4*>(p) = make_float4(f[u][0], f[u][1], f[u][2], f[u][3]);
        *reinterpret_cast<float4*>(p + 4) = make_float4(f[u][4], f[u][5], f[u][6], f[u][7]);
      }
    }
    __syncthreads();
    const int count = P.m - m0 < BM ? P.m - m0 : BM;
    const int col = tid % BN, grp = tid / BN;
    if (grp < NG) {
      float s = 0.f;
      for (int r = grp; r < count; r += NG) s += red[r * LD + col];
      s_col[grp][col] = s;
    }
    __syncthreads();
    if (tid < BN) {
      float s = 0.f;
#pragma unroll
      for (int g = 0; g < NG; ++g) s += s_col[g][tid];
      s_mean[tid] = s / (float)count;
    }
    __syncthreads();
    if (grp < NG) {
      const float mu = s_mean[col];
      float q = 0.f;
      for (int r = grp; r < count; r += NG) {
        const float d = red[r * LD + col] - mu;
        q += d * d;
      }
      s_col[grp][col] = q;
    }
    __syncthreads();
    if (tid < BN && n0 + tid < nout) {
      float q = 0.f;
#pragma unroll
      for (int g = 0; g < NG; ++g) q += s_col[g][tid];
      a.stats_part[(int64_t)mt * nout + n0 + tid] = make_float2(s_mean[tid], q);
    }
  }

  // ---- output vectors
#pragma unroll
  for (int u = 0; u < Sh::VPT; ++u) {
    const int v = tid + u * NT;
    if (v >= Sh::VEC) continue;
    const int row = v / VPR, col = n0 + (v - row * VPR) * 8;
    const int64_t d = s_dst[row];
    if (col >= nout || d < 0) continue;
    if (a.post == kPostBias) {
#pragma unroll
      for (int e = 0; e < 8; ++e) f[u][e] += a.post_bias[col + e];
    } else if (a.post == kPostBnSilu) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float sc, sh;
        bn_fold(a.post_gamma[col + e], a.post_beta[col + e], a.post_mean[col + e], a.post_var[col + e], a.post_eps, sc,
                sh);
        f[u][e] = bn_silu_apply(f[u][e], sc, sh);
      }
    }
    uint4* p = reinterpret_cast<uint4*>(a.dst + d + col);
    if (a.accumulate) {
      float o[8];
      unpack8(*p, o);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[u][e] += o[e];
    }
    *p = pack8(f[u]);
  }
}

struct SInst {
  int tm, tn, nw;
};
constexpr SInst kS[] = {
    {1, 1, 8},  // 0: 32 x 32
    {1, 2, 4},  // 1: 32 x 64
    {2, 2, 4},  // 2: 64 x 64
};
constexpr int kNumS = sizeof(kS) / sizeof(kS[0]);

template <int I>
hipError_t launch_s(const ConvGemmArgs& a, int mmax, hipStream_t s) {
  constexpr SInst c = kS[I];
  using Sh = SplitShape<c.tm, c.tn, c.nw>;
  const dim3 grid((unsigned)((mmax + Sh::BM - 1) / Sh::BM), (unsigned)((a.nout + Sh::BN - 1) / Sh::BN),
                  (unsigned)a.nphase);
  const FastDiv dcs = make_fastdiv((uint32_t)a.cs);
  if (a.bt)
    NUMBAT_LAUNCH((convsplit_kernel<c.tm, c.tn, c.nw, true>), grid, dim3(Sh::NT), 0, s, a, dcs);
  else
    NUMBAT_LAUNCH((convsplit_kernel<c.tm, c.tn, c.nw, false>), grid, dim3(Sh::NT), 0, s, a, dcs);
  return hipGetLastError();
}

}  // namespace

// The smallest tile whose grid fits one block per CU (a second round doubles the time), where
// the reduction is long enough to pay for the meeting of the waves' sums.  Measured alone
// (forward without the statistics merge, us; this kernel against the better of the halo and
// the direct-to-LDS kernel): 32 x 32 tiles, one image of 20 x 20: 576 -> 64 (K 5184) 11.1
// against 21.2, 288 -> 288 (2592) 9.9 against 17.0, 1 x 1 1152 -> 576 8.8 against 11.2,
// 64 -> 64 (576) 7.8 against 6.2; 32 x 64 tiles, 4 images of 576 -> 192 15.5 against 28.0, 40 x
// 40 x 192 (1728) 10.2 against 13.3, 8 images of 26 x 26 x 128 (1152) in a second round 16
// against 9.8; 64 x 64 tiles, 8 images of 576 -> 192 20.9 against 28.9, 8 of 20 x 20 x 288 17.6
// against 17.5.  Data gradients (bt) read their weights through transposing reads and compete
// with the halo kernel on every stride-1 grid: 32 x 32 tiles 288 -> 288 9.3 against 16.7, but
// the larger ones 4 x 21 x 21 x 352 24.5 against 22.0 and 12 x 13 x 13 x 256 16.0 against 14.4;
// of a stride-2 one's four phases 64 x 64 tiles are the better (384 <- 576, one image of 40 x
// 40: 17.5 against 19.9).
TileCfg convsplit_pick(int64_t m_max, int nout, int cs, int ktot, int nphase, bool bt) {
  const TileCfg none{0, 0, -1, kVariantGeneric};
  if (cs % 8 != 0) return none;
#ifdef NUMBAT_TUNING
  if (const char* e = getenv("NUMBAT_SPLIT")) {
    const int id = atoi(e);
    if (id < 0 || id >= kNumS) return none;
    return TileCfg{32 * kS[id].tm, 32 * kS[id].tn, id, kVariantSplit};
  }
#endif
  constexpr int kMinK[kNumS] = {1024, 1536, 2304};
  for (int i = 0; i < kNumS; ++i) {
    const int bm = 32 * kS[i].tm, bn = 32 * kS[i].tn;
    const int64_t blocks = ((m_max + bm - 1) / bm) * ((nout + bn - 1) / bn) * nphase;
    if (blocks > 256 || (bt && i == 1)) continue;
    if (bt && i == 2 && nphase == 1) continue;
    return ktot >= kMinK[i] ? TileCfg{bm, bn, i, kVariantSplit} : none;
  }
  return none;
}

hipError_t convsplit_launch(const ConvGemmArgs& args, const TileCfg& t, hipStream_t s, int cls) {
  ConvGemmArgs a = args;
  if (t.variant != kVariantSplit || t.id < 0 || t.id >= kNumS || a.cs % 8 != 0 || a.nout % 8 != 0)
    return hipErrorInvalidValue;
  if (!convgemm_taps(a, t.bm)) return hipErrorInvalidValue;
  int mmax = 0;
  for (int p = 0; p < a.nphase; ++p) mmax = a.ph[p].m > mmax ? a.ph[p].m : mmax;
  a.remap = 1;
#ifdef NUMBAT_TUNING
  if (const char* e = getenv("NUMBAT_REMAP_CONV")) a.remap = atoi(e);
#endif
  trace_begin(cls);
  hipError_t e;
  switch (t.id) {
    case 0: e = launch_s<0>(a, mmax, s); break;
    case 1: e = launch_s<1>(a, mmax, s); break;
    default: e = launch_s<2>(a, mmax, s); break;
  }
  trace_end(cls);
  return e;
}

}  // namespace numbat
