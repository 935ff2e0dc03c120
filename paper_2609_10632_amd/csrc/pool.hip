// The glue between conv blocks on gfx950: the SPPF block's 5x5 stride-1 max pool (padding
// 2, never winning) and the neck's nearest 2x upsampling, forward and backward, NHWC bf16
// with pixel strides (so inputs and outputs can be channel slices of concatenation
// buffers).  A thread works on 16-byte vectors of 8 channels of one pixel.
//
// Max pool, where tiles are the better (pool_tiles; elsewhere a thread reads each of its vector's
// 25 window positions from memory): a block takes a tile of kTileRows output rows by up to kTileCols columns of one
// image for four vectors (64 bytes of every pixel) and stages the tile and its border of two
// pixels in LDS, so an element is read from memory about twice and not 25 times.
//  * Forward: the window's first maximum in row-major order wins (a later equal value does
//    not replace it); its window position (0 .. 24) is stored per element as one byte.  The
//    search is split into rows: the first maximum of every row of five, then the first
//    maximum of five rows, which is the same element with 10 comparisons instead of 25 (14
//    with the border rows' share).
//  * Backward: a gather: an input pixel visits the 25 windows that contain it in a fixed order
//    and adds the dy of those whose stored position is its own, in fp32, rounded once
//    (deterministic).
// Both are bound by their vector instructions (the compares and selects of 8 elements per
// vector) on top of the 3.9 us of an empty launch.  16 x 20 x 20 x 288 slices: forward 15.8 -> 11.2
// us, backward 18.8 -> 14.0 against one thread per output vector with 25 loads each.
#include "kernels.h"

namespace numbat {

namespace {

constexpr int kPoolThreads = 256;
constexpr int kTileRows = 5, kTileVecs = 4;
constexpr int kTileThreads = 512;  // at most; a block has a thread per output vector, in whole waves
constexpr int kTileCols = 32, kWholeCols = 40;  // images up to kWholeCols wide take one column tile

// tile t of the grid: vector group fastest, then column tile, row band, image
struct PoolTiles {
  int32_t tw;      // columns per tile
  int32_t threads; // per block
  uint32_t count;  // tiles
  FastDiv dvec, dcol, dband;
};
struct PoolTile {
  int img, p0, q0, v0;
};
__device__ __forceinline__ PoolTile pool_tile(uint32_t t, const PoolTiles& T) {
  const uint32_t a = fdiv(t, T.dvec), b = fdiv(a, T.dcol), c = fdiv(b, T.dband);
  return PoolTile{(int)c, (int)(b - c * T.dband.d) * kTileRows, (int)(a - b * T.dcol.d) * T.tw,
                  (int)(t - a * T.dvec.d) * kTileVecs};
}

// LDS: the staged border tile as [row][column][vector] 16-byte values, then (forward) every row's
// first maxima as values and positions, or (backward) the positions of the staged windows
__global__ __launch_bounds__(kTileThreads) void maxpool5_fwd_kernel(PoolArgs a, PoolTiles T, const bf16_t* x, bf16_t* y,
                                                                    uint8_t* idx) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s_pool[];
  const int cv = a.c / 8, tw = T.tw, sw = tw + 4;
  uint4* s_in = reinterpret_cast<uint4*>(s_pool);
  uint4* s_row = s_in + (kTileRows + 4) * sw * kTileVecs;
  uint2* s_at = reinterpret_cast<uint2*>(s_row + (kTileRows + 4) * tw * kTileVecs);
  const PoolTile t = pool_tile(blockIdx.x, T);
  const int c = threadIdx.x % kTileVecs, e0 = threadIdx.x / kTileVecs;
  const int step = blockDim.x / kTileVecs;
  const int ch = (t.v0 + c) * 8;
  const bool chok = t.v0 + c < cv;
  // (the row and column of an element advance without a division)
  {
    int r = e0 / sw, q = e0 - r * sw;
    const int dr = step / sw, dq = step - dr * sw;
    for (int e = e0; e < (kTileRows + 4) * sw; e += step) {
      const int i = t.p0 + r - 2, j = t.q0 + q - 2;
      uint4 v = make_uint4(0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u);  // -inf: never wins
      if (chok && (unsigned)i < (unsigned)a.h && (unsigned)j < (unsigned)a.w)
        v = *reinterpret_cast<const uint4*>(x + (((int64_t)t.img * a.h + i) * a.w + j) * a.x_pix + ch);
      s_in[e * kTileVecs + c] = v;
      r += dr;
      q += dq;
      if (q >= sw) q -= sw, ++r;
    }
  }
  __syncthreads();
  const int r0 = e0 / tw, q0 = e0 - r0 * tw, dr = step / tw, dq = step - dr * tw;
  {
    int r = r0, q = q0;
    for (int e = e0; e < (kTileRows + 4) * tw; e += step) {
      float best[8];
      uint32_t at[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        best[k] = -__builtin_huge_valf();
        at[k] = 0;
      }
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        float f[8];
        unpack8(s_in[(r * sw + q + s) * kTileVecs + c], f);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const bool better = f[k] > best[k];
          best[k] = better ? f[k] : best[k];
          at[k] = better ? (uint32_t)s : at[k];
        }
      }
      s_row[e * kTileVecs + c] = pack8(best);  // bf16 values: exact
      s_at[e * kTileVecs + c] = make_uint2(at[0] | (at[1] << 8) | (at[2] << 16) | (at[3] << 24),
                                           at[4] | (at[5] << 8) | (at[6] << 16) | (at[7] << 24));
      r += dr;
      q += dq;
      if (q >= tw) q -= tw, ++r;
    }
  }
  __syncthreads();
  int r = r0, q = q0;
  for (int e = e0; e < kTileRows * tw; e += step) {
    const int p = t.p0 + r, j = t.q0 + q;
    if (chok && p < a.h && j < a.w) {
      float best[8];
      uint32_t at[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        best[k] = -__builtin_huge_valf();
        at[k] = 0;
      }
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int o = ((r + s) * tw + q) * kTileVecs + c;
        float f[8];
        unpack8(s_row[o], f);
        const uint2 b = s_at[o];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const bool better = f[k] > best[k];
          best[k] = better ? f[k] : best[k];
          at[k] = better ? 5u * s + (((k < 4 ? b.x : b.y) >> (8 * (k & 3))) & 0xffu) : at[k];
        }
      }
      const int64_t pix = ((int64_t)t.img * a.h + p) * a.w + j;
      *reinterpret_cast<uint4*>(y + pix * a.y_pix + ch) = pack8(best);
      if (idx != nullptr)
        *reinterpret_cast<uint2*>(idx + pix * a.c + ch) =
            make_uint2(at[0] | (at[1] << 8) | (at[2] << 16) | (at[3] << 24),
                       at[4] | (at[5] << 8) | (at[6] << 16) | (at[7] << 24));
    }
    r += dr;
    q += dq;
    if (q >= tw) q -= tw, ++r;
  }
}

__global__ __launch_bounds__(kTileThreads) void maxpool5_bwd_kernel(PoolArgs a, PoolTiles T, const bf16_t* dy,
                                                                    const uint8_t* idx, bf16_t* dx, int accumulate) {
  extern __shared__ __attribute__((aligned(16))) unsigned char s_pool[];
  const int cv = a.c / 8, tw = T.tw, sw = tw + 4;
  uint4* s_dy = reinterpret_cast<uint4*>(s_pool);
  uint2* s_at = reinterpret_cast<uint2*>(s_dy + (kTileRows + 4) * sw * kTileVecs);
  const PoolTile t = pool_tile(blockIdx.x, T);
  const int c = threadIdx.x % kTileVecs, e0 = threadIdx.x / kTileVecs;
  const int step = blockDim.x / kTileVecs;
  const int ch = (t.v0 + c) * 8;
  const bool chok = t.v0 + c < cv;
  {
    int r = e0 / sw, q = e0 - r * sw;
    const int dr = step / sw, dq = step - dr * sw;
    for (int e = e0; e < (kTileRows + 4) * sw; e += step) {
      const int i = t.p0 + r - 2, j = t.q0 + q - 2;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      uint2 b = make_uint2(~0u, ~0u);  // outside the image: no position matches
      if (chok && (unsigned)i < (unsigned)a.h && (unsigned)j < (unsigned)a.w) {
        const int64_t pix = ((int64_t)t.img * a.h + i) * a.w + j;
        v = *reinterpret_cast<const uint4*>(dy + pix * a.y_pix + ch);
        b = *reinterpret_cast<const uint2*>(idx + pix * a.c + ch);
      }
      s_dy[e * kTileVecs + c] = v;
      s_at[e * kTileVecs + c] = b;
      r += dr;
      q += dq;
      if (q >= sw) q -= sw, ++r;
    }
  }
  __syncthreads();
  int r = e0 / tw, q = e0 - r * tw;
  const int dr = step / tw, dq = step - dr * tw;
  for (int e = e0; e < kTileRows * tw; e += step) {
    const int i = t.p0 + r, j = t.q0 + q;
    if (chok && i < a.h && j < a.w) {
      uint4* o = reinterpret_cast<uint4*>(dx + (((int64_t)t.img * a.h + i) * a.w + j) * a.x_pix + ch);
      uint4 old = make_uint4(0u, 0u, 0u, 0u);
      if (accumulate) old = *o;
      float acc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = 0.f;
      // window of output (p, q) holds this pixel at position (u, v) = (i - p + 2, j - q + 2)
#pragma unroll
      for (int u = 0; u < 5; ++u)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const int at = ((r + 4 - u) * sw + q + 4 - v) * kTileVecs + c;
          const uint2 b = s_at[at];
          float g[8];
          unpack8(s_dy[at], g);
#pragma unroll
          for (int k = 0; k < 8; ++k)
            acc[k] += (((k < 4 ? b.x : b.y) >> (8 * (k & 3))) & 0xffu) == (uint32_t)(u * 5 + v) ? g[k] : 0.f;
        }
      if (accumulate) {
        float f[8];
        unpack8(old, f);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] += f[k];
      }
      *o = pack8(acc);
    }
    r += dr;
    q += dq;
    if (q >= tw) q -= tw, ++r;
  }
}

// the max pools one output (or input) vector per thread, its window read from memory
__global__ __launch_bounds__(kPoolThreads) void maxpool5_fwd_direct_kernel(PoolArgs a, const bf16_t* x, bf16_t* y,
                                                                           uint8_t* idx) {
  const int cv = a.c / 8;
  const int64_t nvec = (int64_t)a.n * a.h * a.w * cv;
  for (int64_t v = (int64_t)blockIdx.x * kPoolThreads + threadIdx.x; v < nvec; v += (int64_t)gridDim.x * kPoolThreads) {
    const int64_t pix = v / cv;
    const int ch = (int)(v - pix * cv) * 8;
    const int64_t img = pix / ((int64_t)a.h * a.w);
    const int rem = (int)(pix - img * a.h * a.w);
    const int p = rem / a.w, q = rem - p * a.w;
    float best[8];
    uint32_t at[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      best[e] = -__builtin_huge_valf();
      at[e] = 0;
    }
    for (int r = 0; r < 5; ++r) {
      const int i = p + r - 2;
      if ((unsigned)i >= (unsigned)a.h) continue;
      for (int s = 0; s < 5; ++s) {
        const int j = q + s - 2;
        if ((unsigned)j >= (unsigned)a.w) continue;
        float f[8];
        unpack8(*reinterpret_cast<const uint4*>(x + ((img * a.h + i) * a.w + j) * a.x_pix + ch), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool better = f[e] > best[e];
          best[e] = better ? f[e] : best[e];
          at[e] = better ? (uint32_t)(r * 5 + s) : at[e];
        }
      }
    }
    *reinterpret_cast<uint4*>(y + pix * a.y_pix + ch) = pack8(best);  // bf16 values: exact
    if (idx != nullptr) {
      uint2 b;
      b.x = at[0] | (at[1] << 8) | (at[2] << 16) | (at[3] << 24);
      b.y = at[4] | (at[5] << 8) | (at[6] << 16) | (at[7] << 24);
      *reinterpret_cast<uint2*>(idx + pix * a.c + ch) = b;
    }
  }
}

__global__ __launch_bounds__(kPoolThreads) void maxpool5_bwd_direct_kernel(PoolArgs a, const bf16_t* dy, const uint8_t* idx,
                                                                           bf16_t* dx, int accumulate) {
  const int cv = a.c / 8;
  const int64_t nvec = (int64_t)a.n * a.h * a.w * cv;
  for (int64_t v = (int64_t)blockIdx.x * kPoolThreads + threadIdx.x; v < nvec; v += (int64_t)gridDim.x * kPoolThreads) {
    const int64_t pix = v / cv;
    const int ch = (int)(v - pix * cv) * 8;
    const int64_t img = pix / ((int64_t)a.h * a.w);
    const int rem = (int)(pix - img * a.h * a.w);
    const int i = rem / a.w, j = rem - i * a.w;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    // window of output (p, q) holds this pixel at position (r, s) = (i - p + 2, j - q + 2)
    for (int r = 0; r < 5; ++r) {
      const int p = i - r + 2;
      if ((unsigned)p >= (unsigned)a.h) continue;
      for (int s = 0; s < 5; ++s) {
        const int q = j - s + 2;
        if ((unsigned)q >= (unsigned)a.w) continue;
        const int64_t op = (img * a.h + p) * a.w + q;
        const uint2 b = *reinterpret_cast<const uint2*>(idx + op * a.c + ch);
        float g[8];
        unpack8(*reinterpret_cast<const uint4*>(dy + op * a.y_pix + ch), g);
        const uint32_t pos = (uint32_t)(r * 5 + s);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t w = ((e < 4 ? b.x : b.y) >> (8 * (e & 3))) & 0xffu;
          acc[e] += w == pos ? g[e] : 0.f;
        }
      }
    }
    uint4* o = reinterpret_cast<uint4*>(dx + pix * a.x_pix + ch);
    if (accumulate) {
      float f[8];
      unpack8(*o, f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += f[e];
    }
    *o = pack8(acc);
  }
}

// vector index -> pixel and image row
struct UpDiv {
  int32_t small;  // every index below 2^31
  FastDiv dcv, dw;
};

// nearest 2x: input pixel (i, j) -> output pixels (2i + a, 2j + b)
__global__ __launch_bounds__(kPoolThreads) void upsample2x_fwd_kernel(PoolArgs a, UpDiv D, const bf16_t* x, bf16_t* y) {
  const int cv = a.c / 8;
  const int64_t nvec = (int64_t)a.n * a.h * a.w * cv;
  for (int64_t v = (int64_t)blockIdx.x * kPoolThreads + threadIdx.x; v < nvec; v += (int64_t)gridDim.x * kPoolThreads) {
    int64_t pix, row;  // image-major pixel and image row (img * h + i)
    int ch, j;
    if (D.small) {  // 32-bit divisions by multiplication: a 64-bit one is over a hundred instructions
      const uint32_t p32 = fdiv((uint32_t)v, D.dcv), r32 = fdiv(p32, D.dw);
      pix = p32;
      row = r32;
      ch = (int)((uint32_t)v - p32 * D.dcv.d) * 8;
      j = (int)(p32 - r32 * D.dw.d);
    } else {
      pix = v / cv;
      row = pix / a.w;
      ch = (int)(v - pix * cv) * 8;
      j = (int)(pix - row * a.w);
    }
    const uint4 val = *reinterpret_cast<const uint4*>(x + pix * a.x_pix + ch);
    const int64_t o0 = 2 * row * (2 * (int64_t)a.w) + 2 * j;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int s = 0; s < 2; ++s)
        *reinterpret_cast<uint4*>(y + (o0 + r * 2 * (int64_t)a.w + s) * a.y_pix + ch) = val;
  }
}

__global__ __launch_bounds__(kPoolThreads) void upsample2x_bwd_kernel(PoolArgs a, UpDiv D, const bf16_t* dy,
                                                                      bf16_t* dx, int accumulate) {
  const int cv = a.c / 8;
  const int64_t nvec = (int64_t)a.n * a.h * a.w * cv;
  for (int64_t v = (int64_t)blockIdx.x * kPoolThreads + threadIdx.x; v < nvec; v += (int64_t)gridDim.x * kPoolThreads) {
    int64_t pix, row;  // image-major pixel and image row (img * h + i)
    int ch, j;
    if (D.small) {  // 32-bit divisions by multiplication: a 64-bit one is over a hundred instructions
      const uint32_t p32 = fdiv((uint32_t)v, D.dcv), r32 = fdiv(p32, D.dw);
      pix = p32;
      row = r32;
      ch = (int)((uint32_t)v - p32 * D.dcv.d) * 8;
      j = (int)(p32 - r32 * D.dw.d);
    } else {
      pix = v / cv;
      row = pix / a.w;
      ch = (int)(v - pix * cv) * 8;
      j = (int)(pix - row * a.w);
    }
    const int64_t o0 = 2 * row * (2 * (int64_t)a.w) + 2 * j;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        float g[8];
        unpack8(*reinterpret_cast<const uint4*>(dy + (o0 + r * 2 * (int64_t)a.w + s) * a.y_pix + ch), g);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += g[e];
      }
    uint4* o = reinterpret_cast<uint4*>(dx + pix * a.x_pix + ch);
    if (accumulate) {
      float f[8];
      unpack8(*o, f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += f[e];
    }
    *o = pack8(acc);
  }
}

int pool_blocks(const PoolArgs& a) {
  const int64_t nvec = (int64_t)a.n * a.h * a.w * (a.c / 8);
  int64_t b = (nvec + kPoolThreads - 1) / kPoolThreads;
  if (b > 8192) b = 8192;
  return (int)(b < 1 ? 1 : b);
}

UpDiv up_div(const PoolArgs& a) {
  UpDiv d;
  d.small = (int64_t)a.n * a.h * a.w * (a.c / 8) < (1ll << 31);
  d.dcv = make_fastdiv((uint32_t)(a.c / 8));
  d.dw = make_fastdiv((uint32_t)a.w);
  return d;
}

// Whether a max pool runs on tiles, and its tiles.  A tile leaves idle the lanes of missing
// vectors (c = 8: three of four) and of columns past the image (41 wide: 23 of 64), walks at most
// 512 threads twice over its vectors from 26 columns up, and has a border to stage; the direct
// kernel reads a window's vectors from the caches.  Tiles against direct, us, forward / backward:
// 8 images of 20 x 20 x 192 5.9 : 8.7 / 7.5 : 10.1, 32 of 64 x 64 x 192 69 : 95 / 92 : 123, but 32 of
// 80 x 80 x 8 22.4 : 12.2 / 29.0 : 12.4, 41 x 41 x 192 46.6 : 43.1 / 59.9 : 55.1.  So tiles where at
// least three quarters of their vectors exist (forward also up to 32 columns: 8 images of 26 x 26 x
// 8 5.9 : 6.9), and backward past 20 columns from 600000 vectors up (40 x 40 x 288, one image 11.4 :
// 9.7, 8 25.6 : 23.6, 32 58.2 : 77.3).  One column: 4.1 : 3.6 / 6.4 : 4.1.  A launch holds below 2^32
// threads, which 2^22 tiles stay under; the direct kernel walks over any size.
bool pool_tiles(const PoolArgs& a, bool backward, PoolTiles* T) {
  const int64_t cv = a.c / 8, nvec = (cv + kTileVecs - 1) / kTileVecs;
  T->tw = a.w <= kWholeCols ? a.w : kTileCols;
  const int64_t ncol = (a.w + T->tw - 1) / T->tw, nband = (a.h + kTileRows - 1) / kTileRows;
  const int64_t count = nvec * ncol * nband * a.n;
  const bool full = 4 * a.w * cv >= 3 * ncol * T->tw * nvec * kTileVecs;
  const bool on = backward ? full && (a.w <= 20 || (int64_t)a.n * a.h * a.w * cv >= 600000) : full || a.w <= 32;
  if (!on || a.w == 1 || count > (1ll << 22)) return false;
  T->count = (uint32_t)count;
  const int work = kTileRows * T->tw * kTileVecs;
  T->threads = work < kTileThreads ? (work + 63) / 64 * 64 : kTileThreads;
  T->dvec = make_fastdiv((uint32_t)nvec);
  T->dcol = make_fastdiv((uint32_t)ncol);
  T->dband = make_fastdiv((uint32_t)nband);
  return true;
}

}  // namespace

hipError_t maxpool5_fwd_launch(const PoolArgs& a, const bf16_t* x, bf16_t* y, uint8_t* idx, hipStream_t s) {
  PoolTiles T;
  trace_begin(KC_POOL);
  if (pool_tiles(a, false, &T)) {
    const size_t smem = (size_t)(kTileRows + 4) * kTileVecs * ((T.tw + 4) * 16 + T.tw * 24);
    NUMBAT_LAUNCH(maxpool5_fwd_kernel, dim3(T.count), dim3(T.threads), smem, s, a, T, x, y, idx);
  } else {
    NUMBAT_LAUNCH(maxpool5_fwd_direct_kernel, dim3(pool_blocks(a)), dim3(kPoolThreads), 0, s, a, x, y, idx);
  }
  trace_end(KC_POOL);
  return hipGetLastError();
}

hipError_t maxpool5_bwd_launch(const PoolArgs& a, const bf16_t* dy, const uint8_t* idx, bf16_t* dx, int accumulate,
                               hipStream_t s) {
  PoolTiles T;
  trace_begin(KC_POOL);
  if (pool_tiles(a, true, &T)) {
    const size_t smem = (size_t)(kTileRows + 4) * kTileVecs * (T.tw + 4) * 24;
    NUMBAT_LAUNCH(maxpool5_bwd_kernel, dim3(T.count), dim3(T.threads), smem, s, a, T, dy, idx, dx, accumulate);
  } else {
    NUMBAT_LAUNCH(maxpool5_bwd_direct_kernel, dim3(pool_blocks(a)), dim3(kPoolThreads), 0, s, a, dy, idx, dx,
                  accumulate);
  }
  trace_end(KC_POOL);
  return hipGetLastError();
}

hipError_t upsample2x_fwd_launch(const PoolArgs& a, const bf16_t* x, bf16_t* y, hipStream_t s) {
  trace_begin(KC_POOL);
  NUMBAT_LAUNCH(upsample2x_fwd_kernel, dim3(pool_blocks(a)), dim3(kPoolThreads), 0, s, a, up_div(a), x, y);
  trace_end(KC_POOL);
  return hipGetLastError();
}

hipError_t upsample2x_bwd_launch(const PoolArgs& a, const bf16_t* dy, bf16_t* dx, int accumulate, hipStream_t s) {
  trace_begin(KC_POOL);
  NUMBAT_LAUNCH(upsample2x_bwd_kernel, dim3(pool_blocks(a)), dim3(kPoolThreads), 0, s, a, up_div(a), dy, dx, accumulate);
  trace_end(KC_POOL);
  return hipGetLastError();
}

}  // namespace numbat
