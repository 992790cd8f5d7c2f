// Warm-start network (include/wf_nn.h): bfloat16 matrix-core convolutions
// with float32 accumulation, the encoder-decoder's forward and backward
// passes, Adam, and the C ABI.
//
// Every 3x3 convolution is an implicit GEMM on v_mfma_f32_16x16x32_bf16:
// output pixels are the rows, output channels the columns and (tap, input
// channel) the reduction.  Activations are [pixel][channel] bfloat16 so that
// one lane's eight consecutive reduction values are one 16-byte load; a block
// stages its pixels with their periodic border in LDS.  The weight gradient is
// the same product with pixels as the reduction: 64-pixel slabs of the input and of the output gradient are
// staged in LDS and read transposed, each block sums one pixel chunk, and a
// second kernel adds the chunks in a fixed order (deterministic).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "wf.h"
#include "wf_nn.h"

namespace wfnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kLevels = 4;
constexpr int kChan[kLevels] = {32, 64, 96, 128};
constexpr int kLayers = 4 * kLevels - 1;
constexpr int kPad = 32;  // channels of the padded input and output
constexpr int kFew = 8;   // those of them that are stored (the rest are zero)

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round to nearest even (v_cvt_pk_bf16_f32); NaN stays NaN
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// eight bfloat16 values <-> float
__device__ __forceinline__ void unpack8(u32x4 v, float* f) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(v[e] << 16);
    f[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
  }
}
__device__ __forceinline__ u32x4 pack8(const float* f) {
  u32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (uint32_t)f2bf(f[2 * e]) | ((uint32_t)f2bf(f[2 * e + 1]) << 16);
  return v;
}
// channels c .. c + 7 of a pixel of which cs are stored and the rest are zero
__device__ __forceinline__ u32x4 few_channels(const uint16_t* px, int c, int cs) {
  const u32x4 v = *(const u32x4*)(px + (c < cs ? c : 0));
  return c < cs ? v : u32x4{0u, 0u, 0u, 0u};
}
// v where m > 0, else 0, on 8 bfloat16 values
__device__ __forceinline__ u32x4 mask8(u32x4 v, u32x4 m) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = __uint_as_float(m[e] << 16) > 0.f ? 0xffffu : 0u;
    const uint32_t hi = __uint_as_float(m[e] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u;
    v[e] &= lo | hi;
  }
  return v;
}

// ---------------------------------------------------------------------------
// convolution (forward, and the input adjoint with mirrored taps)
// ---------------------------------------------------------------------------

struct ConvArgs {
  const uint16_t* in;    // [P][CIN]; with up: [P/4][CIN], read at (y/2, x/2)
  const uint16_t* wt;    // [9][cout][CIN]: reduction dimension contiguous
  const float* bias;     // [cout] or null
  uint16_t* out;         // [P][cout] or null: v = conv + bias (ReLU with relu)
  uint16_t* out2;        // [P][cout] or null: v + skip, or v where mask > 0
  const uint16_t* skip;  // [P][cout] or null
  const uint16_t* mask;  // [P][cout] or null; without out2 it applies to out
  float* out_f32;        // [P]: channel 0 in float32, or null
  int h, w, cout;
  int cs;                // channels of a pixel in memory: CIN, or kFew (the rest are zero)
  int up;
  int flip;              // 1: tap (dy, dx) reads the pixel at (-dy, -dx)
  int relu;
};

// Tile of one block (256 threads): 4 MT sixteen-pixel rows of the product, as
// TH image rows of TW pixels, times COT output channels; wave v owns MT of the
// sixteen-pixel rows and every column tile.  The tile's input with its
// one-pixel border is staged in LDS once, whole, and each of the nine taps
// reads it shifted (a tap per global read took the input nine times through
// the caches and waited for it each time); the weights of NTB taps at a time
// are staged beside it, the next group's loads in flight meanwhile.  Both are
// padded by 16 bytes per row: sixteen lanes' 16-byte reads fall on distinct
// banks.  Bound: at full resolution (32 channels) memory, one read and one
// write of the activations: four 1024^2 maps 269 to 166 us per launch (0.54
// GB, 3.2 TB/s); with more channels LDS reads and matrix instructions, about
// level.  Products are summed tap by tap, then channel by channel.
template <int CIN, int COT, int TW, int MT>
struct conv_tile {
  static constexpr int TH = 4 * MT * 16 / TW;
  static constexpr int HP = (TH + 2) * (TW + 2);  // staged pixels
  static constexpr int PS = CIN + 8;              // LDS row of a pixel or of a weight
  static constexpr int TAP = COT * PS;            // one tap's weights
  static constexpr int room = 78 * 1024 / 2 - HP * PS;
  static constexpr int NTB = 9 * TAP <= room ? 9 : (3 * TAP <= room ? 3 : 1);
  static constexpr int OS = COT + 8;              // LDS row of an output pixel
  static constexpr int main = HP * PS + NTB * TAP, epi = TH * TW * OS;
  static constexpr int lds = main > epi ? main : epi;
};

template <int CIN, int COT, int TW, int MT>
__global__ __launch_bounds__(256) void conv_kernel(ConvArgs a) {
  using C = conv_tile<CIN, COT, TW, MT>;
  constexpr int NJ = COT / 16, TH = C::TH, PS = C::PS, NTB = C::NTB, U = CIN / 8;
  __shared__ __attribute__((aligned(16))) uint16_t sm[C::lds];
  uint16_t* xs = sm;
  uint16_t* ws = sm + C::HP * PS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int co0 = blockIdx.y * COT;
  // consecutive tiles of an image run on one XCD (their borders overlap)
  const int nt = gridDim.x;
  const int tile = nt % 8 == 0 ? (int)(blockIdx.x & 7) * (nt / 8) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int tx = a.w / TW, ty = a.h / TH;
  const int img = tile / (tx * ty), rem = tile - img * (tx * ty);
  const int y0 = rem / tx * TH, x0 = (rem - rem / tx * tx) * TW;
  const int hw = a.h * a.w;

  // weights of taps NTB s .. NTB s + NTB - 1, in flight in registers
  constexpr int WN = NTB * COT * U, WU = (WN + 255) / 256;
  u32x4 wr[WU];
  auto wload = [&](int s) {
#pragma unroll
    for (int k = 0; k < WU; ++k) {
      const int i = min(tid + k * 256, WN - 1);
      const int row = i / U, cc = i - row * U, t = row / COT, co = row - t * COT;
      wr[k] = *(const u32x4*)(a.wt + ((int64_t)(NTB * s + t) * a.cout + co0 + co) * CIN + cc * 8);
    }
  };
  auto wstore = [&]() {
#pragma unroll
    for (int k = 0; k < WU; ++k) {
      const int i = tid + k * 256;
      const int row = i / U, cc = i - row * U;
      if (i < WN) *(u32x4*)&ws[row * PS + cc * 8] = wr[k];
    }
  };
  wload(0);
  {
    constexpr int N = C::HP * U, NU = (N + 255) / 256, G = 6;
    const int ih = a.up ? a.h >> 1 : a.h, iw = a.up ? a.w >> 1 : a.w;
    const uint16_t* src = a.in + (int64_t)img * ih * iw * a.cs;
#pragma unroll
    for (int k0 = 0; k0 < NU; k0 += G) {
      u32x4 v[G];
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const int i = min(tid + (k0 + k) * 256, N - 1);
        const int px = i / U, cc = i - px * U;
        const int yy = wrap(y0 - 1 + px / (TW + 2), a.h), xx = wrap(x0 - 1 + px % (TW + 2), a.w);
        if (k0 + k < NU)
          v[k] = few_channels(src + ((int64_t)(yy >> a.up) * iw + (xx >> a.up)) * a.cs, cc * 8, a.cs);
      }
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const int i = tid + (k0 + k) * 256;
        const int px = i / U, cc = i - px * U;
        if (k0 + k < NU && i < N) *(u32x4*)&xs[px * PS + cc * 8] = v[k];
      }
    }
  }
  f32x4 acc[MT][NJ];
#pragma unroll
  for (int u = 0; u < MT; ++u)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // staged pixel of this lane's row of product row u, before the tap's shift
  int prow[MT];
#pragma unroll
  for (int u = 0; u < MT; ++u) {
    const int m = wave * MT + u;  // product row: 16 / TW image rows
    prow[u] = (1 + m * (16 / TW) + r / TW) * (TW + 2) + 1 + r % TW;
  }
#pragma unroll 1
  for (int s = 0; s < 9 / NTB; ++s) {
    if (s > 0) __syncthreads();  // the previous taps' weights have been consumed
    wstore();
    __syncthreads();
    if (s + 1 < 9 / NTB) wload(s + 1);
#pragma unroll
    for (int tt = 0; tt < NTB; ++tt) {
      const int t = NTB * s + tt;
      int dy = t / 3 - 1, dx = t % 3 - 1;
      if (a.flip) {
        dy = -dy;
        dx = -dx;
      }
      const int sh = dy * (TW + 2) + dx;
#pragma unroll
      for (int c = 0; c < CIN; c += 32) {
        bf16x8 av[MT];
#pragma unroll
        for (int u = 0; u < MT; ++u)
          av[u] = __builtin_bit_cast(bf16x8, *(const u32x4*)&xs[(prow[u] + sh) * PS + c + kq * 8]);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const bf16x8 bv = __builtin_bit_cast(
              bf16x8, *(const u32x4*)&ws[(tt * COT + 16 * j + r) * PS + c + kq * 8]);
#pragma unroll
          for (int u = 0; u < MT; ++u)
            acc[u][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u], bv, acc[u][j], 0, 0, 0);
        }
      }
    }
  }
  // lane holds rows 4 kq + v (pixels) of column r (channel) of each tile; the
  // bfloat16 tile goes through LDS so that memory sees whole 16-byte vectors
  __syncthreads();
  constexpr int OS = C::OS;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int co = co0 + 16 * j + r;
    const float bb = a.bias ? a.bias[co] : 0.f;
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int pp = (wave * MT + u) * 16 + 4 * kq + v;  // pixel of the tile, row-major
        float val = acc[u][j][v] + bb;
        if (a.relu) val = fmaxf(val, 0.f);
        sm[pp * OS + 16 * j + r] = f2bf(val);
        if (a.out_f32 && co == 0)
          a.out_f32[(int64_t)img * hw + (int64_t)(y0 + pp / TW) * a.w + x0 + pp % TW] = val;
      }
  }
  if (!a.out && !a.out2) return;
  __syncthreads();
  constexpr int VN = TH * TW * (COT / 8);
#pragma unroll 2
  for (int i = tid; i < VN; i += 256) {
    const int pp = i / (COT / 8), cc = i - pp * (COT / 8);
    const int64_t g = ((int64_t)img * hw + (int64_t)(y0 + pp / TW) * a.w + x0 + pp % TW) * a.cout +
                      co0 + cc * 8;
    const u32x4 v = *(const u32x4*)&sm[pp * OS + cc * 8];
    u32x4 q = v;
    if (a.skip) {
      float f[8], k[8];
      unpack8(v, f);
      unpack8(*(const u32x4*)(a.skip + g), k);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] += k[e];
      q = pack8(f);
    } else if (a.mask) {
      q = mask8(v, *(const u32x4*)(a.mask + g));
    }
    if (a.out2) {
      *(u32x4*)(a.out2 + g) = q;
      if (a.out) *(u32x4*)(a.out + g) = v;
    } else {
      *(u32x4*)(a.out + g) = q;
    }
  }
}

// ---------------------------------------------------------------------------
// weight gradient: part[chunk][t][ci][co] = sum over the chunk's pixels p of
// in[p + tap t][ci] g[p][co]
// ---------------------------------------------------------------------------

struct WgradArgs {
  const uint16_t* in;  // [P][cin]
  const uint16_t* g;   // [P][cout]
  float* part;         // [nch][9][cin][cout]
  float* part_b;       // [chunks of the bias sums][cout]
  int h, w, cin, cout;
  int cs, gcs;         // channels of a pixel of in and g in memory (see ConvArgs)
  int up;              // in is at half resolution, read at (y/2, x/2)
  int nch;             // pixel chunks of the weight gradient
  int64_t chunk;       // pixels per chunk, a multiple of 64
  int64_t chunk_b;     // pixels per chunk of the bias sums
};

// bias gradient partials: part[chunk][co] = sum over the chunk of g[p][co].
// A thread reads 8 channels of one pixel per step (16-byte loads, whole
// pixels per step across the block); the per-thread sums are then added
// over the block's pixel lanes in LDS (red: 2048 floats).
__device__ __forceinline__ void column_sums(const uint16_t* __restrict__ g, int cout, int gcs, int64_t chunk, int c,
                                            float* __restrict__ part, float* red) {
  const int vpp = cout / 8;            // 16-byte vectors per pixel
  const int ppi = 256 / vpp;           // pixels per step
  const int lp = threadIdx.x / vpp, v = threadIdx.x - lp * vpp;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int64_t pbeg = (int64_t)c * chunk;
  if (lp < ppi) {
    for (int64_t p = pbeg + lp; p < pbeg + chunk; p += ppi) {
      float f[8];
      unpack8(few_channels(g + p * gcs, 8 * v, gcs), f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += f[e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[threadIdx.x * 8 + e] = acc[e];
  __syncthreads();
  for (int co = threadIdx.x; co < cout; co += blockDim.x) {
    const int vv = co / 8, e = co - vv * 8;
    float sum = 0.f;
    for (int l = 0; l < ppi; ++l) sum += red[(l * vpp + vv) * 8 + e];
    part[(int64_t)c * cout + co] = sum;
  }
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
// Four pixels of one channel: LDS holds [pixel][channel]; each lane of a group
// of sixteen gives the address of a 4-channel run of one pixel (lane i: pixel
// i / 4, channels 4 (i % 4)), and gets its own channel's (lane % 16) values of
// the four pixels (ds_read_b64_tr_b16).
__device__ __forceinline__ s16x4 read_tr(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
}
__device__ __forceinline__ bf16x8 join8(s16x4 lo, s16x4 hi) {
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Blocks 0 .. nch * tiles - 1: one 32 x 32 (ci, co) tile of all nine taps over
// one pixel chunk.  Per 64-pixel slab (a run of a row, or whole rows of WR < 64
// pixels) the block stages the input with its border and the output gradient
// as they lie in memory, [pixel][channel], and reads them transposed: a tap is
// an offset of the address.  (Transposing on the way in took 80 two-byte LDS
// writes per thread and slab, and nine reads of the input.)  The next slab's
// loads are in flight meanwhile.  Wave w owns the 16 x 16 sub-tile (w / 2,
// w % 2) of every tap.  Bound: LDS reads, 20 of 8 bytes per lane for 9 matrix
// instructions; 32 -> 32 channels over a million pixels 102 to 53 us.
// The blocks after them sum the bias gradient.
template <int WR>
__global__ __launch_bounds__(256) void wgrad_kernel(WgradArgs a) {
  constexpr int R = 64 / WR, HP = (R + 2) * (WR + 2), PS = 40;
  constexpr int NL = (HP * 4 + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t sm[(HP + 64) * PS];
  uint16_t* xs = sm;
  uint16_t* gs = sm + HP * PS;
  static_assert((HP + 64) * PS * 2 >= 256 * 8 * 4, "the bias sums' scratch");
  const int ntc = a.cout / 32, tiles = (a.cin / 32) * ntc;
  const int blk = blockIdx.x;
  if (blk >= a.nch * tiles) {
    column_sums(a.g, a.cout, a.gcs, a.chunk_b, blk - a.nch * tiles, a.part_b, (float*)sm);
    return;
  }
  const int ch = blk % a.nch, tile = blk / a.nch;
  const int ci0 = (tile / ntc) * 32, co0 = (tile % ntc) * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int si = (wave >> 1) * 16, sj = (wave & 1) * 16;
  const int hw = a.h * a.w;
  const int ih = a.h >> a.up, iw = a.w >> a.up;
  f32x4 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 xv[NL], gv;
  auto load = [&](int64_t pb) {
    const int img = (int)(pb / hw), rem = (int)(pb - (int64_t)img * hw);
    const int y0 = rem / a.w, x0 = rem - y0 * a.w;
    const uint16_t* src = a.in + (int64_t)img * ih * iw * a.cs;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int i = min(tid + k * 256, HP * 4 - 1);
      const int px = i >> 2, cc = i & 3;
      const int yy = wrap(y0 - 1 + px / (WR + 2), a.h), xx = wrap(x0 - 1 + px % (WR + 2), a.w);
      xv[k] = few_channels(src + ((int64_t)(yy >> a.up) * iw + (xx >> a.up)) * a.cs, ci0 + cc * 8, a.cs);
    }
    gv = few_channels(a.g + (pb + (tid >> 2)) * a.gcs, co0 + (tid & 3) * 8, a.gcs);
  };
  // this lane's addresses in the two transposing reads of each half slab
  int xo[2][2], go[2][2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = 32 * ks + 8 * kq + 4 * h + (r >> 2);
      xo[ks][h] = ((i / WR + 1) * (WR + 2) + i % WR + 1) * PS + si + (r & 3) * 4;
      go[ks][h] = i * PS + sj + (r & 3) * 4;
    }
  const int64_t pbeg = (int64_t)ch * a.chunk, pend = pbeg + a.chunk;
  load(pbeg);
  for (int64_t pb = pbeg; pb < pend; pb += 64) {
    __syncthreads();  // the previous slab has been consumed
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int i = tid + k * 256;
      if (i < HP * 4) *(u32x4*)&xs[(i >> 2) * PS + (i & 3) * 8] = xv[k];
    }
    *(u32x4*)&gs[(tid >> 2) * PS + (tid & 3) * 8] = gv;
    __syncthreads();
    if (pb + 64 < pend) load(pb + 64);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8 bv = join8(read_tr(&gs[go[ks][0]]), read_tr(&gs[go[ks][1]]));
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int sh = ((t / 3 - 1) * (WR + 2) + t % 3 - 1) * PS;
        const bf16x8 av = join8(read_tr(&xs[xo[ks][0] + sh]), read_tr(&xs[xo[ks][1] + sh]));
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[t], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    float* dst = a.part + (((int64_t)ch * 9 + t) * a.cin + ci0 + si) * a.cout + co0 + sj;
#pragma unroll
    for (int v = 0; v < 4; ++v) dst[(int64_t)(4 * kq + v) * a.cout + r] = acc[t][v];
  }
}

// out[i] = sum_c part[c][i] in a fixed order.  A block takes 32 consecutive
// i and 8 groups of chunks (group g sums chunks g, g+8, ..., loading sixteen
// before it adds the first); the 8 group sums are then added in order.  The
// blocks from nb on do the same for the second pair of arrays.
struct SumArgs {
  const float* part;
  float* out;
  int64_t n;
  int nchunk;
};
__global__ __launch_bounds__(256) void chunk_sum_kernel(SumArgs a, SumArgs b, int nb) {
  __shared__ float sh[8][32];
  const bool second = (int)blockIdx.x >= nb;
  const SumArgs s_ = second ? b : a;
  const int li = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int64_t n = s_.n, i = (int64_t)(blockIdx.x - (second ? nb : 0)) * 32 + li;
  float s = 0.f;
  if (i < n) {
    constexpr int U = 16;
    for (int c0 = grp; c0 < s_.nchunk; c0 += 8 * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = s_.part[(int64_t)min(c0 + 8 * u, s_.nchunk - 1) * n + i];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + 8 * u < s_.nchunk) s += v[u];
    }
  }
  sh[grp][li] = s;
  __syncthreads();
  if (grp == 0 && i < n) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 8; ++g) t += sh[g][li];
    s_.out[i] = t;
  }
}

// ---------------------------------------------------------------------------
// resampling and elementwise work on [P][C] bfloat16 (8 channels per thread)
// ---------------------------------------------------------------------------

enum Ew { EW_POOL = 0, EW_UP_ADJ = 1, EW_ADD_POOL_ADJ = 2 };

// One thread per 8 channels of one output pixel.  Sizes (oh, ow) are the
// output's; the coarse/fine partner is at half/double resolution.
//   POOL         out[y][x] = mean of in[2y+a][2x+b]
//   UP_ADJ       out[y][x] = sum of in[2y+a][2x+b], where mask > 0
//   ADD_POOL_ADJ out[y][x] = out[y][x] + in[y/2][x/2] / 4, where mask > 0
__global__ void ew_kernel(int op, const uint16_t* in, const uint16_t* mask, uint16_t* out, int64_t npix,
                          int oh, int ow, int c) {
  const int c8 = c / 8;
  const int64_t total = npix * c8;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = i / c8;
    const int cc = (int)(i - p * c8) * 8;
    const int64_t img = p / ((int64_t)oh * ow);
    const int rem = (int)(p - img * oh * ow);
    const int y = rem / ow, x = rem - (rem / ow) * ow;
    float f[8], g[8];
    if (op == EW_POOL || op == EW_UP_ADJ) {
      const int ih = 2 * oh, iw = 2 * ow;
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = 0.f;
#pragma unroll
      for (int a2 = 0; a2 < 2; ++a2)
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
          const int64_t q = (img * ih + 2 * y + a2) * iw + 2 * x + b2;
          unpack8(*(const u32x4*)(in + q * c + cc), g);
#pragma unroll
          for (int e = 0; e < 8; ++e) f[e] += g[e];
        }
      if (op == EW_POOL)
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] *= 0.25f;
    } else {
      const int ih = oh / 2, iw = ow / 2;
      const int64_t q = (img * ih + y / 2) * iw + x / 2;
      unpack8(*(const u32x4*)(in + q * c + cc), f);
      unpack8(*(const u32x4*)(out + p * c + cc), g);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = g[e] + 0.25f * f[e];
    }
    u32x4 v = pack8(f);
    if (mask) v = mask8(v, *(const u32x4*)(mask + p * c + cc));
    *(u32x4*)(out + p * c + cc) = v;
  }
}

// ---------------------------------------------------------------------------
// features, targets, loss, output scaling
// ---------------------------------------------------------------------------

// per-block partial sums of N_pix and of the observed count over a slice
// of map blockIdx.x (gridDim.y slices per map): part[m][slice][2]
template <class T>
__global__ __launch_bounds__(256) void sigma_kernel(const T* __restrict__ npix,
                                                    const uint8_t* __restrict__ mask, int64_t hw,
                                                    double* __restrict__ part) {
  __shared__ double ss[256], sc[256];
  const int64_t base = (int64_t)blockIdx.x * hw;
  const int64_t len = hw / gridDim.y, beg = (int64_t)blockIdx.y * len;
  double s = 0.0, c = 0.0;
  for (int64_t i = beg + threadIdx.x; i < beg + len; i += blockDim.x) {
    const bool o = mask ? mask[base + i] != 0 : true;
    if (o) {
      s += (double)npix[base + i];
      c += 1.0;
    }
  }
  ss[threadIdx.x] = s;
  sc[threadIdx.x] = c;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) {
      ss[threadIdx.x] += ss[threadIdx.x + k];
      sc[threadIdx.x] += sc[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* o = part + 2 * ((int64_t)blockIdx.x * gridDim.y + blockIdx.y);
    o[0] = ss[0];
    o[1] = sc[0];
  }
}

// sig2[m] = (sum of N_pix) / (observed count) over map m's slices, in order
__global__ void sigma_final_kernel(const double* __restrict__ part, int slices, int nb,
                                   double* __restrict__ sig2) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nb) return;
  double s = 0.0, c = 0.0;
  for (int k = 0; k < slices; ++k) {
    s += part[2 * ((int64_t)m * slices + k)];
    c += part[2 * ((int64_t)m * slices + k) + 1];
  }
  sig2[m] = c > 0 ? s / c : 1.0;
}

// rowm[r] = mean over the observed pixels of row r (of all maps) of d, or 0
template <class T>
__global__ __launch_bounds__(256) void rowmean_kernel(const T* __restrict__ d,
                                                      const uint8_t* __restrict__ mask, int w,
                                                      double* __restrict__ rowm) {
  __shared__ double ss[256], sc[256];
  const int64_t base = (int64_t)blockIdx.x * w;
  double s = 0.0, c = 0.0;
  for (int i = threadIdx.x; i < w; i += blockDim.x) {
    if (mask ? mask[base + i] != 0 : true) {
      s += (double)d[base + i];
      c += 1.0;
    }
  }
  ss[threadIdx.x] = s;
  sc[threadIdx.x] = c;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) {
      ss[threadIdx.x] += ss[threadIdx.x + k];
      sc[threadIdx.x] += sc[threadIdx.x + k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) rowm[blockIdx.x] = sc[0] > 0 ? ss[0] / sc[0] : 0.0;
}

// x [P][8] bf16: d/sigma, log(N/sigma^2), mask, row mean of d/sigma, zeros;
// tgt[p] = s/sigma
template <class T>
__global__ void features_kernel(const T* __restrict__ d, const T* __restrict__ npix,
                                const uint8_t* __restrict__ mask, const T* __restrict__ s,
                                const double* __restrict__ sig2, const double* __restrict__ rowm,
                                int w, int64_t hw, int64_t P, uint16_t* __restrict__ x,
                                float* __restrict__ tgt) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P;
       p += (int64_t)gridDim.x * blockDim.x) {
    const double v2 = sig2[p / hw];
    const double sg = sqrt(v2);
    const bool o = mask ? mask[p] != 0 : true;
    float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f[3] = (float)(rowm[p / w] / sg);
    if (o) {
      f[0] = (float)((double)d[p] / sg);
      f[1] = (float)log((double)npix[p] / v2);
      f[2] = 1.f;
    }
    *(u32x4*)(x + p * kFew) = pack8(f);
    if (s && tgt) tgt[p] = (float)((double)s[p] / sg);
  }
}

// x [P][8] bf16 from caller features [P][4] float
__global__ void raw_features_kernel(const float* __restrict__ f4, int64_t P, uint16_t* __restrict__ x) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P;
       p += (int64_t)gridDim.x * blockDim.x) {
    float f[8] = {f4[4 * p], f4[4 * p + 1], f4[4 * p + 2], f4[4 * p + 3], 0.f, 0.f, 0.f, 0.f};
    *(u32x4*)(x + p * kFew) = pack8(f);
  }
}

// partial sums of (y - t)^2 and the output gradient g [P][8] (channel 0)
__global__ __launch_bounds__(256) void loss_kernel(const float* __restrict__ y, const float* __restrict__ t,
                                                   int64_t P, uint16_t* __restrict__ g,
                                                   double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0.0;
  const float sc = (float)(2.0 / (double)P);
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P;
       p += (int64_t)gridDim.x * blockDim.x) {
    const float e = y[p] - t[p];
    s += (double)e * (double)e;
    float f[8] = {sc * e, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    *(u32x4*)(g + p * kFew) = pack8(f);
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// one block of 256 threads: strided partial sums, then a fixed-order tree
__global__ __launch_bounds__(256) void loss_final_kernel(const double* __restrict__ part, int n, int64_t P,
                                                         double* out) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0] / (double)P;
}

template <class T>
__global__ void scale_out_kernel(const float* __restrict__ y, const double* __restrict__ sig2,
                                 int64_t hw, int64_t P, T* __restrict__ s) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < P;
       p += (int64_t)gridDim.x * blockDim.x)
    s[p] = (T)(sqrt(sig2[p / hw]) * (double)y[p]);
}

// ---------------------------------------------------------------------------
// optimiser and weight packing
// ---------------------------------------------------------------------------

// where each layer's weights lie in the parameter vector and in the two
// bfloat16 copies that the convolutions read
struct PackArgs {
  struct Item {
    int64_t w_off;
    int ci, co;
    uint16_t* w_orig;  // [9][ci][co]
    uint16_t* wt;      // [9][co][ci]
  } l[kLayers];
  int64_t n;           // parameters
};

// Adam on every parameter (or, step 0, none), and the bfloat16 copies of the
// weights; one launch for all layers.
__global__ void adam_pack_kernel(PackArgs a, int step, float* __restrict__ prm, const float* __restrict__ g,
                                 float* __restrict__ m, float* __restrict__ v, float lr, float c1, float c2) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    float p = prm[i];
    if (step) {
      const float gi = g[i];
      const float mi = b1 * m[i] + (1.f - b1) * gi;
      const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
      m[i] = mi;
      v[i] = vi;
      p -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
      prm[i] = p;
    }
    int k = 0;
#pragma unroll
    for (int j = 1; j < kLayers; ++j) k = i >= a.l[j].w_off ? j : k;
    const PackArgs::Item& ly = a.l[k];
    const int64_t o = i - ly.w_off;
    if (o < (int64_t)9 * ly.ci * ly.co) {  // a weight, not a bias
      const int t = (int)(o / ((int64_t)ly.ci * ly.co));
      const int rem = (int)(o - (int64_t)t * ly.ci * ly.co);
      const int ci = rem / ly.co, co = rem - ci * ly.co;
      const uint16_t h = f2bf(p);
      ly.w_orig[o] = h;
      ly.wt[((int64_t)t * ly.co + co) * ly.ci + ci] = h;
    }
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

wf_status from_hip(hipError_t e) {
  if (e == hipSuccess) return WF_OK;
  if (e == hipErrorOutOfMemory) return WF_ENOMEM;
  return WF_EDEVICE;
}

#define NN_TRY(expr)                                \
  do {                                              \
    hipError_t e_ = (expr);                         \
    if (e_ != hipSuccess) return from_hip(e_);      \
  } while (0)

int grid_for(int64_t n, int block = 256, int cap = 8192) {
  int64_t g = (n + block - 1) / block;
  return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

// What a convolution does with its result (see ConvArgs).
struct ConvOut {
  uint16_t* out = nullptr;
  uint16_t* out2 = nullptr;
  const uint16_t* skip = nullptr;
  const uint16_t* mask = nullptr;
  float* f32 = nullptr;
  bool relu = false;
};

template <int CIN, int COT>
hipError_t conv_tiles(const ConvArgs& a, int64_t P, int ny, hipStream_t st) {
  // tiles of 16 x 16 pixels (8 x 16 from 96 input channels on, whose border
  // takes the LDS of two blocks otherwise), smaller ones where the image is
  // smaller or the launch would leave CUs idle
  if (a.w < 16) {
    if (a.w != 8 || a.h % 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL((conv_kernel<CIN, COT, 8, 1>), dim3((unsigned)(P / 64), ny), dim3(256), 0, st, a);
  } else if (CIN <= 64 && a.h % 16 == 0 && P / 256 * ny >= 512) {
    if constexpr (CIN <= 64)
      hipLaunchKernelGGL((conv_kernel<CIN, COT, 16, 4>), dim3((unsigned)(P / 256), ny), dim3(256), 0, st, a);
  } else if (a.h % 8 == 0) {
    hipLaunchKernelGGL((conv_kernel<CIN, COT, 16, 2>), dim3((unsigned)(P / 128), ny), dim3(256), 0, st, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int CIN>
hipError_t conv_cin(const ConvArgs& a, int64_t P, hipStream_t st) {
  if (!a.out && !a.out2) {  // channel 0 alone
    if constexpr (CIN == kChan[0]) return conv_tiles<CIN, 16>(a, P, 1, st);
    return hipErrorInvalidValue;
  }
  if (a.cout == 96) return conv_tiles<CIN, 96>(a, P, 1, st);
  if (a.cout % 64 == 0) return conv_tiles<CIN, 64>(a, P, a.cout / 64, st);
  return conv_tiles<CIN, 32>(a, P, a.cout / 32, st);
}

hipError_t conv(const uint16_t* in, const uint16_t* wt, const float* bias, const ConvOut& o, int64_t P, int h,
                int w, int cin, int cout, bool flip, bool up, hipStream_t st, bool few = false) {
  const ConvArgs a{in, wt, bias, o.out, o.out2, o.skip, o.mask, o.f32, h, w, cout, few ? kFew : cin,
                   up ? 1 : 0, flip ? 1 : 0, o.relu ? 1 : 0};
  switch (cin) {
    case 32: return conv_cin<32>(a, P, st);
    case 64: return conv_cin<64>(a, P, st);
    case 96: return conv_cin<96>(a, P, st);
    case 128: return conv_cin<128>(a, P, st);
    default: return hipErrorInvalidValue;
  }
}

// number of pixel chunks: the largest divisor of the 64-pixel slab count
// that is at most cap, so every chunk is a whole number of slabs
int chunks(int64_t P, int cap) {
  const int64_t slabs = P / 64;
  for (int c = cap; c > 1; --c)
    if (slabs % c == 0) return c;
  return 1;
}
// capacity of the weight-gradient partial buffer, in floats
constexpr int64_t kPartFloats = (int64_t)64 * 9 * 128 * 128;

// pixel chunks of the weight gradient: about 1024 blocks in all (more
// chunks mean more partial sums to add afterwards), within the partial buffer
int wgrad_chunks(int64_t P, int cin, int cout) {
  const int tiles = (cin / 32) * (cout / 32);
  const int64_t want = (1024 + tiles - 1) / tiles;
  const int64_t cap = kPartFloats / ((int64_t)9 * cin * cout);
  return chunks(P, (int)std::min(want, cap));
}

// weight gradient, and with db the bias gradient
hipError_t wgrad(const uint16_t* in, const uint16_t* g, float* part, float* dw, float* db, int64_t P, int h,
                 int w, int cin, int cout, bool up, hipStream_t st, int cs = 0, int gcs = 0) {
  const int nch = wgrad_chunks(P, cin, cout), tiles = (cin / 32) * (cout / 32);
  const int nchb = db ? chunks(P, 256) : 0;
  const int64_t n = (int64_t)9 * cin * cout;
  float* part_b = part + (int64_t)nch * n;
  const WgradArgs a{in, g, part, part_b, h, w, cin, cout, cs ? cs : cin, gcs ? gcs : cout,
                    up ? 1 : 0, nch, P / nch, db ? P / nchb : 0};
  const dim3 grid(nch * tiles + nchb);
  if (w >= 64)
    hipLaunchKernelGGL(wgrad_kernel<64>, grid, dim3(256), 0, st, a);
  else if (w == 32)
    hipLaunchKernelGGL(wgrad_kernel<32>, grid, dim3(256), 0, st, a);
  else if (w == 16)
    hipLaunchKernelGGL(wgrad_kernel<16>, grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(wgrad_kernel<8>, grid, dim3(256), 0, st, a);
  const int nb = (int)((n + 31) / 32), nbb = db ? (cout + 31) / 32 : 0;
  hipLaunchKernelGGL(chunk_sum_kernel, dim3(nb + nbb), dim3(256), 0, st, SumArgs{part, dw, n, nch},
                     SumArgs{part_b, db, cout, nchb}, nb);
  return hipGetLastError();
}

hipError_t ew(int op, const uint16_t* in, const uint16_t* mask, uint16_t* out, int64_t npix, int oh, int ow,
              int c, hipStream_t st) {
  hipLaunchKernelGGL(ew_kernel, dim3(grid_for(npix * (c / 8))), dim3(256), 0, st, op, in, mask, out, npix,
                     oh, ow, c);
  return hipGetLastError();
}

struct Layer {
  int ci, co;
  int64_t w_off, b_off;
  uint16_t* w_orig = nullptr;  // [9][ci][co]
  uint16_t* wt = nullptr;      // [9][co][ci]
};

std::vector<Layer> layer_table(int64_t* total) {
  std::vector<std::pair<int, int>> s;
  s.push_back({kPad, kChan[0]});
  s.push_back({kChan[0], kChan[0]});
  for (int l = 1; l < kLevels; ++l) {
    s.push_back({kChan[l - 1], kChan[l]});
    s.push_back({kChan[l], kChan[l]});
  }
  for (int l = kLevels - 2; l >= 0; --l) {
    s.push_back({kChan[l + 1], kChan[l]});
    s.push_back({kChan[l], kChan[l]});
  }
  s.push_back({kChan[0], kPad});
  std::vector<Layer> L;
  int64_t off = 0;
  for (auto& pr : s) {
    Layer ly;
    ly.ci = pr.first;
    ly.co = pr.second;
    ly.w_off = off;
    off += (int64_t)9 * ly.ci * ly.co;
    ly.b_off = off;
    off += ly.co;
    L.push_back(ly);
  }
  *total = off;
  return L;
}

struct Net {
  int h = 0, w = 0, nmax = 0, prec = 0;
  std::vector<Layer> L;
  int64_t nparam = 0;
  int adam_t = 0;
  float* prm = nullptr;
  float* grad = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  // activations per level (P_l = nmax * (h >> l) * (w >> l) pixels)
  uint16_t* x = nullptr;                 // features [P_0][8]
  uint16_t* ein[kLevels] = {};           // encoder input (l > 0: pooled)
  uint16_t* eh[kLevels] = {};
  uint16_t* ee[kLevels] = {};
  uint16_t* db[kLevels] = {};            // decoder (l < L-1)
  uint16_t* dc[kLevels] = {};
  uint16_t* du[kLevels] = {};
  uint16_t* gen[kLevels] = {};           // gradient with respect to e_l
  uint16_t* g1[kLevels] = {};            // gradient scratch, 128 channels
  uint16_t* g2[kLevels] = {};
  uint16_t* gy = nullptr;                // [P_0][8]
  float* yf = nullptr;                   // [P_0]
  float* tgt = nullptr;                  // [P_0]
  double* sig2 = nullptr;                // [nmax]
  double* rowm = nullptr;                // [nmax * h] row means of d
  float* part = nullptr;                 // weight-gradient chunk partials
  double* lpart = nullptr;               // loss partials
  double* loss = nullptr;
  double* h_loss = nullptr;              // pinned
  std::vector<void*> owned;
};

void free_net(Net* n) {
  for (void* p : n->owned)
    if (p) (void)hipFree(p);
  if (n->h_loss) (void)hipHostFree(n->h_loss);
  delete n;
}

template <class P>
wf_status nalloc(Net* n, P** ptr, size_t bytes) {
  void* q = nullptr;
  hipError_t e = hipMalloc(&q, bytes);
  if (e != hipSuccess) return from_hip(e);
  n->owned.push_back(q);
  *ptr = (P*)q;
  return WF_OK;
}

wf_status create_net(const wf_nn_shape* s, Net** out) {
  Net* n = new (std::nothrow) Net();
  if (!n) return WF_ENOMEM;
  n->h = s->h;
  n->w = s->w;
  n->nmax = s->batch_max;
  n->prec = s->precision;
  n->L = layer_table(&n->nparam);
  wf_status st = WF_OK;
#define NA(ptr, bytes)                                  \
  if ((st = nalloc(n, &(ptr), (bytes))) != WF_OK) {     \
    free_net(n);                                        \
    return st;                                          \
  }
  NA(n->prm, n->nparam * 4);
  NA(n->grad, n->nparam * 4);
  NA(n->m, n->nparam * 4);
  NA(n->v, n->nparam * 4);
  for (auto& ly : n->L) {
    NA(ly.w_orig, (size_t)9 * ly.ci * ly.co * 2);
    NA(ly.wt, (size_t)9 * ly.ci * ly.co * 2);
  }
  const int64_t P0 = (int64_t)n->nmax * n->h * n->w;
  NA(n->x, P0 * kFew * 2);
  for (int l = 0; l < kLevels; ++l) {
    const int64_t Pl = P0 >> (2 * l);
    const int c = kChan[l];
    const int cprev = l > 0 ? kChan[l - 1] : kPad;
    if (l > 0) NA(n->ein[l], Pl * cprev * 2);
    NA(n->eh[l], Pl * c * 2);
    NA(n->ee[l], Pl * c * 2);
    if (l < kLevels - 1) {
      NA(n->db[l], Pl * c * 2);
      NA(n->dc[l], Pl * c * 2);
      NA(n->du[l], Pl * c * 2);
    }
    NA(n->gen[l], Pl * c * 2);
    NA(n->g1[l], Pl * 128 * 2);
    NA(n->g2[l], Pl * 128 * 2);
  }
  n->ein[0] = n->x;
  NA(n->gy, P0 * kFew * 2);
  NA(n->yf, P0 * 4);
  NA(n->tgt, P0 * 4);
  NA(n->sig2, n->nmax * 8);
  NA(n->rowm, (size_t)n->nmax * n->h * 8);
  NA(n->part, (size_t)(kPartFloats + 256 * 128) * 4);  // and the bias sums' partials
  NA(n->lpart, 1024 * 8);
  NA(n->loss, 8);
#undef NA
  hipError_t e = hipHostMalloc((void**)&n->h_loss, 8, hipHostMallocDefault);
  if (e == hipSuccess) e = hipMemset(n->prm, 0, n->nparam * 4);
  if (e == hipSuccess) e = hipMemset(n->m, 0, n->nparam * 4);
  if (e == hipSuccess) e = hipMemset(n->v, 0, n->nparam * 4);
  if (e != hipSuccess) {
    free_net(n);
    return from_hip(e);
  }
  *out = n;
  return WF_OK;
}

// one Adam step with learning rate lr (or, lr = 0, none) and the weights' copies
hipError_t adam_pack(Net* n, float lr, hipStream_t st) {
  PackArgs a;
  for (int k = 0; k < kLayers; ++k) a.l[k] = {n->L[k].w_off, n->L[k].ci, n->L[k].co, n->L[k].w_orig, n->L[k].wt};
  a.n = n->nparam;
  float c1 = 0.f, c2 = 0.f;
  if (lr > 0.f) {
    n->adam_t += 1;
    c1 = (float)(1.0 / (1.0 - std::pow(0.9, n->adam_t)));
    c2 = (float)(1.0 / (1.0 - std::pow(0.999, n->adam_t)));
  }
  hipLaunchKernelGGL(adam_pack_kernel, dim3(grid_for(n->nparam)), dim3(256), 0, st, a, lr > 0.f ? 1 : 0, n->prm,
                     n->grad, n->m, n->v, lr, c1, c2);
  return hipGetLastError();
}

// forward pass of nb maps from n->x into n->yf; keep: every activation that the
// backward pass needs is stored (the decoder's b_l among them)
wf_status forward(Net* n, int nb, bool keep, hipStream_t st) {
  const int64_t P0 = (int64_t)nb * n->h * n->w;
  int k = 0;
  auto relu = [](uint16_t* out) {
    ConvOut o;
    o.out = out;
    o.relu = true;
    return o;
  };
  for (int l = 0; l < kLevels; ++l) {
    const int64_t Pl = P0 >> (2 * l);
    const int hl = n->h >> l, wl = n->w >> l;
    const int cin = l > 0 ? kChan[l - 1] : kPad;
    if (l > 0) NN_TRY(ew(EW_POOL, n->ee[l - 1], nullptr, n->ein[l], Pl, hl, wl, cin, st));
    const Layer& a = n->L[k];
    const Layer& b = n->L[k + 1];
    NN_TRY(conv(n->ein[l], a.wt, n->prm + a.b_off, relu(n->eh[l]), Pl, hl, wl, a.ci, a.co, false, false, st,
                l == 0));
    NN_TRY(conv(n->eh[l], b.wt, n->prm + b.b_off, relu(n->ee[l]), Pl, hl, wl, b.ci, b.co, false, false, st));
    k += 2;
  }
  const uint16_t* u = n->ee[kLevels - 1];
  for (int l = kLevels - 2; l >= 0; --l) {
    const int64_t Pl = P0 >> (2 * l);
    const int hl = n->h >> l, wl = n->w >> l;
    const Layer& a = n->L[k];
    const Layer& b = n->L[k + 1];
    // b_l = R(conv(up(u))), c_l = b_l + e_l
    ConvOut o = relu(keep ? n->db[l] : nullptr);
    o.out2 = n->dc[l];
    o.skip = n->ee[l];
    NN_TRY(conv(u, a.wt, n->prm + a.b_off, o, Pl, hl, wl, a.ci, a.co, false, true, st));
    NN_TRY(conv(n->dc[l], b.wt, n->prm + b.b_off, relu(n->du[l]), Pl, hl, wl, b.ci, b.co, false, false, st));
    u = n->du[l];
    k += 2;
  }
  const Layer& y = n->L[k];
  ConvOut o;
  o.f32 = n->yf;
  NN_TRY(conv(u, y.wt, n->prm + y.b_off, o, P0, n->h, n->w, y.ci, y.co, false, false, st));
  return WF_OK;
}

// loss against n->tgt and the gradient of every parameter into n->grad.  A
// gradient is masked by its layer's ReLU where it is formed: in the adjoint
// convolution that makes it, or in the resampling's adjoint.
wf_status backward(Net* n, int nb, hipStream_t st) {
  const int64_t P0 = (int64_t)nb * n->h * n->w;
  const int nlp = grid_for(P0, 256, 1024);
  hipLaunchKernelGGL(loss_kernel, dim3(nlp), dim3(256), 0, st, n->yf, n->tgt, P0, n->gy, n->lpart);
  hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, st, n->lpart, nlp, P0, n->loss);
  NN_TRY(hipGetLastError());
  // adjoint of layer ly in its input, masked where the activation is not positive
  auto adjoint = [&](const Layer& ly, const uint16_t* g, uint16_t* out, uint16_t* masked,
                     const uint16_t* act, int64_t P, int h, int w, bool few = false) {
    ConvOut o;
    o.out = out ? out : masked;
    o.out2 = out ? masked : nullptr;
    o.mask = act;
    return conv(g, ly.w_orig, nullptr, o, P, h, w, ly.co, ly.ci, true, false, st, few);
  };
  int k = kLayers - 1;
  uint16_t* gu = n->g1[0];  // gradient of u_l's pre-activation
  {
    const Layer& o = n->L[k];
    NN_TRY(wgrad(n->du[0], n->gy, n->part, n->grad + o.w_off, n->grad + o.b_off, P0, n->h, n->w, o.ci, o.co, false,
                 st, 0, kFew));
    NN_TRY(adjoint(o, n->gy, nullptr, gu, n->du[0], P0, n->h, n->w, true));
  }
  k -= 1;
  for (int l = 0; l < kLevels - 1; ++l) {
    const int64_t Pl = P0 >> (2 * l);
    const int hl = n->h >> l, wl = n->w >> l;
    const Layer& b = n->L[k];      // second convolution of decoder level l
    const Layer& a = n->L[k - 1];  // first one
    NN_TRY(wgrad(n->dc[l], gu, n->part, n->grad + b.w_off, n->grad + b.b_off, Pl, hl, wl, b.ci, b.co, false, st));
    // gradient with respect to c_l = b_l + e_l: to the skip, and to b_l
    uint16_t* gb = n->g2[l];
    NN_TRY(adjoint(b, gu, n->gen[l], gb, n->db[l], Pl, hl, wl));
    NN_TRY(wgrad(l + 1 < kLevels - 1 ? n->du[l + 1] : n->ee[l + 1], gb, n->part, n->grad + a.w_off, n->grad + a.b_off, Pl, hl, wl,
                 a.ci, a.co, true, st));
    uint16_t* ga = n->g1[l];
    NN_TRY(adjoint(a, gb, ga, nullptr, nullptr, Pl, hl, wl));
    // adjoint of the upsampling: gradient with respect to u_{l+1}
    const bool top = l + 1 == kLevels - 1;
    gu = top ? n->gen[l + 1] : n->g1[l + 1];
    NN_TRY(ew(EW_UP_ADJ, ga, top ? n->ee[l + 1] : n->du[l + 1], gu, Pl >> 2, hl / 2, wl / 2, kChan[l + 1], st));
    k -= 2;
  }
  // gen[l]: gradient of e_l's pre-activation
  for (int l = kLevels - 1; l >= 0; --l) {
    const int64_t Pl = P0 >> (2 * l);
    const int hl = n->h >> l, wl = n->w >> l;
    const Layer& a = n->L[2 * l];
    const Layer& b = n->L[2 * l + 1];
    NN_TRY(wgrad(n->eh[l], n->gen[l], n->part, n->grad + b.w_off, n->grad + b.b_off, Pl, hl, wl, b.ci, b.co, false, st));
    NN_TRY(adjoint(b, n->gen[l], nullptr, n->g1[l], n->eh[l], Pl, hl, wl));
    NN_TRY(wgrad(n->ein[l], n->g1[l], n->part, n->grad + a.w_off, n->grad + a.b_off, Pl, hl, wl, a.ci, a.co, false, st,
                 l == 0 ? kFew : 0));
    if (l > 0) {
      NN_TRY(adjoint(a, n->g1[l], n->g2[l], nullptr, nullptr, Pl, hl, wl));
      NN_TRY(ew(EW_ADD_POOL_ADJ, n->g2[l], n->ee[l - 1], n->gen[l - 1], Pl << 2, hl * 2, wl * 2, kChan[l - 1], st));
    }
  }
  return WF_OK;
}

template <class T>
wf_status prepare(Net* n, int nb, const void* d, const void* npix, const uint8_t* mask, const void* s,
                  hipStream_t st) {
  const int64_t hw = (int64_t)n->h * n->w, P0 = nb * hw;
  constexpr int kSlices = 128;  // divides every supported map size
  hipLaunchKernelGGL(sigma_kernel<T>, dim3(nb, kSlices), dim3(256), 0, st, (const T*)npix, mask, hw,
                     (double*)n->part);
  hipLaunchKernelGGL(sigma_final_kernel, dim3((nb + 63) / 64), dim3(64), 0, st, (const double*)n->part,
                     kSlices, nb, n->sig2);
  hipLaunchKernelGGL(rowmean_kernel<T>, dim3(nb * n->h), dim3(256), 0, st, (const T*)d, mask, n->w, n->rowm);
  hipLaunchKernelGGL(features_kernel<T>, dim3(grid_for(P0)), dim3(256), 0, st, (const T*)d, (const T*)npix,
                     mask, (const T*)s, n->sig2, n->rowm, n->w, hw, P0, n->x, s ? n->tgt : nullptr);
  NN_TRY(hipGetLastError());
  return WF_OK;
}

wf_status read_loss(Net* n, double* loss, hipStream_t st) {
  NN_TRY(hipMemcpyAsync(n->h_loss, n->loss, 8, hipMemcpyDeviceToHost, st));
  NN_TRY(hipStreamSynchronize(st));
  if (loss) *loss = *n->h_loss;
  return WF_OK;
}

bool shape_ok(int h, int w) {
  auto p2 = [](int v) { return v >= 64 && v <= 2048 && (v & (v - 1)) == 0; };
  return p2(h) && p2(w);
}

}  // namespace wfnn

using namespace wfnn;

extern "C" {

int64_t wf_nn_param_count(void) {
  int64_t total = 0;
  (void)layer_table(&total);
  return total;
}

wf_status wf_nn_create(const wf_nn_shape* s, void** out) {
  if (!s || !out) return WF_EINVAL;
  *out = nullptr;
  if (s->precision != WF_F32 && s->precision != WF_F64) return WF_EINVAL;
  if (s->batch_max < 1 || s->batch_max > 4096) return WF_EINVAL;
  if (!shape_ok(s->h, s->w)) return WF_EUNSUPPORTED;
  Net* n = nullptr;
  wf_status st = create_net(s, &n);
  if (st == WF_OK) *out = n;
  return st;
}

void wf_nn_destroy(void* net) {
  if (net) free_net((Net*)net);
}

wf_status wf_nn_set_params(void* net, const float* params, hipStream_t stream) {
  Net* n = (Net*)net;
  if (!n || !params) return WF_EINVAL;
  NN_TRY(hipMemcpyAsync(n->prm, params, n->nparam * 4, hipMemcpyDeviceToDevice, stream));
  NN_TRY(hipMemsetAsync(n->m, 0, n->nparam * 4, stream));
  NN_TRY(hipMemsetAsync(n->v, 0, n->nparam * 4, stream));
  n->adam_t = 0;
  NN_TRY(adam_pack(n, 0.f, stream));
  NN_TRY(hipStreamSynchronize(stream));
  return WF_OK;
}

wf_status wf_nn_get_params(void* net, float* params, hipStream_t stream) {
  Net* n = (Net*)net;
  if (!n || !params) return WF_EINVAL;
  NN_TRY(hipMemcpyAsync(params, n->prm, n->nparam * 4, hipMemcpyDeviceToDevice, stream));
  NN_TRY(hipStreamSynchronize(stream));
  return WF_OK;
}

wf_status wf_nn_predict(void* net, int32_t nb, const void* d, const void* n_pix, const uint8_t* mask,
                        void* s_out, hipStream_t stream) {
  Net* n = (Net*)net;
  if (!n || !d || !n_pix || !s_out || nb < 1 || nb > n->nmax) return WF_EINVAL;
  const int64_t hw = (int64_t)n->h * n->w, P0 = nb * hw;
  wf_status st = n->prec == WF_F64 ? prepare<double>(n, nb, d, n_pix, mask, nullptr, stream)
                                   : prepare<float>(n, nb, d, n_pix, mask, nullptr, stream);
  if (st != WF_OK) return st;
  st = forward(n, nb, false, stream);
  if (st != WF_OK) return st;
  if (n->prec == WF_F64)
    hipLaunchKernelGGL(scale_out_kernel<double>, dim3(grid_for(P0)), dim3(256), 0, stream, n->yf, n->sig2, hw,
                       P0, (double*)s_out);
  else
    hipLaunchKernelGGL(scale_out_kernel<float>, dim3(grid_for(P0)), dim3(256), 0, stream, n->yf, n->sig2, hw,
                       P0, (float*)s_out);
  NN_TRY(hipGetLastError());
  NN_TRY(hipStreamSynchronize(stream));
  return WF_OK;
}

wf_status wf_nn_train_step(void* net, int32_t nb, const void* d, const void* n_pix, const uint8_t* mask,
                           const void* s_target, float lr, double* loss, hipStream_t stream) {
  Net* n = (Net*)net;
  if (!n || !d || !n_pix || !s_target || nb < 1 || nb > n->nmax) return WF_EINVAL;
  if (!(lr > 0.f) || !std::isfinite(lr)) return WF_EINVAL;
  wf_status st = n->prec == WF_F64 ? prepare<double>(n, nb, d, n_pix, mask, s_target, stream)
                                   : prepare<float>(n, nb, d, n_pix, mask, s_target, stream);
  if (st != WF_OK) return st;
  if ((st = forward(n, nb, true, stream)) != WF_OK) return st;
  if ((st = backward(n, nb, stream)) != WF_OK) return st;
  NN_TRY(adam_pack(n, lr, stream));
  return read_loss(n, loss, stream);
}

wf_status wf_nn_forward_features(void* net, int32_t nb, const float* x, float* y, hipStream_t stream) {
  Net* n = (Net*)net;
  if (!n || !x || !y || nb < 1 || nb > n->nmax) return WF_EINVAL;
  const int64_t P0 = (int64_t)nb * n->h * n->w;
  hipLaunchKernelGGL(raw_features_kernel, dim3(grid_for(P0)), dim3(256), 0, stream, x, P0, n->x);
  NN_TRY(hipGetLastError());
  wf_status st = forward(n, nb, false, stream);
  if (st != WF_OK) return st;
  NN_TRY(hipMemcpyAsync(y, n->yf, P0 * 4, hipMemcpyDeviceToDevice, stream));
  NN_TRY(hipStreamSynchronize(stream));
  return WF_OK;
}

wf_status wf_nn_gradient_features(void* net, int32_t nb, const float* x, const float* target, float* grad,
                                  double* loss, hipStream_t stream) {
  Net* n = (Net*)net;
  if (!n || !x || !target || !grad || nb < 1 || nb > n->nmax) return WF_EINVAL;
  const int64_t P0 = (int64_t)nb * n->h * n->w;
  hipLaunchKernelGGL(raw_features_kernel, dim3(grid_for(P0)), dim3(256), 0, stream, x, P0, n->x);
  NN_TRY(hipGetLastError());
  NN_TRY(hipMemcpyAsync(n->tgt, target, P0 * 4, hipMemcpyDeviceToDevice, stream));
  wf_status st = forward(n, nb, true, stream);
  if (st != WF_OK) return st;
  if ((st = backward(n, nb, stream)) != WF_OK) return st;
  NN_TRY(hipMemcpyAsync(grad, n->grad, n->nparam * 4, hipMemcpyDeviceToDevice, stream));
  return read_loss(n, loss, stream);
}

wf_status wf_nn_conv3x3(int32_t mode, int32_t nb, int32_t h, int32_t w, int32_t ci, int32_t co,
                        const uint16_t* in, const uint16_t* wt, const float* b, const uint16_t* g, void* out,
                        hipStream_t stream) {
  if (mode < 0 || mode > 3 || nb < 1 || !in || !out) return WF_EINVAL;
  if (ci < 32 || co < 32 || ci % 32 || co % 32 || ci > 128 || co > 128) return WF_EINVAL;
  if (h < 8 || w < 8 || (h & (h - 1)) || (w & (w - 1))) return WF_EINVAL;
  const int64_t P = (int64_t)nb * h * w;
  if (P % 64) return WF_EINVAL;
  if (mode == 3) {
    if (!g) return WF_EINVAL;
    float* part = nullptr;
    NN_TRY(hipMalloc((void**)&part, (size_t)wgrad_chunks(P, ci, co) * 9 * ci * co * 4));
    hipError_t e = wgrad(in, g, part, (float*)out, nullptr, P, h, w, ci, co, false, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    (void)hipFree(part);
    return from_hip(e);
  }
  if (!wt) return WF_EINVAL;
  if (mode == 2) {
    // input adjoint: the [9][ci][co] weights are already [tap][out = ci][reduction = co]
    ConvOut o;
    o.out = (uint16_t*)out;
    NN_TRY(conv(in, wt, nullptr, o, P, h, w, co, ci, true, false, stream));
    NN_TRY(hipStreamSynchronize(stream));
    return WF_OK;
  }
  // forward needs [9][co][ci]
  uint16_t* tmp = nullptr;
  NN_TRY(hipMalloc((void**)&tmp, (size_t)9 * ci * co * 2));
  std::vector<uint16_t> hw_((size_t)9 * ci * co), ht((size_t)9 * ci * co);
  hipError_t e = hipMemcpyAsync(hw_.data(), wt, hw_.size() * 2, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e == hipSuccess) {
    for (int t = 0; t < 9; ++t)
      for (int a = 0; a < ci; ++a)
        for (int c = 0; c < co; ++c) ht[((size_t)t * co + c) * ci + a] = hw_[((size_t)t * ci + a) * co + c];
    e = hipMemcpyAsync(tmp, ht.data(), ht.size() * 2, hipMemcpyHostToDevice, stream);
  }
  ConvOut o;
  o.out = (uint16_t*)out;
  o.relu = mode == 1;
  if (e == hipSuccess) e = conv(in, tmp, b, o, P, h, w, ci, co, false, false, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  (void)hipFree(tmp);
  return from_hip(e);
}

}  // extern "C"
