// Learned surrogate of the ILS output: training and inference kernels plus
// the C ABI declared in include/ils_net.h, and the residual-gated inference
// that falls back to plain ILS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/ils.h"
#include "../../include/ils_net.h"
#include "net_kernels.hpp"

// The stream a plan currently enqueues on (library-internal, ils_api.cpp).
void* ilsk_plan_stream(ils_plan* plan);

using namespace ilsn;

namespace {

// ---------------------------------------------------------------- network
struct Layer {
  int ci, co;    // real channels
  int cip, cop;  // padded channels of the forward convolution
  int w_off, b_off;  // offsets (floats) in the master parameter array
};

// Layer i: 5 -> 32, four times 32 -> 32, 32 -> 3.  Parameters are stored
// layer by layer as w[co][ci][3][3] followed by b[co].
__host__ __device__ constexpr Layer layer_def(int i) {
  int off = 0;
  Layer L{0, 0, 0, 0, 0, 0};
  for (int k = 0; k <= i; ++k) {
    const int ci = (k == 0) ? 5 : 32, co = (k == 5) ? 3 : 32;
    L = Layer{ci, co, ci == 5 ? 8 : 32, co == 3 ? 16 : 32, off, off + co * ci * 9};
    off += co * ci * 9 + co;
  }
  return L;
}

struct Net {
  Layer L[6];
  size_t nparams;
  Net() {
    for (int i = 0; i < 6; ++i) L[i] = layer_def(i);
    nparams = (size_t)L[5].b_off + L[5].co;
  }
};
const Net kNet;

// channels of the gradient tensor flowing into the output of layer i
inline int gchan(int i) { return kNet.L[i].co == 3 ? 8 : 32; }

inline size_t al(size_t v) { return (v + 255) / 256 * 256; }

constexpr int kWgradBlocks = 512;  // most blocks of a backward kernel (each writes a row of partial sums)
constexpr int kPartialRows = 256;  // rows of a 32 -> 32 layer that the workspace holds (see net_layout)
constexpr int kLossBlocks = 256;

// --------------------------------------------------------- small kernels
// dst[0] = a, dst[1] = b (a frame's lambda and p for the input maps)
__global__ void k_set_pair(float* dst, float a, float b) {
  if (threadIdx.x == 0) {
    dst[0] = a;
    dst[1] = b;
  }
}

__global__ void __launch_bounds__(256) k_pack_input(const float* f, const float* lam, const float* p, bf16* x0,
                                                   int B, int H, int W) {
  const size_t plane = (size_t)H * W;
  const size_t n = (size_t)B * plane;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const size_t img = i / plane, pix = i - img * plane;
    const float* fi = f + img * 3 * plane + pix;
    bf16 o[8];
    o[0] = f2bf(fi[0]);
    o[1] = f2bf(fi[plane]);
    o[2] = f2bf(fi[2 * plane]);
    o[3] = f2bf(lam[img]);
    o[4] = f2bf(p[img]);
    o[5] = o[6] = o[7] = f2bf(0.0f);
    *reinterpret_cast<uint4*>(&x0[i * 8]) = *reinterpret_cast<const uint4*>(o);
  }
}

// g6 = d(mean squared error)/dv = 2 (v - t) / n, NHWC bf16 (8 channels);
// per-block partial sums of (v - t)^2 in double.
__global__ void __launch_bounds__(256) k_loss_grad(const float* v, const float* t, bf16* g, double* partial,
                                                  int B, int H, int W) {
  const size_t plane = (size_t)H * W;
  const size_t n = (size_t)B * plane;
  const float scale = (float)(2.0 / (3.0 * (double)n));
  double acc = 0.0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const size_t img = i / plane, pix = i - img * plane;
    const size_t base = img * 3 * plane + pix;
    bf16 o[8];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float d = v[base + c * plane] - t[base + c * plane];
      acc += (double)d * d;
      o[c] = f2bf(scale * d);
    }
    o[3] = o[4] = o[5] = o[6] = o[7] = f2bf(0.0f);
    *reinterpret_cast<uint4*>(&g[i * 8]) = *reinterpret_cast<const uint4*>(o);
  }
  __shared__ double red[256];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// One block: a thread per partial, then a tree (one thread summing all of
// them waited for a load at a time: 15 us).
__global__ void __launch_bounds__(kLossBlocks) k_loss_final(const double* partial, double n, float* loss) {
  __shared__ double red[kLossBlocks];
  red[threadIdx.x] = partial[threadIdx.x];
  __syncthreads();
  for (int s = kLossBlocks / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(red[0] / n);
}

// Partial weight and bias gradients of a convolution on the MFMA units:
//   dW[co][ci][tap] = sum_pixels g[pixel][co] x[pixel + shift(tap)][ci]
// is, for each tap, D[co][ci] += sum_k G[co][k] X_tap[k][ci] with k running
// over the 32 pixels of one tile row (one K block of v_mfma_f32_16x16x32_bf16).
// The (16-row co block, 16-column ci block) pairs are dealt to the four
// waves; when there are two pairs (first and last layers), two waves share a
// pair, taking alternate tile rows, and add up through LDS at the end.
// db[co] is one more product, with a column of ones.  Blocks stride over TH x
// TW pixel tiles and write one partial row each (reduced in a fixed order
// afterwards: deterministic).
//
// The tensors are NHWC, while both operands want eight consecutive pixels of
// a channel per lane.  A thread loads four pixels x eight channels, turns
// them round in registers and writes them to LDS channel by channel; a
// fragment is then one 16-byte read, the tap one column on is the same ten
// pixels shifted by 16 bits, and a row of x serves three rows of taps.  The
// next tile's loads are in flight during a tile's products.  (Fragments read
// element by element from NHWC tiles took 110 us a 32-channel layer for 16
// crops of 256 x 256.)
//
// PixTile: in LDS a row of a block of MW channels is one MW x 16 byte piece
// per eight pixels, channel c of piece k in place c ^ k.  A 16-byte LDS read
// serves sixteen lanes together that are not consecutive (0-3, 12-15, 20-27
// and so on): with lane l reading channel l % 16 of piece l / 16, these have
// sixteen places of their own, as have the 8-byte stores of 32 lanes.
template <int C, int ROWS, int QUADS, bool PIXELS = false>
struct PixTile {  // ROWS x 4 QUADS pixels of C channels, held channel-major in LDS
  static constexpr int CG = C / 8;                        // channel groups of 8
  static constexpr int ITEMS = ROWS * QUADS * CG;         // (row, 4 pixels, 8 channels)
  static constexpr int NIT = (ITEMS + 255) / 256;         // items per thread
  static constexpr int MW = C < 16 ? C : 16;              // channels of a block
  static constexpr int RP = (QUADS + 1) / 2 * MW * 16;    // bytes of a block's row
  static constexpr int BS = ROWS * RP + 64;               // bytes from one block to the next
  static constexpr int BYTES = (C / MW - 1) * BS + ROWS * RP;
  u32x4 v[NIT][4];  // v[j][p] is pixel p ^ turn() of item j

  // Byte offset, within its row, of pixels 8 k .. 8 k + 7 of channel c.
  __device__ __forceinline__ static int at(int c, int k) {
    return c / MW * BS + k * (MW * 16) + (((c % MW) ^ k) % MW << 4);
  }
  // The order of an item's pixels: lanes that store together take different
  // ones, or store_pixels() would send them to the same banks.
  __device__ __forceinline__ static int turn(int i) {
    const int q = i / CG;
    return !PIXELS ? 0 : CG > 1 ? q & 3 : (q >> 2) & 3;
  }

  __device__ __forceinline__ static void place(int i, int& row, int& px, int& cg) {
    cg = i % CG;
    const int q = i / CG;
    row = q / QUADS;
    px = 4 * (q - row * QUADS);
  }
  // pixel (row, px) of the tile is image pixel (y0 + row, x0 + px); WRAP: periodic, else zero outside
  template <bool WRAP>
  __device__ __forceinline__ void fetch(const bf16* img, int H, int W, int y0, int x0) {
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
      const int i = imin(threadIdx.x + j * 256, ITEMS - 1);
      int row, px, cg;
      place(i, row, px, cg);
      const int gy = WRAP ? wrap_near(y0 + row, H) : y0 + row;
      const int gx = x0 + px;
      const bool rowin = gy < H;
      const bf16* src = img + (size_t)(rowin ? gy : 0) * W * C + cg * 8;
      const int tn = turn(i);
      if (rowin && gx >= 0 && gx + 4 <= W) {
#pragma unroll
        for (int p = 0; p < 4; ++p) v[j][p] = *reinterpret_cast<const u32x4*>(src + (size_t)(gx + (p ^ tn)) * C);
      } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int gp = gx + (p ^ tn);
          const bool in = WRAP || (rowin && gp < W);
          const u32x4 r = *reinterpret_cast<const u32x4*>(src + (size_t)(in ? wrap_near(gp, W) : 0) * C);
          v[j][p] = in ? r : u32x4{0, 0, 0, 0};
        }
      }
    }
  }
  __device__ __forceinline__ void store(unsigned char* lds) const {
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
      const int i = threadIdx.x + j * 256;
      if (j * 256 + 256 > ITEMS && i >= ITEMS) continue;
      int row, px, cg;
      place(i, row, px, cg);
      const int tn = turn(i);
      const unsigned low = tn & 1 ? 0x01000504 : 0x05040100, high = tn & 1 ? 0x03020706 : 0x07060302;
      unsigned char* dst = lds + row * RP + (px & 4) * 2;
#pragma unroll
      for (int c = 0; c < 4; ++c) {  // channels 2 c (low halves) and 2 c + 1 (high halves)
        const u32x4 d = {__builtin_amdgcn_perm(v[j][1][c], v[j][0][c], low), __builtin_amdgcn_perm(v[j][3][c], v[j][2][c], low),
                         __builtin_amdgcn_perm(v[j][1][c], v[j][0][c], high), __builtin_amdgcn_perm(v[j][3][c], v[j][2][c], high)};
        *reinterpret_cast<uint2*>(dst + at(cg * 8 + 2 * c, px >> 3)) = tn & 2 ? make_uint2(d[1], d[0]) : make_uint2(d[0], d[1]);
        *reinterpret_cast<uint2*>(dst + at(cg * 8 + 2 * c + 1, px >> 3)) = tn & 2 ? make_uint2(d[3], d[2]) : make_uint2(d[2], d[3]);
      }
    }
  }
  // the first LW columns as they came, pixel by pixel
  template <int LW>
  __device__ __forceinline__ void store_pixels(bf16* tile) const {
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
      const int i = threadIdx.x + j * 256;
      if (j * 256 + 256 > ITEMS && i >= ITEMS) continue;
      int row, px, cg;
      place(i, row, px, cg);
      const int tn = turn(i);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int x = px + (p ^ tn);
        if (4 * QUADS <= LW || x < LW) *reinterpret_cast<u32x4*>(&tile[(row * LW + x) * C + pixel_chunk<C>(x, cg) * 8]) = v[j][p];
      }
    }
  }
};

// Pixels 0 .. 7, 1 .. 8 and 2 .. 9 from a chunk of a channel-major row and the next one.
__device__ __forceinline__ void row_taps(const unsigned char* at, const unsigned char* next, bf16x8 (&f)[3]) {
  const u32x4 d = *reinterpret_cast<const u32x4*>(at);
  const unsigned e = *reinterpret_cast<const unsigned*>(next);
  f[0] = __builtin_bit_cast(bf16x8, d);
  f[1] = __builtin_bit_cast(bf16x8, u32x4{__builtin_amdgcn_alignbit(d[1], d[0], 16), __builtin_amdgcn_alignbit(d[2], d[1], 16),
                                          __builtin_amdgcn_alignbit(d[3], d[2], 16), __builtin_amdgcn_alignbit(e, d[3], 16)});
  f[2] = __builtin_bit_cast(bf16x8, u32x4{d[1], d[2], d[3], e});
}

// Sums of a block's waves over (16-row co block mb, 16-column ci block nb)
// to its partial row; waves of a second row group hand theirs to the first.
template <int PAIRS, int RG>
__device__ __forceinline__ void write_partial(const f32x4 (&acc)[9], const f32x4& accb, unsigned char* lds, int pair,
                                              int rg, int mb, int nb, int gcr, int xcr, float* out) {
  const int lane = threadIdx.x & 63, m = lane & 15, kc = lane >> 4;
  float* red = reinterpret_cast<float*>(lds);
  if (RG == 2 && rg == 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) red[((pair * 10 + tap) * 4 + i) * 64 + lane] = acc[tap][i];
      red[((pair * 10 + 9) * 4 + i) * 64 + lane] = accb[i];
    }
  }
  if (RG == 2) __syncthreads();
  if (rg != 0) return;
  const int ci = nb * 16 + m;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int co = mb * 16 + 4 * kc + i;
    if (co >= gcr) continue;
    if (ci < xcr) {
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        float v = acc[tap][i];
        if (RG == 2) v += red[((pair * 10 + tap) * 4 + i) * 64 + lane];
        out[((size_t)co * xcr + ci) * 9 + tap] = v;
      }
    }
    if (nb == 0 && m == 0) {
      float v = accb[i];
      if (RG == 2) v += red[((pair * 10 + 9) * 4 + i) * 64 + lane];
      out[(size_t)gcr * xcr * 9 + co] = v;
    }
  }
}
constexpr int kPartialLds = 2 * 64 * 40 * 4;  // bytes the above needs where RG is 2

// The first layer, whose input needs no gradient: 32 channels of g, 8 of x.
// 23 us for 16 crops of 256 x 256 (84 MB).
__global__ void __launch_bounds__(256) k_wgrad_first(const bf16* g, const bf16* x, float* partial, int gcr, int xcr,
                                                     int B, int H, int W) {
  constexpr int GC = 32, XC = 8, PAIRS = 2, RG = 2;  // RG: waves per pair
  static_assert(TH == 8 && TW == 32, "one K block per tile row");
  using GT = PixTile<GC, TH, TW / 4>;
  using XT = PixTile<XC, TH + 2, (TW + 4) / 4>;  // columns x0 - 1 .. x0 + 34 (the last two are not used)
  constexpr int TILE_BYTES = GT::BYTES + XT::BYTES;
  __shared__ __attribute__((aligned(16))) unsigned char lds[TILE_BYTES > kPartialLds ? TILE_BYTES : kPartialLds];
  unsigned char* gl = lds;
  unsigned char* xl = lds + GT::BYTES;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int mb = wave % PAIRS, rg = wave / PAIRS;
  const int m = lane & 15, kc = lane >> 4;
  // channels beyond the tensor's give columns that are not written
  const unsigned char* ga = gl + GT::at(mb * 16 + m, kc);
  const unsigned char* xa = xl + XT::at(m % XC, kc);
  const unsigned char* xb = xl + XT::at(m % XC, kc + 1);
  f32x4 acc[9], accb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) acc[tap] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bf16x8 ones = {(bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f, (bf16)1.0f};

  const TileGrid tg(B, H, W, TH, TW);
  const size_t plane = (size_t)H * W;
  GT gt;
  XT xt;
  auto fetch = [&](int tile) {
    int img, y0, x0;
    tg.origin(tile, img, y0, x0);
    gt.template fetch<false>(g + (size_t)img * plane * GC, H, W, y0, x0);
    xt.template fetch<true>(x + (size_t)img * plane * XC, H, W, y0 - 1, x0 - 1);
  };
  int t, t_end, step;
  tg.span(t, t_end, step);
  if (t < t_end) fetch(t);
  for (; t < t_end; t += step) {
    gt.store(gl);
    xt.store(xl);
    __syncthreads();
    if (t + step < t_end) fetch(t + step);
#pragma unroll
    for (int p = 0; p < TH / RG; ++p) {
      const int py = RG * p + rg;
      bf16x8 xf[3][3];
#pragma unroll
      for (int ta = 0; ta < 3; ++ta) row_taps(xa + (py + ta) * XT::RP, xb + (py + ta) * XT::RP, xf[ta]);
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(ga + py * GT::RP);
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
        acc[tap] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, xf[tap / 3][tap % 3], acc[tap], 0, 0, 0);
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, accb, 0, 0, 0);
    }
    __syncthreads();
  }
  write_partial<PAIRS, RG>(acc, accb, lds, mb, rg, mb, 0, gcr, xcr,
                           partial + (size_t)blockIdx.x * (size_t)(gcr * xcr * 9 + gcr));
}

// Backward of layers 1 .. 5 in one pass over g and x: the gradient flowing
// into the layer before,
//   out[q][ci] = [x[q][ci] > 0] sum_{co, tap} w[co][ci][tap] g[q - shift(tap)][co],
// and the partial weight and bias gradients
//   dW[co][ci][tap] = sum_q g[q - shift(tap)][co] x[q][ci].
// Both read g around a tile of x, so that g and its halo are loaded once (as
// two kernels they move 335 MB a 32-channel layer of 16 crops of 256 x 256,
// as one 201 MB), and held twice in LDS: pixel by pixel as the operand of
// the convolution, channel by channel as that of the weight gradient, of which
// row p of x meets rows p .. p + 2.  x lies there channel by channel too, and
// pixel by pixel as the mask.  80 256 B, of which two blocks fit a CU's 160 KB
// (8 tiles a block: 256 blocks 45.5 us, 512 56.9), so that one's loads and
// stores run beside the other's products.  Two waves share rows and halve
// the channels of the convolution, which leaves its weights 36 registers; with
// 72 the kernel spilled and took 78 us.  A 32-channel layer of those crops
// took 40 us for the gradient of x and 41 for that of the weights; this takes
// 63 (the 8-channel one 26 + 31, now 37): the products alone are 19 us, their
// operands' packing as much again, and the LDS 20.
struct BwdArgs {
  const bf16* g;      // NHWC, GC channels
  const bf16* x;      // NHWC, 32 channels: the layer's input, an activation after its ReLU
  const bf16* wfrag;  // 32 x kpad(GC)
  bf16* out;          // NHWC, 32 channels
  float* partial;
  int gcr;            // real channels of g
  int B, H, W;
};

template <int GC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_bwd(BwdArgs a) {
  constexpr int XC = 32, LH = TH + 2, LW = TW + 2;
  constexpr int MB = (GC + 15) / 16, PAIRS = 2 * MB, RG = 4 / PAIRS;
  using GT = PixTile<GC, LH, (TW + 4) / 4, true>;
  using XT = PixTile<XC, TH, TW / 4, true>;
  constexpr int GPIX = LH * LW * GC * 2, XPIX = TH * TW * XC * 2;
  constexpr int BYTES = GT::BYTES + XT::BYTES + GPIX + XPIX;
  static_assert(BYTES <= 80 * 1024 && BYTES >= kPartialLds, "two blocks per CU");
  __shared__ __attribute__((aligned(16))) unsigned char lds[BYTES];
  unsigned char* gl = lds;
  unsigned char* xl = gl + GT::BYTES;
  bf16* gpix = reinterpret_cast<bf16*>(xl + XT::BYTES);
  bf16* xpix = reinterpret_cast<bf16*>(xl + XT::BYTES + GPIX);
  const int H = a.H, W = a.W;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int pair = wave % PAIRS, rg = wave / PAIRS;
  const int mb = pair / 2, nb = pair % 2;
  const int m = lane & 15, kc = lane >> 4;
  const unsigned char* ga = gl + GT::at((mb * 16 + m) % GC, kc);
  const unsigned char* gb = gl + GT::at((mb * 16 + m) % GC, kc + 1);
  const unsigned char* xa = xl + XT::at(nb * 16 + m, kc);
  const int cb = 16 * (wave & 1), row0 = 4 * (wave >> 1);  // this wave's channels and rows of the gradient of x
  bf16x8 wf[1][kpad(GC) / 32];
  load_wfrag<GC, 16>(a.wfrag + cb * kpad(GC), wf);
  f32x4 acc[9], accb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) acc[tap] = f32x4{0.f, 0.f, 0.f, 0.f};

  const TileGrid tg(a.B, H, W, TH, TW);
  const size_t plane = (size_t)H * W;
  int t, t_end, step;
  tg.span(t, t_end, step);
  GT gt;
  XT xt;
  auto fetch = [&](int tile) {
    int img, y0, x0;
    tg.origin(tile, img, y0, x0);
    gt.template fetch<true>(a.g + (size_t)img * plane * GC, H, W, y0 - 1, x0 - 1);
    xt.template fetch<false>(a.x + (size_t)img * plane * XC, H, W, y0, x0);
  };
  if (t < t_end) fetch(t);
  for (; t < t_end; t += step) {
    gt.store(gl);
    gt.template store_pixels<LW>(gpix);
    xt.store(xl);
    xt.template store_pixels<TW>(xpix);
    __syncthreads();
    int img, y0, x0;
    tg.origin(t, img, y0, x0);

    // the gradient of x
#pragma unroll 1  // unrolled, it spills
    for (int h = 0; h < 4; h += 2) {
      f32x4 d[2][2][1];
      conv_mfma<GC, 16, LW, true>(gpix, wf, row0 + h, d);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int ly = row0 + h + r, y = y0 + ly;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int px = c * 16 + m;
          if (y >= H || x0 + px >= W) continue;
          const uint2 mraw = *reinterpret_cast<const uint2*>(&xpix[(ly * TW + px) * XC + pixel_chunk<XC>(px, (cb >> 3) + (kc >> 1)) * 8 + 4 * (kc & 1)]);
          const bf16* mk = reinterpret_cast<const bf16*>(&mraw);
          bf16 o[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = f2bf(bf2f(mk[i]) > 0.0f ? d[r][c][0][i] : 0.0f);
          *reinterpret_cast<uint2*>(&a.out[((size_t)img * plane + (size_t)y * W + x0 + px) * XC + cb + 4 * kc]) =
              *reinterpret_cast<const uint2*>(o);
        }
      }
    }
    if (t + step < t_end) fetch(t + step);
    // the gradient of the weights; pixels outside the image have x = 0, and
    // are left out of the bias's by the column of ones
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (bf16)(x0 + kc * 8 + i < W ? 1.0f : 0.0f);
    bf16x8 gf[3][3];
    if constexpr (RG == 1) {
      row_taps(ga, gb, gf[0]);
      row_taps(ga + GT::RP, gb + GT::RP, gf[1]);
    }
#pragma unroll
    for (int p = 0; p < TH / RG; ++p) {
      __builtin_amdgcn_sched_barrier(0);
      const int py = RG * p + rg;
      if constexpr (RG == 1) {
        row_taps(ga + (p + 2) * GT::RP, gb + (p + 2) * GT::RP, gf[(p + 2) % 3]);
      } else {
#pragma unroll
        for (int r = 0; r < 3; ++r) row_taps(ga + (py + r) * GT::RP, gb + (py + r) * GT::RP, gf[(p + r) % 3]);
      }
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(xa + py * XT::RP);
      // tap (ta, tc) pairs x[q] with g[q - (ta - 1, tc - 1)]
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
        acc[tap] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[(p + 2 - tap / 3) % 3][2 - tap % 3], b, acc[tap], 0, 0, 0);
      if (nb == 0 && y0 + py < H)
        accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[(p + 1) % 3][1], ones, accb, 0, 0, 0);
    }
    __syncthreads();
  }
  write_partial<PAIRS, RG>(acc, accb, lds, pair, rg, mb, nb, a.gcr, XC,
                           a.partial + (size_t)blockIdx.x * (size_t)(a.gcr * XC * 9 + a.gcr));
}

// grad[k] = sum over blocks (fixed order) of partial[b][k].  A block sums 32
// columns, eight threads to a column (one thread per column left 37 blocks
// with a chain of 256 loads each: 62 us a layer).
constexpr int kRedCols = 32, kRedRows = 8;
__global__ void __launch_bounds__(kRedCols * kRedRows) k_reduce_partials(const float* partial, int nblocks, int len,
                                                                        float* grad) {
  const int c = threadIdx.x % kRedCols, r = threadIdx.x / kRedCols;
  const int k = blockIdx.x * kRedCols + c;
  double s = 0.0;
  if (k < len) {
#pragma unroll 8
    for (int b = r; b < nblocks; b += kRedRows) s += partial[(size_t)b * len + k];
  }
  __shared__ double red[kRedRows][kRedCols];
  red[r][c] = s;
  __syncthreads();
  if (r == 0 && k < len) {
    for (int i = 1; i < kRedRows; ++i) s += red[i][c];
    grad[k] = (float)s;
  }
}

// Adam with bias correction (Kingma & Ba): fp32 master parameters.
__global__ void __launch_bounds__(256) k_adam(float* prm, float* m, float* v, const float* g, int n, float lr,
                                             float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mhat = mi / c1, vhat = vi / c2;
  prm[i] -= lr * mhat / (sqrtf(vhat) + eps);
}

// Pack master fp32 weights into the bf16 fragment layouts.
//   forward WF[co][tap*CIP + ci]    = w[co][ci][tap]
//   dgrad   WD[ci][tap'*COPg + co]  = w[co][ci][8 - tap']   (flipped, transposed)
// and the padded fp32 biases.
struct PackArgs {
  const float* master;
  bf16* wf[6];
  bf16* wd[6];
  float* bias[6];
};

__global__ void __launch_bounds__(256) k_pack_weights(PackArgs a) {
  const int layer = blockIdx.y;
  const Layer L = layer_def(layer);
  const float* w = a.master + L.w_off;
  const float* b = a.master + L.b_off;
  const int kpf = kpad(L.cip);
  const int nf = L.cop * kpf;
  const int gcp = (L.co == 3) ? 8 : 32;  // channels of the gradient tensor
  const int kpd = kpad(gcp);
  const int nd = 32 * kpd;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < nf + nd + L.cop; i += gridDim.x * 256) {
    if (i < nf) {
      const int co = i / kpf, k = i - co * kpf;
      const int tap = k / L.cip, ci = k - tap * L.cip;
      float val = 0.0f;
      if (co < L.co && ci < L.ci && tap < 9) val = w[((size_t)co * L.ci + ci) * 9 + tap];
      a.wf[layer][i] = f2bf(val);
    } else if (i < nf + nd) {
      if (layer == 0) continue;  // the image gradient is never needed
      const int j = i - nf;
      const int ci = j / kpd, k = j - ci * kpd;
      const int tapd = k / gcp, co = k - tapd * gcp;
      float val = 0.0f;
      if (co < L.co && ci < L.ci && tapd < 9) val = w[((size_t)co * L.ci + ci) * 9 + (8 - tapd)];
      a.wd[layer][j] = f2bf(val);
    } else {
      const int co = i - nf - nd;
      a.bias[layer][co] = co < L.co ? b[co] : 0.0f;
    }
  }
}

}  // namespace

// ------------------------------------------------------------------ state
struct ils_net {
  int max_B, max_H, max_W;
  hipStream_t stream;
  char* ws;
  size_t ws_bytes;
  int last_error;
  long long step;
  // device buffers (carved from the workspace)
  float* master;
  float* adam_m;
  float* adam_v;
  float* grad;
  bf16* wf[6];
  bf16* wd[6];
  float* bias[6];
  bf16* act[6];   // act[0] = x0 (8 ch), act[1..5] = a1..a5 (32 ch)
  bf16* gbuf[2];  // gradient ping-pong (32 ch)
  float* zbuf;    // v (B, 3, H, W) scratch
  // rows of partial sums: of layer 5, and of the layers before it
  float* partial;
  float* partial_wide;
  size_t partial_bytes, partial_wide_bytes;
  double* lpart;  // loss partials
  float* loss;
};

namespace {

size_t net_layout(int B, int H, int W, ils_net* n) {
  const size_t px = (size_t)B * H * W;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = al(off + bytes);
    return o;
  };
  size_t o_master = take(kNet.nparams * 4), o_m = take(kNet.nparams * 4), o_v = take(kNet.nparams * 4),
         o_g = take(kNet.nparams * 4);
  size_t o_wf[6], o_wd[6], o_b[6];
  for (int i = 0; i < 6; ++i) {
    o_wf[i] = take((size_t)kNet.L[i].cop * kpad(kNet.L[i].cip) * 2);
    o_wd[i] = take((size_t)32 * kpad(gchan(i)) * 2);
    o_b[i] = take((size_t)kNet.L[i].cop * 4);
  }
  size_t o_act[6];
  o_act[0] = take(px * 8 * 2);
  for (int i = 1; i < 5; ++i) o_act[i] = take(px * 32 * 2);
  size_t o_gb0 = take(px * 32 * 2), o_gb1 = take(px * 32 * 2);
  size_t o_lp = take(kLossBlocks * 8);
  size_t o_loss = take(4);
  // The last activation, v and the partial sums lie together: behind layer 5
  // the first two are spent, and the partial sums of the layers before it
  // start where they did, so that kWgradBlocks rows of a 32 -> 32 layer fit
  // an area of kPartialRows of them for any batch of so many full tiles.  The
  // partial sums end the workspace and take what it holds beyond the minimum:
  // many images smaller than a tile have more tiles than the minimum has rows
  // (64 crops of 9 x 93: 183 us with it, 167 with kWgradBlocks rows).
  o_act[5] = take(px * 32 * 2);
  size_t o_z = take(px * 3 * 4);
  size_t o_part = take((size_t)kPartialRows * (32 * 32 * 9 + 32) * 4);
  if (n) {
    char* b = n->ws;
    n->master = (float*)(b + o_master);
    n->adam_m = (float*)(b + o_m);
    n->adam_v = (float*)(b + o_v);
    n->grad = (float*)(b + o_g);
    for (int i = 0; i < 6; ++i) {
      n->wf[i] = (bf16*)(b + o_wf[i]);
      n->wd[i] = (bf16*)(b + o_wd[i]);
      n->bias[i] = (float*)(b + o_b[i]);
      n->act[i] = (bf16*)(b + o_act[i]);
    }
    n->gbuf[0] = (bf16*)(b + o_gb0);
    n->gbuf[1] = (bf16*)(b + o_gb1);
    n->zbuf = (float*)(b + o_z);
    n->partial = (float*)(b + o_part);
    n->partial_bytes = n->ws_bytes - o_part;
    n->partial_wide = (float*)(b + o_act[5]);
    n->partial_wide_bytes = n->ws_bytes - o_act[5];
    n->lpart = (double*)(b + o_lp);
    n->loss = (float*)(b + o_loss);
  }
  return off;
}

int rec(ils_net* n, hipError_t e) {
  if (e == hipSuccess) return ILS_OK;
  if (n && n->last_error == ILS_OK) n->last_error = (int)e;
  return ILS_ERR_HIP;
}

// Workgroups of `kernel` the current device holds at once (the convolution
// kernels loop over tiles, so a larger grid only adds weight reloads).
int resident_blocks(const void* kernel, int threads = NTHREADS) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1024;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 1024;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu <= 0)
    per_cu = 1;
  return cus * per_cu;
}

int conv_grid(long long tiles, int cap) { return (int)(tiles < cap ? tiles : cap); }

template <int CIP, int COP, int MODE>
hipError_t conv(const ConvArgs& a, hipStream_t st) {
  static const int cap_near = resident_blocks(reinterpret_cast<const void*>(&k_conv<CIP, COP, MODE, true>));
  static const int cap_any = resident_blocks(reinterpret_cast<const void*>(&k_conv<CIP, COP, MODE, false>));
  const long long tiles = (long long)a.B * ((a.H + TH - 1) / TH) * ((a.W + TW - 1) / TW);
  if (a.H >= TH + 2 && a.W >= TW + 2)
    hipLaunchKernelGGL((k_conv<CIP, COP, MODE, true>), dim3(conv_grid(tiles, cap_near)), dim3(NTHREADS), 0, st, a);
  else
    hipLaunchKernelGGL((k_conv<CIP, COP, MODE, false>), dim3(conv_grid(tiles, cap_any)), dim3(NTHREADS), 0, st, a);
  return hipGetLastError();
}

// forward through the six layers; v written to `v` (planar fp32)
hipError_t run_forward(ils_net* n, const float* f, const float* lam, const float* p, int B, int H, int W, float* v) {
  hipStream_t st = n->stream;
  const size_t px = (size_t)B * H * W;
  int blocks = (int)((px + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_pack_input, dim3(blocks), dim3(256), 0, st, f, lam, p, n->act[0], B, H, W);
  hipError_t e = hipGetLastError();
  for (int i = 0; i < 6 && e == hipSuccess; ++i) {
    ConvArgs a{};
    a.in = n->act[i];
    a.wfrag = n->wf[i];
    a.bias = n->bias[i];
    a.B = B;
    a.H = H;
    a.W = W;
    if (i == 0) {
      a.out = n->act[1];
      e = conv<8, 32, CONV_RELU>(a, st);
    } else if (i < 5) {
      a.out = n->act[i + 1];
      e = conv<32, 32, CONV_RELU>(a, st);
    } else {
      a.f = f;
      a.v = v;
      e = conv<32, 16, CONV_LAST>(a, st);
    }
  }
  return e;
}

// The network without its hidden activations (inference): strips of SW
// columns, each cut into segments down the image so that the chip's compute
// units (one workgroup each) all have the same number of steps.  A segment of
// r rows takes r / 2 + 12 steps (the rows its halo recomputes and the depth of
// the pipeline), so more segments than it takes to fill the rounds cost time:
// the cheapest number, the chip taking its blocks in rounds.  At least 16 are
// looked at: 16 frames of 1080p are 576 strips, which whole (2 1/4 rounds) took
// 3670 us and in four segments each (9 rounds) take 2780.
struct StreamPlan {
  int strips, segs;
  long long rounds, steps;  // of one launch, and of one of its rounds
};
StreamPlan stream_plan(int B, int H, int W, int cus) {
  StreamPlan s{(W + SW - 1) / SW, 1, 1, 0};
  const long long units = (long long)B * s.strips;
  for (int g = 1; g <= (H + 1) / 2 && (g <= 16 || units * g <= 4LL * cus); ++g) {
    const long long rounds = (units * g + cus - 1) / cus;
    const long long steps = ((H + g - 1) / g + 1) / 2 + 12;
    if (g > 1 && rounds * steps >= s.rounds * s.steps) continue;
    s.segs = g;
    s.rounds = rounds;
    s.steps = steps;
  }
  return s;
}

// Whether the network runs faster layer by layer than as strips: for many
// images of few rows, where the pipeline's 12 steps are most of a segment's, or
// of a few columns or a little over one strip's.  Both times in microseconds,
// fitted to 780 sizes of 1 to 512 images of 2 to 64 rows and 2 to 256 columns
// (per compute unit: tiles and pixels of the layers, of which images smaller
// than a tile take the halo by division): strips within 7 %, layers within 11.
// Over 320 further sizes up to 8 M pixels the choice is within 6 % of the faster
// one; strips alone took up to 1.5 times the layers' time.  267 images of 327 x
// 5: strips 457 us, layers 299; 512 of 8 x 55: 91, 75; of 32 x 55: 191, 171; of
// 64 x 64: 221, 262; one 256 x 256: 19, 34; 8 of 720 x 1280: 650, 1222.
bool stream_loses(const StreamPlan& s, int B, int H, int W, int cus) {
  const double strips = s.rounds * (1.97 * s.steps - 9.7) + 1.3;
  const double tiles = (double)B * ((H + TH - 1) / TH) * ((W + TW - 1) / TW) / cus;
  const double full = (double)B * H * W / ((double)TH * TW * cus);  // tiles' worth of pixels
  const bool near = H >= TH + 2 && W >= TW + 2;
  const double layers = near ? 30.0 + 5.25 * tiles + 4.44 * full : 36.0 + 6.06 * tiles + 3.76 * full;
  return strips > 1.02 * layers;
}

// In place, where other strips' halos would be overwritten, layer by layer.
hipError_t run_stream(ils_net* n, const float* f, const float* lam, const float* p, int B, int H, int W, float* v) {
  const size_t vals = (size_t)B * 3 * H * W;
  static const int cus = resident_blocks(reinterpret_cast<const void*>(&k_net_stream), 512);
  const StreamPlan sp = stream_plan(B, H, W, cus);
  if ((f < v + vals && v < f + vals) || stream_loses(sp, B, H, W, cus)) return run_forward(n, f, lam, p, B, H, W, v);
  StreamArgs a{};
  a.f = f;
  a.lam = lam;
  a.p = p;
  a.v = v;
  for (int i = 0; i < 6; ++i) {
    a.wfrag[i] = n->wf[i];
    a.bias[i] = n->bias[i];
  }
  a.H = H;
  a.W = W;
  a.strips = sp.strips;
  a.segs = sp.segs;
  hipLaunchKernelGGL(k_net_stream, dim3((unsigned)((long long)B * sp.strips * sp.segs)), dim3(512), 0, n->stream, a);
  return hipGetLastError();
}

// gradients of the loss for the batch whose forward pass is in n->act / zbuf
hipError_t run_backward(ils_net* n, const float* t, int B, int H, int W) {
  hipStream_t st = n->stream;
  const size_t px = (size_t)B * H * W;
  hipLaunchKernelGGL(k_loss_grad, dim3(kLossBlocks), dim3(256), 0, st, n->zbuf, t, n->gbuf[0], n->lpart, B, H, W);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(kLossBlocks), 0, st, n->lpart, 3.0 * (double)px, n->loss);
  e = hipGetLastError();
  const long long tiles = (long long)B * ((H + TH - 1) / TH) * ((W + TW - 1) / TW);
  int cur = 0;
  for (int i = 5; i >= 0 && e == hipSuccess; --i) {
    const Layer& L = kNet.L[i];
    const int len = L.co * L.ci * 9 + L.co;
    // no more blocks (partial rows to write and to sum) than there are tiles,
    // nor than rows fit
    float* partial = i == 5 ? n->partial : n->partial_wide;
    const long long rows = (long long)((i == 5 ? n->partial_bytes : n->partial_wide_bytes) / ((size_t)len * 4));
    const int nblk = (int)std::min({tiles, rows, (long long)kWgradBlocks});
    if (i == 0) {
      hipLaunchKernelGGL(k_wgrad_first, dim3(nblk), dim3(256), 0, st, n->gbuf[cur], n->act[0], partial, L.co,
                         L.ci, B, H, W);
    } else {
      BwdArgs a{};
      a.g = n->gbuf[cur];
      a.x = n->act[i];
      a.wfrag = n->wd[i];
      a.out = n->gbuf[1 - cur];
      a.partial = partial;
      a.gcr = L.co;
      a.B = B;
      a.H = H;
      a.W = W;
      if (i == 5)
        hipLaunchKernelGGL(k_bwd<8>, dim3(nblk), dim3(256), 0, st, a);
      else
        hipLaunchKernelGGL(k_bwd<32>, dim3(nblk), dim3(256), 0, st, a);
      cur = 1 - cur;
    }
    e = hipGetLastError();
    if (e != hipSuccess) break;
    hipLaunchKernelGGL(k_reduce_partials, dim3((len + kRedCols - 1) / kRedCols), dim3(kRedCols * kRedRows), 0, st,
                       partial, nblk, len, n->grad + L.w_off);
    e = hipGetLastError();
  }
  return e;
}

hipError_t pack_weights(ils_net* n) {
  PackArgs pa;
  pa.master = n->master;
  for (int i = 0; i < 6; ++i) {
    pa.wf[i] = n->wf[i];
    pa.wd[i] = n->wd[i];
    pa.bias[i] = n->bias[i];
  }
  hipLaunchKernelGGL(k_pack_weights, dim3(16, 6), dim3(256), 0, n->stream, pa);
  return hipGetLastError();
}

int check_batch(const ils_net* n, int B, int H, int W) {
  if (B < 1 || H < 2 || W < 2 || B > n->max_B || H > n->max_H || W > n->max_W) return ILS_ERR_INVALID_ARG;
  if (B > 512) return ILS_ERR_INVALID_ARG;
  return ILS_OK;
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" {

int ils_net_param_count(void) { return (int)kNet.nparams; }

size_t ils_net_workspace_bytes(int max_B, int max_H, int max_W) {
  if (max_B < 1 || max_H < 2 || max_W < 2) return 0;
  return net_layout(max_B, max_H, max_W, nullptr);
}

int ils_net_create(ils_net** out, int max_B, int max_H, int max_W, void* workspace, size_t ws_bytes,
                   void* hip_stream) {
  if (!out) return ILS_ERR_INVALID_ARG;
  *out = nullptr;
  if (max_B < 1 || max_H < 2 || max_W < 2) return ILS_ERR_INVALID_ARG;
  if (!workspace || ((uintptr_t)workspace & 255)) return ILS_ERR_WORKSPACE;
  if (ws_bytes < ils_net_workspace_bytes(max_B, max_H, max_W)) return ILS_ERR_WORKSPACE;
  ils_net* n = new (std::nothrow) ils_net();
  if (!n) return ILS_ERR_HIP;
  n->max_B = max_B;
  n->max_H = max_H;
  n->max_W = max_W;
  n->stream = static_cast<hipStream_t>(hip_stream);
  n->ws = static_cast<char*>(workspace);
  n->ws_bytes = ws_bytes;
  n->last_error = ILS_OK;
  n->step = 0;
  net_layout(max_B, max_H, max_W, n);
  *out = n;
  return ILS_OK;
}

int ils_net_set_stream(ils_net* n, void* hip_stream) {
  if (!n) return ILS_ERR_INVALID_ARG;
  n->stream = static_cast<hipStream_t>(hip_stream);
  return ILS_OK;
}

int ils_net_set_state(ils_net* n, const float* params, const float* m, const float* v, long long step) {
  if (!n || !params || step < 0) return ILS_ERR_INVALID_ARG;
  const size_t bytes = kNet.nparams * 4;
  hipError_t e = hipMemcpy(n->master, params, bytes, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = m ? hipMemcpy(n->adam_m, m, bytes, hipMemcpyHostToDevice) : hipMemset(n->adam_m, 0, bytes);
  if (e == hipSuccess) e = v ? hipMemcpy(n->adam_v, v, bytes, hipMemcpyHostToDevice) : hipMemset(n->adam_v, 0, bytes);
  if (e == hipSuccess) e = pack_weights(n);
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  n->step = step;
  return rec(n, e);
}

int ils_net_get_state(ils_net* n, float* params, float* m, float* v, long long* step) {
  if (!n) return ILS_ERR_INVALID_ARG;
  const size_t bytes = kNet.nparams * 4;
  hipError_t e = hipStreamSynchronize(n->stream);
  if (e == hipSuccess && params) e = hipMemcpy(params, n->master, bytes, hipMemcpyDeviceToHost);
  if (e == hipSuccess && m) e = hipMemcpy(m, n->adam_m, bytes, hipMemcpyDeviceToHost);
  if (e == hipSuccess && v) e = hipMemcpy(v, n->adam_v, bytes, hipMemcpyDeviceToHost);
  if (step) *step = n->step;
  return rec(n, e);
}

int ils_net_forward(ils_net* n, const float* f, const float* lam, const float* p, int B, int H, int W, float* v) {
  if (!n || !f || !lam || !p || !v) return ILS_ERR_INVALID_ARG;
  int rc = check_batch(n, B, H, W);
  if (rc != ILS_OK) return rc;
  return rec(n, run_stream(n, f, lam, p, B, H, W, v));
}

int ils_net_gradients(ils_net* n, const float* f, const float* lam, const float* p, const float* target, int B, int H,
                      int W, float* grad, float* loss) {
  if (!n || !f || !lam || !p || !target || !grad || !loss) return ILS_ERR_INVALID_ARG;
  int rc = check_batch(n, B, H, W);
  if (rc != ILS_OK) return rc;
  hipError_t e = run_forward(n, f, lam, p, B, H, W, n->zbuf);
  if (e == hipSuccess) e = run_backward(n, target, B, H, W);
  if (e == hipSuccess) e = hipMemcpyAsync(grad, n->grad, kNet.nparams * 4, hipMemcpyDeviceToDevice, n->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(loss, n->loss, 4, hipMemcpyDeviceToDevice, n->stream);
  return rec(n, e);
}

int ils_net_train_step(ils_net* n, const float* f, const float* lam, const float* p, const float* target, int B,
                       int H, int W, float lr, float* loss) {
  if (!n || !f || !lam || !p || !target) return ILS_ERR_INVALID_ARG;
  if (!(lr > 0.0f) || !std::isfinite(lr)) return ILS_ERR_INVALID_ARG;
  int rc = check_batch(n, B, H, W);
  if (rc != ILS_OK) return rc;
  hipError_t e = run_forward(n, f, lam, p, B, H, W, n->zbuf);
  if (e == hipSuccess) e = run_backward(n, target, B, H, W);
  if (e == hipSuccess) {
    n->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = (float)(1.0 - std::pow(0.9, (double)n->step));
    const float c2 = (float)(1.0 - std::pow(0.999, (double)n->step));
    const int np = (int)kNet.nparams;
    hipLaunchKernelGGL(k_adam, dim3((np + 255) / 256), dim3(256), 0, n->stream, n->master, n->adam_m, n->adam_v,
                       n->grad, np, lr, b1, b2, 1e-8f, c1, c2);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = pack_weights(n);
  if (e == hipSuccess && loss) e = hipMemcpyAsync(loss, n->loss, 4, hipMemcpyDeviceToDevice, n->stream);
  return rec(n, e);
}

int ils_net_last_error(ils_net* n) {
  if (!n) return ILS_ERR_INVALID_ARG;
  int r = n->last_error;
  n->last_error = ILS_OK;
  return r;
}

int ils_net_destroy(ils_net* n) {
  delete n;
  return ILS_OK;
}

// Residual-gated surrogate inference.  v = net(f); for every image
// T(v) = one ILS iteration from u^0 = v with data term f; R = rms(T(v) - v);
// images with R > tau are recomputed with plain ILS (N iterations) into out.
// The gated pipeline proper; the plan is already bound to the network's stream.
static int surrogate_infer_bound(ils_net* n, ils_plan* plan, const float* f, const float* lam_dev, const float* p_dev,
                                 const float* lam_host, const float* p_host, float eps, int N, int B, int H, int W,
                                 float tau, float* out, float* tv_scratch, float* residual_host, int* fallback_host) {
  int rc = ILS_OK;
  hipError_t e = run_stream(n, f, lam_dev, p_dev, B, H, W, out);
  if (e != hipSuccess) return rec(n, e);
  const size_t img = (size_t)3 * H * W;
  std::vector<const float*> pa(B), pb(B);
  std::vector<long long> cnt(B, (long long)img);
  // T(v) for every image: one batched call when the plan holds B frames of
  // this size (every argument was checked above, so a refusal can only be
  // the plan's frame count or workspace), else image by image; both give
  // the same bits.
  std::vector<ils_frame> tv(B);
  for (int b = 0; b < B; ++b) {
    tv[b] = ils_frame{f + b * img, tv_scratch + b * img, H, W, 3, lam_host[b], p_host[b], eps, 1, out + b * img,
                      ILS_PENALTY_CHARBONNIER, 0.0f};
    pa[b] = tv_scratch + b * img;
    pb[b] = out + b * img;
  }
  rc = ils_smooth_batch(plan, tv.data(), B);
  if (rc == ILS_ERR_WORKSPACE || rc == ILS_ERR_INVALID_ARG) {
    for (int b = 0; b < B; ++b) {
      rc = ils_iterate_from(plan, f + b * img, out + b * img, H, W, 3, lam_host[b], p_host[b], eps, 1,
                            tv_scratch + b * img);
      if (rc != ILS_OK) return rc;
    }
  }
  if (rc != ILS_OK) return rc;
  // per-image residuals go to the loss-partial area of the network workspace
  float* rms_dev = reinterpret_cast<float*>(n->lpart);
  rc = ils_rms_diff(plan, pa.data(), pb.data(), cnt.data(), B, rms_dev);
  if (rc != ILS_OK) return rc;
  e = hipMemcpyAsync(residual_host, rms_dev, B * sizeof(float), hipMemcpyDeviceToHost, n->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  if (e != hipSuccess) return rec(n, e);
  std::vector<ils_frame> fb;
  for (int b = 0; b < B; ++b) {
    fallback_host[b] = !(residual_host[b] <= tau);  // NaN residual also falls back
    if (fallback_host[b])
      fb.push_back(ils_frame{f + b * img, out + b * img, H, W, 3, lam_host[b], p_host[b], eps, N, nullptr,
                             ILS_PENALTY_CHARBONNIER, 0.0f});
  }
  if (fb.empty()) return ILS_OK;
  // plain ILS for the images that fall back, batched like T(v) when the plan allows
  rc = ils_smooth_batch(plan, fb.data(), (int)fb.size());
  if (rc == ILS_ERR_WORKSPACE || rc == ILS_ERR_INVALID_ARG) {
    for (const ils_frame& fr : fb) {
      rc = ils_smooth(plan, fr.f, H, W, 3, fr.lambda, fr.p, eps, N, fr.out);
      if (rc != ILS_OK) return rc;
    }
    rc = ILS_OK;
  }
  return rc;
}

// Frame-list gate: the network frame by frame (its lambda and p maps from two
// scalars that a one-thread kernel writes into the workspace, so the host
// stages nothing), then T(v), the residuals and the fallback over the whole
// list, as in surrogate_infer_bound.
static int surrogate_infer_frames_bound(ils_net* n, ils_plan* plan, const ils_frame* frames, int nf, float tau,
                                        float* tv_scratch, float* residual_host, int* fallback_host) {
  float* lp = reinterpret_cast<float*>(n->lpart);  // lambda, p of the frame in flight
  std::vector<ils_frame> tv(nf);
  std::vector<const float*> pa(nf), pb(nf);
  std::vector<long long> cnt(nf);
  size_t off = 0;
  for (int i = 0; i < nf; ++i) {
    const ils_frame& fr = frames[i];
    hipLaunchKernelGGL(k_set_pair, dim3(1), dim3(64), 0, n->stream, lp, fr.lambda, fr.p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = run_stream(n, fr.f, lp, lp + 1, 1, fr.H, fr.W, fr.out);
    if (e != hipSuccess) return rec(n, e);
    const size_t img = (size_t)3 * fr.H * fr.W;
    tv[i] = ils_frame{fr.f, tv_scratch + off, fr.H, fr.W, 3, fr.lambda, fr.p, fr.eps, 1, fr.out,
                      ILS_PENALTY_CHARBONNIER, 0.0f};
    pa[i] = tv_scratch + off;
    pb[i] = fr.out;
    cnt[i] = (long long)img;
    off += img;
  }
  int rc = ils_smooth_batch(plan, tv.data(), nf);
  if (rc == ILS_ERR_WORKSPACE || rc == ILS_ERR_INVALID_ARG) {
    for (const ils_frame& t : tv) {
      rc = ils_iterate_from(plan, t.f, t.u0, t.H, t.W, 3, t.lambda, t.p, t.eps, 1, t.out);
      if (rc != ILS_OK) return rc;
    }
  }
  if (rc != ILS_OK) return rc;
  float* rms_dev = reinterpret_cast<float*>(n->lpart);
  rc = ils_rms_diff(plan, pa.data(), pb.data(), cnt.data(), nf, rms_dev);
  if (rc != ILS_OK) return rc;
  hipError_t e = hipMemcpyAsync(residual_host, rms_dev, nf * sizeof(float), hipMemcpyDeviceToHost, n->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  if (e != hipSuccess) return rec(n, e);
  std::vector<ils_frame> fb;
  for (int i = 0; i < nf; ++i) {
    fallback_host[i] = !(residual_host[i] <= tau);  // NaN residual also falls back
    if (fallback_host[i]) {
      const ils_frame& fr = frames[i];
      fb.push_back(ils_frame{fr.f, fr.out, fr.H, fr.W, 3, fr.lambda, fr.p, fr.eps, fr.N, nullptr,
                             ILS_PENALTY_CHARBONNIER, 0.0f});
    }
  }
  if (fb.empty()) return ILS_OK;
  rc = ils_smooth_batch(plan, fb.data(), (int)fb.size());
  if (rc == ILS_ERR_WORKSPACE || rc == ILS_ERR_INVALID_ARG) {
    for (const ils_frame& fr : fb) {
      rc = ils_smooth(plan, fr.f, fr.H, fr.W, 3, fr.lambda, fr.p, fr.eps, fr.N, fr.out);
      if (rc != ILS_OK) return rc;
    }
    rc = ILS_OK;
  }
  return rc;
}

int ils_surrogate_infer_frames(ils_net* n, ils_plan* plan, const ils_frame* frames, int nframes, float tau,
                               float* tv_scratch, float* residual_host, int* fallback_host) {
  if (!n || !plan || !frames || !tv_scratch || !residual_host || !fallback_host) return ILS_ERR_INVALID_ARG;
  if (nframes < 1 || nframes > n->max_B) return ILS_ERR_INVALID_ARG;
  if (!std::isfinite(tau)) return ILS_ERR_NOT_CALIBRATED;
  for (int i = 0; i < nframes; ++i) {
    const ils_frame& fr = frames[i];
    if (!fr.f || !fr.out || fr.C != 3 || fr.penalty != ILS_PENALTY_CHARBONNIER || (fr.u0 && fr.u0 != fr.f))
      return ILS_ERR_INVALID_ARG;
    int rc = check_batch(n, 1, fr.H, fr.W);
    if (rc == ILS_OK) rc = ils_check_args(fr.H, fr.W, 3, fr.lambda, fr.p, fr.eps, fr.N);
    if (rc != ILS_OK) return rc;
  }
  void* saved = ilsk_plan_stream(plan);
  int rc = ils_plan_set_stream(plan, n->stream);
  if (rc != ILS_OK) return rc;
  rc = surrogate_infer_frames_bound(n, plan, frames, nframes, tau, tv_scratch, residual_host, fallback_host);
  (void)ils_plan_set_stream(plan, saved);
  return rc;
}

int ils_surrogate_infer(ils_net* n, ils_plan* plan, const float* f, const float* lam_dev, const float* p_dev,
                        const float* lam_host, const float* p_host, float eps, int N, int B, int H, int W,
                        float tau, float* out, float* tv_scratch, float* residual_host, int* fallback_host) {
  if (!n || !plan || !f || !lam_dev || !p_dev || !lam_host || !p_host || !out || !tv_scratch || !residual_host ||
      !fallback_host)
    return ILS_ERR_INVALID_ARG;
  if (!std::isfinite(tau)) return ILS_ERR_NOT_CALIBRATED;
  int rc = check_batch(n, B, H, W);
  if (rc != ILS_OK) return rc;
  for (int b = 0; b < B; ++b) {
    rc = ils_check_args(H, W, 3, lam_host[b], p_host[b], eps, N);
    if (rc != ILS_OK) return rc;
  }
  // the plan's own work goes on the network's stream for the call and back
  // to the caller's stream on every return path
  void* saved = ilsk_plan_stream(plan);
  rc = ils_plan_set_stream(plan, n->stream);
  if (rc != ILS_OK) return rc;
  rc = surrogate_infer_bound(n, plan, f, lam_dev, p_dev, lam_host, p_host, eps, N, B, H, W, tau, out, tv_scratch,
                             residual_host, fallback_host);
  (void)ils_plan_set_stream(plan, saved);
  return rc;
}

}  // extern "C"
