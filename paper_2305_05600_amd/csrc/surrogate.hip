// Convolutional neural operator for the magnetic-field subcycle
// (libhvpic.so, gfx950).
//
// A stand-in for the subcycled Faraday/Ohm advance of arXiv 2305.05600,
// Sec. II.A, on 2D periodic grids: four periodic 3x3 convolutions
// 7 -> 32 -> 32 -> 32 -> 3 channels with tanh between them map the
// normalised (B^n, n^{n+1/2}, J_i^{n+1/2}) to the normalised increment
// B^{n+1} - B^n.  Inference and training run here: BF16 operands on the
// matrix cores (v_mfma_f32_16x16x32_bf16) with FP32 accumulation, FP32 master
// weights and Adam.
//
// Layout: activations are pixel-major with the channels contiguous ([pixel]
// [channel], BF16), so that one lane's 8 consecutive channels are one 16-byte
// load; a layer is an implicit GEMM (out channels) x (pixels) with K = 9 taps
// x in channels, the taps wrapping around each image.  Channel counts are
// padded to 16 (7 inputs, 3 outputs) with zero weights.  The weight gradient
// has its K along the pixels: it stages pixel-major tiles in LDS and reads its
// operands through the transposing LDS load; blocks leave partial sums that
// one pass adds in a fixed order.
#include <string.h>

#include <algorithm>

#include "hvpic_internal.hpp"
#include "pixel_groups.hpp"

namespace hvpic {
namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
// 16-byte global accesses at 8-byte aligned addresses
typedef uint32_t u4a8 __attribute__((ext_vector_type(4), aligned(8)));

constexpr int kNL = 4;
constexpr int kCin[kNL] = {7, 32, 32, 32}, kCout[kNL] = {32, 32, 32, 3};
constexpr int kCinP[kNL] = {16, 32, 32, 32}, kCoutP[kNL] = {32, 32, 32, 16};
constexpr int wsize(int l) { return kCoutP[l] * 9 * kCinP[l]; }
constexpr int woff(int l) { return l == 0 ? 0 : woff(l - 1) + wsize(l - 1); }
constexpr int boff(int l) { return l == 0 ? 0 : boff(l - 1) + kCoutP[l - 1]; }
constexpr int kW = woff(kNL), kB = boff(kNL);  // 27648 weights, 112 biases (padded)
constexpr int bwoff(int l) { return l <= 1 ? 0 : bwoff(l - 1) + wsize(l - 1); }  // layers 1..3
constexpr int kWb = bwoff(kNL);

// The parameter block (device, caller-owned), byte offsets.
struct PB {
  static constexpr size_t w = 0;                         // f32 [kW] master weights
  static constexpr size_t b = w + 4 * kW;                // f32 [kB]
  static constexpr size_t mw = b + 4 * kB;               // Adam moments
  static constexpr size_t vw = mw + 4 * kW;
  static constexpr size_t mb = vw + 4 * kW;
  static constexpr size_t vb = mb + 4 * kB;
  static constexpr size_t gw = vb + 4 * kB;              // gradient accumulators
  static constexpr size_t gb = gw + 4 * kW;
  static constexpr size_t norm = gb + 4 * kB;            // f32 mean[8], std[8], out_std[16]
  static constexpr size_t step = norm + 4 * 32;          // int32 Adam step count
  static constexpr size_t wf = step + 256;               // bf16 [kW] forward weights
  static constexpr size_t wb = wf + 2 * kW;              // bf16 [kWb] backward-data weights
  static constexpr size_t total = (wb + 2 * kWb + 255) & ~(size_t)255;
};

__device__ __forceinline__ uint16_t f2bf(float f) {
  // round to nearest even of the upper 16 bits (finite inputs)
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// tanh in FP32.  Below 1: x + x^3 p(x^2), p fitted for the least relative error,
// its coefficients rounded one after the other with the rest fitted again.
// Above: 1 - 2 / (1 + exp(2|x|)) with the sign of x, by the hardware's exp2 and
// reciprocal (1 ulp each).  A NaN takes the polynomial.  Over all floats of
// [2^-12, 12): at most 1.35 ulp, 0.290 on average (root mean square); the
// math library's 1.41 and 0.295, at twice the time of the layer's matrix
// instructions.
__device__ __forceinline__ float tanh_f32(float x) {
  const float a = fabsf(x), s = x * x;
  const float e = __builtin_amdgcn_exp2f(2.88539008f * a);
  const float big = copysignf(fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + e), 1.0f), x);
  float p = fmaf(s, 0x1.e77086p-14f, -0x1.ae8e98p-11f);
  p = fmaf(s, p, 0x1.8f86c0p-9f);
  p = fmaf(s, p, -0x1.18db78p-7f);
  p = fmaf(s, p, 0x1.64c046p-6f);
  p = fmaf(s, p, -0x1.b9f6dap-5f);
  p = fmaf(s, p, 0x1.11103cp-3f);
  p = fmaf(s, p, -0x1.555552p-2f);
  return a >= 1.0f ? big : fmaf(x * s, p, x);
}

// One periodic 3x3 layer over N = nimg*ny*nx pixels.  W: bf16
// [COUTP][9][CINP].  MODE 0: out bf16 = tanh(acc + bias); 1: out f32 = acc +
// bias; 2: out bf16 = acc * (1 - h^2) with h from H [N][COUTP] (the
// backward-data product of a tanh layer, no bias).
//
// A wavefront takes tiles of 16 consecutive pixels; lane (ln, lq) = (lane %
// 16, lane / 16) holds, of each group of 32 k, the k 8 lq .. 8 lq + 7 of pixel
// ln for the B operand and of output row ln for the A operand, and receives
// out channels 4lq..4lq+3 of pixel ln.  A group is one tap's 32 channels, or
// two taps' 16 (of the tenth tap both operands are zero, so that an infinite
// input stays infinite there).  What bounds it: the activations
// cross HBM once (a 32-channel layer of a million pixels moves 134 MB), and
// each is read nine times from L1 and L2.  The weights stay in registers (72
// of them at 32 x 32 channels) over all tiles of the wavefront: read from LDS
// for every tile they took one LDS access per matrix instruction.  The next
// tile's nine loads go out before the current tile's products.
// 32 -> 32 at 1,048,576 pixels: 125 to 53 us (2.5 TB/s of HBM); at 131,072 29 to
// 12 us.
template <int CINP, int COUTP, int MODE>
__global__ __launch_bounds__(256, 2) void k_conv3x3(const uint16_t* __restrict__ X,
                                                    const uint16_t* __restrict__ W,
                                                    const float* __restrict__ bias,
                                                    const uint16_t* __restrict__ Hact,
                                                    void* __restrict__ out, uint32_t N, int nx,
                                                    int ny, FastDiv fP, FastDiv fnx) {
  constexpr int MT = COUTP / 16, TPG = 32 / CINP, NG = (9 + TPG - 1) / TPG;  // taps per group, groups
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int ln = lane & 15, lq = lane >> 4;
  const int sub = lq * 8 / CINP, ch = lq * 8 % CINP;  // the lane's tap in a group, and channels
  v8b w[NG][MT];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    const int t = q * TPG + sub;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      u4a8 v = {0u, 0u, 0u, 0u};
      if (t < 9) v = *reinterpret_cast<const u4a8*>(W + ((mt * 16 + ln) * 9 + t) * CINP + ch);
      w[q][mt] = __builtin_bit_cast(v8b, v);
    }
  }
  float bs[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) bs[mt][i] = MODE == 2 ? 0.0f : bias[mt * 16 + lq * 4 + i];
  const uint32_t ntiles = (uint32_t)(((uint64_t)N + 15) / 16);
  // block b's tiles are contiguous (neighbouring rows share its L1), and an
  // XCD's blocks take a contiguous eighth of them (they share its L2)
  const uint32_t nb = gridDim.x, per8 = nb / 8, rem8 = nb % 8, xcd = blockIdx.x % 8;
  const uint32_t blk = xcd * per8 + min(xcd, rem8) + blockIdx.x / 8;
  const uint32_t t1 = (uint32_t)((uint64_t)(blk + 1) * ntiles / nb);
  uint32_t tile = (uint32_t)((uint64_t)blk * ntiles / nb) + (uint32_t)wid;
  auto load = [&](uint32_t tl, u4a8* v) {
    // a lane past the end reads the last pixel (never stored)
    const uint32_t p = min(tl * 16 + (uint32_t)ln, N - 1);
    const uint32_t img = fdiv(p, fP), r = p - img * fP.d;
    const int y = (int)fdiv(r, fnx), x = (int)(r - (uint32_t)y * fnx.d);
    const int yy[3] = {(y == 0 ? ny : y) - 1, y, y == ny - 1 ? 0 : y + 1};
    const int xx[3] = {(x == 0 ? nx : x) - 1, x, x == nx - 1 ? 0 : x + 1};
    const uint16_t* base = X + (int64_t)img * fP.d * CINP + ch;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      int yt, xt;
      if (TPG == 1) {
        yt = yy[q / 3];
        xt = xx[q % 3];
      } else {  // two taps a group: the lane's own (the tenth tap reads the last one's pixel)
        constexpr int last = 8;
        const int ta = q * TPG < last ? q * TPG : last, tb = q * TPG + 1 < last ? q * TPG + 1 : last;
        yt = sub == 0 ? yy[ta / 3] : yy[tb / 3];
        xt = sub == 0 ? xx[ta % 3] : xx[tb % 3];
      }
      v[q] = *reinterpret_cast<const u4a8*>(base + ((int64_t)yt * nx + xt) * CINP);
    }
  };
  u4a8 cur[NG], nxt[NG];
  if (tile < t1) load(tile, cur);
  for (; tile < t1; tile += 4) {
    if (tile + 4 < t1) load(tile + 4, nxt);
    const uint32_t p = tile * 16 + (uint32_t)ln;
    const bool live = p < N;
    uint2 hv[MT];
    if (MODE == 2)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        hv[mt] = *reinterpret_cast<const uint2*>(Hact + (int64_t)min(p, N - 1) * COUTP + mt * 16 +
                                                 lq * 4);
    v4f acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = v4f{0.f, 0.f, 0.f, 0.f};
    if (TPG == 2 && sub == 1) cur[NG - 1] = u4a8{0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[q][mt], __builtin_bit_cast(v8b, cur[q]),
                                                          acc[mt], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NG; ++q) cur[q] = nxt[q];
    if (!live) continue;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int co = mt * 16 + lq * 4;
      if (MODE == 1) {
        float4 v;
        v.x = acc[mt][0] + bs[mt][0];
        v.y = acc[mt][1] + bs[mt][1];
        v.z = acc[mt][2] + bs[mt][2];
        v.w = acc[mt][3] + bs[mt][3];
        *reinterpret_cast<float4*>(static_cast<float*>(out) + (int64_t)p * COUTP + co) = v;
      } else {
        // (the conversion rounds to nearest even, two values an instruction)
        typedef __bf16 v4b __attribute__((ext_vector_type(4)));
        v4b o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v;
          if (MODE == 0) {
            v = tanh_f32(acc[mt][i] + bs[mt][i]);
          } else {
            const uint32_t hw = i < 2 ? hv[mt].x : hv[mt].y;
            const float h = bf2f((uint16_t)(i & 1 ? hw >> 16 : hw & 0xFFFFu));
            v = acc[mt][i] * (1.0f - h * h);
          }
          o[i] = (__bf16)v;
        }
        const uint2 pk = __builtin_bit_cast(uint2, o);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(out) + (int64_t)p * COUTP + co) = pk;
      }
    }
  }
}

// Weight gradient of a periodic 3x3 layer: dW[co][t][ci] = sum_p dZ[p][co]
// X[p + off(t)][ci], db[co] = sum_p dZ[p][co], as per-block partials
// part[block][COUTP*9*CINP + COUTP].
//
// A block takes tiles of 32 x 8 pixels, one row per wavefront: dZ and X with a
// one-pixel rim go to LDS as they lie in memory (pixel-major), each X once
// instead of once per tap.  K runs along the 32 pixels of a row: both operands
// come through the transposing LDS load, whose 16 lanes read 4 pixels x 16
// channels and each receive one channel of the 4 pixels (the same pixels in
// the same places for A and B, so their order does not matter); a tap is an
// offset of the X address.  A wavefront keeps all 9 * (COUTP/16) * (CINP/16)
// output tiles and the sums of dZ (a product with ones) in registers, and the
// eight wavefronts' are added in order at the end.  The pixel stride (80 or 48
// bytes) spreads the 16 pixels of an access over all banks.  The next tile's
// loads go out before the current tile's products.
// 32 x 32 channels, 1,048,576 pixels: 763 to 43 us (134 MB, 19.3 GFLOP).
constexpr int kSegX = 32, kSegY = 8, kWgThreads = 64 * kSegY;
template <int CINP, int COUTP>
__global__ __launch_bounds__(kWgThreads, 2) void k_conv3x3_wgrad(const uint16_t* __restrict__ X,
                                                                 const uint16_t* __restrict__ dZ,
                                                                 float* __restrict__ part, int nimg,
                                                                 int nx, int ny) {
  constexpr int MT = COUTP / 16, NT = CINP / 16, NWT = COUTP * 9 * CINP;
  constexpr int XW = kSegX + 2, XH = kSegY + 2;              // X tile with its rim
  constexpr int XS = CINP + 8, ZS = COUTP + 8;               // pixel strides
  constexpr int XC = CINP / 8, ZC = COUTP / 8;               // 16-byte chunks per pixel
  constexpr int XN = XW * XH * XC, ZN = kSegX * kSegY * ZC;
  constexpr int XL = (XN + kWgThreads - 1) / kWgThreads, ZL = (ZN + kWgThreads - 1) / kWgThreads;
  constexpr int LX = XW * XH * XS, LZ = kSegX * kSegY * ZS;  // halves
  // a wavefront's sums of one tap (rows of RS: the four quarters of an access
  // fall on different banks) and of dZ
  constexpr int RS = CINP + 4, RW = COUTP * RS + COUTP;
  constexpr int LB = 2 * (LX + LZ);
  static_assert(4 * RW * kSegY <= LB, "two buffers of sums in the tiles' place (halves)");
  __shared__ __attribute__((aligned(16))) uint16_t lds[LB];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 15, lq = lane >> 4;
  const int64_t P = (int64_t)nx * ny;
  const int nsx = (nx + kSegX - 1) / kSegX, nsy = (ny + kSegY - 1) / kSegY;
  const int64_t steps = (int64_t)nimg * nsx * nsy;
  const int64_t s0 = steps * blockIdx.x / gridDim.x, s1 = steps * (blockIdx.x + 1) / gridDim.x;
  u4a8 gx[XL], gz[ZL];
  struct Tile {
    int64_t img;
    int x0, y0, w, h;
  };
  auto tile_at = [&](int64_t st) {
    Tile T;
    T.img = st / ((int64_t)nsx * nsy);
    const int r = (int)(st - T.img * nsx * nsy), sx = r / nsy, sy = r - sx * nsy;
    T.x0 = sx * kSegX;
    T.y0 = sy * kSegY;
    T.w = min(kSegX, nx - T.x0);
    T.h = min(kSegY, ny - T.y0);
    return T;
  };
  auto load = [&](const Tile& T) {
    const int64_t img = T.img;
    const int x0 = T.x0, y0 = T.y0, w = T.w, h = T.h;
#pragma unroll
    for (int u = 0; u < XL; ++u) {
      const int e = (int)threadIdx.x + u * kWgThreads;
      const int c = e % XC, px = (e / XC) % XW, row = e / (XC * XW);
      gx[u] = u4a8{0u, 0u, 0u, 0u};
      if (px < w + 2 && row < h + 2) {
        int xx = x0 + px - 1, yy = y0 + row - 1;
        xx = xx < 0 ? nx - 1 : (xx >= nx ? 0 : xx);
        yy = yy < 0 ? ny - 1 : (yy >= ny ? 0 : yy);
        gx[u] = *reinterpret_cast<const u4a8*>(X + (img * P + (int64_t)yy * nx + xx) * CINP + c * 8);
      }
    }
#pragma unroll
    for (int u = 0; u < ZL; ++u) {
      const int e = (int)threadIdx.x + u * kWgThreads;
      const int c = e % ZC, px = (e / ZC) % kSegX, row = e / (ZC * kSegX);
      gz[u] = u4a8{0u, 0u, 0u, 0u};
      if (px < w && row < h)
        gz[u] = *reinterpret_cast<const u4a8*>(
            dZ + (img * P + (int64_t)(y0 + row) * nx + x0 + px) * COUTP + c * 8);
    }
  };
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  auto stage = [&](uint16_t* sx, uint16_t* sz) {
#pragma unroll
    for (int u = 0; u < XL; ++u) {
      const int e = (int)threadIdx.x + u * kWgThreads;
      if (e < XN) *reinterpret_cast<u4*>(sx + (e / XC) * XS + (e % XC) * 8) = (u4)gx[u];
    }
#pragma unroll
    for (int u = 0; u < ZL; ++u) {
      const int e = (int)threadIdx.x + u * kWgThreads;
      if (e < ZN) *reinterpret_cast<u4*>(sz + (e / ZC) * ZS + (e % ZC) * 8) = (u4)gz[u];
    }
  };
  // 32 pixels (k) x 16 channels at `at` (pixel stride S): the lane's 8 k
  auto frag = [&](const uint16_t* at, int S) {
    typedef __attribute__((address_space(3))) v4s* Lp;
    const uint16_t* q = at + (4 * lq + ln / 4) * S + (ln % 4) * 4;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lp)q);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lp)(q + 16 * S));
    return __builtin_bit_cast(v8b, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  v4f acc[9][MT][NT], sum[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    sum[mt] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[t][mt][nt] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  v8b ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;
  Tile next{};
  if (s0 < s1) load(next = tile_at(s0));
  int buf = 0;
  for (int64_t st = s0; st < s1; ++st, buf ^= 1) {
    // one barrier a tile: its buffer was last read two tiles ago, before the
    // barrier of the tile in between
    uint16_t* sx = lds + buf * (LX + LZ);
    uint16_t* sz = sx + LX;
    const Tile cur = next;
    stage(sx, sz);
    __syncthreads();
    if (st + 1 < s1) load(next = tile_at(st + 1));
    // pixels of the row that are missing (their dZ is zero) have their X zeroed
    // too: a pixel of the rim may lie there, and 0 times an infinite X is NaN
    const int w = wid < cur.h ? cur.w : 0;
    u4 keep;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int px = 16 * (i / 2) + 4 * lq + 2 * (i % 2);  // and the one after
      keep[i] = (px < w ? 0xFFFFu : 0u) | (px + 1 < w ? 0xFFFF0000u : 0u);
    }
    v8b a[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      a[mt] = frag(sz + wid * kSegX * ZS + mt * 16, ZS);
      sum[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], ones, sum[mt], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const v8b x = frag(sx + ((wid + t / 3) * XW + t % 3) * XS + nt * 16, XS);
        const v8b b = __builtin_bit_cast(v8b, __builtin_bit_cast(u4, x) & keep);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[t][mt][nt] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], b, acc[t][mt][nt], 0, 0, 0);
      }
  }
  // The eight wavefronts' sums, added in order, a tap at a time: all leave
  // theirs in LDS and every thread adds up two or one of the outputs, with two
  // buffers and one barrier a tap (one wavefront after the other adding all of
  // its sums to the block's took 17 us more of every launch: training steps of
  // three 8 x 8 grids 148 to 79 us, of eight 512 x 256 ones 619 to 550).
  float* red = reinterpret_cast<float*>(lds);
  float* mine = part + (size_t)blockIdx.x * (NWT + COUTP);
  __syncthreads();  // the last tile is read
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    float* r = red + (t & 1) * RW * kSegY;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int co = mt * 16 + lq * 4 + i;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) r[wid * RW + co * RS + nt * 16 + ln] = acc[t][mt][nt][i];
        if (t == 0 && ln == 0) r[wid * RW + COUTP * RS + co] = sum[mt][i];
      }
    __syncthreads();
    auto total = [&](int at) {
      float v = r[at];
#pragma unroll
      for (int wv = 1; wv < kSegY; ++wv) v += r[wv * RW + at];
      return v;
    };
    for (int o = threadIdx.x; o < COUTP * CINP; o += kWgThreads)
      mine[(o / CINP * 9 + t) * CINP + o % CINP] = total(o / CINP * RS + o % CINP);
    if (t == 0 && threadIdx.x < COUTP) mine[NWT + threadIdx.x] = total(COUTP * RS + threadIdx.x);
  }
}

// gw[i] += sum over nb blocks of part[b][i] (fixed order: four quarters of the
// blocks, each in order, then their sum); i < n weights followed by nbias
// biases of the layer.  A block takes 64 outputs, a wavefront one quarter of
// the partials (one thread for all 256 took 61 us, this 5).
__global__ __launch_bounds__(256) void k_wgrad_reduce(const float* __restrict__ part, int nb,
                                                      int nwt, int nbias, float* __restrict__ gw,
                                                      float* __restrict__ gb) {
  __shared__ float s_q[4][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const int n = nwt + nbias;
  const int b0 = nb * wid / 4, b1 = nb * (wid + 1) / 4;
  float s = 0.f;
  if (i < n) {
    int b = b0;
    for (; b + 8 <= b1; b += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(b + u) * n + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < b1; ++b) s += part[(size_t)b * n + i];
  }
  s_q[wid][lane] = s;
  __syncthreads();
  if (wid != 0 || i >= n) return;
  s = (s_q[0][lane] + s_q[1][lane]) + (s_q[2][lane] + s_q[3][lane]);
  if (i < nwt)
    gw[i] += s;
  else
    gb[i - nwt] += s;
}

// The 7 normalised input channels (padded to 16) of sample idx[s] (s if idx
// is null) at every pixel: X0[s*P + r][c].
__global__ void k_no_pack(const float* __restrict__ B, const float* __restrict__ n,
                          const float* __restrict__ J, const int32_t* __restrict__ idx, int S,
                          int64_t P, const float* __restrict__ norm, uint16_t* __restrict__ X0) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (int64_t)S * P) return;
  const int s = (int)(p / P);
  const int64_t r = p - (int64_t)s * P;
  const int64_t smp = idx ? idx[s] : s;
  const float v[7] = {B[smp * 3 * P + r], B[smp * 3 * P + P + r], B[smp * 3 * P + 2 * P + r],
                      n[smp * P + r],   J[smp * 3 * P + r], J[smp * 3 * P + P + r],
                      J[smp * 3 * P + 2 * P + r]};
  uint16_t o[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) o[c] = c < 7 ? f2bf((v[c] - norm[c]) / norm[8 + c]) : (uint16_t)0;
  uint4* dst = reinterpret_cast<uint4*>(X0 + p * 16);
  uint4 a, b;
  a.x = o[0] | ((uint32_t)o[1] << 16);
  a.y = o[2] | ((uint32_t)o[3] << 16);
  a.z = o[4] | ((uint32_t)o[5] << 16);
  a.w = o[6] | ((uint32_t)o[7] << 16);
  b.x = o[8] | ((uint32_t)o[9] << 16);
  b.y = o[10] | ((uint32_t)o[11] << 16);
  b.z = o[12] | ((uint32_t)o[13] << 16);
  b.w = o[14] | ((uint32_t)o[15] << 16);
  dst[0] = a;
  dst[1] = b;
}

// Loss of the normalised increment and its gradient: d = D[p][c] - (Bt - B)
// / out_std for c < 3; dZ4 = bf16(2 d / (3 S P)); per-block FP64 partials of
// sum d^2.
__global__ __launch_bounds__(256) void k_no_loss(const float* __restrict__ D,
                                                 const float* __restrict__ B,
                                                 const float* __restrict__ Bt,
                                                 const int32_t* __restrict__ idx, int S, int64_t P,
                                                 const float* __restrict__ norm,
                                                 uint16_t* __restrict__ dZ, double* part) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double v[1] = {0.0};
  if (p < (int64_t)S * P) {
    const int s = (int)(p / P);
    const int64_t r = p - (int64_t)s * P;
    const int64_t smp = idx ? idx[s] : s;
    const float scale = 2.0f / (float)(3.0 * (double)S * (double)P);
    uint16_t o[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) o[c] = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float tgt = (Bt[smp * 3 * P + c * P + r] - B[smp * 3 * P + c * P + r]) / norm[16 + c];
      const float d = D[p * 16 + c] - tgt;
      v[0] += (double)d * (double)d;
      o[c] = f2bf(scale * d);
    }
    uint4* dst = reinterpret_cast<uint4*>(dZ + p * 16);
    uint4 a, b;
    a.x = o[0] | ((uint32_t)o[1] << 16);
    a.y = o[2] | ((uint32_t)o[3] << 16);
    a.z = a.w = 0u;
    b.x = b.y = b.z = b.w = 0u;
    dst[0] = a;
    dst[1] = b;
  }
  block_partial<1, 1>(v, part);
}

__global__ void k_no_loss_final(const double* part, int nb, int64_t count, double* out) {
  double r[1];
  sum_partials<1, 1>(part, nb, r);
  if (threadIdx.x == 0) out[0] = r[0] / (double)count;
}

// mask of the real (unpadded) entries of weight i of the concatenated
// padded array (layer l, out co, in ci)
__device__ __forceinline__ bool weight_live(int i, int& l, int& co, int& t, int& ci) {
  l = 0;
  while (l < kNL - 1 && i >= woff(l + 1)) ++l;
  const int j = i - woff(l);
  co = j / (9 * kCinP[l]);
  t = (j / kCinP[l]) % 9;
  ci = j % kCinP[l];
  return co < kCout[l] && ci < kCin[l];
}

// One Adam step (bias-corrected) over the padded weights and biases, the
// gradient accumulators cleared, the BF16 forward copies and the flipped,
// transposed backward-data copies (layers 1..3) rewritten.  With lr = 0 only
// the copies are refreshed (after loading weights).
__global__ void k_no_adam(char* pb, float lr, float b1, float b2, float eps, int do_update) {
  float* w = reinterpret_cast<float*>(pb + PB::w);
  float* b = reinterpret_cast<float*>(pb + PB::b);
  float* mw = reinterpret_cast<float*>(pb + PB::mw);
  float* vw = reinterpret_cast<float*>(pb + PB::vw);
  float* mb = reinterpret_cast<float*>(pb + PB::mb);
  float* vb = reinterpret_cast<float*>(pb + PB::vb);
  float* gw = reinterpret_cast<float*>(pb + PB::gw);
  float* gb = reinterpret_cast<float*>(pb + PB::gb);
  uint16_t* wf = reinterpret_cast<uint16_t*>(pb + PB::wf);
  uint16_t* wbk = reinterpret_cast<uint16_t*>(pb + PB::wb);
  const int step = *reinterpret_cast<const int*>(pb + PB::step) + (do_update ? 1 : 0);
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  auto upd = [&](float& p, float& m, float& v, float& g) {
    m = b1 * m + (1.0f - b1) * g;
    v = b2 * v + (1.0f - b2) * g * g;
    p -= lr * (m / c1) / (sqrtf(v / c2) + eps);
    g = 0.0f;
  };
  if (i < kW) {
    int l, co, t, ci;
    const bool live = weight_live(i, l, co, t, ci);
    if (!live) {
      w[i] = 0.0f;
      gw[i] = 0.0f;
    } else if (do_update) {
      upd(w[i], mw[i], vw[i], gw[i]);
    }
    const uint16_t h = f2bf(w[i]);
    wf[i] = h;
    if (l >= 1) {
      // backward data of layer l: [CINP_l][9][COUTP_l], tap flipped
      wbk[bwoff(l) + (ci * 9 + (8 - t)) * kCoutP[l] + co] = h;
    }
  } else if (i < kW + kB) {
    const int j = i - kW;
    int l = 0;
    while (l < kNL - 1 && j >= boff(l + 1)) ++l;
    const bool live = j - boff(l) < kCout[l];
    if (!live) {
      b[j] = 0.0f;
      gb[j] = 0.0f;
    } else if (do_update) {
      upd(b[j], mb[j], vb[j], gb[j]);
    }
  }
  if (i == 0 && do_update) *reinterpret_cast<int*>(pb + PB::step) = step;
}

// Loads logical weights w_l [Cout][9][Cin] (concatenated), biases and the
// normalisation (mean[7], std[7], out_std[3]) into the padded block; clears
// Adam's state and the gradients.
__global__ void k_no_load(char* pb, const float* __restrict__ wl, const float* __restrict__ bl,
                          const float* __restrict__ norm) {
  float* w = reinterpret_cast<float*>(pb + PB::w);
  float* b = reinterpret_cast<float*>(pb + PB::b);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kW) {
    int l, co, t, ci;
    const bool live = weight_live(i, l, co, t, ci);
    int lo = 0;
    for (int k = 0; k < l; ++k) lo += kCout[k] * 9 * kCin[k];
    w[i] = live ? wl[lo + (co * 9 + t) * kCin[l] + ci] : 0.0f;
    reinterpret_cast<float*>(pb + PB::mw)[i] = 0.0f;
    reinterpret_cast<float*>(pb + PB::vw)[i] = 0.0f;
    reinterpret_cast<float*>(pb + PB::gw)[i] = 0.0f;
  } else if (i < kW + kB) {
    const int j = i - kW;
    int l = 0;
    while (l < kNL - 1 && j >= boff(l + 1)) ++l;
    int lo = 0;
    for (int k = 0; k < l; ++k) lo += kCout[k];
    const int co = j - boff(l);
    b[j] = co < kCout[l] ? bl[lo + co] : 0.0f;
    reinterpret_cast<float*>(pb + PB::mb)[j] = 0.0f;
    reinterpret_cast<float*>(pb + PB::vb)[j] = 0.0f;
    reinterpret_cast<float*>(pb + PB::gb)[j] = 0.0f;
  } else if (i < kW + kB + 32) {
    const int k = i - kW - kB;
    float v = 0.0f;
    if (k < 7) v = norm[k];
    else if (k >= 8 && k < 15) v = norm[7 + k - 8];
    else if (k >= 16 && k < 19) v = norm[14 + k - 16];
    else if (k >= 8) v = 1.0f;  // scale slots of padding channels
    reinterpret_cast<float*>(pb + PB::norm)[k] = v;
  }
  if (i == 0) *reinterpret_cast<int*>(pb + PB::step) = 0;
}

__global__ void k_no_store(const char* pb, float* __restrict__ wl, float* __restrict__ bl) {
  const float* w = reinterpret_cast<const float*>(pb + PB::w);
  const float* b = reinterpret_cast<const float*>(pb + PB::b);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kW) {
    int l, co, t, ci;
    if (weight_live(i, l, co, t, ci)) {
      int lo = 0;
      for (int k = 0; k < l; ++k) lo += kCout[k] * 9 * kCin[k];
      wl[lo + (co * 9 + t) * kCin[l] + ci] = w[i];
    }
  } else if (i < kW + kB) {
    const int j = i - kW;
    int l = 0;
    while (l < kNL - 1 && j >= boff(l + 1)) ++l;
    int lo = 0;
    for (int k = 0; k < l; ++k) lo += kCout[k];
    const int co = j - boff(l);
    if (co < kCout[l]) bl[lo + co] = b[j];
  }
}

// B_out[c][r] = B[c][r] + out_std[c] * D[r][c] (one sample)
__global__ void k_no_out(const float* __restrict__ B, const float* __restrict__ D, int64_t P,
                         const float* __restrict__ norm, float* __restrict__ Bo) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= P) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) Bo[c * P + r] = B[c * P + r] + norm[16 + c] * D[r * 16 + c];
}

// activation buffers of a workspace for S samples of P pixels
struct Acts {
  uint16_t *x0, *h1, *h2, *h3, *dz4, *dza, *dzb;
  float* d4;
  float* part;    // weight-gradient partials
  double* lpart;  // loss partials
};
constexpr int kWgradBlocks = 256;
int64_t lpart_slots(int64_t N) { return ceil_div(N, 256); }

size_t acts_bytes(int64_t N) {
  size_t off = 0;
  auto take = [&](size_t b) { off += (b + 255) & ~(size_t)255; };
  take(2 * 16 * N);                                    // x0
  for (int k = 0; k < 3; ++k) take(2 * 32 * N);        // h1..h3
  take(2 * 16 * N);                                    // dz4
  take(2 * 32 * N);                                    // dza
  take(2 * 32 * N);                                    // dzb
  take(4 * 16 * N);                                    // d4
  take(4 * (size_t)kWgradBlocks * (32 * 9 * 32 + 32)); // partials
  take(8 * lpart_slots(N));
  return off;
}

Acts acts_of(void* ws, int64_t N) {
  char* base = static_cast<char*>(ws);
  size_t off = 0;
  auto take = [&](size_t b) {
    char* p = base + off;
    off += (b + 255) & ~(size_t)255;
    return p;
  };
  Acts a;
  a.x0 = (uint16_t*)take(2 * 16 * N);
  a.h1 = (uint16_t*)take(2 * 32 * N);
  a.h2 = (uint16_t*)take(2 * 32 * N);
  a.h3 = (uint16_t*)take(2 * 32 * N);
  a.dz4 = (uint16_t*)take(2 * 16 * N);
  a.dza = (uint16_t*)take(2 * 32 * N);
  a.dzb = (uint16_t*)take(2 * 32 * N);
  a.d4 = (float*)take(4 * 16 * N);
  a.part = (float*)take(4 * (size_t)kWgradBlocks * (32 * 9 * 32 + 32));
  a.lpart = (double*)take(8 * lpart_slots(N));
  return a;
}

// two blocks (eight wavefronts) per CU hold the layers' weights; fewer tiles
// take a wavefront each
int conv_grid(int64_t N) { return (int)std::min<int64_t>(ceil_div(ceil_div(N, 16), 4), 512); }

template <int CINP, int COUTP, int MODE>
void conv(hipStream_t s, const uint16_t* X, const uint16_t* W, const float* bias,
          const uint16_t* H, void* out, int64_t N, int nx, int ny) {
  constexpr int kOutBytes = COUTP * (MODE == 1 ? sizeof(float) : sizeof(uint16_t));
  for_pixel_groups(N, (int64_t)nx * ny, [&](int64_t p, int64_t n) {
    hipLaunchKernelGGL((k_conv3x3<CINP, COUTP, MODE>), dim3(conv_grid(n)), dim3(256), 0, s,
                       X + p * CINP, W, bias, H ? H + p * COUTP : nullptr,
                       static_cast<void*>(static_cast<char*>(out) + p * kOutBytes), (uint32_t)n,
                       nx, ny, make_fastdiv((uint32_t)(nx * ny)), make_fastdiv((uint32_t)nx));
  });
}

template <int CINP, int COUTP>
void wgrad(hipStream_t s, const uint16_t* X, const uint16_t* dZ, float* part, float* gw,
           float* gb, int64_t N, int nx, int ny) {
  const int nimg = (int)(N / ((int64_t)nx * ny));
  const int64_t tiles = nimg * ceil_div(nx, kSegX) * ceil_div(ny, kSegY);
  const int nb = (int)std::min<int64_t>(tiles, kWgradBlocks);
  hipLaunchKernelGGL((k_conv3x3_wgrad<CINP, COUTP>), dim3(nb), dim3(kWgThreads), 0, s, X, dZ, part,
                     nimg, nx, ny);
  const int n = COUTP * 9 * CINP + COUTP;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)ceil_div(n, 64)), dim3(256), 0, s,
                     (const float*)part, nb, COUTP * 9 * CINP, COUTP, gw, gb);
}

// the forward pass of S samples: X0 -> d4 (normalised increment)
void forward(hipStream_t s, const char* pb, const Acts& a, int64_t N, int nx, int ny) {
  const uint16_t* wf = reinterpret_cast<const uint16_t*>(pb + PB::wf);
  const float* b = reinterpret_cast<const float*>(pb + PB::b);
  conv<16, 32, 0>(s, a.x0, wf + woff(0), b + boff(0), nullptr, a.h1, N, nx, ny);
  conv<32, 32, 0>(s, a.h1, wf + woff(1), b + boff(1), nullptr, a.h2, N, nx, ny);
  conv<32, 32, 0>(s, a.h2, wf + woff(2), b + boff(2), nullptr, a.h3, N, nx, ny);
  conv<32, 16, 1>(s, a.h3, wf + woff(3), b + boff(3), nullptr, a.d4, N, nx, ny);
}

bool grid_ok(int nx, int ny) { return nx >= 1 && ny >= 1 && (int64_t)nx * ny < (1ll << 28); }

}  // namespace

size_t no_params_bytes() { return PB::total; }

// The proposal B_out of the operator for one sample (B, n, J on an nx x ny
// grid), enqueued on s.
int no_predict(hipStream_t s, const void* params, void* ws, int nx, int ny, const float* B,
               const float* n, const float* J, float* B_out) {
  const int64_t P = (int64_t)nx * ny;
  const Acts a = acts_of(ws, P);
  const char* pb = static_cast<const char*>(params);
  const float* norm = reinterpret_cast<const float*>(pb + PB::norm);
  hipLaunchKernelGGL(k_no_pack, dim3((unsigned)ceil_div(P, 256)), dim3(256), 0, s, B, n, J,
                     (const int32_t*)nullptr, 1, P, norm, a.x0);
  forward(s, pb, a, P, nx, ny);
  hipLaunchKernelGGL(k_no_out, dim3((unsigned)ceil_div(P, 256)), dim3(256), 0, s, B,
                     (const float*)a.d4, P, norm, B_out);
  return hipGetLastError() == hipSuccess ? HVPIC_OK : HVPIC_EHIP;
}

}  // namespace hvpic

using namespace hvpic;

extern "C" {

int hvpic_no_params_bytes(size_t* bytes) {
  if (!bytes) return HVPIC_EINVAL;
  *bytes = PB::total;
  return HVPIC_OK;
}

int hvpic_no_workspace_bytes(int nx, int ny, int batch, size_t* bytes) {
  if (!bytes || !grid_ok(nx, ny) || batch < 1 || batch > 4096) return HVPIC_EINVAL;
  *bytes = acts_bytes((int64_t)nx * ny * batch);
  return HVPIC_OK;
}

int hvpic_no_load(void* params, const float* w, const float* b, const float* norm,
                  void* hip_stream) {
  if (!params || !w || !b || !norm) return HVPIC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int n = kW + kB + 32;
  hipLaunchKernelGGL(k_no_load, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, s,
                     static_cast<char*>(params), w, b, norm);
  hipLaunchKernelGGL(k_no_adam, dim3((unsigned)ceil_div(kW + kB, 256)), dim3(256), 0, s,
                     static_cast<char*>(params), 0.0f, 0.9f, 0.999f, 1e-8f, 0);
  return hipGetLastError() == hipSuccess ? HVPIC_OK : HVPIC_EHIP;
}

int hvpic_no_store(const void* params, float* w, float* b, void* hip_stream) {
  if (!params || !w || !b) return HVPIC_EINVAL;
  hipLaunchKernelGGL(k_no_store, dim3((unsigned)ceil_div(kW + kB, 256)), dim3(256), 0,
                     static_cast<hipStream_t>(hip_stream), static_cast<const char*>(params), w, b);
  return hipGetLastError() == hipSuccess ? HVPIC_OK : HVPIC_EHIP;
}

int hvpic_no_predict(const void* params, void* workspace, int nx, int ny, const float* B,
                     const float* n, const float* J, float* B_out, void* hip_stream) {
  if (!params || !workspace || !grid_ok(nx, ny) || !B || !n || !J || !B_out) return HVPIC_EINVAL;
  return no_predict(static_cast<hipStream_t>(hip_stream), params, workspace, nx, ny, B, n, J,
                    B_out);
}

int hvpic_no_train_step(void* params, void* workspace, int nx, int ny, const float* B,
                        const float* n, const float* J, const float* B_target, const int32_t* idx,
                        int batch, float lr, double* loss_out, void* hip_stream) {
  if (!params || !workspace || !grid_ok(nx, ny) || !B || !n || !J || !B_target || batch < 1 ||
      batch > 4096 || !(lr >= 0.0f))
    return HVPIC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int64_t P = (int64_t)nx * ny, N = P * batch;
  const Acts a = acts_of(workspace, N);
  char* pb = static_cast<char*>(params);
  const float* norm = reinterpret_cast<const float*>(pb + PB::norm);
  const uint16_t* wbk = reinterpret_cast<const uint16_t*>(pb + PB::wb);
  float* gw = reinterpret_cast<float*>(pb + PB::gw);
  float* gb = reinterpret_cast<float*>(pb + PB::gb);
  const unsigned pix = (unsigned)ceil_div(N, 256);
  hipLaunchKernelGGL(k_no_pack, dim3(pix), dim3(256), 0, s, B, n, J, idx, batch, P, norm, a.x0);
  forward(s, pb, a, N, nx, ny);
  hipLaunchKernelGGL(k_no_loss, dim3(pix), dim3(256), 0, s, (const float*)a.d4, B, B_target, idx,
                     batch, P, norm, a.dz4, a.lpart);
  // layer 3 (32 -> 16): weights, then the gradient at its input through tanh
  wgrad<32, 16>(s, a.h3, a.dz4, a.part, gw + woff(3), gb + boff(3), N, nx, ny);
  conv<16, 32, 2>(s, a.dz4, wbk + bwoff(3), nullptr, a.h3, a.dza, N, nx, ny);
  wgrad<32, 32>(s, a.h2, a.dza, a.part, gw + woff(2), gb + boff(2), N, nx, ny);
  conv<32, 32, 2>(s, a.dza, wbk + bwoff(2), nullptr, a.h2, a.dzb, N, nx, ny);
  wgrad<32, 32>(s, a.h1, a.dzb, a.part, gw + woff(1), gb + boff(1), N, nx, ny);
  conv<32, 32, 2>(s, a.dzb, wbk + bwoff(1), nullptr, a.h1, a.dza, N, nx, ny);
  wgrad<16, 32>(s, a.x0, a.dza, a.part, gw + woff(0), gb + boff(0), N, nx, ny);
  if (loss_out)
    hipLaunchKernelGGL(k_no_loss_final, dim3(1), dim3(1024), 0, s, (const double*)a.lpart,
                       (int)pix, (int64_t)(3 * N), loss_out);
  hipLaunchKernelGGL(k_no_adam, dim3((unsigned)ceil_div(kW + kB, 256)), dim3(256), 0, s, pb, lr,
                     0.9f, 0.999f, 1e-8f, 1);
  return hipGetLastError() == hipSuccess ? HVPIC_OK : HVPIC_EHIP;
}

int hvpic_field_advance_no(hvpic_ctx* ctx, const void* params, void* workspace, float* B,
                           const float* n_half, const float* J_half, const float* n_prev,
                           const float* J_prev, float* E_out, double* diag_out, float tol,
                           double* stats) {
  if (!ctx || ctx->magic != kMagic) return HVPIC_ESTATE;
  const hvpic_params& p = ctx->p;
  if (p.ndim != 2 || p.energy_eq || p.open_x || p.eta_h != 0.0 || p.nsub < 1) return HVPIC_EINVAL;
  if (!params || !workspace || !B || !n_half || !J_half || !n_prev || !J_prev || !E_out ||
      !(tol >= 0.0f))
    return HVPIC_EINVAL;
  float* Bno = ctx->fscratch + 22ll * ctx->ncell;  // the proposal [3][ncell]
  int rc = no_predict(ctx->stream, params, workspace, p.nx, p.ny, B, n_half, J_half, Bno);
  if (rc != HVPIC_OK) return rc;
  return launch_field_advance_no(ctx, B, n_half, J_half, n_prev, J_prev, E_out, diag_out, Bno,
                                 tol, stats);
}

// Single layers, for checking the kernels: a periodic 3x3 layer over nimg
// images (x bf16 [N][cinp], w bf16 [coutp][9][cinp]) and its weight gradient
// (added to dw [coutp][9][cinp] and db [coutp]).
int hvpic_no_conv3x3(int nimg, int nx, int ny, int cinp, int coutp, int mode, const void* x,
                     const void* w, const float* bias, const void* h, void* out,
                     void* hip_stream) {
  if (nimg < 1 || !grid_ok(nx, ny) || !x || !w || !out) return HVPIC_EINVAL;
  if (mode < 0 || mode > 2 || (mode != 2 && !bias) || (mode == 2 && !h)) return HVPIC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int64_t N = (int64_t)nx * ny * nimg;
  const uint16_t* X = static_cast<const uint16_t*>(x);
  const uint16_t* W = static_cast<const uint16_t*>(w);
  const uint16_t* H = static_cast<const uint16_t*>(h);
  const int key = cinp * 1000 + coutp * 10 + mode;
  switch (key) {
    case 16320: conv<16, 32, 0>(s, X, W, bias, H, out, N, nx, ny); break;
    case 32320: conv<32, 32, 0>(s, X, W, bias, H, out, N, nx, ny); break;
    case 32161: conv<32, 16, 1>(s, X, W, bias, H, out, N, nx, ny); break;
    case 16322: conv<16, 32, 2>(s, X, W, bias, H, out, N, nx, ny); break;
    case 32322: conv<32, 32, 2>(s, X, W, bias, H, out, N, nx, ny); break;
    default: return HVPIC_EINVAL;
  }
  return hipGetLastError() == hipSuccess ? HVPIC_OK : HVPIC_EHIP;
}

int hvpic_no_conv3x3_wgrad(int nimg, int nx, int ny, int cinp, int coutp, const void* x,
                           const void* dz, float* dw, float* db, void* workspace,
                           void* hip_stream) {
  if (nimg < 1 || !grid_ok(nx, ny) || !x || !dz || !dw || !db || !workspace) return HVPIC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int64_t N = (int64_t)nx * ny * nimg;
  const Acts a = acts_of(workspace, N);
  const uint16_t* X = static_cast<const uint16_t*>(x);
  const uint16_t* Z = static_cast<const uint16_t*>(dz);
  if (cinp == 32 && coutp == 16)
    wgrad<32, 16>(s, X, Z, a.part, dw, db, N, nx, ny);
  else if (cinp == 32 && coutp == 32)
    wgrad<32, 32>(s, X, Z, a.part, dw, db, N, nx, ny);
  else if (cinp == 16 && coutp == 32)
    wgrad<16, 32>(s, X, Z, a.part, dw, db, N, nx, ny);
  else
    return HVPIC_EINVAL;
  return hipGetLastError() == hipSuccess ? HVPIC_OK : HVPIC_EHIP;
}

}  // extern "C"
