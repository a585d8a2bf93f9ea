// Kernels of the warm-start network: MFMA implicit-GEMM convolutions (forward
// and, with flipped taps and transposed weights, backward-data), MFMA weight
// gradients with a fixed-order reduction, pooling / upsampling / skip
// kernels, the loss, parameter packing and Adam.
//
// The 3x3x3 convolutions read their input 27 times; from the caches that took
// 50 us for 16 channels at 64x64x128, where the bytes of one pass take 7 us
// and the matrix instructions 6.  They therefore stage a tile with its
// one-site ring in LDS (k_conv3), and take the element-wise passes around
// them along: the input's normalisation or the upsampled skip sum on the way
// in, the pooling, the 1x1x1 layer D or the children's sum on the way out.
// The weight gradients stage both operands once for all 27 taps (k_wgrad3).
//
// Convolution as a matrix product per 16 output sites:
//   D[co][site] = sum_k W[co][k] X[k][site],  k = (tap, input channel).
// The A operand (weights) is read as 8 or 4 consecutive input channels of one
// output channel, the B operand (activations) as 8 or 4 consecutive channels
// of one site; both are single vector loads in channels-last order.  The
// result lane holds 4 consecutive output channels of one site, stored as one
// 8-byte vector.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "ek_internal.h"
#include "reduce.h"
#include "unet.h"

namespace ek {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));

constexpr uint16_t BF_ONE = 0x3F80;

__device__ __forceinline__ uint16_t f2bf(float v) {
  return __builtin_bit_cast(uint16_t, (__bf16)v);
}
__device__ __forceinline__ float bf2f(uint16_t u) {
  return __builtin_bit_cast(float, uint32_t(u) << 16);
}

__device__ __forceinline__ void decode(const Grid3& g, int r, int& x, int& y, int& z) {
  const unsigned q = unsigned(r) / unsigned(g.nx);
  x = r - int(q) * g.nx;
  z = int(q / unsigned(g.ny));
  y = int(q) - z * g.ny;
}

// ---------------------------------------------------------------------------
// Convolution (forward, or backward-data with the flipped weight set)
// ---------------------------------------------------------------------------
enum Epi { EPI_RELU = 0, EPI_LINEAR = 1, EPI_MASK = 2, EPI_PLAIN = 3, EPI_OUT = 4 };

struct ConvIO {
  const uint16_t* in;       // [n][CIN]
  const uint16_t* w;        // [T][COUT][CIN]
  const float* bias;        // [COUT] (EPI_RELU, EPI_LINEAR, EPI_OUT)
  const uint16_t* act;      // [n][COUT]: ReLU gate (EPI_MASK)
  uint16_t* out;            // [n][COUT]
  float* out32;             // [n]: channel 0 (EPI_OUT)
  double* guess;            // [n]: channel 0 times the output scale (EPI_OUT, optional)
  const UNetScalars* sc;
  // sources and tails of k_conv3 / k_conv1
  const uint32_t* pair;     // [n]: two channels
  const double* b;          // [n]: right-hand side
  const void* solid;
  uint32_t* pair_out;       // [n]: the input formed from b and solid (optional)
  const uint16_t* up;       // [coarse n][CIN]: to be upsampled
  uint16_t* sum;            // [n][CIN]: the skip sum (optional)
  uint16_t* pool;           // [coarse n][COUT], or layer D's output [n][32]
  const uint16_t* w2;       // layer D
  const float* bias2;
};

__device__ __forceinline__ void unpack8(const uint4 q, float (&f)[8]) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = bf2f(uint16_t(w[e >> 1] >> (16 * (e & 1))));
}
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = uint32_t(f2bf(f[2 * e])) | (uint32_t(f2bf(f[2 * e + 1])) << 16);
  return uint4{w[0], w[1], w[2], w[3]};
}

__device__ __forceinline__ int parent(const Grid3& fine, const Grid3& coarse, int rf) {
  int x, y, z;
  decode(fine, rf, x, y, z);
  return ((z >> 1) * coarse.ny + (y >> 1)) * coarse.nx + (x >> 1);
}

// ReLU(a + b) of 8 channels.
__device__ __forceinline__ uint4 up_sum(const uint4 up, const uint4 skip) {
  float a[8], b[8];
  unpack8(up, a);
  unpack8(skip, b);
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = fmaxf(a[e] + b[e], 0.f);
  return pack8(a);
}

// Gradient at a pooled-and-skipped activation: (g + dp / 8) * [act > 0].
__device__ __forceinline__ uint4 skip_grad8(const uint4 g, const uint4 dp, const uint4 act) {
  float a[8], b[8], m[8];
  unpack8(g, a);
  unpack8(dp, b);
  unpack8(act, m);
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = m[e] > 0.f ? a[e] + 0.125f * b[e] : 0.f;
  return pack8(a);
}

// The network's two input channels at a site: ((b - mean) / s, solid).
__device__ __forceinline__ uint32_t input_pair(double b, bool solid, const UNetScalars* sc) {
  const float v = float((b - sc->mean) * sc->inv_s);
  return uint32_t(f2bf(v)) | (uint32_t(solid ? BF_ONE : 0) << 16);
}

// Four output channels of a site: bias, ReLU or gate, stored (and returned).
template <int COUT, int EPI>
__device__ __forceinline__ uint2 store4(const ConvIO& io, const f4& acc, size_t r, int co) {
  float v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = acc[i];
    if constexpr (EPI == EPI_RELU || EPI == EPI_LINEAR) v[i] += io.bias[co + i];
    if constexpr (EPI == EPI_RELU) v[i] = fmaxf(v[i], 0.f);
  }
  if constexpr (EPI == EPI_MASK) {
    const uint2 a = *(const uint2*)(io.act + r * COUT + co);
    if ((a.x & 0xFFFFu) == 0 || (a.x & 0x8000u)) v[0] = 0.f;
    if ((a.x >> 16) == 0 || (a.x & 0x80000000u)) v[1] = 0.f;
    if ((a.y & 0xFFFFu) == 0 || (a.y & 0x8000u)) v[2] = 0.f;
    if ((a.y >> 16) == 0 || (a.y & 0x80000000u)) v[3] = 0.f;
  }
  uint2 o;
  o.x = uint32_t(f2bf(v[0])) | (uint32_t(f2bf(v[1])) << 16);
  o.y = uint32_t(f2bf(v[2])) | (uint32_t(f2bf(v[3])) << 16);
  *(uint2*)(io.out + r * COUT + co) = o;
  return o;
}

// The 1x1x1 layers: a product per site.  With UP (layer E forward) the input
// is ReLU(upsample(u) + in), the skip sum of the finer level `in`, which goes
// to io.sum where that is given.
template <int CIN, int COUT, int EPI, bool UP>
__global__ __launch_bounds__(256) void k_conv1(ConvIO io, Grid3 g, Grid3 coarse) {
  constexpr int NC = COUT / 16;
  constexpr int KB = CIN == 16 ? 1 : CIN / 32;
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int site = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + col;
  const int r = site < g.n ? site : g.n - 1;
  f4 acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = f4{0.f, 0.f, 0.f, 0.f};
  if constexpr (CIN == 16) {
    const s4 bf = *(const s4*)(io.in + (size_t)r * CIN + grp * 4);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const s4 af = *(const s4*)(io.w + (size_t)(c * 16 + col) * CIN + grp * 4);
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af, bf, acc[c], 0, 0, 0);
    }
  } else {
    b8 bf[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      uint4 q = *(const uint4*)(io.in + (size_t)r * CIN + kb * 32 + grp * 8);
      if constexpr (UP) {
        q = up_sum(*(const uint4*)(io.up + (size_t)parent(g, coarse, r) * CIN + kb * 32 + grp * 8), q);
        if (io.sum && site < g.n) *(uint4*)(io.sum + (size_t)r * CIN + kb * 32 + grp * 8) = q;
      }
      bf[kb] = __builtin_bit_cast(b8, q);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const b8 af = *(const b8*)(io.w + (size_t)(c * 16 + col) * CIN + kb * 32 + grp * 8);
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf[kb], acc[c], 0, 0, 0);
      }
  }
  if (site >= g.n) return;
#pragma unroll
  for (int c = 0; c < NC; ++c) store4<COUT, EPI>(io, acc[c], (size_t)r, c * 16 + grp * 4);
}

// ---------------------------------------------------------------------------
// 3x3x3 convolution of a tile of 16 x TY x TZ sites staged in LDS with its
// one-site ring (periodic).  The four waves share the tile's x-runs of 16
// sites, or with WC > 1 also the output channels.  The taps are added in the
// order of the packed weights, one matrix instruction each (and per 32 input
// channels), whatever the tile.
// ---------------------------------------------------------------------------
enum Source {
  SRC_PLAIN = 0,    // io.in, CIN channels
  SRC_PAIR = 1,     // io.pair: the first two of 16 channels, the rest 0
  SRC_INPUT = 2,    // the network's input from b and the byte mask (a pair; to io.pair_out
                    // where that is given)
  SRC_LINK = 3,     // the same from b and link words
  SRC_UP = 4        // ReLU(upsample(io.up) + io.in) (to io.sum where that is given)
};
// What follows on the tile's output: nothing, the average or the sum of each
// 2x2x2 block (io.pool), or layer D (io.w2, io.bias2, io.pool: 32 channels)
enum Tail { TAIL_NONE = 0, TAIL_POOL = 1, TAIL_SUM = 2, TAIL_D = 3 };

// Tile -> workgroup so that each XCD holds a contiguous share of the tiles.
__device__ __forceinline__ int xcd_tile(int b, int n) {
  return (n & 7) == 0 ? (b & 7) * (n >> 3) + (b >> 3) : b;
}
__device__ __forceinline__ int wrap_at(int v, int n) {
  v = v < 0 ? v + n : v;
  return v < n ? v : v % n;
}

// Taps per matrix instruction.  One by one keeps the order of the additions;
// where no bfloat16 rounding follows that a forward pass hands on (the last
// layer, the data gradients of a pair) two taps of 16 channels or sixteen
// taps of a pair fill an instruction of 32 products: 14 or 2 instead of 27.
enum Taps { TAPS_ONE = 0, TAPS_TWO = 1, TAPS_ALL = 2 };

template <int SRC, int CIN, int COUT, int TY, int TZ, int WC, int EPI, int TAIL, int TAPS = TAPS_ONE>
__global__ __launch_bounds__(256) void k_conv3(ConvIO io, Grid3 g, Grid3 coarse) {
  constexpr bool PAIR = SRC == SRC_PAIR || SRC == SRC_INPUT || SRC == SRC_LINK;
  constexpr int RX = 18, RY = TY + 2, RZ = TZ + 2, RING = RX * RY * RZ;
  constexpr int SB = PAIR ? 4 : CIN * 2;                      // bytes of a staged site
  constexpr int RUNS = TY * TZ, WS = 4 / WC, NS = RUNS / WS, NC = COUT / 16 / WC;
  constexpr int KB = CIN == 16 ? 1 : CIN / 32;
  constexpr int OUT_BYTES = TAIL == TAIL_NONE ? 0 : RUNS * 16 * COUT * 2;
  static_assert(RUNS % WS == 0 && (COUT / 16) % WC == 0, "whole shares per wave");
  __shared__ __align__(16) unsigned char lds[RING * SB > OUT_BYTES ? RING * SB : OUT_BYTES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int ntx = (g.nx + 15) / 16, nty = (g.ny + TY - 1) / TY;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int x0 = tile % ntx * 16, y0 = tile / ntx % nty * TY, z0 = tile / (ntx * nty) * TZ;

  // every weight fragment of this wave, in flight while the tile is staged
  // (read a row of taps ahead instead, the small levels waited for the caches
  // nine times: 15 us for the quarter level's layers)
  static_assert(TAPS == TAPS_ONE || (CIN == 16 && COUT == 16 && PAIR == (TAPS == TAPS_ALL)), "schedules");
  const int ws = wave % WS, wc = wave / WS;
  constexpr int STEPS = TAPS == TAPS_ONE ? 27 : TAPS == TAPS_TWO ? 14 : 2;
  using Frag = std::conditional_t<CIN == 16 && TAPS == TAPS_ONE, s4, b8>;
  Frag w[STEPS][NC][KB];
  if constexpr (TAPS == TAPS_TWO) {          // lanes of group 2, 3: the second tap
    const uint16_t* wl = io.w + (size_t)col * CIN + (grp & 1) * 8;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      uint4 q{0u, 0u, 0u, 0u};
      if (2 * t + (grp >> 1) < 27) q = *(const uint4*)(wl + (size_t)(2 * t + (grp >> 1)) * COUT * CIN);
      w[t][0][0] = __builtin_bit_cast(b8, q);
    }
  } else if constexpr (TAPS == TAPS_ALL) {   // four taps per lane
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      uint32_t q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tap = 16 * t + 4 * grp + i;
        q[i] = tap < 27 ? *(const uint32_t*)(io.w + (size_t)(tap * COUT + col) * CIN) : 0u;
      }
      w[t][0][0] = __builtin_bit_cast(b8, uint4{q[0], q[1], q[2], q[3]});
    }
  } else {
    const uint16_t* wl = io.w + (size_t)(wc * NC * 16 + col) * CIN + grp * (CIN == 16 ? 4 : 8);
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          w[t][c][kb] = *(const Frag*)(wl + (size_t)(t * COUT + c * 16) * CIN + kb * 32);
  }

  // the tile and its ring, 16 bytes (or one pair) per thread and round
  constexpr int PER = PAIR ? 1 : CIN / 8;
#pragma unroll 4
  for (int t = tid; t < RING * PER; t += 256) {
    const int s = t / PER, v = t % PER;
    const int lx = s % RX, ly = s / RX % RY, lz = s / (RX * RY);
    const int x = wrap_at(x0 + lx - 1, g.nx), y = wrap_at(y0 + ly - 1, g.ny),
              z = wrap_at(z0 + lz - 1, g.nz);
    const size_t r = (size_t)(z * g.ny + y) * g.nx + x;
    const bool own = lx > 0 && lx < RX - 1 && ly > 0 && ly < RY - 1 && lz > 0 && lz < RZ - 1 &&
                     x0 + lx - 1 < g.nx && y0 + ly - 1 < g.ny && z0 + lz - 1 < g.nz;
    if constexpr (PAIR) {
      uint32_t q;
      if constexpr (SRC == SRC_PAIR) {
        q = io.pair[r];
      } else {
        bool solid;
        if constexpr (SRC == SRC_LINK) solid = (((const uint32_t*)io.solid)[r] & MASK_SOLID) != 0;
        else solid = ((const uint8_t*)io.solid)[r] != 0;
        q = input_pair(io.b[r], solid, io.sc);
        if (io.pair_out && own) io.pair_out[r] = q;
      }
      *(uint32_t*)(lds + s * 4) = q;
    } else {
      uint4 q = *(const uint4*)(io.in + r * CIN + v * 8);
      if constexpr (SRC == SRC_UP) {
        q = up_sum(*(const uint4*)(io.up + (size_t)((z >> 1) * coarse.ny + (y >> 1)) * coarse.nx * CIN +
                                   (size_t)(x >> 1) * CIN + v * 8),
                   q);
        if (io.sum && own) *(uint4*)(io.sum + r * CIN + v * 8) = q;
      }
      *(uint4*)(lds + s * SB + v * 16) = q;
    }
  }
  __syncthreads();

  int base[NS];                        // LDS byte of tap (-1, -1, -1) for this lane's site
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int run = ws * NS + j;
    base[j] = ((run / TY * RY + run % TY) * RX + col) * SB +
              (PAIR ? 0 : CIN > 16 ? grp * 16 : TAPS == TAPS_TWO ? (grp & 1) * 16 : grp * 8);
  }
  f4 acc[NC][NS];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int j = 0; j < NS; ++j) acc[c][j] = f4{0.f, 0.f, 0.f, 0.f};
  auto tap_at = [&](int t) { return ((t / 9 * RY + t / 3 % 3) * RX + t % 3) * SB; };
  int tap_lane[TAPS == TAPS_ALL ? STEPS : 1][4];   // this lane's taps (past the last: weight 0)
  if constexpr (TAPS == TAPS_ALL)
#pragma unroll
    for (int t = 0; t < STEPS; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) tap_lane[t][i] = tap_at(min(16 * t + 4 * grp + i, 26));
#pragma unroll
  for (int t = 0; t < STEPS; ++t) {
    if constexpr (TAPS == TAPS_ALL) {
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        uint32_t q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = *(const uint32_t*)(lds + base[j] + tap_lane[t][i]);
        acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            w[t][0][0], __builtin_bit_cast(b8, uint4{q[0], q[1], q[2], q[3]}), acc[0][j], 0, 0, 0);
      }
      continue;
    }
    if constexpr (TAPS == TAPS_TWO) {
      const int at = grp < 2 ? tap_at(2 * t) : tap_at(2 * t + 1 < 27 ? 2 * t + 1 : 26);
      b8 bf[NS];
#pragma unroll
      for (int j = 0; j < NS; ++j) bf[j] = *(const b8*)(lds + base[j] + at);
#pragma unroll
      for (int j = 0; j < NS; ++j)
        acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][0][0], bf[j], acc[0][j], 0, 0, 0);
      continue;
    }
    const unsigned char* src = lds + tap_at(t);
    if constexpr (CIN == 16 && TAPS == TAPS_ONE) {
      s4 bf[NS];
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        if constexpr (PAIR) {
          const uint32_t q = *(const uint32_t*)(src + base[j]);
          bf[j] = __builtin_bit_cast(s4, uint2{grp == 0 ? q : 0u, 0u});
        } else {
          bf[j] = *(const s4*)(src + base[j]);
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int j = 0; j < NS; ++j)
          acc[c][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[t][c][0], bf[j], acc[c][j], 0, 0, 0);
    } else if constexpr (CIN > 16) {
      b8 bf[NS][KB];
#pragma unroll
      for (int j = 0; j < NS; ++j)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) bf[j][kb] = *(const b8*)(src + base[j] + kb * 64);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int j = 0; j < NS; ++j)
            acc[c][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][c][kb], bf[j][kb], acc[c][j], 0, 0, 0);
    }
  }

  if constexpr (TAIL != TAIL_NONE) __syncthreads();   // the staged input is no longer read
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int run = ws * NS + j, x = x0 + col, y = y0 + run % TY, z = z0 + run / TY;
    const bool in_box = x < g.nx && y < g.ny && z < g.nz;
    const size_t r = (size_t)(z * g.ny + y) * g.nx + x;
    if constexpr (EPI == EPI_OUT) {
      if (grp == 0 && in_box) {
        const float v = acc[0][j][0] + io.bias[0];
        io.out32[r] = v;
        if (io.guess) io.guess[r] = double(v) * io.sc->scale;
      }
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int co = (wc * NC + c) * 16 + grp * 4;
        uint2 o{0u, 0u};
        if (in_box) o = store4<COUT, EPI>(io, acc[c][j], r, co);
        if constexpr (TAIL != TAIL_NONE)
          *(uint2*)(lds + (size_t)((run * 16 + col) * COUT + co) * 2) = o;
      }
    }
  }
  if constexpr (TAIL == TAIL_POOL || TAIL == TAIL_SUM) {
    __syncthreads();
    constexpr int G = COUT / 8, PX = 8, PY = TY / 2, PZ = TZ / 2;
    for (int t = tid; t < PX * PY * PZ * G; t += 256) {
      const int v = t % G, px = t / G % PX, py = t / (G * PX) % PY, pz = t / (G * PX * PY);
      const int X = x0 / 2 + px, Y = y0 / 2 + py, Z = z0 / 2 + pz;
      if (X >= coarse.nx || Y >= coarse.ny || Z >= coarse.nz) continue;
      float sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int run = (2 * pz + (k >> 2)) * TY + 2 * py + ((k >> 1) & 1);
        float f[8];
        unpack8(*(const uint4*)(lds + (size_t)((run * 16 + 2 * px + (k & 1)) * COUT + v * 8) * 2), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[e] += f[e];
      }
      if constexpr (TAIL == TAIL_POOL)
#pragma unroll
        for (int e = 0; e < 8; ++e) sum[e] *= 0.125f;
      *(uint4*)(io.pool + ((size_t)(Z * coarse.ny + Y) * coarse.nx + X) * COUT + v * 8) = pack8(sum);
    }
  }
  if constexpr (TAIL == TAIL_D) {      // a 1x1x1 product of the tile's 64 channels into 32
    static_assert(COUT == 64 && RUNS == 4, "a run per wave");
    __syncthreads();
    f4 u[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const b8 af = *(const b8*)(io.w2 + (size_t)(c * 16 + col) * 64 + kb * 32 + grp * 8);
        const b8 bf = *(const b8*)(lds + (size_t)((wave * 16 + col) * 64 + kb * 32 + grp * 8) * 2);
        u[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, u[c], 0, 0, 0);
      }
    const int x = x0 + col, y = y0 + wave % TY, z = z0 + wave / TY;
    if (x < g.nx && y < g.ny && z < g.nz) {
      ConvIO d = io;
      d.bias = io.bias2;
      d.out = io.pool;
#pragma unroll
      for (int c = 0; c < 2; ++c)
        store4<32, EPI_LINEAR>(d, u[c], (size_t)(z * g.ny + y) * g.nx + x, c * 16 + grp * 4);
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradient of the 1x1x1 layers: dW[ci][co] = sum_r in(r)[ci] dy(r)[co]
// and, as an extra tap, the bias gradient sum_r dy(r)[co] in row ci = 0.  A
// block owns `subs` consecutive chunks of 256 sites; per tap it stages the
// input (or ones) and dy of a chunk transposed in LDS ([channel][site]) so
// both MFMA operands are 16-byte LDS reads, sums over its chunks in registers,
// then over its 4 waves in LDS, and writes one partial per tap:
// part[block][t][ci][co].
// ---------------------------------------------------------------------------
constexpr int WG_LD = 264;     // LDS row length (256 sites + 8 padding)

template <int CIN, int COUT>
__global__ __launch_bounds__(256) void k_wgrad1(const uint16_t* __restrict__ in,
                                               const uint16_t* __restrict__ dy,
                                               float* __restrict__ part, Grid3 g, int subs) {
  constexpr int NI = CIN / 16, NO = COUT / 16;
  static_assert(4 * CIN * COUT * 4 <= (CIN + COUT) * WG_LD * 2, "reduction buffer");
  __shared__ __align__(16) uint16_t lds[(CIN + COUT) * WG_LD];
  uint16_t* a_l = lds;
  uint16_t* d_l = lds + CIN * WG_LD;
  float* red = (float*)lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int col = lane & 15, grp = lane >> 4;

  for (int t = 0; t <= 1; ++t) {
    f4 acc[NI][NO];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int o = 0; o < NO; ++o) acc[i][o] = f4{0.f, 0.f, 0.f, 0.f};
    for (int sc = 0; sc < subs; ++sc) {
      const long long site = ((long long)blockIdx.x * subs + sc) * 256 + tid;
      __syncthreads();
      if (site < g.n) {
        if (t < 1) {
#pragma unroll
          for (int v = 0; v < CIN / 8; ++v) {
            const uint4 q = *(const uint4*)(in + (size_t)site * CIN + v * 8);
            const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
              a_l[(v * 8 + e) * WG_LD + tid] = uint16_t(w4[e >> 1] >> (16 * (e & 1)));
          }
        } else {
#pragma unroll
          for (int c = 0; c < CIN; ++c) a_l[c * WG_LD + tid] = c == 0 ? BF_ONE : 0;
        }
#pragma unroll
        for (int v = 0; v < COUT / 8; ++v) {
          const uint4 q = *(const uint4*)(dy + (size_t)site * COUT + v * 8);
          const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            d_l[(v * 8 + e) * WG_LD + tid] = uint16_t(w4[e >> 1] >> (16 * (e & 1)));
        }
      } else {
#pragma unroll
        for (int c = 0; c < CIN; ++c) a_l[c * WG_LD + tid] = 0;
#pragma unroll
        for (int c = 0; c < COUT; ++c) d_l[c * WG_LD + tid] = 0;
      }
      __syncthreads();
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int k0 = wv * 64 + kb * 32 + grp * 8;
        b8 af[NI], bf[NO];
#pragma unroll
        for (int i = 0; i < NI; ++i) af[i] = *(const b8*)(a_l + (i * 16 + col) * WG_LD + k0);
#pragma unroll
        for (int o = 0; o < NO; ++o) bf[o] = *(const b8*)(d_l + (o * 16 + col) * WG_LD + k0);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int o = 0; o < NO; ++o)
            acc[i][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[o], acc[i][o], 0, 0, 0);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          red[(wv * CIN + i * 16 + grp * 4 + q) * COUT + o * 16 + col] = acc[i][o][q];
    __syncthreads();
    float* dst = part + ((size_t)blockIdx.x * 2 + t) * CIN * COUT;
    for (int e = tid; e < CIN * COUT; e += 256)
      dst[e] = (red[e] + red[CIN * COUT + e]) + (red[2 * CIN * COUT + e] + red[3 * CIN * COUT + e]);
  }
}

// ---------------------------------------------------------------------------
// Weight gradient of a 3x3x3 layer, 16 input by 16 output channels per
// workgroup (blockIdx.y picks them): dW[t][ci][co] = sum_r in(r + d_t)[ci]
// dy(r)[co], and as tap 27 the bias gradient in row ci = 0.  A workgroup walks
// over tiles of 32 x 4 x 4 sites, staging the input with its ring and dy
// transposed ([channel][row][x]), so that a matrix instruction contracts a row
// of 32 sites; the three taps of a row shift the input by one element in
// registers, and all 28 sums stay there (112 registers) until the end: the
// operands are staged once, not once per tap.  Then the waves are added in
// LDS, and part[block][t][ci][co] gets the block's sums.
// ---------------------------------------------------------------------------
constexpr int WT_X = 32, WT_Y = 4, WT_Z = 4, WT_ROWS = WT_Y * WT_Z;
constexpr int WI_ROWS = (WT_Y + 2) * (WT_Z + 2);
constexpr int WI_LD = 48;                         // x = 0 at element 8: 16-byte reads stay aligned
constexpr int WI_CH = WI_ROWS * WI_LD + 96;       // channel strides of 16 (mod 64) words:
constexpr int WD_CH = WT_ROWS * WT_X + 32;        // the lanes' reads spread over the banks
constexpr int WG3_TAPS_AT_ONCE = 7;

// Channels of two neighbouring sites as words of LDS, two or eight of them.
__device__ __forceinline__ void put2(uint16_t* dst, int ch_stride, uint32_t a, uint32_t b) {
  *(uint32_t*)dst = (a & 0xFFFFu) | (b << 16);
  *(uint32_t*)(dst + ch_stride) = (a >> 16) | (b & 0xFFFF0000u);
}
__device__ __forceinline__ void put8(uint16_t* dst, int ch_stride, const uint4 p, const uint4 q) {
  put2(dst, ch_stride, p.x, q.x);
  put2(dst + 2 * ch_stride, ch_stride, p.y, q.y);
  put2(dst + 4 * ch_stride, ch_stride, p.z, q.z);
  put2(dst + 6 * ch_stride, ch_stride, p.w, q.w);
}

__global__ __launch_bounds__(256) void k_wgrad3(const uint16_t* __restrict__ in, int cin,
                                                const uint16_t* __restrict__ dy, int cout,
                                                float* __restrict__ part, Grid3 g, int tiles) {
  __shared__ __align__(16) uint16_t lds[16 * (WI_CH + WD_CH)];
  static_assert(4 * WG3_TAPS_AT_ONCE * 256 * 4 <= sizeof(lds), "reduction buffer");
  uint16_t* a_l = lds;
  uint16_t* d_l = lds + 16 * WI_CH;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int ni = cin / 16, ci0 = int(blockIdx.y) % ni * 16, co0 = int(blockIdx.y) / ni * 16;
  const int ntx = (g.nx + WT_X - 1) / WT_X, nty = (g.ny + WT_Y - 1) / WT_Y;
  for (int t = tid; t < 8 * (WI_CH + WD_CH); t += 256) ((uint32_t*)lds)[t] = 0;
  f4 acc[27], accb = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int x0 = tile % ntx * WT_X, y0 = tile / ntx % nty * WT_Y, z0 = tile / (ntx * nty) * WT_Z;
    __syncthreads();
    constexpr int PAIRS = WT_X / 2 + 2;   // sites -2 .. 33 of a row
    for (int t = tid; t < WI_ROWS * PAIRS * 2; t += 256) {
      const int half = t % 2, k = t / 2;
      const int pr = k % PAIRS, row = k / PAIRS;
      const int y = wrap_at(y0 + row % (WT_Y + 2) - 1, g.ny), z = wrap_at(z0 + row / (WT_Y + 2) - 1, g.nz);
      const int xa = x0 + 2 * pr - 2;
      const size_t base = (size_t)(z * g.ny + y) * g.nx;
      const size_t ra = base + wrap_at(xa < 0 ? xa + 2 * g.nx : xa, g.nx);
      const size_t rb = base + wrap_at(xa + 1 < 0 ? xa + 1 + 2 * g.nx : xa + 1, g.nx);
      uint16_t* dst = a_l + row * WI_LD + 6 + 2 * pr;
      const uint16_t* src = in + ci0 + half * 8;
      put8(dst + half * 8 * WI_CH, WI_CH, *(const uint4*)(src + ra * cin), *(const uint4*)(src + rb * cin));
    }
    for (int t = tid; t < WT_ROWS * WT_X; t += 256) {
      const int half = t % 2, k = t / 2;
      const int pr = k % (WT_X / 2), row = k / (WT_X / 2);
      const int x = x0 + 2 * pr, y = y0 + row % WT_Y, z = z0 + row / WT_Y;
      const bool rows = y < g.ny && z < g.nz;
      const bool va = rows && x < g.nx, vb = rows && x + 1 < g.nx;
      const size_t r = (size_t)(z * g.ny + y) * g.nx + x;
      uint16_t* dst = d_l + row * WT_X + 2 * pr;
      const uint16_t* src = dy + co0 + half * 8;
      uint4 p{0u, 0u, 0u, 0u}, q{0u, 0u, 0u, 0u};
      if (va) p = *(const uint4*)(src + r * cout);
      if (vb) q = *(const uint4*)(src + (r + 1) * cout);
      put8(dst + half * 8 * WD_CH, WD_CH, p, q);
    }
    __syncthreads();
#pragma unroll 1
    for (int row = wave; row < WT_ROWS; row += 4) {
      const b8 bf = *(const b8*)(d_l + col * WD_CH + row * WT_X + grp * 8);
      const uint32_t one = col == 0 ? 0x3F803F80u : 0u;
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, uint4{one, one, one, one}),
                                                     bf, accb, 0, 0, 0);
      const uint16_t* src = a_l + col * WI_CH + (row / WT_Y * (WT_Y + 2) + row % WT_Y) * WI_LD + 8 + grp * 8;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const uint16_t* p = src + (k / 3 * (WT_Y + 2) + k % 3) * WI_LD;
        const uint4 c = *(const uint4*)p;
        const uint32_t l = *(const uint32_t*)(p - 2), r = *(const uint32_t*)(p + 8);
        const uint4 m{__builtin_amdgcn_alignbit(c.x, l, 16), __builtin_amdgcn_alignbit(c.y, c.x, 16),
                      __builtin_amdgcn_alignbit(c.z, c.y, 16), __builtin_amdgcn_alignbit(c.w, c.z, 16)};
        const uint4 n{m.y, m.z, m.w, __builtin_amdgcn_alignbit(r, c.w, 16)};
        acc[3 * k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, m), bf, acc[3 * k], 0, 0, 0);
        acc[3 * k + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, c), bf, acc[3 * k + 1], 0, 0, 0);
        acc[3 * k + 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, n), bf, acc[3 * k + 2], 0, 0, 0);
      }
    }
  }
  float* red = (float*)lds;
#pragma unroll
  for (int t0 = 0; t0 < 28; t0 += WG3_TAPS_AT_ONCE) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WG3_TAPS_AT_ONCE; ++k) {
      const f4 v = t0 + k < 27 ? acc[t0 + k < 27 ? t0 + k : 0] : accb;
#pragma unroll
      for (int q = 0; q < 4; ++q) red[((k * 4 + wave) * 16 + grp * 4 + q) * 16 + col] = v[q];
    }
    __syncthreads();
    for (int e = tid; e < WG3_TAPS_AT_ONCE * 256; e += 256) {
      const int k = e / 256, m = e % 256;
      const float* s = red + k * 1024 + m;
      part[(((size_t)blockIdx.x * 28 + t0 + k) * cin + ci0 + m / 16) * cout + co0 + m % 16] =
          (s[0] + s[256]) + (s[512] + s[768]);
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradient of the layers with CH = 1 or 2 channels on one side (thin, a
// pair per site) and 16 on the other (wide): the taps and thin channels are the
// rows of the product, sum_s thin(s + d_t or s - d_t)[ch] wide(s)[c], so that two
// or four matrix instructions cover the 27 taps of 32 sites, and only the thin
// side has a ring to stage, in three copies shifted along x (12 us for F and 16
// for A at 64x64x128; by k_wgrad3, padded to 16 channels, 28 and 25, and A's dy
// in a pass of its own).
//   THIN_OUT: layer F, thin = dy (CH = 1), wide = the input; dW[t][c][0] with
//   dy(s - d_t), the bias gradient the sum of dy
//   else: layer A, thin = the input (CH = 2), wide = dy, formed on the way in
//   as [act > 0] (skip + up / 8) (k_skip_grad); dW[t][ch][c] with in(s + d_t)
// part[block][t][ci][co] with the layer's own channel numbers.
// ---------------------------------------------------------------------------
template <bool THIN_OUT>
__global__ __launch_bounds__(256) void k_wgrad_thin(const uint32_t* __restrict__ thin,
                                                    const uint16_t* __restrict__ wide,
                                                    const uint16_t* __restrict__ up,
                                                    const uint16_t* __restrict__ act,
                                                    float* __restrict__ part, Grid3 g, Grid3 coarse,
                                                    int tiles) {
  constexpr int CH = THIN_OUT ? 1 : 2, ROWS = 27 * CH, MT = (ROWS + 15) / 16;
  constexpr int COPY = WI_ROWS * WT_X + 32, CHS = 3 * COPY;
  __shared__ __align__(16) uint16_t lds[16 * WD_CH + CH * CHS];
  static_assert(4 * (MT + 1) * 256 * 4 <= sizeof(lds), "reduction buffer");
  uint16_t* d_l = lds;
  uint16_t* t_l = lds + 16 * WD_CH;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int ntx = (g.nx + WT_X - 1) / WT_X, nty = (g.ny + WT_Y - 1) / WT_Y;
  f4 acc[MT], accb = f4{0.f, 0.f, 0.f, 0.f};
  int from[MT];                       // LDS element of this lane's row (tap, channel) at run (0, 0)
  bool real[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    acc[m] = f4{0.f, 0.f, 0.f, 0.f};
    const int e = m * 16 + col, t = min(e / CH, 26), ch = e % CH;
    real[m] = e < ROWS;
    const int dz = t / 9, dy = t / 3 % 3, dx = t % 3;
    // copy k holds thin(x + k - 1); rows are those of the ring
    const int k = THIN_OUT ? 2 - dx : dx, ry = THIN_OUT ? 2 - dy : dy, rz = THIN_OUT ? 2 - dz : dz;
    from[m] = ch * CHS + k * COPY + (rz * (WT_Y + 2) + ry) * WT_X + grp * 8;
  }
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int x0 = tile % ntx * WT_X, y0 = tile / ntx % nty * WT_Y, z0 = tile / (ntx * nty) * WT_Z;
    __syncthreads();
    for (int t = tid; t < WI_ROWS * (WT_X + 2); t += 256) {
      const int i = t % (WT_X + 2), row = t / (WT_X + 2);   // site x0 + i - 1
      const int y = y0 + row % (WT_Y + 2) - 1, z = z0 + row / (WT_Y + 2) - 1, x = x0 + i - 1;
      const uint32_t q = thin[(size_t)(wrap_at(z, g.nz) * g.ny + wrap_at(y, g.ny)) * g.nx + wrap_at(x, g.nx)];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (i - k >= 0 && i - k < WT_X) {
          t_l[k * COPY + row * WT_X + i - k] = uint16_t(q);
          if constexpr (CH == 2) t_l[CHS + k * COPY + row * WT_X + i - k] = uint16_t(q >> 16);
        }
    }
#pragma unroll 2
    for (int t = tid; t < WT_ROWS * WT_X; t += 256) {
      const int half = t % 2, pr = t / 2 % (WT_X / 2), row = t / WT_X;
      const int x = x0 + 2 * pr, y = y0 + row % WT_Y, z = z0 + row / WT_Y;
      uint4 p{0u, 0u, 0u, 0u}, q{0u, 0u, 0u, 0u};
      if (y < g.ny && z < g.nz && x < g.nx) {   // nx is even: both sites
        const size_t r = ((size_t)(z * g.ny + y) * g.nx + x) * 16 + half * 8;
        p = *(const uint4*)(wide + r);
        q = *(const uint4*)(wide + r + 16);
        if constexpr (!THIN_OUT) {
          const uint4 u = *(const uint4*)(up + ((size_t)((z >> 1) * coarse.ny + (y >> 1)) * coarse.nx + (x >> 1)) * 16 + half * 8);
          p = skip_grad8(p, u, *(const uint4*)(act + r));
          q = skip_grad8(q, u, *(const uint4*)(act + r + 16));
        }
      }
      put8(d_l + half * 8 * WD_CH + row * WT_X + 2 * pr, WD_CH, p, q);
    }
    __syncthreads();
#pragma unroll 1
    for (int row = wave; row < WT_ROWS; row += 4) {
      const b8 bf = *(const b8*)(d_l + col * WD_CH + row * WT_X + grp * 8);
      const uint16_t* src = t_l + (row / WT_Y * (WT_Y + 2) + row % WT_Y) * WT_X;
      const uint4 ones{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u}, none{0u, 0u, 0u, 0u};
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const uint4 v = *(const uint4*)(src + from[m]);
        const uint4 a = real[m] ? v : none;
        acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), bf, acc[m], 0, 0, 0);
        // F's bias gradient: the centre tap (row 13, m = 0) against ones; its
        // sites are the tile's own, those outside the box masked below
        if constexpr (THIN_OUT) {
          if (m == 0) {
            const bool in_row = y0 + row % WT_Y < g.ny && z0 + row / WT_Y < g.nz;
            const int left = g.nx - x0 - grp * 8;      // sites of this lane's eight inside the box
            auto keep = [&](uint32_t w, int k) {
              return in_row ? (2 * k + 1 < left ? w : 2 * k < left ? w & 0xFFFFu : 0u) : 0u;
            };
            const uint4 c{keep(a.x, 0), keep(a.y, 1), keep(a.z, 2), keep(a.w, 3)};
            accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, c),
                                                           __builtin_bit_cast(b8, ones), accb, 0, 0, 0);
          }
        }
      }
      if constexpr (!THIN_OUT)         // A's: ones (row 0) against dy
        accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, col == 0 ? ones : none),
                                                       bf, accb, 0, 0, 0);
    }
  }
  float* red = (float*)lds;
  __syncthreads();
#pragma unroll
  for (int m = 0; m <= MT; ++m) {
    const f4 v = m < MT ? acc[m < MT ? m : 0] : accb;
#pragma unroll
    for (int q = 0; q < 4; ++q) red[((m * 4 + wave) * 16 + grp * 4 + q) * 16 + col] = v[q];
  }
  __syncthreads();
  constexpr int CIN = THIN_OUT ? 16 : 2, COUT = THIN_OUT ? 1 : 16;
  float* dst = part + (size_t)blockIdx.x * 28 * CIN * COUT;
  for (int e = tid; e < (MT + 1) * 256; e += 256) {
    const int m = e / 256, r = e / 16 % 16, c = e % 16;
    const float* p = red + m * 1024 + e % 256;
    const float v = (p[0] + p[256]) + (p[512] + p[768]);
    if (m == MT) {
      if (THIN_OUT ? (r == 13 && c == 0) : r == 0) dst[(27 * CIN) * COUT + (THIN_OUT ? 0 : c)] = v;
      continue;
    }
    const int row = m * 16 + r, t = row / CH, ch = row % CH;
    if (row >= ROWS) continue;
    if (THIN_OUT) dst[(t * CIN + c) * COUT] = v;
    else dst[(t * CIN + ch) * COUT + c] = v;
  }
}

// Sums of the per-block partials of all layers added to the flat gradient at
// the real (unpadded) positions.  A block of 1024 threads owns 64 consecutive
// elements of one layer; its 16 waves take every 16th partial block and the 16
// sums are added in a fixed order, so the result does not depend on timing.
struct WReduce {
  const float* part[UNET_LAYERS];
  int nblk[UNET_LAYERS];
  int cinp[UNET_LAYERS], coutp[UNET_LAYERS];   // channels in the partials
  int first[UNET_LAYERS + 1];                  // first block of a layer
};

__global__ __launch_bounds__(1024) void k_wreduce(WReduce w, float* __restrict__ grad) {
  __shared__ float sh[16][64];
  int l = 0;
  while (l + 1 < UNET_LAYERS && int(blockIdx.x) >= w.first[l + 1]) ++l;
  const UNetLayer L = UNET[l];
  const int cinp = w.cinp[l], coutp = w.coutp[l], nblk = w.nblk[l];
  const float* part = w.part[l];
  const int per = (L.taps + 1) * cinp * coutp;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int e = (blockIdx.x - w.first[l]) * 64 + lane;
  const int co = e % coutp, ci = e / coutp % cinp, tap = e / (coutp * cinp);
  const bool mine = e < per && co < L.cout && (tap < L.taps ? ci < L.cin : ci == 0);
  float s = 0.f;
  if (mine) {
#pragma unroll 8
    for (int b = wv; b < nblk; b += 16) s += part[(size_t)b * per + e];
  }
  sh[wv][lane] = s;
  __syncthreads();
  if (wv != 0 || !mine) return;
  float t = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) t += sh[k][lane];
  if (tap < L.taps) grad[L.woff + (tap * L.cin + ci) * L.cout + co] += t;
  else grad[L.boff + co] += t;
}

// ---------------------------------------------------------------------------
// Elementwise kernels on channels-last bfloat16 tensors, 8 channels a thread
// ---------------------------------------------------------------------------
// Site index of child (cx, cy, cz) in {0,1}^3 of coarse site rc.
__device__ __forceinline__ size_t child(const Grid3& fine, const Grid3& coarse, int rc, int k) {
  int x, y, z;
  decode(coarse, rc, x, y, z);
  return ((size_t)(2 * z + (k >> 2)) * fine.ny + 2 * y + ((k >> 1) & 1)) * fine.nx + 2 * x + (k & 1);
}
// Sum of the 8 children (upsample backward)
__global__ __launch_bounds__(256) void k_down(const uint16_t* __restrict__ in,
                                              uint16_t* __restrict__ out, int C, Grid3 fine,
                                              Grid3 coarse) {
  const int groups = C / 8;
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= (long long)coarse.n * groups) return;
  const int rc = int(id / groups), v = int(id % groups);
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int k = 0; k < 8; ++k) {
    float f[8];
    unpack8(*(const uint4*)(in + child(fine, coarse, rc, k) * C + v * 8), f);
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] += f[e];
  }
  *(uint4*)(out + (size_t)rc * C + v * 8) = pack8(s);
}

// Gradient at a pooled-and-skipped activation: (g + dp(parent) / 8) * [act > 0]
__global__ __launch_bounds__(256) void k_skip_grad(const uint16_t* __restrict__ gsk,
                                                   const uint16_t* __restrict__ dp,
                                                   const uint16_t* __restrict__ act,
                                                   uint16_t* __restrict__ out, int C, Grid3 fine,
                                                   Grid3 coarse) {
  const int groups = C / 8;
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= (long long)fine.n * groups) return;
  const int rf = int(id / groups), v = int(id % groups);
  *(uint4*)(out + (size_t)rf * C + v * 8) =
      skip_grad8(*(const uint4*)(gsk + (size_t)rf * C + v * 8),
                 *(const uint4*)(dp + (size_t)parent(fine, coarse, rf) * C + v * 8),
                 *(const uint4*)(act + (size_t)rf * C + v * 8));
}

// ---------------------------------------------------------------------------
// Input normalisation, loss
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_in_stats(const double* __restrict__ b,
                                                  double* __restrict__ partials, int n) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  double v[2] = {0.0, 0.0};
  if (r < n) {
    v[0] = b[r];
    v[1] = b[r] * b[r];
  }
  block_partials<2>(v, partials, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(1024) void k_in_final(const double* __restrict__ partials,
                                                   int nblocks, int n, double out_scale,
                                                   UNetScalars* __restrict__ sc) {
  double t[2];
  block_sums_1024<2>(partials, nblocks, t);
  if (threadIdx.x == 0) {
    const double mean = t[0] / n;
    const double var = t[1] / n - mean * mean;
    const double s = var > 0.0 ? sqrt(var) : 1.0;
    sc->mean = mean;
    sc->s = s;
    sc->inv_s = 1.0 / s;
    sc->scale = s * out_scale;
    sc->inv_scale = 1.0 / (s * out_scale);
  }
}

// d0[r] = 2 (out - target / scale) / n (a pair with 0); partial sums of the squared error
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ out,
                                              const double* __restrict__ target,
                                              const UNetScalars* __restrict__ sc,
                                              uint32_t* __restrict__ d0,
                                              double* __restrict__ partials, int n) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  double v[1] = {0.0};
  if (r < n) {
    const double diff = double(out[r]) - target[r] * sc->inv_scale;
    v[0] = diff * diff;
    const float gval = float(2.0 * diff / n);
    d0[r] = uint32_t(f2bf(gval));
  }
  block_partials<1>(v, partials, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(1024) void k_loss_final(const double* __restrict__ partials,
                                                     int nblocks, int n,
                                                     UNetScalars* __restrict__ sc) {
  double t[1];
  block_sums_1024<1>(partials, nblocks, t);
  if (threadIdx.x == 0) {
    sc->loss_sum += t[0] / n;
    sc->loss_count += 1;
  }
}

// ---------------------------------------------------------------------------
// Parameters
// ---------------------------------------------------------------------------
// Packed forward weights wf[t][co][ci], backward-data weights wb[t][ci][co] =
// w[taps-1-t][ci][co] (the flipped kernel), padded bias; padding is zero.
__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ p, uint16_t* __restrict__ wf,
                                              uint16_t* __restrict__ wb, float* __restrict__ bias) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < UNET_BIAS_PADDED) {
    int l = 0;
    while (l + 1 < UNET_LAYERS && UNET[l + 1].pb <= e) ++l;
    const int co = e - UNET[l].pb;
    bias[e] = co < UNET[l].cout ? p[UNET[l].boff + co] : 0.f;
  }
  if (e >= UNET_PACKED) return;
  int l = 0;
  while (l + 1 < UNET_LAYERS && UNET[l + 1].pw <= e) ++l;
  const UNetLayer L = UNET[l];
  const int k = e - L.pw;
  {   // forward: k = (t * coutp + co) * cinp + ci
    const int ci = k % L.cinp, co = (k / L.cinp) % L.coutp, t = k / (L.cinp * L.coutp);
    const bool real = ci < L.cin && co < L.cout;
    wf[e] = real ? f2bf(p[L.woff + (t * L.cin + ci) * L.cout + co]) : 0;
  }
  if (wb) {   // backward-data: k = (t * cinp + ci) * coutp + co
    const int co = k % L.coutp, ci = (k / L.coutp) % L.cinp, t = k / (L.cinp * L.coutp);
    const int tf = L.taps - 1 - t;
    const bool real = ci < L.cin && co < L.cout;
    wb[e] = real ? f2bf(p[L.woff + (tf * L.cin + ci) * L.cout + co]) : 0;
  }
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v,
                                              float lr, float b1, float b2, float eps, float c1,
                                              float c2, float gscale) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= UNET_PARAMS) return;
  const float gr = g[e] * gscale;
  const float mm = b1 * m[e] + (1.f - b1) * gr;
  const float vv = b2 * v[e] + (1.f - b2) * gr * gr;
  m[e] = mm;
  v[e] = vv;
  p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  g[e] = 0.f;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
namespace {

inline int blocks_for(long long n) { return int((n + 255) / 256); }

constexpr int WG_MAX_BLOCKS = 1024;

inline int wgrad_subs(int n) {
  const int chunks = (n + 255) / 256;
  return (chunks + WG_MAX_BLOCKS - 1) / WG_MAX_BLOCKS;
}
inline int wgrad_blocks(int n) {
  const int chunks = (n + 255) / 256;
  const int subs = wgrad_subs(n);
  return (chunks + subs - 1) / subs;
}

template <int CIN, int COUT, int EPI, bool UP = false>
void conv1(const ConvIO& io, const Grid3& g, const Grid3& coarse, hipStream_t s) {
  hipLaunchKernelGGL((k_conv1<CIN, COUT, EPI, UP>), dim3((g.n + 63) / 64), dim3(256), 0, s, io, g,
                     coarse);
}

// Tiles of 16 x 4 x 4 sites (16 x 4 x 8, which reads a smaller ring, leaves
// fewer workgroups to overlap staging and products: 25 against 20 us for layer
// A at 64x64x128, 16 x 8 x 8 33 us), 16 x 2 x 2 on the quarter level (its 8,192
// sites there are 32 of the former tiles).
template <int SRC, int CIN, int COUT, int TY, int TZ, int WC, int EPI, int TAIL, int TAPS = TAPS_ONE>
void conv3(const ConvIO& io, const Grid3& g, const Grid3& coarse, hipStream_t s) {
  const int tiles = (g.nx + 15) / 16 * ((g.ny + TY - 1) / TY) * ((g.nz + TZ - 1) / TZ);
  hipLaunchKernelGGL((k_conv3<SRC, CIN, COUT, TY, TZ, WC, EPI, TAIL, TAPS>), dim3(tiles), dim3(256), 0, s,
                     io, g, coarse);
}

constexpr int WG3_MAX_BLOCKS = 512;   // two workgroups on each of 256 compute units
int wgrad3_tiles(const Grid3& g) {
  return (g.nx + WT_X - 1) / WT_X * ((g.ny + WT_Y - 1) / WT_Y) * ((g.nz + WT_Z - 1) / WT_Z);
}
// Blocks of a layer's weight gradient, and its channels in the partials (the
// layers A and F keep their own numbers, see k_wgrad_thin).
int wgrad_parts(int l, const Grid3& g) {
  return UNET[l].taps == 1 ? wgrad_blocks(g.n) : std::min(wgrad3_tiles(g), WG3_MAX_BLOCKS);
}
int level_of(int l) { return l == 0 || l == 5 ? 0 : (l == 1 || l == 4 ? 1 : 2); }
int part_cin(int l) { return l == 0 ? UNET[l].cin : UNET[l].cinp; }
int part_cout(int l) { return l == 5 ? UNET[l].cout : UNET[l].coutp; }
size_t part_floats(int l, const Grid3& g) {
  return ((size_t)wgrad_parts(l, g) * (UNET[l].taps + 1) * part_cin(l) * part_cout(l) + 63) / 64 * 64;
}

template <int CIN, int COUT>
void wgrad1(const uint16_t* in, const uint16_t* dy, float* part, const Grid3& g, hipStream_t s) {
  hipLaunchKernelGGL((k_wgrad1<CIN, COUT>), dim3(wgrad_blocks(g.n)), dim3(256), 0, s, in, dy, part, g,
                     wgrad_subs(g.n));
}

void wgrad3(const uint16_t* in, const uint16_t* dy, float* part, int l, const Grid3& g, hipStream_t s) {
  const UNetLayer& L = UNET[l];
  hipLaunchKernelGGL(k_wgrad3, dim3(wgrad_parts(l, g), (L.cinp / 16) * (L.coutp / 16)), dim3(256), 0, s,
                     in, L.cinp, dy, L.coutp, part, g, wgrad3_tiles(g));
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

}  // namespace

bool UNet::shape_ok(int nx, int ny, int nz) {
  return nx >= 4 && ny >= 4 && nz >= 4 && nx % 4 == 0 && ny % 4 == 0 && nz % 4 == 0 &&
         (long long)nx * ny * nz < (1ll << 31);
}

namespace {
struct UNetCarve {
  char* base;
  size_t off = 0;
  template <typename T>
  T* take(size_t count) {
    T* p = base ? (T*)(base + off) : nullptr;
    off += align256(count * sizeof(T));
    return p;
  }
};

void carve_all(UNet& u, UNetCarve& c, int nx, int ny, int nz, bool training) {
  const size_t n0 = (size_t)nx * ny * nz, n1 = n0 / 8, n2 = n0 / 64;
  // x0, c1 and c2 are written in training only, but have their place in either
  // layout: the workspace holds every layer's activations
  uint32_t* x0 = c.take<uint32_t>(n0);
  u.x0 = training ? x0 : nullptr;
  u.a1 = c.take<uint16_t>(n0 * 16);
  u.p1 = c.take<uint16_t>(n1 * 16);
  u.a2 = c.take<uint16_t>(n1 * 32);
  u.p2 = c.take<uint16_t>(n2 * 32);
  u.a3 = c.take<uint16_t>(n2 * 64);
  u.u3 = c.take<uint16_t>(n2 * 32);
  uint16_t* c2 = c.take<uint16_t>(n1 * 32);
  u.c2 = training ? c2 : nullptr;
  u.u2 = c.take<uint16_t>(n1 * 16);
  uint16_t* c1 = c.take<uint16_t>(n0 * 16);
  u.c1 = training ? c1 : nullptr;
  u.out = c.take<float>(n0);
  u.params = c.take<float>(UNET_PARAMS);
  u.wf = c.take<uint16_t>(UNET_PACKED);
  u.bias = c.take<float>(UNET_BIAS_PADDED);
  u.sc = c.take<UNetScalars>(1);
  u.red = c.take<double>(2 * ((n0 + 255) / 256));
  if (training) {
    u.wb = c.take<uint16_t>(UNET_PACKED);
    u.grad = c.take<float>(UNET_PARAMS);
    u.adam_m = c.take<float>(UNET_PARAMS);
    u.adam_v = c.take<float>(UNET_PARAMS);
    u.d0 = c.take<uint32_t>(n0);
    u.g1 = c.take<uint16_t>(n0 * 16);
    u.du2 = c.take<uint16_t>(n1 * 16);
    u.g2 = c.take<uint16_t>(n1 * 32);
    u.du3 = c.take<uint16_t>(n2 * 32);
    u.g3 = c.take<uint16_t>(n2 * 64);
    u.dp2 = c.take<uint16_t>(n2 * 32);
    u.gb = c.take<uint16_t>(n1 * 32);
    u.dp1 = c.take<uint16_t>(n1 * 16);
    size_t part = 0;
    for (int l = 0; l < UNET_LAYERS; ++l) {
      const int v = level_of(l);
      part += part_floats(l, Grid3{nx >> v, ny >> v, nz >> v, int(n0 >> (3 * v))});
    }
    u.wpart = c.take<float>(part);
  }
}
}  // namespace

size_t UNet::bytes(int nx, int ny, int nz, bool training) {
  UNet u;
  UNetCarve c{nullptr};
  carve_all(u, c, nx, ny, nz, training);
  return c.off;
}

void UNet::carve(char* base, int nx, int ny, int nz, bool train) {
  UNetCarve c{base};
  carve_all(*this, c, nx, ny, nz, train);
  training = train;
  for (int l = 0; l < 3; ++l) g[l] = Grid3{nx >> l, ny >> l, nz >> l, (nx >> l) * (ny >> l) * (nz >> l)};
}

hipError_t UNet::init_state() {
  adam_t = 0;
  hipError_t e = hipMemsetAsync(sc, 0, sizeof(UNetScalars), stream);
  if (e == hipSuccess && training) {
    e = hipMemsetAsync(grad, 0, UNET_PARAMS * 4, stream);
    if (e == hipSuccess) e = hipMemsetAsync(adam_m, 0, UNET_PARAMS * 4, stream);
    if (e == hipSuccess) e = hipMemsetAsync(adam_v, 0, UNET_PARAMS * 4, stream);
  }
  return e;
}

void UNet::pack() {
  hipLaunchKernelGGL(k_pack, dim3(blocks_for(UNET_PACKED)), dim3(256), 0, stream, params, wf,
                     training ? wb : nullptr, bias);
}

void UNet::forward(const double* b, const void* solid, bool link, double* guess) {
  hipStream_t s = stream;
  const Grid3 G0 = g[0], G1 = g[1], G2 = g[2];
  const int nb = blocks_for(G0.n);
  hipLaunchKernelGGL(k_in_stats, dim3(nb), dim3(256), 0, s, b, red, G0.n);
  hipLaunchKernelGGL(k_in_final, dim3(1), dim3(1024), 0, s, red, nb, G0.n, double(out_scale), sc);
  ConvIO io{};
  io.sc = sc;
  // A from b and the mask, pooled to p1
  io.b = b; io.solid = solid; io.pair_out = x0;
  io.w = wf + UNET[0].pw; io.bias = bias + UNET[0].pb; io.out = a1; io.pool = p1;
  if (link) conv3<SRC_LINK, 16, 16, 4, 4, 1, EPI_RELU, TAIL_POOL>(io, G0, G1, s);
  else conv3<SRC_INPUT, 16, 16, 4, 4, 1, EPI_RELU, TAIL_POOL>(io, G0, G1, s);
  // B, pooled to p2
  io.in = p1; io.w = wf + UNET[1].pw; io.bias = bias + UNET[1].pb; io.out = a2; io.pool = p2;
  conv3<SRC_PLAIN, 16, 32, 4, 4, 1, EPI_RELU, TAIL_POOL>(io, G1, G2, s);
  // C and D
  io.in = p2; io.w = wf + UNET[2].pw; io.bias = bias + UNET[2].pb; io.out = a3;
  io.w2 = wf + UNET[3].pw; io.bias2 = bias + UNET[3].pb; io.pool = u3;
  conv3<SRC_PLAIN, 32, 64, 2, 2, 4, EPI_RELU, TAIL_D>(io, G2, G2, s);
  // E of c2 = ReLU(upsample(u3) + a2)
  io.in = a2; io.up = u3; io.sum = c2;
  io.w = wf + UNET[4].pw; io.bias = bias + UNET[4].pb; io.out = u2;
  conv1<32, 16, EPI_LINEAR, true>(io, G1, G2, s);
  // F of c1 = ReLU(upsample(u2) + a1)
  io.in = a1; io.up = u2; io.sum = c1;
  io.w = wf + UNET[5].pw; io.bias = bias + UNET[5].pb; io.out = nullptr;
  io.out32 = out; io.guess = guess;
  conv3<SRC_UP, 16, 16, 4, 4, 1, EPI_OUT, TAIL_NONE, TAPS_TWO>(io, G0, G1, s);
}

void UNet::accumulate(const double* b, const void* solid, const double* target) {
  hipStream_t s = stream;
  forward(b, solid, false, nullptr);
  const Grid3 G0 = g[0], G1 = g[1], G2 = g[2];
  const int nb = blocks_for(G0.n);
  hipLaunchKernelGGL(k_loss, dim3(nb), dim3(256), 0, s, out, target, sc, d0, red, G0.n);
  hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(1024), 0, s, red, nb, G0.n, sc);
  ConvIO io{};
  io.sc = sc;
  WReduce w{};
  float* at = wpart;
  float* part[UNET_LAYERS];
  for (int l = 0; l < UNET_LAYERS; ++l) {
    const Grid3& G = g[level_of(l)];
    part[l] = at;
    at += part_floats(l, G);
    w.part[l] = part[l];
    w.nblk[l] = wgrad_parts(l, G);
    w.cinp[l] = part_cin(l);
    w.coutp[l] = part_cout(l);
    w.first[l + 1] = w.first[l] + ((UNET[l].taps + 1) * w.cinp[l] * w.coutp[l] + 63) / 64;
  }
  // F: weight gradient from (c1, d0); data gradient through the ReLU of c1,
  // and E's output gradient, the sum of g1 over the 8 children
  hipLaunchKernelGGL(k_wgrad_thin<true>, dim3(w.nblk[5]), dim3(256), 0, s, d0, c1, nullptr, nullptr,
                     part[5], G0, G1, wgrad3_tiles(G0));
  io.pair = d0; io.w = wb + UNET[5].pw; io.act = c1; io.out = g1; io.pool = du2;
  conv3<SRC_PAIR, 16, 16, 4, 4, 1, EPI_MASK, TAIL_SUM, TAPS_ALL>(io, G0, G1, s);
  // E: input c2
  wgrad1<32, 16>(c2, du2, part[4], G1, s);
  io.in = du2; io.w = wb + UNET[4].pw; io.act = c2; io.out = g2;
  conv1<16, 32, EPI_MASK>(io, G1, G2, s);
  // D: input a3, output gradient = sum of g2 over the children
  hipLaunchKernelGGL(k_down, dim3(blocks_for((long long)G2.n * 4)), dim3(256), 0, s, g2, du3, 32, G1, G2);
  wgrad1<64, 32>(a3, du3, part[3], G2, s);
  io.in = du3; io.w = wb + UNET[3].pw; io.act = a3; io.out = g3;
  conv1<32, 64, EPI_MASK>(io, G2, G2, s);
  // C: input p2
  wgrad3(p2, g3, part[2], 2, G2, s);
  io.in = g3; io.w = wb + UNET[2].pw; io.act = nullptr; io.out = dp2;
  conv3<SRC_PLAIN, 64, 32, 2, 2, 2, EPI_PLAIN, TAIL_NONE>(io, G2, G2, s);
  // a2 gets the skip gradient g2 and the pooled gradient dp2 / 8, then its ReLU
  hipLaunchKernelGGL(k_skip_grad, dim3(blocks_for((long long)G1.n * 4)), dim3(256), 0, s, g2, dp2, a2, gb, 32, G1, G2);
  // B: input p1
  wgrad3(p1, gb, part[1], 1, G1, s);
  io.in = gb; io.w = wb + UNET[1].pw; io.out = dp1;
  conv3<SRC_PLAIN, 32, 16, 4, 4, 1, EPI_PLAIN, TAIL_NONE>(io, G1, G1, s);
  // A: input x0, output gradient from g1 and dp1 as for a2
  hipLaunchKernelGGL(k_wgrad_thin<false>, dim3(w.nblk[0]), dim3(256), 0, s, x0, g1, dp1, a1, part[0],
                     G0, G1, wgrad3_tiles(G0));
  hipLaunchKernelGGL(k_wreduce, dim3(w.first[UNET_LAYERS]), dim3(1024), 0, s, w, grad);
}

void UNet::adam(float lr, float beta1, float beta2, float eps, float grad_scale) {
  ++adam_t;
  const float c1 = float(1.0 - std::pow(double(beta1), double(adam_t)));
  const float c2 = float(1.0 - std::pow(double(beta2), double(adam_t)));
  hipLaunchKernelGGL(k_adam, dim3(blocks_for(UNET_PARAMS)), dim3(256), 0, stream, params, grad,
                     adam_m, adam_v, lr, beta1, beta2, eps, c1, c2, grad_scale);
  pack();
}

}  // namespace ek
