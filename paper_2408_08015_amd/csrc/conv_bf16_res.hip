// 3x3 'same' stride-1 convolution of NHWC bf16 images (forward, and the input gradient: the same product on the output gradient
// with point-reflected taps) whose channels or pixels do not fill the persistent tiles of conv_bf16_halo.hip.
//
//   y[p][n] = sum_{c, tap} x[p + shift(tap)][c] * w[n][c][tap]     p = flattened (image, row, column)
//
// A block takes 32 * PG (32 or 64) consecutive pixels and stages them WITH THEIR HALO (W + 1 pixels before and after) and ALL channels in
// LDS once: one barrier, then every wavefront runs through its 32 output channels without another.  The pixel operand of
// tap (u, v) is the same LDS tile read u*W + v rows further down; a pixel whose neighbour lies outside the image reads a row
// of zeros.  Rows are an odd number of 16-byte chunks apart, so the reads of 16 rows fall into different banks.  The weights
// come from a copy in the order of the matrix instruction's operand ([32 channels][16 contracted][tap]: 1 KB per fragment),
// straight from L2 into registers.  (The nine fragments of the next 16 contracted channels are written as requested one by one,
// as those of the present ones are used up; in the code as built the requests stand behind the last products of a step,
// and each pixel operand is waited for where it is read.)
//
// Bound by those waits, for L2 and for LDS, with few blocks (6 x 45x45 pixels, 96 -> 96 channels: 7.4 us, the general product
// kernel 14) and with many (32 x 56x56, 96 -> 96: 26 and 50 us, where products, LDS and L2 take about 7 each; 160 -> 224: 73
// and 132, 0.89 PFLOP/s).  Four groups of pixels, or two tiles of channels, per wavefront leave fewer blocks and were slower nearly everywhere (28 and 37 us for 26).
#include "device_utils.h"
#include "kernels_bf16.h"
#include "prof.h"

#include <algorithm>

namespace ast {

namespace {

struct ResArgs {
  const bf16_t* x;     // [M][C]
  const bf16_t* w;     // [N/32][C/16][9][64 lanes][8]
  bf16_t* y;           // [M][N]
  const float* bias;   // [N] or NULL
  const bf16_t* mask;  // [M][N] or NULL: the output is zeroed where mask <= 0
  int M, H, W, C, N, act;
  int KS;              // steps of 16 contracted channels
  int pitch;           // bytes between rows in LDS
  int rows;            // staged pixels
  int blocks_n;        // blocks side by side over the output channels
  unsigned m_chunks;   // reciprocal of 2 * KS
  unsigned x_bytes, w_bytes;
};

constexpr unsigned RES_OOB = 0x80000000u;  // buffer offset beyond every extent: the load returns zeros
typedef unsigned int res_u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t res_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

template <int PG>
__device__ __forceinline__ void conv_res_body(const ResArgs& g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, nthreads = blockDim.x, waves = nthreads >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 31, lgrp = lane >> 5;
  const int bid = (int)xcd_grouped(blockIdx.x, gridDim.x);
  const int blk_m = bid / g.blocks_n, blk_n = bid - blk_m * g.blocks_n;
  const int m0 = blk_m * (32 * PG), n0 = blk_n * (waves * 32);
  const int W = g.W, KS = g.KS, HW = g.H * W;
  const __amdgpu_buffer_rsrc_t rx = res_rsrc(g.x, g.x_bytes), rw = res_rsrc(g.w, g.w_bytes);

  // ---- the weight fragments of the first step.  (Offsets stay inside the copy: a wavefront past the last tile of channels takes
  // the last one, the request behind the last step repeats it.  Neither is used.)
  const int tile = min((n0 >> 5) + wave, (g.N + 31) / 32 - 1);
  auto weight = [&](int ks, int t) __attribute__((always_inline)) -> bf16x8 {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, (unsigned)lane * 16u,
                                                                            (unsigned)((tile * KS + ks) * 9 + t) * 1024u, 0));
  };
  bf16x8 fw[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) fw[t] = weight(0, t);

  // ---- the pixels: 16-byte chunks, eight of a thread in flight
  const int total = g.rows * 2 * KS;
  for (int i0 = tid; i0 < total; i0 += 8 * nthreads) {
    res_u32x4 v[8];
    int at[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = i0 + k * nthreads;
      const int row = (int)__umulhi((unsigned)i, g.m_chunks), c = i - row * 2 * KS, p = m0 - (W + 1) + row;
      const bool ok = i < total && p >= 0 && p < g.M && c * 8 < g.C;
      v[k] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? (unsigned)((p * g.C + c * 8) * 2) : RES_OOB, 0, 0);
      at[k] = row * g.pitch + c * 16;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (i0 + k * nthreads < total) *reinterpret_cast<res_u32x4*>(smem + at[k]) = v[k];
  }
  const int zero_row = g.rows * g.pitch;
  for (int i = tid; i < 2 * KS; i += nthreads) *reinterpret_cast<res_u32x4*>(smem + zero_row + i * 16) = res_u32x4{0, 0, 0, 0};

  // ---- where the lane's pixels read each tap
  int addr[9][PG];
#pragma unroll
  for (int i = 0; i < PG; ++i) {
    const int o = i * 32 + lrow, rem = (m0 + o) % HW, yy = rem / W, xx = rem - yy * W;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int ty = t / 3, tx = t - ty * 3;
      const bool in = (unsigned)(yy + ty - 1) < (unsigned)g.H && (unsigned)(xx + tx - 1) < (unsigned)W;
      addr[t][i] = (in ? (o + ty * W + tx) * g.pitch : zero_row) + lgrp * 16;
    }
  }
  floatx16 acc[PG];
#pragma unroll
  for (int i = 0; i < PG; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  __syncthreads();

  for (int ks = 0; ks < KS; ++ks) {
    const int next = min(ks + 1, KS - 1);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      bf16x8 fa[PG];
#pragma unroll
      for (int i = 0; i < PG; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(smem + addr[t][i] + ks * 32);
#pragma unroll
      for (int i = 0; i < PG; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[t], fa[i], acc[i], 0, 0, 0);
      fw[t] = weight(next, t);
    }
  }

  // ---- out through LDS: rows of the block's channels, 16 bytes of padding
  const int cols = waves * 32, op = cols * 2 + 16;
  __syncthreads();
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    const int c4 = wave * 32 + 8 * r4 + 4 * lgrp;  // four consecutive channels
    float b[4] = {0.f, 0.f, 0.f, 0.f};
    if (g.bias && n0 + c4 < g.N) {
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = g.bias[n0 + c4 + e];
    }
#pragma unroll
    for (int i = 0; i < PG; ++i) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = acc[i][4 * r4 + e] + b[e];
        if (g.act == ACT_RELU) v[e] = fmaxf(v[e], 0.f);
      }
      uint2 pk;
      pk.x = f2bf_pk(v[0], v[1]);
      pk.y = f2bf_pk(v[2], v[3]);
      *reinterpret_cast<uint2*>(smem + (i * 32 + lrow) * op + c4 * 2) = pk;
    }
  }
  __syncthreads();
  const int per_row = cols >> 3;
  for (int i = tid; i < 32 * PG * per_row; i += nthreads) {
    const int row = i / per_row, ch = i - row * per_row, m = m0 + row, n = n0 + ch * 8;
    if (m >= g.M || n >= g.N) continue;
    const size_t at = (size_t)m * g.N + n;
    res_u32x4 v = *reinterpret_cast<const res_u32x4*>(smem + row * op + ch * 16);
    if (g.mask) {
      const res_u32x4 mk = *reinterpret_cast<const res_u32x4*>(g.mask + at);
#pragma unroll
      for (int e = 0; e < 4; ++e) {  // bf16 > 0: sign clear and not zero
        const uint32_t lo = mk[e] & 0xffffu, hi = mk[e] >> 16;
        v[e] &= ((lo != 0u && lo < 0x8000u) ? 0x0000ffffu : 0u) | ((hi != 0u && hi < 0x8000u) ? 0xffff0000u : 0u);
      }
    }
    *reinterpret_cast<res_u32x4*>(g.y + at) = v;
  }
}

__global__ __launch_bounds__(512) void conv_res_kernel_p32(ResArgs g) { conv_res_body<1>(g); }
__global__ __launch_bounds__(512) void conv_res_kernel_p64(ResArgs g) { conv_res_body<2>(g); }

constexpr size_t kResLds = 160 * 1024;
constexpr int kResUnits = 256;  // compute units that the choice of the tile aims at
inline long rcdiv(long a, long b) { return (a + b - 1) / b; }

struct ResPick {
  int pg = 0, waves = 0;  // groups of 32 pixels per block, wavefronts (of 32 output channels); pg = 0: no block fits
  size_t lds = 0;
  ResArgs g{};
};
// us of the launch, with those waits in it: a group's step costs a lone wavefront 41 ns, and w of them on a SIMD 28 ns each where a weight fragment
// serves one group of pixels (it comes from L2), 18 where it serves two.  Fitted to 416 sizes (16 to 256 channels, 400 to
// 144000 pixels): the choice by it costs 0.2 % over the faster one of both, 18 % at most.
double res_cost(const ResPick& p) {
  const long blocks = rcdiv(p.g.M, 32 * p.pg) * p.g.blocks_n, n = rcdiv(blocks, kResUnits);
  const long r = std::max(1L, std::min({n, (long)(kResLds / p.lds), 20L / p.waves}));
  const double body = p.g.KS * 9 * p.pg * std::max(0.041, (p.pg == 1 ? 0.028 : 0.018) * r * p.waves / 4) + 2.0 +
                      2e-5 * p.g.rows * p.g.pitch * r;
  return 2.0 + 0.5 * rcdiv(2 * n, r) * body;
}
ResPick res_pick_pg(int pg, int N, int H, int W, int Cin, int Cout) {
  ResPick p;
  ResArgs& g = p.g;
  g.M = N * H * W; g.H = H; g.W = W; g.C = Cin; g.N = Cout;
  g.KS = (int)rcdiv(Cin, 16);
  g.pitch = (2 * g.KS | 1) * 16;
  g.rows = 32 * pg + 2 * (W + 1);
  g.m_chunks = (unsigned)((1ull << 32) / (2 * g.KS)) + 1u;  // exact below 2^32 / (2 * KS): a block stages at most kResLds / 16 chunks
  const long units = rcdiv(Cout, 32);
  g.blocks_n = (int)rcdiv(units, 8);
  p.waves = (int)rcdiv(units, g.blocks_n);
  p.lds = std::max((size_t)(g.rows + 1) * g.pitch, (size_t)32 * pg * (p.waves * 64 + 16));
  if (p.lds <= kResLds) p.pg = pg;
  return p;
}
ResPick res_pick(int N, int H, int W, int Cin, int Cout) {
  const ResPick a = res_pick_pg(1, N, H, W, Cin, Cout), b = res_pick_pg(2, N, H, W, Cin, Cout);
  return a.pg && b.pg ? (res_cost(a) <= res_cost(b) ? a : b) : a;
}

}  // namespace

bool conv_res_supported(int N, int H, int W, int Cin, int Cout) {
  const long M = (long)N * H * W;
  return Cin % 8 == 0 && Cout % 8 == 0 && M * Cin * 2 < (1L << 31) && M * Cout * 2 < (1L << 31) &&
         (long)conv_res_pack_elems(Cin, Cout) * 2 < (1L << 31) && res_pick(N, H, W, Cin, Cout).pg;
}
size_t conv_res_pack_elems(int Cin, int Cout) { return (size_t)rcdiv(Cout, 32) * rcdiv(Cin, 16) * 9 * 512; }
hipError_t conv_res_allow() {
  const hipError_t e =
      hipFuncSetAttribute((const void*)conv_res_kernel_p32, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds);
  return e ? e : hipFuncSetAttribute((const void*)conv_res_kernel_p64, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds);
}
void conv_res_bf16(hipStream_t st, const bf16_t* x, const bf16_t* w, const float* bias, const bf16_t* mask, bf16_t* y, int N,
                   int H, int W, int Cin, int Cout, int act) {
  ResPick p = res_pick(N, H, W, Cin, Cout);
  ResArgs& g = p.g;
  g.x = x; g.w = w; g.y = y; g.bias = bias; g.mask = mask; g.act = act;
  g.x_bytes = (unsigned)((size_t)g.M * Cin * 2);
  g.w_bytes = (unsigned)(conv_res_pack_elems(Cin, Cout) * 2);
  KLAUNCH_NAMED(p.pg == 2 ? "conv_res_kernel_p64" : "conv_res_kernel_p32", p.pg == 2 ? conv_res_kernel_p64 : conv_res_kernel_p32,
                dim3((unsigned)(rcdiv(g.M, 32 * p.pg) * g.blocks_n)), dim3(p.waves * 64), p.lds, st, g);
}

}  // namespace ast

// The choice above, for tests: groups of 32 pixels, wavefronts, blocks over the output channels.  0: the kernel does not take
// these sizes.
extern "C" int ast_conv_res_choice(int N, int H, int W, int Cin, int Cout, int out[3]) {
  using namespace ast;
  if (!conv_res_supported(N, H, W, Cin, Cout)) return 0;
  const ResPick p = res_pick(N, H, W, Cin, Cout);
  out[0] = p.pg; out[1] = p.waves; out[2] = p.g.blocks_n;
  return 1;
}
