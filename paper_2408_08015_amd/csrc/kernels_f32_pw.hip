// fp32 pointwise (1x1) convolution: forward product, input gradient, weight gradient, and the packed weight copies.
//
// The products run on the bf16 matrix cores with their operands split in three (kernels_f32_x3.h).  In NCHW a channel plane is
// contiguous, so pixels go on the MFMA N dimension: lane l supplies eight channels B[k = 8*(l/32) + 0..7] of pixel l%32 with
// coalesced loads and splits them in registers, the weights are A[m = l%32][k], read from a copy that is split and packed in
// exactly that lane order, and accumulator register r of lane l is D[8*(r/4) + 4*(l/32) + r%4][l%32].  No LDS and no barrier
// in front of the products: a wavefront waits for its own loads alone, and the others of its SIMD fill the gaps.  (A version
// that staged the split pixels of a block in LDS needed half the loads and took as long as the fp32 kernels: 64 -> 256
// channels at 32 x 56x56 52 us against 45, 24 -> 144 31 us against 17; two wavefronts per SIMD ran in step.)
#include <algorithm>

#include "device_utils.h"
#include "kernels.h"
#include "kernels_f32_x3.h"
#include "prof.h"

namespace ast {

static inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

struct WgArgs {  // one pointwise-conv weight-gradient launch (partials only)
  const float* g;
  const float* x;
  float* part;
  long NQ;
  int Cin, Cout, HW, splits;
  unsigned rHW;  // plane_reciprocal(HW)
  int tile_order;  // 1: the (ci, co) tiles of one pixel range run side by side on one XCD
};

// Block coordinates of a product grid of gx pixel blocks x gy channel tiles from the flat block id:
// pixel blocks fastest, or (tile_order) channel tiles fastest within XCD-grouped ids, so that the
// gy blocks that read the same pixels of X hit one L2.
__device__ __forceinline__ void pw_block_xy(unsigned id, unsigned gx, unsigned gy, int tile_order, int& bx, int& by) {
  if (tile_order) {
    id = xcd_grouped(id, gx * gy);
    by = (int)(id % gy);
    bx = (int)(id / gy);
  } else {
    bx = (int)(id % gx);
    by = (int)(id / gx);
  }
}

// ============================================================== product (forward / input gradient)
// Y[n][m][p] = sum_k A[m][k] X[n][k][p] (+ bias[m]) (+ add[n][m][p]); A from its split copy (x3_pack layout).
struct PwArgs {
  const uint4* Wp;
  const float* X;
  float* Y;
  const float* bias;
  const float* add;
  double* stats;  // or NULL: per block (sum, sum of squares) of the output per channel, stats[m][pixel blocks][2]
  size_t x_words, y_words;
  unsigned NQ;    // pixels of all samples
  unsigned rHW;   // plane_reciprocal(HW)
  int HW, Kdim, Mdim, KG, gy;
  int mper;       // the wide kernel: row tiles of a wavefront
  int order;      // 1: the channel tiles of one pixel block run side by side on one XCD (they share X), 0: the pixel blocks
                  // of one channel tile (they share the weights)
};

// Block coordinates of a product grid from the flat block id.  (Both from one division, in scalar registers: everything
// that follows from them is uniform.)
__device__ __forceinline__ void pw_product_xy(unsigned id, unsigned n, const PwArgs& a, int& bx, int& by) {
  id = xcd_grouped(id, n);
  const unsigned d = a.order ? (unsigned)a.gy : n / (unsigned)a.gy, hi = id / d, lo = id - hi * d;
  bx = __builtin_amdgcn_readfirstlane(a.order ? hi : lo);
  by = __builtin_amdgcn_readfirstlane(a.order ? lo : hi);
}

template <int PXL> struct PxVec { float v[PXL]; };  // PXL neighbouring pixels
template <int PXL>
__device__ __forceinline__ PxVec<PXL> px_load(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
  PxVec<PXL> o;
  if constexpr (PXL == 1) {
    o.v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
  } else {
    const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
    o.v[0] = __uint_as_float(u[0]);
    o.v[1] = __uint_as_float(u[1]);
  }
  return o;
}
template <int PXL>
__device__ __forceinline__ void px_store(__amdgpu_buffer_rsrc_t r, unsigned vo, const PxVec<PXL>& p) {
  if constexpr (PXL == 1) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(p.v[0]), r, vo, 0, 0);
  } else {
    typedef uint32_t uint2_t __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(uint2_t{__float_as_uint(p.v[0]), __float_as_uint(p.v[1])}, r, vo, 0, 0);
  }
}

// Where the 32 * PXL pixels from q0 on of a wavefront lie: descriptors of operand and result from the first pixel's sample
// on, and the lane's byte offsets in them (kOutside for pixels past the last).
template <int PXL>
struct PwLane {
  unsigned n0, k, p;  // first sample; the lane's sample from there and its pixel
  bool valid;
  unsigned vx, vy;    // channel 8 * (l/32) of X, row m0 + 4 * (l/32) of Y
  __device__ __forceinline__ const float* pixel(const PwArgs& a) const {  // channel 0 of X
    return valid ? a.X + xo + (size_t)k * a.Kdim * a.HW + p : a.X;
  }
  size_t xo, yo;
  __amdgpu_buffer_rsrc_t rx, ry;
  __device__ __forceinline__ PwLane(const PwArgs& a, unsigned q0, int m0) {
    const unsigned HW = (unsigned)a.HW, lane = threadIdx.x & 63, half = lane >> 5;
    n0 = __builtin_amdgcn_readfirstlane(min(q0, a.NQ - 1) / HW);
    const unsigned q = q0 + (lane & 31) * PXL, r = q - n0 * HW;
    k = plane_of(r, HW, a.rHW);
    p = r - k * HW;
    valid = q < a.NQ;  // (HW % PXL == 0: the pixels of a lane are valid together)
    xo = (size_t)n0 * a.Kdim * HW;
    yo = ((size_t)n0 * a.Mdim + m0) * HW;
    rx = rsrc_words(a.X + xo, a.x_words - xo);
    ry = rsrc_words(a.Y + yo, a.y_words - yo);
    vx = valid ? (k * (unsigned)a.Kdim * HW + p + 8u * half * HW) * 4u : kOutside;
    vy = valid ? (k * (unsigned)a.Mdim * HW + p + 4u * half * HW) * 4u : kOutside;
  }
};
// row of accumulator register i, without the lane's 4 * (l/32)
__device__ __forceinline__ constexpr int acc_row(int i) { return 8 * (i >> 2) + (i & 3); }

// acc + acs += A X over the groups [gbeg, gend) of 16 channels, at least one; PXL column tiles (column j of tile t is pixel PXL*j + t of
// the wavefront), MT row tiles.  The next group is in flight while one is multiplied; the loads past the last group are
// outside every extent, and channels past Kdim meet zero weights.
template <int PXL, int MT>
__device__ __forceinline__ void pw_contract(const uint4* wl, size_t wt, __amdgpu_buffer_rsrc_t rx, unsigned vx, unsigned row_bytes,
                                            int gbeg, int gend, floatx16 (&acc)[MT][PXL], floatx16 (&acs)[MT][PXL]) {
  uint4 a0[MT][3], a1[MT][3];
  PxVec<PXL> b0[8], b1[8];
  auto load = [&](uint4 (&a)[MT][3], PxVec<PXL> (&b)[8], int g) __attribute__((always_inline)) {
    const unsigned v = g < gend ? vx : kOutside;
    const int gg = min(g, gend - 1);
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = px_load<PXL>(rx, v, (unsigned)(gg * 16 + j) * row_bytes);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int p = 0; p < 3; ++p) a[m][p] = wl[m * wt + (size_t)(gg * 3 + p) * 64];
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mma = [&](const uint4 (&a)[MT][3], const PxVec<PXL> (&b)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < PXL; ++t) {
      float v[8];
      uint4 x[3];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = b[j].v[t];
      split3(v, x);
#pragma unroll
      for (int m = 0; m < MT; ++m) acs[m][t] = mfma_bf16(a[m][2], x[0], acs[m][t]);
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m][t] = mfma_bf16(a[m][0], x[0], acc[m][t]);
#pragma unroll
      for (int m = 0; m < MT; ++m) acs[m][t] = mfma_bf16(a[m][1], x[0], acs[m][t]);
#pragma unroll
      for (int m = 0; m < MT; ++m) acs[m][t] = mfma_bf16(a[m][1], x[1], acs[m][t]);
#pragma unroll
      for (int m = 0; m < MT; ++m) acs[m][t] = mfma_bf16(a[m][0], x[1], acs[m][t]);
#pragma unroll
      for (int m = 0; m < MT; ++m) acs[m][t] = mfma_bf16(a[m][0], x[2], acs[m][t]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  load(a0, b0, gbeg);
  int g = gbeg;
  do {
    load(a1, b1, g + 1);
    mma(a0, b0);
    if (g + 1 < gend) {
      load(a0, b0, g + 2);
      mma(a1, b1);
    }
    g += 2;
  } while (g < gend);
}

// acc += A X over the groups [gbeg, gend) for one row tile and the pixel at xq of each lane, on the fp32 matrix instructions
// (kernels_f32_x3.h: where the pieces gave no finite sum)
__device__ __forceinline__ void pw_contract_f32(const uint4* wl, const float* xq, bool valid, size_t HW, int Kdim, int gbeg,
                                                int gend, floatx16& acc) {
  const int half = threadIdx.x >> 5 & 1;
#pragma unroll 1
  for (int g = gbeg; g < gend; ++g) {
    uint4 p[3];
    float w[8], x[8];
    const int k = g * 16 + 8 * half;
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = wl[(size_t)(g * 3 + i) * 64];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = valid && k + j < Kdim ? xq[(size_t)(k + j) * HW] : 0.f;
    join3(p, w);
    acc = mfma_f32(w, x, acc);
  }
}

// Sum over the 32 lanes of a half of each of 16 values: lane l ends with that of value 8*l4 + 4*l3 + 2*l2 + l1 (bits of l).
// Every step halves the number of values, so it takes 39 instructions instead of 80.
__device__ __forceinline__ float half_sums(const float (&v)[16]) {
  const int lane = threadIdx.x & 63;
  float a[8], b[4], c[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {  // even rows of 16 lanes keep value i, odd ones value i + 8
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    a[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = (b3 ? a[i + 4] : a[i]) + dpp_move<DPP_ROW_MIRROR>(b3 ? a[i] : a[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = (b2 ? b[i + 2] : b[i]) + dpp_move<DPP_HALF_MIRROR>(b2 ? b[i] : b[i + 2]);
  float d = (b1 ? c[1] : c[0]) + dpp_move<DPP_QUAD_MIRROR>(b1 ? c[0] : c[1]);
  d += dpp_move<DPP_QUAD_SWAP1>(d);
  return d;
}
// The statistics of one row tile, one wavefront's pixels: sums to sd[32] in row order
__device__ __forceinline__ void tile_stats(const float (&s)[16], const float (&q)[16], float2* sd) {
  const int lane = threadIdx.x & 63, i = 8 * (lane >> 4 & 1) + 4 * (lane >> 3 & 1) + 2 * (lane >> 2 & 1) + (lane >> 1 & 1);
  const float a = half_sums(s), b = half_sums(q);
  if (!(lane & 1)) sd[8 * (i >> 2) + (i & 3) + 4 * (lane >> 5)] = make_float2(a, b);
}
// ... and the sums of all wavefronts of a block to stats[m][P][2]; sd[waves][rows] in LDS, m0: the block's first channel
__device__ __forceinline__ void block_stats(const float2* sd, int waves, int rows, double* stats, int m0, int Mdim, int bx, int P) {
  __syncthreads();
  for (int c = threadIdx.x; c < rows && m0 + c < Mdim; c += blockDim.x) {
    double s = 0.0, q = 0.0;
    for (int w = 0; w < waves; ++w) {
      s += sd[w * rows + c].x;
      q += sd[w * rows + c].y;
    }
    double* o = stats + ((size_t)(m0 + c) * P + bx) * 2;
    o[0] = s;
    o[1] = q;
  }
}

// The results of rows [m0, m1) of the wavefront's pixels that are not finite once more, over what was stored, and the
// statistics of those rows.  (Behind everything else: a branch in front of the stores costs the wide form its registers.)
template <int PXL>
__device__ __forceinline__ void pw_again(const PwArgs& a, const PwLane<PXL>& L, const uint4* wl, int m0, int m1, float2* sd) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores in front
  const int half = threadIdx.x >> 5 & 1;
  const unsigned row_bytes = (unsigned)a.HW * 4u;
  const __amdgpu_buffer_rsrc_t ra = rsrc_words(a.add ? a.add + L.yo : a.Y, a.add ? a.y_words - L.yo : 0);
#pragma unroll 1
  for (int m = m0; m < m1; m += 32) {
    float s[16], q[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = q[i] = 0.f;
#pragma unroll 1
    for (int t = 0; t < PXL; ++t) {
      floatx16 v = zero16();
      pw_contract_f32(wl + (size_t)(m - m0) / 32 * a.KG * 192, L.pixel(a) + t, L.valid, a.HW, a.Kdim, 0, a.KG, v);
      const int rows = L.valid ? m1 - m - 4 * half : 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const unsigned at = acc_row(i) < rows ? L.vy + (unsigned)(m - m0 + acc_row(i)) * row_bytes + 4u * t : kOutside;
        const float y = px_load<1>(L.ry, at, 0).v[0];
        float o = v[i];
        if (a.bias) o += a.bias[min(m + acc_row(i) + 4 * half, m1 - 1)];
        if (a.add) o += px_load<1>(ra, at, 0).v[0];
        o = finite_f(y) ? y : o;
        px_store<1>(L.ry, at, {o});
        s[i] += o;
        q[i] = fmaf(o, o, q[i]);
      }
    }
    if (a.stats) tile_stats(s, q, sd + (m - m0));  // uniform
  }
}

// A wavefront: 32 * PXL pixels x MT 32-row tiles, blocks of any number of wavefronts side by side over the pixels.  More
// pixels and tiles per wavefront read and split the operands less often, and leave fewer wavefronts: 94 registers at 1 x 1
// (five wavefronts per SIMD), 142 at 2 x 1, 153 at 1 x 2, 233 at 2 x 2.
// us, forward, fp32 matrix instructions / now: 256 -> 64 channels at 32 x 56x56 50 / 36 (2 x 2), 256 -> 128 at 8 x 56x56 30 /
// 16, 144 -> 24 at 32 x 56x56 20 / 14 (2 x 1), 240 -> 40 at 32 x 30x30 16 / 10, 64 -> 64 at 32 x 56x56 18 / 13 (1 x 1).
template <int PXL, int MT>
__device__ __forceinline__ void pw_body(const PwArgs& a, int bx, int by, float2* sd, int P) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, Mdim = a.Mdim, KG = a.KG, m0 = by * 32 * MT;
  const unsigned row_bytes = (unsigned)a.HW * 4u;
  const PwLane<PXL> L(a, ((unsigned)bx * (blockDim.x >> 6) + wave) * (32u * PXL), m0);
  const uint4* wl = a.Wp + (size_t)by * MT * KG * 192 + lane;
  const size_t wt = MT > 1 && m0 + 32 < Mdim ? (size_t)KG * 192 : 0;  // the second tile, where it exists
  floatx16 acc[MT][PXL], acs[MT][PXL];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < PXL; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[m][t][i] = acs[m][t][i] = 0.f;
  pw_contract<PXL, MT>(wl, wt, L.rx, L.vx, row_bytes, 0, KG, acc, acs);
  float bad = 0.f;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < PXL; ++t) bad = add_small(acc[m][t], acs[m][t], bad);
  if (a.stats) {  // uniform; only without bias and addend; pixels past the last hold zeros
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      float s[16], q[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = acc[m][0][i];
        q[i] = s[i] * s[i];
        if constexpr (PXL == 2) {
          s[i] += acc[m][1][i];
          q[i] = fmaf(acc[m][1][i], acc[m][1][i], q[i]);
        }
      }
      tile_stats(s, q, sd + (wave * MT + m) * 32);
    }
  }
  if (a.bias || a.add) {  // uniform
    const __amdgpu_buffer_rsrc_t ra = rsrc_words(a.add ? a.add + L.yo : a.Y, a.add ? a.y_words - L.yo : 0);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i0 = 0; i0 < 16; i0 += 8) {  // eight rows at a time are requested before the first is used
        PxVec<PXL> kv[8];
        float bv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int r = 32 * m + acc_row(i0 + i);
          bv[i] = a.bias ? a.bias[min(m0 + r + 4 * half, Mdim - 1)] : 0.f;
          kv[i] = px_load<PXL>(ra, L.vy, (unsigned)r * row_bytes);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int t = 0; t < PXL; ++t) acc[m][t][i0 + i] += bv[i] + kv[i].v[t];
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  const int rows = Mdim - m0 - 4 * half;   // of the lane, in acc_row's numbering
  const bool full = m0 + 32 * MT <= Mdim;  // uniform
  unsigned vo = L.vy;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      PxVec<PXL> v;
#pragma unroll
      for (int t = 0; t < PXL; ++t) v.v[t] = acc[m][t][i];
      px_store<PXL>(L.ry, full || 32 * m + acc_row(i) < rows ? vo : kOutside, v);
      vo += (i & 3) == 3 ? 5 * row_bytes : row_bytes;
    }
  if (any_not_finite(bad)) pw_again<PXL>(a, L, wl, m0, min(m0 + 32 * MT, Mdim), sd + wave * MT * 32);
  if (a.stats) block_stats(sd, blockDim.x >> 6, 32 * MT, a.stats, m0, Mdim, bx, P);
}
template <int PXL, int MT>
__global__ __launch_bounds__(512, PXL * MT == 1 ? 4 : 2) void pw_conv_f32_kernel(PwArgs a) {
  __shared__ float2 sd[8 * 32 * MT];
  int bx, by;
  pw_product_xy(blockIdx.x, gridDim.x, a, bx, by);
  pw_body<PXL, MT>(a, bx, by, sd, gridDim.x / a.gy);
}

// Few pixels, long K (the 14x14 / 7x7 layers of a whole network): the WK wavefronts of a block share one tile of 32 pixels
// x MT * 32 channels and split K between them, so there are WK times as many wavefronts and a WK-th of the dependent
// passes; their tiles are added through LDS in a fixed order.
// us, fp32 matrix instructions / now: 1024 -> 256 channels at 8 x 14x14 18.5 / 11.3 (WK 4, MT 2), 512 -> 2048 at 8 x 7x7
// 18.1 / 11.6, 960 -> 160 at 8 x 7x7 9.5 / 7.4 (WK 8, MT 1), 576 -> 96 at 8 x 14x14 7.5 / 5.6.
template <int MT, int WK>
__device__ __forceinline__ void pw_ks_body(const PwArgs& a, int bx, int by, float (*sR)[16][64]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, Mdim = a.Mdim, KG = a.KG, m0 = by * 32 * MT;
  const unsigned row_bytes = (unsigned)a.HW * 4u;
  const PwLane<1> L(a, (unsigned)bx * 32u, m0);
  const uint4* wl = a.Wp + (size_t)by * MT * KG * 192 + lane;
  const size_t wt = MT > 1 && m0 + 32 < Mdim ? (size_t)KG * 192 : 0;  // the second tile, where it exists
  floatx16 acc[MT][1], acs[MT][1];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[m][0][i] = acs[m][0][i] = 0.f;
  const int gper = (KG + WK - 1) / WK, gbeg = wave * gper, gend = min(gbeg + gper, KG);
  if (gbeg < gend) pw_contract<1, MT>(wl, wt, L.rx, L.vx, row_bytes, gbeg, gend, acc, acs);  // uniform
  float bad = 0.f;
#pragma unroll
  for (int m = 0; m < MT; ++m) bad = add_small(acc[m][0], acs[m][0], bad);
  if (any_not_finite(bad)) {  // the wavefront's share again
#pragma unroll 1
    for (int m = 0; m < MT; ++m) {
      floatx16 again = zero16();
      pw_contract_f32(wl + m * wt, L.pixel(a), L.valid, a.HW, a.Kdim, gbeg, gend, again);
#pragma unroll
      for (int j = 0; j < MT; ++j)
        if (m == j) take_not_finite(acc[j][0], again);
    }
  }
  constexpr int RW = 16 / WK;  // rows of the register layout that each wavefront finishes
  const __amdgpu_buffer_rsrc_t ra = rsrc_words(a.add ? a.add + L.yo : a.Y, a.add ? a.y_words - L.yo : 0);
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (m) __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) sR[wave][i][lane] = acc[m][0][i];
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < RW; ++rr) {
      const int i = RW * wave + rr, r = 32 * m + acc_row(i), mm = m0 + r + 4 * half;
      float v = 0.f;
#pragma unroll
      for (int s = 0; s < WK; s += 4)  // fixed order
        v += (sR[s][i][lane] + sR[s + 1][i][lane]) + (sR[s + 2][i][lane] + sR[s + 3][i][lane]);
      const unsigned vo = L.valid && mm < Mdim ? L.vy + (unsigned)r * row_bytes : kOutside;
      if (a.bias) v += a.bias[min(mm, Mdim - 1)];
      if (a.add) v += px_load<1>(ra, vo, 0).v[0];
      px_store<1>(L.ry, vo, {v});
    }
  }
}
template <int MT, int WK>
__global__ __launch_bounds__(64 * WK) void pw_conv_f32_ks_kernel(PwArgs a) {
  __shared__ float sR[WK][16][64];
  int bx, by;
  pw_product_xy(blockIdx.x, gridDim.x, a, bx, by);
  pw_ks_body<MT, WK>(a, bx, by, sR);
}

// Short contractions into many channels (at most 16 * G of them in): a wavefront reads and splits its 32 pixels once and
// walks the row tiles [by * mper, (by + 1) * mper), the weights one tile ahead.  These products write several times what they
// read, so what counts is that stores never wait for anything.
// us, fp32 matrix instructions / now: 24 -> 144 channels at 32 x 56x56 21.8 / 17.5 (copy of its bytes 13.8), at 32 x 60x60
// 29.3 / 19.6, 40 -> 240 at 32 x 30x30 15.7 / 12.4, 16 -> 96 at 8 x 112x112 15.3 / 10.6, 64 -> 256 at 32 x 56x56 59 / 45.6.
template <int G, bool ADD>
__device__ __forceinline__ void pw_wide_body(const PwArgs& a, int bx, int by, float2* sd) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, Mdim = a.Mdim, KG = a.KG;
  const unsigned row_bytes = (unsigned)a.HW * 4u;
  const int t0 = by * a.mper, t1 = min(t0 + a.mper, (Mdim + 31) / 32);
  const PwLane<1> L(a, ((unsigned)bx * (blockDim.x >> 6) + wave) * 32u, t0 * 32);
  const uint4* wl = a.Wp + lane;
  uint4 a0[G][3], a1[G][3], x[G][3];
  auto loadA = [&](uint4 (&w)[G][3], int t) __attribute__((always_inline)) {
    const uint4* s = wl + (size_t)min(t, t1 - 1) * KG * 192;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int i = 0; i < 3; ++i) w[g][i] = s[(min(g, KG - 1) * 3 + i) * 64];
  };
  float v[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int j = 0; j < 8; ++j) v[g][j] = px_load<1>(L.rx, g < KG ? L.vx : kOutside, (unsigned)(g * 16 + j) * row_bytes).v[0];
  loadA(a0, t0);
#pragma unroll
  for (int g = 0; g < G; ++g) split3(v[g], x[g]);
  float bad = 0.f;
  const __amdgpu_buffer_rsrc_t ra = rsrc_words(a.add ? a.add + L.yo : a.Y, a.add ? a.y_words - L.yo : 0);
  auto tile = [&](const uint4 (&w)[G][3], int t) __attribute__((always_inline)) {
    floatx16 acc, acs;
    const unsigned vt = L.vy + (unsigned)(t - t0) * 32u * row_bytes;
    float kv[16];  // requested in front of the products
    if constexpr (ADD) {
#pragma unroll
      for (int i = 0; i < 16; ++i) kv[i] = px_load<1>(ra, L.valid ? vt : kOutside, (unsigned)acc_row(i) * row_bytes).v[0];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = acs[i] = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      acs = mfma_bf16(w[g][2], x[g][0], acs);
      acc = mfma_bf16(w[g][0], x[g][0], acc);
      acs = mfma_bf16(w[g][1], x[g][0], acs);
      acs = mfma_bf16(w[g][1], x[g][1], acs);
      acs = mfma_bf16(w[g][0], x[g][1], acs);
      acs = mfma_bf16(w[g][0], x[g][2], acs);
    }
    const int rows = L.valid ? Mdim - t * 32 - 4 * half : 0;
    unsigned vo = vt;
    float o[16], q[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      o[i] = acc[i] + acs[i];
      bad = fmaf(o[i], 0.f, bad);
      px_store<1>(L.ry, acc_row(i) < rows ? vo : kOutside, {ADD ? o[i] + kv[i] : o[i]});
      vo += (i & 3) == 3 ? 5 * row_bytes : row_bytes;
    }
    if (a.stats) {  // uniform; pixels past the last hold zeros
#pragma unroll
      for (int i = 0; i < 16; ++i) q[i] = o[i] * o[i];
      tile_stats(o, q, sd + (wave * a.mper + t - t0) * 32);
    }
  };
  for (int t = t0; t < t1; t += 2) {
    loadA(a1, t + 1);
    tile(a0, t);
    if (t + 1 < t1) {
      loadA(a0, t + 2);
      tile(a1, t + 1);
    }
  }
  if (any_not_finite(bad)) pw_again<1>(a, L, wl + (size_t)t0 * KG * 192, t0 * 32, min(t1 * 32, Mdim), sd + wave * a.mper * 32);
}
constexpr int kWideTiles = 8;  // most row tiles of a wavefront
template <int G>
__global__ __launch_bounds__(512, G <= 2 ? 4 : 2) void pw_conv_f32_wide_kernel(PwArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  int bx, by;
  pw_product_xy(blockIdx.x, gridDim.x, a, bx, by);
  const int waves = blockDim.x >> 6, rows = a.mper * 32;
  float2* const sd = reinterpret_cast<float2*>(lds);  // [waves][rows]
  pw_wide_body<G, false>(a, bx, by, sd);
  if (a.stats) block_stats(sd, waves, rows, a.stats, by * rows, a.Mdim, bx, gridDim.x / a.gy);
}

// Planes that 32-bit offsets from a wavefront's first sample do not reach (pw_far): 64-bit addresses, one 32 x 32 tile per
// wavefront on the fp32 matrix instructions, five and more wavefronts per SIMD to hide its loads.
// One sample of 2048x2048, us (the generic kernels): 16 -> 96 channels forward 625 (9060), backward with the weight gradient 900
// (27200); 96 -> 24 950 (13700) and 1160 (42000); 64 -> 128 1590 (47500) and 2570 (126000).
__global__ __launch_bounds__(256, 5) void pw_conv_f32_far_kernel(PwArgs a) {
  int bx, by;
  pw_product_xy(blockIdx.x, gridDim.x, a, bx, by);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned q = ((unsigned)bx * 4u + wave) * 32u + (lane & 31), HW = (unsigned)a.HW;
  const bool valid = q < a.NQ;
  const unsigned n = valid ? q / HW : 0, p = valid ? q - n * HW : 0;
  floatx16 acc = zero16();
  pw_contract_f32(a.Wp + (size_t)by * a.KG * 192 + lane, a.X + (size_t)n * a.Kdim * HW + p, valid, HW, a.Kdim, 0, a.KG, acc);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int m = by * 32 + acc_row(i) + 4 * (lane >> 5);
    if (!valid || m >= a.Mdim) continue;
    const size_t o = ((size_t)n * a.Mdim + m) * HW + p;
    float v = acc[i];
    if (a.bias) v += a.bias[m];
    if (a.add) v += a.add[o];
    a.Y[o] = v;
  }
}

// Split copy of A[m][k] = W[m*lda_m + k*lda_k]: for tile t of 32 rows, group g of 16 columns and piece i, lane l finds
// A[32t + l%32][16g + 8*(l/32) + 0..7] as one 16-byte word at Wp[((t*KG + g)*3 + i)*64 + l]; zero outside.
size_t x3_pack_floats(int Mdim, int Kdim) { return (size_t)cdiv(Mdim, 32) * cdiv(Kdim, 16) * 768; }
// fp32 copy (the other convolutions): Wp[((t*KG + g)*64 + l)*4 + e] = A[32t + l%32][8g + 2e + l/32], zero outside.
size_t pw_pack_floats(int Mdim, int Kdim) { return (size_t)cdiv(Mdim, 32) * cdiv(Kdim, 8) * 256; }

// Block b of a task: 32 rows x 16 columns of all taps of split copies, or 256 words of one fp32 copy.  A split block reads every
// weight once, the taps of a row and column side by side, and writes whole 1 KB pieces.  (A block per piece and tap read and
// split each weight three times.  Both copies of 9.4 M weights of 3x3 convolutions 302 us, now 42; of 4.2 M pointwise ones 54, 21.)
unsigned pack_blocks(const PackTask& t) {
  return (unsigned)(cdiv(t.Mdim, 32) * t.KG * (t.split ? 1 : t.taps));
}
// the pieces of two neighbouring columns' weights (their sum is the weight, also where the first would round to infinity; of one
// that is not finite the first piece is the value, and the others 0)
__device__ __forceinline__ void split_weights(float a, float b, uint32_t (&p)[3]) {
  auto pieces = [](float w, uint32_t (&h)[3]) __attribute__((always_inline)) {
    const bool fin = finite_f(w);
    h[0] = f2bf(w);
    if (fin && !finite_f(bf2f((bf16_t)h[0]))) h[0] = __float_as_uint(w) >> 16;
    w -= bf2f((bf16_t)h[0]);
    h[1] = fin ? f2bf(w) : 0;
    w -= bf2f((bf16_t)h[1]);
    h[2] = fin ? f2bf(w) : 0;
  };
  uint32_t x[3], y[3];
  pieces(a, x);
  pieces(b, y);
#pragma unroll
  for (int i = 0; i < 3; ++i) p[i] = x[i] | y[i] << 16;
}
template <int TAPS>
__device__ __forceinline__ void pack_split(const PackTask& t, unsigned b, float* arena) {
  const int e = threadIdx.x & 3, l = threadIdx.x >> 2;
  const unsigned tile = b / (unsigned)t.KG, g = b - tile * t.KG;
  const int m = (int)(32 * tile) + (l & 31), k = (int)(16 * g) + 8 * (l >> 5) + 2 * e;
  const bool in0 = m < t.Mdim && k < t.Kdim, in1 = m < t.Mdim && k + 1 < t.Kdim;
  const float* const w = t.W + (size_t)m * t.lda_m + (size_t)k * t.lda_k;
  uint32_t* o = reinterpret_cast<uint32_t*>(arena) + t.dst + (size_t)b * 768 + threadIdx.x;
  const size_t tap_words = (size_t)((t.Mdim + 31) / 32 * t.KG) * 768;
  float v[TAPS][2];
#pragma unroll
  for (int i = 0; i < TAPS; ++i) {
    v[i][0] = in0 ? w[i] : 0.f;
    v[i][1] = in1 ? w[t.lda_k + i] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < TAPS; ++i) {
    uint32_t p[3];
    split_weights(v[i][0], v[i][1], p);
#pragma unroll
    for (int q = 0; q < 3; ++q) o[q * 256] = p[q];
    o += tap_words;
  }
}
__device__ __forceinline__ void pack_block(const PackTask& t, unsigned b, float* arena) {
  if (t.split) {  // uniform
    if (t.taps == 9) pack_split<9>(t, b, arena);
    else pack_split<1>(t, b, arena);
    return;
  }
  const int e = threadIdx.x & 3, l = threadIdx.x >> 2;
  const unsigned per = (unsigned)((t.Mdim + 31) / 32 * t.KG), tap = b / per, r = b - tap * per;
  const unsigned tile = r / (unsigned)t.KG, g = r - tile * t.KG;
  const int m = (int)(32 * tile) + (l & 31), k = (int)(8 * g) + 2 * e + (l >> 5);
  arena[t.dst + (size_t)b * 256 + threadIdx.x] =
      m < t.Mdim && k < t.Kdim ? t.W[(size_t)m * t.lda_m + (size_t)k * t.lda_k + tap] : 0.f;
}
__global__ __launch_bounds__(256) void pw_pack_all_kernel(const PackTask* __restrict__ tasks,
                                                          const unsigned short* __restrict__ block_task,
                                                          float* __restrict__ arena) {
  const PackTask t = tasks[block_task[blockIdx.x]];
  pack_block(t, blockIdx.x - t.block0, arena);
}
void pw_pack_all_f32(hipStream_t st, const PackTask* tasks_dev, const unsigned short* block_task_dev, float* arena,
                     int nblocks) {
  KLAUNCH(pw_pack_all_kernel, dim3(nblocks), dim3(256), 0, st, tasks_dev, block_task_dev, arena);
}
__global__ __launch_bounds__(256) void pw_pack_kernel(PackTask t, float* __restrict__ arena) { pack_block(t, blockIdx.x, arena); }
void pw_pack_f32(hipStream_t st, const PackTask& t, float* arena) {
  KLAUNCH(pw_pack_kernel, dim3(pack_blocks(t)), dim3(256), 0, st, t, arena);
}
PackTask pack_task(const float* W, int lda_m, int lda_k, size_t dst, int Mdim, int Kdim, int taps, bool split) {
  PackTask t = {};
  t.W = W; t.dst = dst; t.lda_m = lda_m; t.lda_k = lda_k; t.Mdim = Mdim; t.Kdim = Kdim; t.taps = taps; t.split = split;
  t.KG = cdiv(Kdim, split ? 16 : 8);
  return t;
}

// ---- which product kernel serves a shape, and its grid
enum PwVar { PW_1x1, PW_1x2, PW_2x1, PW_2x2, PW_KS4, PW_KS4x2, PW_KS8, PW_WIDE, PW_FAR };
struct PwPick { PwVar var; int waves, gx, gy, mper; };
// A wavefront's offsets from its first sample are 32-bit: two samples and the rows of a tile past them have to be in reach.
static bool pw_far(int Cin, int Cout, int HW) { return ((size_t)HW + 64) * (std::max(Cin, Cout) + 64) * 4 >= ((size_t)1 << 30); }
// Measured over the layers of MobileNetV2, EfficientNet-B1 and ResNet50 at 1 to 32 samples; `tiles` counts 32 x 32 tiles.
static PwPick pw_pick(long NQ, int HW, int Kdim, int Mdim, bool wide) {
  const int mt = cdiv(Mdim, 32), KG = cdiv(Kdim, 16);
  const long tiles = (long)cdiv(NQ, 32) * mt;
  PwPick p = {PW_1x1, 4, 0, mt, 0};
  if (pw_far(Kdim, Mdim, HW)) {
    p.var = PW_FAR;
    p.gx = cdiv(NQ, 128);
    return p;
  }
  if (tiles < 1024 && KG >= 6) {
    // under one wavefront per SIMD: K is split.  Two row tiles per wavefront where that leaves K long (512 -> 2048 at
    // 8 x 7x7 11.6 us, one tile 13.2), eight shares where there are few tiles (960 -> 160 at 8 x 7x7 7.4 us, four 7.7).
    // Below six groups a share is too short (64 -> 384 at 8 x 14x14: split 4.5 us, not 4.3).
    if (KG >= 32 && mt >= 2 && tiles >= 384) { p.var = PW_KS4x2; p.gy = cdiv(mt, 2); }
    else if (KG >= 16 && tiles < 256) { p.var = PW_KS8; p.waves = 8; }
    else p.var = PW_KS4;
    p.gx = cdiv(NQ, 32);
    return p;
  }
  if (KG <= 4 && mt >= 3 && tiles >= 7000 && wide) {
    // enough wavefronts even with all row tiles in one: below, more and shorter ones win (24 -> 144 at 8 x 56x56 7.7 us, 7.3)
    p.var = PW_WIDE;
    p.mper = std::min(mt, kWideTiles);
    p.gy = cdiv(mt, p.mper);
    p.gx = cdiv(NQ, 128);
    return p;
  }
  // Longer contractions are bound by reading and splitting the pixels once per row tile.
  if (KG > 4 && HW % 2 == 0) {
    // Two row tiles per wavefront read and split half the pixels, but of an odd count the last pair does nothing for its second
    // tile, which is too much below seven: forward, two tiles / one, three of them 128 -> 72 at 32 x 56x56 30 / 25 us, five
    // 256 -> 144 at 32 x 28x28 26.6 / 20.9, seven 256 -> 208 27.0 / 27.4 and 96 -> 200 at 16 x 56x56 24.8 / 23.9.
    if ((mt % 2 == 0 || mt >= 7) && tiles >= 3000) { p.var = PW_2x2; p.gy = cdiv(mt, 2); p.gx = cdiv(NQ, 256); }
    else { p.var = PW_2x1; p.gx = cdiv(NQ, 256); }
    return p;
  }
  if (KG > 4 && mt >= 2) { p.var = PW_1x2; p.gy = cdiv(mt, 2); }
  p.gx = cdiv(NQ, 128);
  return p;
}

static PwArgs pw_args(const float* Wp, const float* X, float* Y, const float* bias, const float* add, int N, int Kdim,
                      int Mdim, int HW, const PwPick& p) {
  PwArgs a;
  a.Wp = reinterpret_cast<const uint4*>(Wp);
  a.X = X; a.Y = Y; a.bias = bias; a.add = add;
  a.stats = nullptr;
  a.NQ = (unsigned)((size_t)N * HW);
  a.x_words = (size_t)a.NQ * Kdim; a.y_words = (size_t)a.NQ * Mdim;
  a.HW = HW; a.rHW = plane_reciprocal(HW); a.Kdim = Kdim; a.Mdim = Mdim; a.KG = cdiv(Kdim, 16);
  a.gy = p.gy; a.mper = p.mper;
  // What the blocks of an XCD share is the larger operand: 2048 -> 512 channels at 8 x 7x7 (6 bytes a weight) 14.1 us with
  // the weights shared, 15.5 with the pixels; 256 -> 64 at 8 x 56x56 11.3 and 10.6.
  a.order = (size_t)Mdim * 3 < (size_t)a.NQ * 2;
  return a;
}

// Partial pairs per channel that the forward product can leave for a BatchNorm behind it: its pixel blocks, of eight
// wavefronts where four would leave more than 256, while they are at most 512; 0 = not offered.  (24 -> 144 channels at
// 32 x 56x56 as 392 blocks of eight wavefronts 19.5 us, as 196 of sixteen 25.9 us: one block on a compute unit, and its loads
// and stores take turns.)
static bool pw_stats_blocks(PwPick& p, long NQ) {
  if (p.var == PW_KS4 || p.var == PW_KS4x2 || p.var == PW_KS8 || p.var == PW_FAR) return false;
  if (p.gx > 256) {
    p.waves = 8;
    p.gx = cdiv(NQ, 256L * (p.var == PW_2x1 || p.var == PW_2x2 ? 2 : 1));
  }
  return p.gx <= 512;
}
int pw_conv_stats_parts(int N, int Kdim, int Mdim, int HW) {
  PwPick p = pw_pick((long)N * HW, HW, Kdim, Mdim, true);
  return pw_stats_blocks(p, (long)N * HW) ? p.gx : 0;
}

template <int G>
static void launch_wide(hipStream_t st, const PwArgs& a, const PwPick& p) {
  const size_t lds = a.stats ? (size_t)p.waves * p.mper * 32 * sizeof(float2) : 0;
  KLAUNCH_NAMED("pw_conv_f32_wide_kernel", (pw_conv_f32_wide_kernel<G>), dim3(p.gx * p.gy), dim3(64 * p.waves), lds, st, a);
}
static void launch_product(hipStream_t st, const PwArgs& a, const PwPick& p) {
  const dim3 grid(p.gx * p.gy), block(64 * p.waves);
  switch (p.var) {
    case PW_1x1: KLAUNCH_NAMED("pw_conv_f32_kernel", (pw_conv_f32_kernel<1, 1>), grid, block, 0, st, a); break;
    case PW_1x2: KLAUNCH_NAMED("pw_conv_f32_kernel", (pw_conv_f32_kernel<1, 2>), grid, block, 0, st, a); break;
    case PW_2x1: KLAUNCH_NAMED("pw_conv_f32_kernel", (pw_conv_f32_kernel<2, 1>), grid, block, 0, st, a); break;
    case PW_2x2: KLAUNCH_NAMED("pw_conv_f32_kernel", (pw_conv_f32_kernel<2, 2>), grid, block, 0, st, a); break;
    case PW_KS4: KLAUNCH_NAMED("pw_conv_f32_ks_kernel", (pw_conv_f32_ks_kernel<1, 4>), grid, block, 0, st, a); break;
    case PW_KS4x2: KLAUNCH_NAMED("pw_conv_f32_ks_kernel", (pw_conv_f32_ks_kernel<2, 4>), grid, block, 0, st, a); break;
    case PW_KS8: KLAUNCH_NAMED("pw_conv_f32_ks_kernel", (pw_conv_f32_ks_kernel<1, 8>), grid, block, 0, st, a); break;
    case PW_WIDE:
      if (a.KG == 1) launch_wide<1>(st, a, p);
      else if (a.KG == 2) launch_wide<2>(st, a, p);
      else launch_wide<4>(st, a, p);
      break;
    case PW_FAR: KLAUNCH(pw_conv_f32_far_kernel, grid, block, 0, st, a); break;
  }
}

void pw_conv_f32(hipStream_t st, const float* Wp, const float* X, float* Y, const float* bias, const float* add,
                 int N, int Kdim, int Mdim, int HW, double* stats) {
  const bool plain = !bias && !add;
  PwPick p = pw_pick((long)N * HW, HW, Kdim, Mdim, plain), q = p;
  const bool given = stats && plain && pw_stats_blocks(q, (long)N * HW);
  if (given) p = q;
  PwArgs a = pw_args(Wp, X, Y, bias, add, N, Kdim, Mdim, HW, p);
  if (given) a.stats = stats;
  launch_product(st, a, p);
}

// ============================================================== weight gradient
// dW[co][ci] = sum over the pixels q of all samples of g[co][q] x[ci][q], with the split operands of the products above.  A
// block owns TCO x TCI tiles of 32 x 32 weights and the pixels of one of `splits` equal ranges of the flattened (sample,
// pixel) index, in steps of 64 of which each of its four wavefronts multiplies 16 for every tile.  A step's rows of g and x
// are loaded in whole 128-byte runs one step ahead, split in registers and copied to LDS as three planes of 128-byte rows; a
// lane reads eight pixels of row l%32 as one 16-byte word.  Which pixels of a step are neighbours in LDS does not matter
// as long as g and x agree: word c of a row holds pixels 4c..4c+3 and 32+4c..32+4c+3, so that eight lanes load whole runs.
// Word c lies at position c ^ (row/2 & 7): the sixteen lanes of one LDS access hit all 64 banks.
//
// Chains of additions: two roundings per 16 pixels (the small products have accumulators of their own), and a range is at most
// WG_CHAIN steps, so no chain grows with the micro-batch; wavefronts and partials are added in 64 bits.  LONG: where there is
// no room for so many partials, a range is longer, and every WG_CHAIN steps of it go to 64-bit sums in registers.
template <int TCO, int TCI>
struct WgTile {
  static constexpr int ROWS = (TCO + TCI) * 32, PLANE = ROWS * 128, LDS = 3 * PLANE / 4;  // bytes, floats
};
// acc += one 32 x 32 tile of dW over a wavefront's pixels of the steps [s0, s1), on the fp32 matrix instructions
// (kernels_f32_x3.h: where the pieces gave no finite sum)
__device__ __forceinline__ void wg_contract_f32(const WgArgs& w, int co, int ci, int wave, int s0, int s1, floatx16& acc) {
  const unsigned HW = (unsigned)w.HW, Q = (unsigned)w.NQ;
  const int half = threadIdx.x >> 5 & 1;
  co += threadIdx.x & 31;
  ci += threadIdx.x & 31;
#pragma unroll 1
  for (int s = s0; s < s1; ++s) {
    const unsigned q0 = (unsigned)s * 64u + 4u * (2 * wave + half), n0 = q0 / HW;  // (word 2 * wave + half of every row)
    float g[8], x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const unsigned q = q0 + 32 * (e >> 2) + (e & 3), r = q - n0 * HW, k = plane_of(r, HW, w.rHW), n = n0 + k, p = r - k * HW;
      g[e] = q < Q && co < w.Cout ? w.g[((size_t)n * w.Cout + co) * HW + p] : 0.f;
      x[e] = q < Q && ci < w.Cin ? w.x[((size_t)n * w.Cin + ci) * HW + p] : 0.f;
    }
    acc = mfma_f32(g, x, acc);
  }
}

constexpr int WG_CHAIN = 32;
template <int TCO, int TCI, bool VEC, bool LONG, bool FAR>
__device__ __forceinline__ void pw_wgrad_body(const WgArgs& w, int split, int bci, int bco, char* __restrict__ lds) {
  using T = WgTile<TCO, TCI>;
  constexpr int NI = TCO + TCI;  // a thread stages eight pixels of one row of each 32-row tile
  const int Cin = w.Cin, Cout = w.Cout;
  const unsigned HW = (unsigned)w.HW, Q = (unsigned)w.NQ;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int co_base = bco * (TCO * 32), ci_base = bci * (TCI * 32);
  const int steps = (int)((Q + 63) / 64);
  const int s0 = (int)((long)steps * split / w.splits), s1 = (int)((long)steps * (split + 1) / w.splits);

  const int sr = t >> 3, sc = t & 7;
  const unsigned row_bytes = HW * 4u;
  float rv[NI][8];
  unsigned q0 = (unsigned)s0 * 64u, n0 = __builtin_amdgcn_readfirstlane(q0 / HW), p0 = q0 - n0 * HW;  // of the step to load
  // (FAR: planes that 32-bit offsets do not reach)
  auto load_far = [&]() __attribute__((always_inline)) {
    constexpr int NV = VEC ? 2 : 8;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const unsigned d = VEC ? 32 * j + 4 * sc : 32 * (j >> 2) + 4 * sc + (j & 3);
      const unsigned k = plane_of(p0 + d, HW, w.rHW), p = p0 + d - k * HW;
      const float* const gp = w.g + ((size_t)(n0 + k) * Cout + co_base + sr) * HW + p;
      const float* const xp = w.x + ((size_t)(n0 + k) * Cin + ci_base + sr) * HW + p;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const bool isg = i < TCO;
        const int row = (isg ? i : i - TCO) * 32;
        const bool in = q0 + d < Q && (isg ? co_base + row + sr < Cout : ci_base + row + sr < Cin);
        const float* const s = (isg ? gp : xp) + (size_t)row * HW;
        if constexpr (VEC) {
          const float4 v = in ? *reinterpret_cast<const float4*>(s) : make_float4(0.f, 0.f, 0.f, 0.f);
          rv[i][4 * j] = v.x; rv[i][4 * j + 1] = v.y; rv[i][4 * j + 2] = v.z; rv[i][4 * j + 3] = v.w;
        } else {
          rv[i][j] = in ? *s : 0.f;
        }
      }
    }
    q0 += 64;
    for (p0 += 64; p0 >= HW; p0 -= HW) ++n0;  // uniform
  };
  auto load = [&]() __attribute__((always_inline)) {
    if constexpr (FAR) {
      load_far();
      return;
    }
    const size_t go = ((size_t)n0 * Cout + co_base) * HW, xo = ((size_t)n0 * Cin + ci_base) * HW;
    const __amdgpu_buffer_rsrc_t rg = rsrc_words(w.g + go, (size_t)Q * Cout - go), rx = rsrc_words(w.x + xo, (size_t)Q * Cin - xo);
    constexpr int NV = VEC ? 2 : 8;  // words of four pixels (HW % 4 == 0: they never leave their sample) or single ones
    unsigned og[NV], ox[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const unsigned d = VEC ? 32 * j + 4 * sc : 32 * (j >> 2) + 4 * sc + (j & 3);
      const unsigned k = plane_of(p0 + d, HW, w.rHW), p = p0 + d - k * HW;
      const bool ok = q0 + d < Q;
      og[j] = ok ? (k * (unsigned)Cout * HW + p + (unsigned)sr * HW) * 4u : kOutside;
      ox[j] = ok ? (k * (unsigned)Cin * HW + p + (unsigned)sr * HW) * 4u : kOutside;
    }
    q0 += 64;
    for (p0 += 64; p0 >= HW; p0 -= HW) ++n0;  // uniform
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bool isg = i < TCO;
      const int tile = isg ? i : i - TCO;
      const bool in = isg ? co_base + tile * 32 + sr < Cout : ci_base + tile * 32 + sr < Cin;
      const unsigned so = (unsigned)tile * 32u * row_bytes;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const unsigned vo = in ? (isg ? og[j] : ox[j]) : kOutside;
        if constexpr (VEC) {
          const auto v = __builtin_amdgcn_raw_buffer_load_b128(isg ? rg : rx, vo, so, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) rv[i][4 * j + e] = __uint_as_float(v[e]);
        } else {
          rv[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(isg ? rg : rx, vo, so, 0));
        }
      }
    }
  };
  char* const st = lds + sr * 128 + ((sc ^ (sr >> 1 & 7)) * 16);
  auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      uint4 p[3];
      split3(rv[i], p);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4*>(st + k * T::PLANE + i * 4096) = p[k];
    }
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the loads of the next step stay in flight)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  const int row = lane & 31, half = lane >> 5;
  const char* const ld = lds + row * 128 + (((2 * wave + half) ^ (row >> 1 & 7)) * 16);
  floatx16 acc[TCO][TCI], acs[TCO][TCI];
#pragma unroll
  for (int i = 0; i < TCO; ++i)
#pragma unroll
    for (int j = 0; j < TCI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = acs[i][j][r] = 0.f;
  double sum[LONG ? TCO : 1][LONG ? TCI : 1][LONG ? 16 : 1];
  if constexpr (LONG) {
#pragma unroll
    for (int i = 0; i < TCO; ++i)
#pragma unroll
      for (int j = 0; j < TCI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[i][j][r] = 0.0;
  }
  if (s0 < s1) load();  // uniform
  for (int s = s0; s < s1; ++s) {
    put();
    barrier();
    if (s + 1 < s1) load();  // uniform
    uint4 f[NI][3];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) f[i][k] = *reinterpret_cast<const uint4*>(ld + k * T::PLANE + i * 4096);
    auto mma = [&](floatx16(&c)[TCO][TCI], int a, int b) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TCO; ++i)
#pragma unroll
        for (int j = 0; j < TCI; ++j) c[i][j] = mfma_bf16(f[i][a], f[TCO + j][b], c[i][j]);
    };
    mma(acs, 2, 0);
    mma(acc, 0, 0);
    mma(acs, 0, 2);
    mma(acs, 1, 1);
    mma(acs, 1, 0);
    mma(acs, 0, 1);
    if constexpr (LONG) {
      if ((s - s0) % WG_CHAIN == WG_CHAIN - 1) {  // uniform
#pragma unroll
        for (int i = 0; i < TCO; ++i)
#pragma unroll
          for (int j = 0; j < TCI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              sum[i][j][r] += (double)acc[i][j][r] + acs[i][j][r];
              acc[i][j][r] = acs[i][j][r] = 0.f;
            }
      }
    }
    if (s + 1 < s1) barrier();  // the buffer has been read
  }
  // the four wavefronts' sums of a tile are added in a fixed order; the staging buffer is free by now
  float* out = w.part + (size_t)split * Cout * Cin;
  float* const red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < TCO; ++i)
#pragma unroll
    for (int j = 0; j < TCI; ++j) {
      __syncthreads();
      float bad = 0.f, *const own = red + wave * 1024 + lane;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v;
        if constexpr (LONG) v = (float)(sum[i][j][r] + ((double)acc[i][j][r] + acs[i][j][r]));
        else v = acc[i][j][r] + acs[i][j][r];
        bad = fmaf(v, 0.f, bad);
        own[r * 64] = v;
      }
      if (any_not_finite(bad)) {
        floatx16 again = zero16();
        wg_contract_f32(w, co_base + i * 32, ci_base + j * 32, wave, s0, s1, again);
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (!finite_f(own[r * 64])) own[r * 64] = again[r];
      }
      __syncthreads();
      const int ci = ci_base + j * 32 + row;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int r = wave * 4 + rr, co = co_base + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        const float* v = red + r * 64 + lane;
        const float d = (float)(((double)v[0] + v[16 * 64]) + ((double)v[2 * 16 * 64] + v[3 * 16 * 64]));
        if (ci < Cin && co < Cout) out[(size_t)co * Cin + ci] = d;
      }
    }
}

// The block shapes of the weight gradient: weight tiles (co x ci) per block, wavefronts per tile
enum { WG_2x2 = 0, WG_2x1 = 1, WG_1x2 = 2, WG_1x1 = 3 };
template <int SHAPE, bool VEC, bool LONG = false, bool FAR = false>
__device__ __forceinline__ void pw_wgrad_shape(const WgArgs& w, int split, int bci, int bco, float* lds) {
  constexpr int TCO = SHAPE == WG_2x2 || SHAPE == WG_2x1 ? 2 : 1, TCI = SHAPE == WG_2x2 || SHAPE == WG_1x2 ? 2 : 1;
  pw_wgrad_body<TCO, TCI, VEC, LONG, FAR>(w, split, bci, bco, reinterpret_cast<char*>(lds));
}
template <int SHAPE>
constexpr int wg_lds_floats() {
  return SHAPE == WG_2x2 ? WgTile<2, 2>::LDS : SHAPE == WG_1x1 ? WgTile<1, 1>::LDS : WgTile<2, 1>::LDS;
}

template <int SHAPE, bool VEC, bool LONG = false, bool FAR = false>
__global__ __launch_bounds__(256, SHAPE == WG_2x2 || LONG ? 2 : 3) void pw_wgrad_f32_kernel(WgArgs w) {
  __shared__ float4 lds[wg_lds_floats<SHAPE>() / 4];
  int bx, t;
  pw_block_xy((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, gridDim.x, gridDim.y * gridDim.z,
              w.tile_order, bx, t);
  pw_wgrad_shape<SHAPE, VEC, LONG, FAR>(w, bx, t % (int)gridDim.y, t / (int)gridDim.y, reinterpret_cast<float*>(lds));
}

// the wide product's forms in the launch below: more than 32 channels in, an addend
constexpr int PW_WIDE4 = PW_FAR + 1, PW_WIDE_ADD = PW_FAR + 2, PW_WIDE4_ADD = PW_FAR + 3;

// Input gradient and weight-gradient partials of one pointwise conv in ONE launch: the two products only share their input
// g, and each alone is too short to fill the chip, so their blocks are dealt from one grid: block ids [0, nA) are those of
// the input-gradient product, the rest the (x, y, z) grid of the weight-gradient kernel.
template <int VAR, int SHAPE, bool VEC>
__global__ __launch_bounds__(256, 2)
void pw_bwd_dual_kernel(PwArgs a, WgArgs w, unsigned nA, unsigned gWx, unsigned gWy) {
  __shared__ float4 lds[wg_lds_floats<SHAPE>() / 4];
  static_assert(wg_lds_floats<SHAPE>() >= 4 * 16 * 64, "the product kernels use 16 KB");
  if (blockIdx.x < nA) {  // uniform per block
    int bx, by;
    pw_product_xy(blockIdx.x, nA, a, bx, by);
    if constexpr (VAR == PW_1x1) pw_body<1, 1>(a, bx, by, nullptr, 0);
    else if constexpr (VAR == PW_1x2) pw_body<1, 2>(a, bx, by, nullptr, 0);
    else if constexpr (VAR == PW_2x1) pw_body<2, 1>(a, bx, by, nullptr, 0);
    else if constexpr (VAR == PW_2x2) pw_body<2, 2>(a, bx, by, nullptr, 0);
    else if constexpr (VAR == PW_KS4) pw_ks_body<1, 4>(a, bx, by, reinterpret_cast<float(*)[16][64]>(lds));
    else if constexpr (VAR == PW_KS4x2) pw_ks_body<2, 4>(a, bx, by, reinterpret_cast<float(*)[16][64]>(lds));
    else if constexpr (VAR == PW_WIDE) pw_wide_body<2, false>(a, bx, by, nullptr);
    else if constexpr (VAR == PW_WIDE4) pw_wide_body<4, false>(a, bx, by, nullptr);
    else if constexpr (VAR == PW_WIDE_ADD) pw_wide_body<2, true>(a, bx, by, nullptr);
    else pw_wide_body<4, true>(a, bx, by, nullptr);
  } else {
    int bx, t;  // the weight-gradient ids start at nA: ids that agree mod 8 still share an XCD
    pw_block_xy(blockIdx.x - nA, gWx, (gridDim.x - nA) / gWx, w.tile_order, bx, t);
    pw_wgrad_shape<SHAPE, VEC>(w, bx, t % (int)gWy, t / (int)gWy, reinterpret_cast<float*>(lds));
  }
}
// G[i] += sum_c part[c][i]: 64 outputs per block, four interleaved part lanes, fixed order
__global__ __launch_bounds__(256) void reduce_parts_acc_kernel(const float* __restrict__ part,
                                                               float* __restrict__ G, size_t n, int parts) {
  __shared__ float sh[4][64];
  const int o = threadIdx.x & 63, q = threadIdx.x >> 6;
  const size_t i = (size_t)blockIdx.x * 64 + o;
  float s = 0.f;
  if (i < n) {
    int c = q;
    for (; c + 28 < parts; c += 32) {  // eight independent loads in flight
      float v0 = part[(size_t)c * n + i], v1 = part[(size_t)(c + 4) * n + i];
      float v2 = part[(size_t)(c + 8) * n + i], v3 = part[(size_t)(c + 12) * n + i];
      float v4 = part[(size_t)(c + 16) * n + i], v5 = part[(size_t)(c + 20) * n + i];
      float v6 = part[(size_t)(c + 24) * n + i], v7 = part[(size_t)(c + 28) * n + i];
      s += ((v0 + v1) + (v2 + v3)) + ((v4 + v5) + (v6 + v7));
    }
    for (; c < parts; c += 4) s += part[(size_t)c * n + i];
  }
  sh[q][o] = s;
  __syncthreads();
  if (q == 0 && i < n) G[i] += (sh[0][o] + sh[1][o]) + (sh[2][o] + sh[3][o]);
}

// Block shape and number of pixel ranges of a weight gradient.  A larger block reads and splits less per product, and leaves
// fewer blocks: 204 registers at 2x2 (two blocks per compute unit), 130 at 2x1, 82 at 1x1 (four and more).  Measured, us:
//   one channel tile on a side: 24 -> 144 at 32 x 56x56 1x1 17.3, 2x1 18.1; 192 -> 32 at 32 x 28x28 9.3, 9.5
//   much work: 64 -> 256 at 32 x 56x56 2x2 33.3, 2x1 35.2; 512 -> 256 at 8 x 28x28 19.9, 20.7; many tiles over few pixels:
//     512 -> 2048 at 8 x 7x7 20.5, 24.0; 256 -> 1024 at 8 x 14x14 13.8, 14.8
//   between: 40 -> 240 at 32 x 30x30 2x1 14.5, 2x2 15.6; 64 -> 64 at 32 x 56x56 14.8, 15.8
//   little (less than two blocks per compute unit): the smallest blocks with one step upwards
// A range is at most WG_CHAIN steps: chains of 64 roundings.  Relative error of dW against 64 bits 5e-8 to 9e-8 over these
// sizes (the fp32 matrix instructions with their sums in two levels: 8e-8 to 1.3e-7).  A cap on the number of ranges that makes
// them longer (chained) takes a shape with registers for 64-bit sums.  far: planes that 32-bit offsets do not reach.
struct WgPick { int shape; dim3 grid; bool chained, far; };
static WgPick wg_pick(int N, int Cin, int Cout, int HW, int cap) {
  const int a = cdiv(Cout, 32), b = cdiv(Cin, 32);
  static const int tco[4] = {2, 2, 1, 1}, tci[4] = {2, 1, 2, 1}, blocks[4] = {512, 768, 768, 1024};
  const long NQ = (long)N * HW;
  WgPick p;
  auto splits = [&](int shape, int px) {
    p.shape = shape;
    const int gy = cdiv(b, tci[shape]), gz = cdiv(a, tco[shape]);
    const long fill = std::min((long)cdiv(blocks[shape], (long)gy * gz), NQ / px);
    const long s = std::min(std::max(fill, (long)cdiv(NQ, WG_CHAIN * 64)), (long)cap);
    p.grid = dim3((unsigned)s, gy, gz);
    return s * gy * gz;
  };
  if (a == 1 || b == 1) splits(WG_1x1, 64);
  else if (NQ * a * b >= 600000 || (NQ < 2048 && a * b >= 256)) splits(WG_2x2, 128);
  else if (splits(a % 2 && b % 2 == 0 ? WG_1x2 : WG_2x1, 128) < 512) splits(WG_1x1, 64);
  p.far = pw_far(Cin, Cout, HW);
  p.chained = cdiv(cdiv(NQ, 64), p.grid.x) > WG_CHAIN;
  if (p.chained && p.shape == WG_2x2) splits(a % 2 && b % 2 == 0 ? WG_1x2 : WG_2x1, 128);
  return p;
}
int pw_wgrad_f32_parts(int N, int Cin, int Cout, int HW, int cap) { return (int)wg_pick(N, Cin, Cout, HW, cap).grid.x; }
// The fewest that a stage is held to where more would not fit the static workspace: one wavefront per SIMD and tile.
int pw_wgrad_f32_compact_parts(int N, int Cin, int Cout, int HW) {
  const long fill = std::min((long)cdiv(768, (long)cdiv(Cin, 32) * cdiv(Cout, 32)), (long)N * HW / 128);
  return (int)std::max(1L, fill);
}
size_t pw_wgrad_f32_ws(int N, int Cin, int Cout, int HW, int cap) {
  return (size_t)pw_wgrad_f32_parts(N, Cin, Cout, HW, cap) * Cin * Cout;
}
static WgArgs wg_args(const float* g, const float* x, float* part, int N, int Cin, int Cout, int HW, const WgPick& p) {
  WgArgs w;
  w.g = g; w.x = x; w.part = part;
  w.Cin = Cin; w.Cout = Cout; w.HW = HW; w.rHW = plane_reciprocal(HW);
  w.NQ = (long)N * HW;
  w.splits = (int)p.grid.x;
  w.tile_order = p.grid.y * p.grid.z > 1;
  return w;
}
template <int SHAPE, bool LONG, bool FAR>
static void launch_wgrad(hipStream_t st, const WgArgs& w, dim3 grid) {
  if (w.HW % 4 == 0) KLAUNCH_NAMED("pw_wgrad_f32_kernel", (pw_wgrad_f32_kernel<SHAPE, true, LONG, FAR>), grid, dim3(256), 0, st, w);
  else KLAUNCH_NAMED("pw_wgrad_f32_kernel", (pw_wgrad_f32_kernel<SHAPE, false, LONG, FAR>), grid, dim3(256), 0, st, w);
}
template <bool LONG, bool FAR>
static void launch_wgrad(hipStream_t st, const WgArgs& w, const WgPick& p) {
  switch (p.shape) {
    case WG_2x2:
      if constexpr (!LONG) launch_wgrad<WG_2x2, LONG, FAR>(st, w, p.grid);
      break;
    case WG_2x1: launch_wgrad<WG_2x1, LONG, FAR>(st, w, p.grid); break;
    case WG_1x2: launch_wgrad<WG_1x2, LONG, FAR>(st, w, p.grid); break;
    default: launch_wgrad<WG_1x1, LONG, FAR>(st, w, p.grid); break;
  }
}
static void launch_wgrad(hipStream_t st, const WgArgs& w, const WgPick& p) {
  if (p.chained && p.far) launch_wgrad<true, true>(st, w, p);
  else if (p.chained) launch_wgrad<true, false>(st, w, p);
  else if (p.far) launch_wgrad<false, true>(st, w, p);
  else launch_wgrad<false, false>(st, w, p);
}
void pw_wgrad_f32(hipStream_t st, const float* g, const float* x, float* part, float* G, int N,
                  int Cin, int Cout, int HW, int cap) {
  const WgPick p = wg_pick(N, Cin, Cout, HW, cap);
  launch_wgrad(st, wg_args(g, x, part, N, Cin, Cout, HW, p), p);
  size_t n = (size_t)Cin * Cout;
  if (G) KLAUNCH(reduce_parts_acc_kernel, dim3(cdiv(n, 64)), dim3(256), 0, st, part, G, n, (int)p.grid.x);
}

template <int VAR, int SHAPE>
static void launch_dual(hipStream_t st, const PwArgs& a, const WgArgs& w, unsigned nA, dim3 gW) {
  const dim3 grid(nA + gW.x * gW.y * gW.z);
  if (w.HW % 4 == 0)
    KLAUNCH_NAMED("pw_bwd_dual_kernel", (pw_bwd_dual_kernel<VAR, SHAPE, true>), grid, dim3(256), 0, st, a, w, nA, gW.x, gW.y);
  else
    KLAUNCH_NAMED("pw_bwd_dual_kernel", (pw_bwd_dual_kernel<VAR, SHAPE, false>), grid, dim3(256), 0, st, a, w, nA, gW.x, gW.y);
}
template <int VAR>
static void launch_dual(hipStream_t st, const PwArgs& a, const WgArgs& w, unsigned nA, const WgPick& p) {
  switch (p.shape) {
    case WG_2x2: launch_dual<VAR, WG_2x2>(st, a, w, nA, p.grid); break;
    case WG_2x1: launch_dual<VAR, WG_2x1>(st, a, w, nA, p.grid); break;
    case WG_1x2: launch_dual<VAR, WG_1x2>(st, a, w, nA, p.grid); break;
    default: launch_dual<VAR, WG_1x1>(st, a, w, nA, p.grid); break;
  }
}

static PwPick bwd_pick(int N, int Cin, int Cout, int HW) {
  PwPick p = pw_pick((long)N * HW, HW, Cout, Cin, true);
  if (p.var == PW_KS8) {  // a launch has blocks of one size: four shares of the contraction cost less than a second launch
    p.var = PW_KS4;
    p.waves = 4;
  }
  return p;
}
void pw_conv_bwd_f32(hipStream_t st, const float* Wp_t, const float* g, float* dx, const float* add, const float* x,
                     float* part, float* G, int N, int Cin, int Cout, int HW, int cap) {
  const PwPick p = bwd_pick(N, Cin, Cout, HW);  // dx = W^T g (+ add)
  const PwArgs a = pw_args(Wp_t, g, dx, nullptr, add, N, Cout, Cin, HW, p);
  const WgPick wp = wg_pick(N, Cin, Cout, HW, cap);
  const WgArgs w = wg_args(g, x, part, N, Cin, Cout, HW, wp);
  const unsigned nA = p.gx * p.gy;
  if (wp.chained || wp.far) {  // (rare, and not worth the forms of the common launch)
    pw_conv_f32(st, Wp_t, g, dx, nullptr, add, N, Cout, Cin, HW, nullptr);
    launch_wgrad(st, w, wp);
  } else switch (p.var) {
    case PW_1x1: launch_dual<PW_1x1>(st, a, w, nA, wp); break;
    case PW_1x2: launch_dual<PW_1x2>(st, a, w, nA, wp); break;
    case PW_2x1: launch_dual<PW_2x1>(st, a, w, nA, wp); break;
    case PW_2x2: launch_dual<PW_2x2>(st, a, w, nA, wp); break;
    case PW_KS4: launch_dual<PW_KS4>(st, a, w, nA, wp); break;
    case PW_KS4x2: launch_dual<PW_KS4x2>(st, a, w, nA, wp); break;
    case PW_WIDE:
      if (a.KG <= 2 && !add) launch_dual<PW_WIDE>(st, a, w, nA, wp);
      else if (!add) launch_dual<PW_WIDE4>(st, a, w, nA, wp);
      else if (a.KG <= 2) launch_dual<PW_WIDE_ADD>(st, a, w, nA, wp);
      else launch_dual<PW_WIDE4_ADD>(st, a, w, nA, wp);
      break;
    default: break;
  }
  size_t n = (size_t)Cin * Cout;
  if (G) KLAUNCH(reduce_parts_acc_kernel, dim3(cdiv(n, 64)), dim3(256), 0, st, part, G, n, (int)wp.grid.x);
}

// (sums in 64 bits: the kernel waits for memory, and adding partials in 32 bits was a third of the rounding error of a
// weight gradient)
__global__ __launch_bounds__(256) void reduce_tasks_kernel(const RedTask* __restrict__ tasks,
                                                           const unsigned short* __restrict__ block_task) {
  __shared__ double sh[4][64];
  const RedTask t = tasks[block_task[blockIdx.x]];
  if (t.wide) {  // uniform per block
    const size_t i4 = ((size_t)(blockIdx.x - t.block0) * 256 + threadIdx.x) * 4;
    if (i4 >= t.n) return;
    const float* p4 = t.part + i4;
    const size_t st4 = t.stride;
    const int parts4 = (int)t.parts;
    double s4[4] = {0.0, 0.0, 0.0, 0.0};
    int c4 = 0;
    for (; c4 + 4 <= parts4; c4 += 4) {
      const float4 v0 = *reinterpret_cast<const float4*>(p4 + (size_t)c4 * st4);
      const float4 v1 = *reinterpret_cast<const float4*>(p4 + (size_t)(c4 + 1) * st4);
      const float4 v2 = *reinterpret_cast<const float4*>(p4 + (size_t)(c4 + 2) * st4);
      const float4 v3 = *reinterpret_cast<const float4*>(p4 + (size_t)(c4 + 3) * st4);
      s4[0] += ((double)v0.x + v1.x) + ((double)v2.x + v3.x);
      s4[1] += ((double)v0.y + v1.y) + ((double)v2.y + v3.y);
      s4[2] += ((double)v0.z + v1.z) + ((double)v2.z + v3.z);
      s4[3] += ((double)v0.w + v1.w) + ((double)v2.w + v3.w);
    }
    for (; c4 < parts4; ++c4) {
      const float4 v = *reinterpret_cast<const float4*>(p4 + (size_t)c4 * st4);
      s4[0] += v.x; s4[1] += v.y; s4[2] += v.z; s4[3] += v.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      size_t out = i4 + e;
      if (t.taps > 1) {
        const size_t tp = out / t.mn;
        out = (out - tp * t.mn) * t.taps + tp;
      }
      t.G[out] = (float)(t.G[out] + s4[e]);
    }
    return;
  }
  const int o = threadIdx.x & 63, q = threadIdx.x >> 6;
  const size_t n = t.n, st = t.stride;
  const size_t i = (size_t)(blockIdx.x - t.block0) * 64 + o;
  const int parts = (int)t.parts;
  const float* p = t.part + i;
  double s = 0.0;
  if (i < n) {
    int c = q;
    for (; c + 28 < parts; c += 32) {  // eight independent loads in flight
      const double v0 = p[(size_t)c * st], v1 = p[(size_t)(c + 4) * st];
      const double v2 = p[(size_t)(c + 8) * st], v3 = p[(size_t)(c + 12) * st];
      const double v4 = p[(size_t)(c + 16) * st], v5 = p[(size_t)(c + 20) * st];
      const double v6 = p[(size_t)(c + 24) * st], v7 = p[(size_t)(c + 28) * st];
      s += ((v0 + v1) + (v2 + v3)) + ((v4 + v5) + (v6 + v7));
    }
    for (; c < parts; c += 4) s += p[(size_t)c * st];
  }
  sh[q][o] = s;
  __syncthreads();
  if (q == 0 && i < n) {
    size_t out = i;
    if (t.taps > 1) {
      const size_t tp = i / t.mn;
      out = (i - tp * t.mn) * t.taps + tp;
    }
    t.G[out] = (float)(t.G[out] + ((sh[0][o] + sh[1][o]) + (sh[2][o] + sh[3][o])));
  }
}
void reduce_tasks_f32(hipStream_t st, const RedTask* tasks_dev, const unsigned short* block_task_dev, int nblocks) {
  KLAUNCH(reduce_tasks_kernel, dim3(nblocks), dim3(256), 0, st, tasks_dev, block_task_dev);
}

void reduce_parts_acc_f32(hipStream_t st, const float* part, float* G, size_t n, int parts) {
  KLAUNCH(reduce_parts_acc_kernel, dim3(cdiv(n, 64)), dim3(256), 0, st, part, G, n, parts);
}

}  // namespace ast

// The choices above, for tests: out = {product's form (PwVar), pixel blocks, row tiles of a block's wavefront walk, wavefronts}
// of a forward product without bias or of an input gradient, and {block shape, ranges, 64-bit sums} of a
// weight gradient.
extern "C" void ast_pw_choice(int dgrad, int N, int Cin, int Cout, int HW, int out[4]) {
  using namespace ast;
  const PwPick p = dgrad ? bwd_pick(N, Cin, Cout, HW) : pw_pick((long)N * HW, HW, Cin, Cout, true);
  out[0] = p.var; out[1] = p.gx; out[2] = p.mper; out[3] = p.waves;
}
extern "C" void ast_pw_wgrad_choice(int N, int Cin, int Cout, int HW, int cap, int out[3]) {
  using namespace ast;
  const WgPick p = wg_pick(N, Cin, Cout, HW, cap);
  out[0] = p.shape; out[1] = (int)p.grid.x; out[2] = p.chained;
}
