// Weight gradient of the 3x3 'same' stride-1 convolution on NHWC bf16 tensors with all nine taps of a 32 x 32 tile of weights in
// one wavefront, for products that do not fill the 256-channel tiles of conv_bf16_wgrad.hip:
//
//   dW[co][tap][ci] = sum_p dy[p][co] * x[p + shift(tap)][ci]
//
// Pixels are walked in a virtual order with a zero behind every row and a row of zeros behind every image, where a tap is one
// constant shift (a pixel's neighbours outside the image are zeros of that order): x is staged once, with its halo, for the nine
// taps, and a dy operand serves nine products.  Rows of 32 channels (64 bytes) go to LDS as they lie in memory; the operands
// are read transposed (ds_read_b64_tr_b16: lane i of a group of 16 gets the four pixels of channel i), four rows of 64
// bytes at a time, which fall into different banks at any shift.
//
// A block owns one 32 x 32 tile and a range of the order; its four wavefronts take every fourth step of 16 pixels, and are added
// through LDS in a fixed order.  Partials [range][tap][co][ci], and the column sums of dy [range][co] from the blocks of the
// first input-channel tile.  The next chunk of both operands (256 pixels, 52 KB of LDS a block) is requested before this one is
// multiplied, but the compiler takes a transposed read for one that may see any copy in flight and waits for all of them
// before the first: a block's copies hide behind the products of the other block on its compute unit, not behind its own.
//
// Bound by that wait and by operand reads and products taking turns.  (The reads alone: one 16-pixel step reads 9 + 1 operands of
// 1 KB for nine products of 32 cycles, 8 us of the 32 below at 128 bytes a clock.)  96 -> 96 at 32 x 56x56: 32 us
// in 51 ranges, 520 TFLOP/s (tiles of 256 channels 74 us), at 6 x 45x45 10.8 us (20); 16 -> 32 at 32 x 56x56 9.8 us (57).
#include "device_utils.h"
#include "kernels_bf16.h"
#include "prof.h"

#include <algorithm>
#include <type_traits>

namespace ast {

namespace {

struct TapsArgs {
  const bf16_t* dy;   // [P][Cout]
  const bf16_t* x;    // [P][Cin]
  float* part;        // [splits][9][Cout][Cin]
  float* bias_part;   // [splits][Cout] or NULL
  int H, W, Cout, Cin, tiles_co, tiles_ci;
  int Q;              // virtual pixels
  int xrows;          // rows of x that a chunk needs, a multiple of 16
  int per_split;      // ... of a range, a multiple of kTapsChunk
  unsigned dy_bytes, x_bytes;
  unsigned m_w, m_h;  // reciprocals of W + 1 and H + 1
};

constexpr int kTapsWaves = 4, kTapsChunk = 256;  // virtual pixels staged at a time
constexpr size_t kTapsLds = 160 * 1024;
constexpr unsigned TAPS_OOB = 0x80000000u;

typedef short taps_short4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) taps_short4 taps_lds_short4;
typedef __attribute__((address_space(3))) void taps_lds_void;
typedef unsigned int taps_u32x4 __attribute__((ext_vector_type(4)));

// eight pixels (k) of one channel: two transposed reads of four rows each
__device__ __forceinline__ bf16x8 taps_read(const unsigned char* smem, int off) {
  const taps_short4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((taps_lds_short4*)(smem + off));
  const taps_short4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((taps_lds_short4*)(smem + off + 4 * 64));
  typedef short short8 __attribute__((ext_vector_type(8)));
  const short8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

__global__ __launch_bounds__(64 * kTapsWaves, 2) void conv_wgrad_taps_kernel(TapsArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int bid = (int)xcd_grouped(blockIdx.x, gridDim.x);
  const int tile_ci = bid % g.tiles_ci; bid /= g.tiles_ci;
  const int tile_co = bid % g.tiles_co, split = bid / g.tiles_co;
  const int co0 = tile_co * 32, ci0 = tile_ci * 32, V = g.W + 1, halo = V + 1;
  const int q_begin = split * g.per_split, q_end = min(q_begin + g.per_split, g.Q);
  const __amdgpu_buffer_rsrc_t rdy = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(g.dy), 0, g.dy_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(g.x), 0, g.x_bytes, 0x00020000);
  // two buffers of [xrows][64 bytes], whose first row is virtual pixel q - halo, and [kTapsChunk][64 bytes] of dy
  const int xrows = g.xrows, buffer = (xrows + kTapsChunk) * 64;

  // the pixel of the tensors that virtual pixel q is, or -1
  auto pixel = [&](int q) __attribute__((always_inline)) -> int {
    const int row = (int)__umulhi((unsigned)q, g.m_w), col = q - row * V;
    const int img = (int)__umulhi((unsigned)row, g.m_h), r = row - img * (g.H + 1);
    return q >= 0 && q < g.Q && col < g.W && r < g.H ? (img * g.H + r) * g.W + col : -1;
  };
  // byte offset of virtual pixel q's chunk c in a tensor of C channels whose tile begins at channel t0; beyond the extent where
  // there is no such pixel or channel
  auto source = [&](int q, int c, int C, int t0) __attribute__((always_inline)) -> unsigned {
    const int p = pixel(q);
    return p >= 0 && t0 + c * 8 < C ? (unsigned)((p * C + t0 + c * 8) * 2) : TAPS_OOB;
  };

  float bsum = 0.f;
  const bool do_bias = g.bias_part != nullptr && tile_ci == 0;

  // lane l of a transposed read: 16-lane group b = l / 16 covers channels 16*(b & 1) .. +15 and pixels 8*(b >> 1) .. +3, lane j
  // of the group pixel j / 4, channels 4*(j % 4) .. +3
  const int j16 = lane & 15, blk = lane >> 4;
  const int lane_off = (8 * (blk >> 1) + (j16 >> 2)) * 64 + (16 * (blk & 1) + 4 * (j16 & 3)) * 2;

  // one instruction of a wavefront copies 16 rows: lane l, piece l % 4 of row l / 4
  auto issue = [&](int q0, int at) __attribute__((always_inline)) {
    for (int i = wave; i < (xrows + kTapsChunk) / 16; i += kTapsWaves) {
      const int row = i * 16 + (lane >> 2), c = lane & 3;
      taps_lds_void* const to = (taps_lds_void*)(smem + at + i * 1024);
      if (i * 16 < xrows) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, to, 16, source(q0 - halo + row, c, g.Cin, ci0), 0, 0, 0);
      } else {
        const int q = q0 + row - xrows;  // (dy is read up to the end of the range only)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rdy, to, 16, q < q_end ? source(q, c, g.Cout, co0) : TAPS_OOB, 0, 0, 0);
      }
    }
  };
  // The products of the range and the partials.  A zero of the virtual order times an infinity or a NaN of the other operand is a
  // NaN in a weight that this pair of pixels has no part in: with `pairs`, both operands are zero where either pixel is none.
  // Returns whether a partial is no finite number.
  const int row = tid >> 3, col = (tid & 7) * 4;
  float* const sums = reinterpret_cast<float*>(smem);
  auto form = [&](auto pairs_c) __attribute__((always_inline)) -> bool {
    constexpr bool pairs = decltype(pairs_c)::value;
    floatx16 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    issue(q_begin, 0);
    __syncthreads();  // (waits for the copies too)
    int at = 0;
    for (int q0 = q_begin; q0 < q_end; q0 += kTapsChunk, at = buffer - at) {
      if (q0 + kTapsChunk < q_end) issue(q0 + kTapsChunk, buffer - at);
      const unsigned char* const sx = smem + at;
      const unsigned char* const sdy = sx + xrows * 64;
#pragma unroll 1
      for (int s = wave; s < kTapsChunk / 16; s += kTapsWaves) {
        const bf16x8 a = taps_read(sdy, s * 16 * 64 + lane_off);
        const int q = q0 + s * 16 + 8 * (lane >> 5);  // (of the lane's first k)
        unsigned have = 0;                            // ... and which of its eight are pixels of dy
        if constexpr (pairs) {
#pragma unroll
          for (int e = 0; e < 8; ++e) have |= (unsigned)(pixel(q + e) >= 0 && q + e < q_end) << e;
        }
        if (do_bias && !pairs) {
          const taps_u32x4 w = __builtin_bit_cast(taps_u32x4, a);
#pragma unroll
          for (int e = 0; e < 4; ++e) bsum += __uint_as_float(w[e] << 16) + __uint_as_float(w[e] & 0xffff0000u);
        }
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          bf16x8 b = taps_read(sx, (s * 16 + (t / 3) * V + t % 3) * 64 + lane_off);
          if constexpr (pairs) {
            bf16x8 ap = a;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const bool both = (have >> e & 1) && pixel(q + e + (t / 3 - 1) * V + t % 3 - 1) >= 0;
              ap[e] = both ? ap[e] : (__bf16)0.f;
              b[e] = both ? b[e] : (__bf16)0.f;
            }
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap, b, acc[t], 0, 0, 0);
          } else {
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[t], 0, 0, 0);
          }
        }
      }
      __syncthreads();
    }

    // ---- the wavefronts' tiles, tap by tap, through LDS: [wavefront][32 co][32 ci], two areas in turn
    float none = 0.f;  // 0 as long as all partials are finite
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      float* const area = sums + (t & 1) * (kTapsWaves * 1024);
#pragma unroll
      for (int r = 0; r < 16; ++r)  // register r of lane l is D[8*(r/4) + 4*(l/32) + r%4][l%32]
        area[wave * 1024 + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[t][r];
      __syncthreads();
      floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kTapsWaves; ++w) s += *reinterpret_cast<const floatx4*>(area + w * 1024 + row * 32 + col);
#pragma unroll
      for (int e = 0; e < 4; ++e) none = fmaf(s[e], 0.f, none);
      if (co0 + row < g.Cout && ci0 + col < g.Cin)
        *reinterpret_cast<floatx4*>(g.part + ((size_t)(split * 9 + t) * g.Cout + co0 + row) * g.Cin + ci0 + col) = s;
    }
    return none != 0.f;
  };
  unsigned* const again = reinterpret_cast<unsigned*>(smem) + 2 * kTapsWaves * 1024;  // behind both areas, in what held the operands
  if (__any(form(std::false_type{}))) again[wave] = 1;
  else again[wave] = 0;
  if (do_bias) {  // (uniform) lane l holds channel l % 32 over its half of the pixels
    __syncthreads();
    sums[tid] = bsum;
    __syncthreads();
    if (tid < 32 && co0 + tid < g.Cout) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < 2 * kTapsWaves; ++w) s += sums[w * 32 + tid];
      g.bias_part[(size_t)split * g.Cout + co0 + tid] = s;
    }
  }
  if (!do_bias) __syncthreads();
  const taps_u32x4 w = *reinterpret_cast<const taps_u32x4*>(again);
  static_assert(kTapsWaves == 4, "one word each");
  if (w[0] | w[1] | w[2] | w[3]) {  // (uniform)
    __syncthreads();
    (void)form(std::true_type{});
  }
}

inline long tcdiv(long a, long b) { return (a + b - 1) / b; }
inline int taps_xrows(int W) { return (kTapsChunk + 2 * (W + 2) + 15) / 16 * 16; }
inline size_t taps_lds(int W) { return std::max((size_t)2 * (taps_xrows(W) + kTapsChunk) * 64, (size_t)2 * kTapsWaves * 4096); }
// ranges that the blocks of `most` make; per_split: virtual pixels of each
inline int taps_splits(int N, int H, int W, int most, int& per_split) {
  const long Q = (long)N * (H + 1) * (W + 1);
  per_split = (int)(tcdiv(tcdiv(Q, most), kTapsChunk) * kTapsChunk);
  return (int)tcdiv(Q, per_split);
}

}  // namespace

// as many ranges as make one round of blocks (two to a compute unit where their LDS allows it), at most `most`
int conv_wgrad_taps_splits(int N, int H, int W, int Cin, int Cout, int most) {
  const long tiles = tcdiv(Cout, 32) * tcdiv(Cin, 32), slots = 256 * std::min((size_t)2, kTapsLds / taps_lds(W));
  int per;
  return taps_splits(N, H, W, (int)std::max(1L, std::min((long)most, slots / tiles)), per);
}
bool conv_wgrad_taps_supported(int N, int H, int W, int Cin, int Cout) {
  const long P = (long)N * H * W, Q = (long)N * (H + 1) * (W + 1);
  return Cin % 8 == 0 && Cout % 8 == 0 && P * Cin * 2 < (1L << 31) && P * Cout * 2 < (1L << 31) &&
         Q * (W + 1) < (1L << 32) && (Q / (W + 1)) * (H + 1) < (1L << 32) && Q < (1L << 30) && taps_lds(W) <= kTapsLds;
}
hipError_t conv_wgrad_taps_allow() {
  return hipFuncSetAttribute((const void*)conv_wgrad_taps_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTapsLds);
}
void conv_wgrad_taps_bf16(hipStream_t st, const bf16_t* dy, const bf16_t* x, float* part, float* bias_part, int N, int H, int W,
                          int Cin, int Cout, int splits) {
  TapsArgs g = {};
  g.dy = dy; g.x = x; g.part = part; g.bias_part = bias_part;
  g.H = H; g.W = W; g.Cout = Cout; g.Cin = Cin;
  g.tiles_co = (int)tcdiv(Cout, 32);
  g.tiles_ci = (int)tcdiv(Cin, 32);
  g.xrows = taps_xrows(W);
  g.Q = N * (H + 1) * (W + 1);
  (void)taps_splits(N, H, W, splits, g.per_split);
  g.dy_bytes = (unsigned)((size_t)N * H * W * Cout * 2);
  g.x_bytes = (unsigned)((size_t)N * H * W * Cin * 2);
  g.m_w = (unsigned)((1ull << 32) / (W + 1)) + 1u;
  g.m_h = (unsigned)((1ull << 32) / (H + 1)) + 1u;
  KLAUNCH(conv_wgrad_taps_kernel, dim3((unsigned)(splits * g.tiles_co * g.tiles_ci)), dim3(64 * kTapsWaves), taps_lds(W), st, g);
}

}  // namespace ast
