// fp32 dense convolutions on the matrix cores with the pixels staged in LDS: 3x3 pad 1 (stride 1 or 2) and 1x1
// stride 2, forward, input gradient and weight gradient.
//
// v_mfma_f32_32x32x2 takes 64 cycles for one word of either operand per lane, so the matrix cores are the bound as soon as
// operands arrive with few instructions: nine taps are nine shifted reads of one LDS copy of the pixels.
//
// LDS copy: "virtual rows".  Row h of sample n of the operand tensor is virtual row n*(XH+1) + h + 1; the rows
// between two samples and around the first and last one are zero, and every row has a zero on either side (pitch
// XW + 2).  A tile of consecutive result pixels needs a contiguous range of virtual rows, whatever samples it
// touches, and a tap is one constant offset from a pixel's position: no border test in the product loop.
#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <map>
#include <type_traits>
#include <utility>

#include "device_utils.h"
#include "kernels.h"
#include "kernels_f32_x3.h"
#include "prof.h"

namespace ast {

namespace {

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
__host__ __device__ constexpr int round_up64(int v) { return (v + 63) & ~63; }
// floor(n / d) = mulhi(n, reciprocal(d)) for d > 1 while n * d < 2^32; reciprocal(1) is 0
inline unsigned reciprocal(unsigned d) { return d == 1 ? 0 : (unsigned)(((1ull << 32) + d - 1) / d); }
constexpr size_t kProductLds = 128 * 1024, kWgradLds = 156 * 1024;
// The copies address a whole tensor in memory with 32-bit byte offsets below kOutside.
inline bool copies_reach(int N, int C, int H, int W) { return (size_t)N * C * H * W * 4 < kOutside; }

// ------------------------------------------------------------------ product (forward / input gradient)
// One class of result pixels: all of them, or (input gradient of a stride-2 conv) those of one row / column
// parity, which are reached by the same taps.  The taps are the product of a row list and a column list: entry k of
// `rows` is the byte (tap row u << 4) | (dr + 1), with dr the shift of the operand row in [-1, 1].
struct LdsClass {
  int PH, PW, oy, ox;     // pixels of the class, first result row / column
  unsigned npix;          // N * PH * PW
  unsigned rows, cols;
  int nr, nc;
};
struct LdsArgs {
  const float4* Wp;       // packed weight copies (pw_pack layout), one per tap, tap_stride words apart
  const float* X;         // operand tensor [N][Kdim][XH][XW], or every XS-th row and column of a larger one
  float* Y;               // result tensor  [N][Mdim][OH][OW]
  const float* bias;
  LdsClass cls[4];
  unsigned tap_stride, x_bytes, XHW;  // XHW: words of an operand plane in memory; XRW of a row
  int N, XH, XW, XS, XRW, OH, OW, SI, SO, Kdim, Mdim, KG, KS;
  int WN, WK, rows, RW, NP, PL, CH;
  unsigned rRW, rXH1;
};

typedef __attribute__((address_space(3))) void lds_void;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ void copy_to_lds(__amdgpu_buffer_rsrc_t r, float* dst, unsigned voff, unsigned soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)dst, 4, voff, soff, 0, 0);
}
// byte offset (without the channel part) of position `pos` of the virtual rows vr0, vr0 + 1, ... (pitch XW + 2), or
// kOutside for the zeros between samples, beside the rows and past the last row.
// rRW, rXH1: reciprocal() of XW + 2 and XH + 1.
__device__ __forceinline__ unsigned virtual_offset(int pos, int vr0, int rows, unsigned rRW, unsigned rXH1, int N, int XH,
                                                   int XW, int XRW, int XS, unsigned sample_words) {
  // (an integer division is about 40 vector instructions; 840 of a stage's 9200 cycles this way, 4200 with them)
  const int r = (int)__umulhi((unsigned)pos, rRW), x = pos - r * (XW + 2) - 1;
  const int v = vr0 + r, n = (int)__umulhi((unsigned)v, rXH1), h = v - n * (XH + 1) - 1;
  const bool in = r < rows && (unsigned)x < (unsigned)XW && h >= 0 && n < N;
  return in ? ((unsigned)n * sample_words + (unsigned)((h * XRW + x) * XS)) * 4u : kOutside;
}

// Block: WN pixel groups of 32 x WK shares of the contraction, one wavefront each, and MT 32-row tiles of result
// channels.  A chunk of CH = 8*WK operand channels is copied to LDS (buffer_load ... lds: no registers, zeros
// from the descriptor's bounds check) while the previous chunk is multiplied; wavefront (wn, wk) multiplies the
// wk-th group of eight channels for every tap.  The weights of a wavefront's taps stay one chunk ahead in registers: their
// loads are issued behind the copies of the next chunk, and vector-memory results return in order, so a weight load waited
// for in the same chunk would wait for the copies too.  The WK partial tiles are added through LDS in fixed order.
template <int MT, int NT>
__device__ __forceinline__ void conv_lds_body(const LdsArgs& a, const LdsClass& c, float* lds, int tile0, unsigned q0) {
  const int tid = threadIdx.x, lane = tid & 63, T = blockDim.x, waves = T >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
  const int col = lane & 31, half = lane >> 5;
  const int WN = a.WN, WK = a.WK, wn = wave % WN, wk = wave / WN;
  const int XH1 = a.XH + 1, RW = a.RW, PL = a.PL, KG = a.KG, NP = a.NP, CH = a.CH;
  const unsigned PHW = (unsigned)(c.PH * c.PW);
  const unsigned n0 = q0 / PHW;
  const int vr0 = (int)n0 * XH1 + a.SI * (int)((q0 - n0 * PHW) / (unsigned)c.PW);
  unsigned* const tabv = reinterpret_cast<unsigned*>(lds);  // [NP * 64] operand offsets of the staged positions
  float* const buf0 = lds + NP * 64;
  const int bufsz = CH * PL;
  for (int pos = tid; pos < NP * 64; pos += T)
    tabv[pos] = virtual_offset(pos, vr0, a.rows, a.rRW, a.rXH1, a.N, a.XH, a.XW, a.XRW, a.XS, (unsigned)a.Kdim * a.XHW);
  const __amdgpu_buffer_rsrc_t rx = rsrc_of(a.X, a.x_bytes);
  // The copies of a chunk are dealt to the wavefronts round robin; a wavefront takes its share up in pieces: `i` is the
  // 64-position block and `cc` the channel of its next copy.
  const int dc = waves / NP, di = waves - dc * NP;
  const int ncopy = (CH * NP - wave + waves - 1) / waves;  // of this wavefront
  struct { int cc, i; } cur = {};
  auto first_copy = [&]() __attribute__((always_inline)) {
    cur.cc = wave / NP;
    cur.i = wave - cur.cc * NP;
  };
  auto copies = [&](int k0, float* dst, int count) __attribute__((always_inline)) {
    for (int n = 0; n < count; ++n) {
      const unsigned k = (unsigned)min(k0 + cur.cc, a.Kdim - 1);  // rows past Kdim meet zero weights
      copy_to_lds(rx, dst + cur.cc * PL + cur.i * 64, tabv[cur.i * 64 + lane], k * a.XHW * 4u);
      cur.cc += dc;
      cur.i += di;
      if (cur.i >= NP) { cur.i -= NP; ++cur.cc; }
    }
  };
  const unsigned q = q0 + wn * 32 + col;
  const bool qv = q < c.npix;
  const unsigned qc = qv ? q : c.npix - 1;
  const unsigned qn = qc / PHW;
  const int qp = (int)(qc - qn * PHW), qi = qp / c.PW, qj = qp - qi * c.PW;
  const int base = ((int)qn * XH1 + a.SI * qi - vr0) * RW + a.SI * qj;

  unsigned woff[NT];   // tap t: offset of its weight copy, and of its shift in LDS (uniform)
  int boff[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int ri = t / c.nc, ci = t - ri * c.nc;
    const unsigned rc = c.rows >> (8 * ri), cc = c.cols >> (8 * ci);
    woff[t] = ((rc >> 4 & 15) * (unsigned)a.KS + (cc >> 4 & 15)) * a.tap_stride;
    boff[t] = (int)(rc & 15) * RW + (int)(cc & 15);
  }
  const float4* wl = a.Wp + (size_t)tile0 * KG * 64 + lane;
  const unsigned t1 = (tile0 + 1) * 32 < a.Mdim ? (unsigned)KG * 64u : 0u;  // the second tile, where it exists
  float4 A[NT][MT];
  auto ldA = [&](int i, int ch) __attribute__((always_inline)) {
    const int g = min(ch * WK + wk, KG - 1);  // groups past KG are not multiplied
    const float4* w = wl + (woff[i] + (unsigned)g * 64u);
    A[i][0] = w[0];
    if (MT > 1) A[i][MT - 1] = w[t1];
  };
#pragma unroll
  for (int i = 0; i < NT; ++i) ldA(i, 0);
  floatx16 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
  __syncthreads();
  first_copy();
  copies(0, buf0, ncopy);
  __syncthreads();  // (waits for the copies)
  const int nchunk = (KG + WK - 1) / WK;
  // The copies of the next chunk leave between the products of the first CT taps, so that their issue and their
  // table reads run beside matrix instructions; the weights of the next chunk follow tap by tap, LATE of them behind the
  // last copy.  Vector-memory results return in order: vmcnt(LATE) at the end of a chunk waits for the copies and leaves
  // those weights in flight over the barrier.
  constexpr int CT = NT == 9 ? 6 : NT == 4 ? 2 : 1, LATE = (NT - CT + 1) * MT;
  const int piece = (ncopy + CT - 1) / CT;
  auto chunk = [&](int ch, auto more_c) __attribute__((always_inline)) {
    constexpr bool more = decltype(more_c)::value;
    const float* lb = buf0 + (ch & 1) * bufsz + (8 * wk + half) * PL + base;
    float* const next = buf0 + ((ch + 1) & 1) * bufsz;
    const bool live = more || ch * WK + wk < KG;  // uniform per wavefront; only the last chunk can be short
    float b[2][4];
    auto ldB = [&](int i) __attribute__((always_inline)) {
      const float* p = lb + boff[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) b[i & 1][e] = p[2 * e * PL];
    };
    if (more) first_copy();
    ldB(0);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (i + 1 < NT) ldB(i + 1);
      if (live) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const float av = e == 0 ? A[i][m].x : e == 1 ? A[i][m].y : e == 2 ? A[i][m].z : A[i][m].w;
            acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, b[i & 1][e], acc[m], 0, 0, 0);
          }
      }
      if constexpr (more) {
        if (i < CT) {
          copies((ch + 1) * CH, next, max(0, min(piece, ncopy - i * piece)));
          asm volatile("" ::: "memory");  // the copies stay in front of the weights of this tap and the next ones
        }
        ldA(i, ch + 1);
      }
    }
    if constexpr (more) {
      // lgkmcnt: this wavefront's reads of the buffer that the next chunk overwrites are done
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LATE) : "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
  };
  for (int ch = 0; ch + 1 < nchunk; ++ch) chunk(ch, std::true_type{});
  chunk(nchunk - 1, std::false_type{});
  if (WK > 1) __syncthreads();  // the partial tiles overwrite the staged pixels

  float* yq = a.Y + (size_t)qn * a.Mdim * a.OH * a.OW + (size_t)(a.SO * qi + c.oy) * a.OW + a.SO * qj + c.ox;
  const size_t OHW = (size_t)a.OH * a.OW;
  if (WK == 1) {
    if (!qv) return;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = (tile0 + mt) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (m < a.Mdim) yq[(size_t)m * OHW] = acc[mt][r] + (a.bias ? a.bias[m] : 0.f);
      }
    return;
  }
  const int rpw = 16 / WK;  // accumulator rows that each of the WK wavefronts finishes
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (mt) __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) lds[(wave * 16 + r) * 64 + lane] = acc[mt][r];
    __syncthreads();
    for (int rr = 0; rr < rpw; ++rr) {
      const int r = wk * rpw + rr;
      const int m = (tile0 + mt) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
      float v = 0.f;
      for (int k = 0; k < WK; k += 2)  // fixed order
        v += lds[((k * WN + wn) * 16 + r) * 64 + lane] + lds[(((k + 1) * WN + wn) * 16 + r) * 64 + lane];
      if (qv && m < a.Mdim) yq[(size_t)m * OHW] = v + (a.bias ? a.bias[m] : 0.f);
    }
  }
}

// ALL: one class reached by all nine taps; else the class decides (1, 2 or 4 taps, or none: zeros)
template <int MT, bool ALL>
__global__ __launch_bounds__((MT == 2 && ALL) ? 512 : 1024) void conv_lds_f32_kernel(LdsArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const LdsClass& c = a.cls[blockIdx.z];
  const unsigned id = xcd_grouped(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int tile0 = (int)(id % gridDim.y) * MT;      // the channel tiles of one pixel block share an L2
  const unsigned q0 = (id / gridDim.y) * (unsigned)(32 * a.WN);
  if (q0 >= c.npix) return;  // uniform: a smaller parity class
  if constexpr (ALL) {
    conv_lds_body<MT, 9>(a, c, lds, tile0, q0);
  } else {
    const int nt = c.nr * c.nc;
    if (nt == 4) conv_lds_body<MT, 4>(a, c, lds, tile0, q0);
    else if (nt == 2) conv_lds_body<MT, 2>(a, c, lds, tile0, q0);
    else if (nt == 1) conv_lds_body<MT, 1>(a, c, lds, tile0, q0);
    else {
      const unsigned PHW = (unsigned)(c.PH * c.PW);
      for (unsigned i = threadIdx.x; i < 32u * a.WN * 32u * MT; i += blockDim.x) {
        const unsigned q = q0 + i % (32u * a.WN), m = tile0 * 32 + i / (32u * a.WN);
        if (q >= c.npix || m >= (unsigned)a.Mdim) continue;
        const unsigned n = q / PHW, p = q - n * PHW, r = p / (unsigned)c.PW;
        a.Y[((size_t)n * a.Mdim + m) * a.OH * a.OW + (size_t)(a.SO * r + c.oy) * a.OW + a.SO * (p - r * c.PW) + c.ox] = 0.f;
      }
    }
  }
}

// virtual rows that P consecutive pixels of a PH x PW class can need
int tile_rows(int P, int PH, int PW, int SI, int XH) {
  const int r = cdiv(P - 1, PW) + 1;
  return SI * (r - 1) + cdiv(r - 1, PH) * std::max(0, XH + 1 - SI * PH) + 3;
}
struct LdsPick { int MT, WN, WK, CH, rows, NP, PL; size_t lds; double cost; };

// The block shape with the least modelled time (cycles of the busiest SIMD): matrix cycles of the waves it is dealt,
// at least the latency of a chunk, plus staging and the reduction over WK.  Wide tiles read less per product; splitting the
// contraction is what fills the chip when there are few pixels.
bool search_product(const LdsArgs& a, int ncls, LdsPick& best) {
  best.cost = 1e30;
  const bool all = ncls == 1 && a.cls[0].nr * a.cls[0].nc == 9;
  for (int MT = 1; MT <= (a.Mdim > 32 ? 2 : 1); ++MT)
    for (int WK = 1; WK <= 16; WK *= 2)
      for (int WN = 1; WN * WK <= (MT == 2 && all ? 8 : 16) && WN <= 8; ++WN) {
        if (WK > 1 && WK > a.KG) continue;
        const int waves = WN * WK, P = 32 * WN;
        LdsPick p;
        p.MT = MT; p.WN = WN; p.WK = WK; p.CH = 8 * WK;
        p.rows = 0;
        for (int i = 0; i < ncls; ++i) p.rows = std::max(p.rows, tile_rows(P, a.cls[i].PH, a.cls[i].PW, a.SI, a.XH));
        p.NP = cdiv(p.rows * a.RW, 64);
        p.PL = p.NP * 64 + 32;
        p.lds = std::max((size_t)2 * p.CH * p.PL + p.NP * 64, WK > 1 ? (size_t)waves * 1024 : (size_t)0) * 4;
        if (p.lds > kProductLds) continue;
        double blocks = 0, mfma = 0;
        for (int i = 0; i < ncls; ++i) {
          if (a.cls[i].nr * a.cls[i].nc == 0) continue;  // zeros only
          const double b = (double)cdiv(a.cls[i].npix, P) * cdiv(a.Mdim, 32 * MT);
          blocks += b;
          mfma += b * a.cls[i].nr * a.cls[i].nc;  // taps, averaged over the blocks below
        }
        const double taps = mfma / blocks;
        const int nchunk = cdiv(a.KG, WK);
        const double per_cu = std::ceil(blocks / 256.0);
        const double simd_waves = std::ceil(per_cu * waves / 4.0);
        const double chunk_mfma = taps * 4 * MT * 64;
        // bytes through L2 per compute unit: staged pixels (with their halo) and weights
        const double traffic = per_cu * ((double)a.KG * 8 * p.NP * 256 + (double)MT * taps * a.KG * 1024);
        const double resident = std::min(std::floor(160.0 * 1024 / p.lds),
                                         std::max(1.0, std::floor((MT == 2 ? 12.0 : 16.0) / waves)));
        const double rounds = std::ceil(per_cu / resident);
        const double stage = 600 + (double)p.CH * p.NP / waves * 30.0;   // not hidden while a block is alone on its CU
        p.cost = simd_waves * nchunk * chunk_mfma + (per_cu > 1 ? 0.3 : 0.6) * rounds * nchunk * stage +
                 rounds * (4000 + (WK > 1 ? MT * (600.0 + WK * 60) : 0)) + simd_waves * nchunk * taps * 4 * 8 + traffic / 40;
        if (p.cost < best.cost) best = p;
      }
  return best.cost < 1e30;
}

// (the choice depends on the sizes alone: looked up after a thread's first call with them)
bool pick_product(const LdsArgs& a, int ncls, LdsPick& p) {
  static thread_local std::map<std::array<int, 9>, LdsPick> seen;
  const std::array<int, 9> key = {a.N, a.XH, a.XW, a.OH, a.OW, a.SI * 2 + a.SO, a.Kdim, a.Mdim, a.KS};
  auto it = seen.find(key);
  if (it == seen.end()) {
    LdsPick q;
    search_product(a, ncls, q);
    if (seen.size() >= 1024) seen.clear();
    it = seen.emplace(key, q).first;
  }
  p = it->second;
  return p.cost < 1e30;
}

template <int MT, bool ALL>
void launch_one(hipStream_t st, const char* name, const LdsArgs& a, const LdsPick& p, dim3 grid) {
  KLAUNCH_NAMED(name, (conv_lds_f32_kernel<MT, ALL>), grid, dim3(64 * p.WN * p.WK), p.lds, st, a);
}

// The sizes of a product and its classes of result pixels; false: the tensors are too large.
bool product_sizes(bool dgrad, int N, int Kdim, int Mdim, int H, int W, int KS, int S, LdsArgs& a, int& ncls) {
  const int pad = KS / 2, Ho = (H + 2 * pad - KS) / S + 1, Wo = (W + 2 * pad - KS) / S + 1;
  a = {};
  a.N = N; a.Kdim = Kdim; a.Mdim = Mdim; a.KG = cdiv(Kdim, 8); a.KS = KS;
  a.tap_stride = (unsigned)(pw_pack_floats(Mdim, Kdim) / 4);
  if (dgrad) { a.XH = Ho; a.XW = Wo; a.OH = H; a.OW = W; a.SI = 1; a.SO = S; }
  else { a.XH = H; a.XW = W; a.OH = Ho; a.OW = Wo; a.SI = S; a.SO = 1; }
  a.XS = 1; a.XRW = a.XW; a.XHW = (unsigned)(a.XH * a.XW);
  if ((size_t)N * (a.XH + 2) * (a.XH + 1) >= ((size_t)1 << 32)) return false;  // reciprocals
  if (!copies_reach(N, Kdim, a.XH, a.XW) || (size_t)a.tap_stride * KS * KS >= kOutside) return false;  // 32-bit offsets
  a.x_bytes = (unsigned)N * Kdim * a.XHW * 4u;
  if (!dgrad && KS == 1 && S > 1) {  // only the pixels a strided 1x1 conv reads: its operand is the subsampled tensor
    a.XH = Ho; a.XW = Wo; a.SI = 1; a.XS = S;
  }
  ncls = 0;
  auto code = [](int u, int d) { return (unsigned)((u << 4) | (d + 1)); };
  // row (or column) taps of a parity class: input row r = S*i + u - pad
  auto taps = [&](int par, unsigned& list) {
    int n = 0;
    list = 0;
    for (int u = 0; u < KS; ++u) {
      int d;
      if (!dgrad) d = u - pad;
      else if (S == 1) d = pad - u;
      else if ((par + pad - u) & 1) continue;
      else d = (par + pad - u) / 2;
      list |= code(u, d) << (8 * n++);
    }
    return n;
  };
  for (int pr = 0; pr < a.SO; ++pr)
    for (int pc = 0; pc < a.SO; ++pc) {
      LdsClass& c = a.cls[ncls];
      c.PH = (a.OH - pr + a.SO - 1) / a.SO;
      c.PW = (a.OW - pc + a.SO - 1) / a.SO;
      if (c.PH <= 0 || c.PW <= 0) continue;
      c.oy = pr; c.ox = pc;
      c.npix = (unsigned)N * c.PH * c.PW;
      c.nr = taps(pr, c.rows);
      c.nc = taps(pc, c.cols);
      ++ncls;
    }
  a.RW = a.XW + 2;
  a.rRW = reciprocal(a.RW); a.rXH1 = reciprocal(a.XH + 1);
  return true;
}
// ... and the block shape; false: no shape fits.
bool plan_product(bool dgrad, int N, int Kdim, int Mdim, int H, int W, int KS, int S, LdsArgs& a, int& ncls, LdsPick& p) {
  if (!product_sizes(dgrad, N, Kdim, Mdim, H, W, KS, S, a, ncls) || !pick_product(a, ncls, p)) return false;
  a.WN = p.WN; a.WK = p.WK; a.rows = p.rows; a.NP = p.NP; a.PL = p.PL; a.CH = p.CH;
  return true;
}

}  // namespace

// Y = conv of X (dgrad: gradient of a conv's input from its output gradient X).  H, W: the conv's INPUT size.
// false: the caller's direct kernel runs instead (very wide rows, operands of 2 GiB and more).
bool conv_lds_product(hipStream_t st, const char* name, bool dgrad, const float* Wp, const float* X, float* Y,
                      const float* bias, int N, int Kdim, int Mdim, int H, int W, int KS, int S) {
  LdsArgs a;
  LdsPick p;
  int ncls;
  if (!plan_product(dgrad, N, Kdim, Mdim, H, W, KS, S, a, ncls, p)) return false;
  a.Wp = reinterpret_cast<const float4*>(Wp);
  a.X = X; a.Y = Y; a.bias = bias;
  unsigned most = 0;
  for (int i = 0; i < ncls; ++i) most = std::max(most, a.cls[i].npix);
  const dim3 grid((unsigned)cdiv(most, 32 * p.WN), (unsigned)cdiv(Mdim, 32 * p.MT), (unsigned)ncls);
  const bool all = ncls == 1 && a.cls[0].nr * a.cls[0].nc == 9;
  if (p.MT == 2) all ? launch_one<2, true>(st, name, a, p, grid) : launch_one<2, false>(st, name, a, p, grid);
  else all ? launch_one<1, true>(st, name, a, p, grid) : launch_one<1, false>(st, name, a, p, grid);
  return true;
}

// ------------------------------------------------------------------ product on the bf16 matrix cores
namespace {

// The same product with its operands split in three (kernels_f32_x3.h).  Pixels are split once per block on their way to
// LDS, where eight channels of a staged position lie together, three planes of 16-byte words [piece][group of 8][position]:
// a tap of 32 pixels and 16 channels is three aligned 16-byte reads per lane, conflict-free (positions of neighbouring pixels
// are neighbours).  They travel through registers, loaded between the taps of the chunk before and split at its end.
//
// Block: WM row tiles x WN groups of 32 * NT pixels x WK shares of the contraction, one wavefront each.  A wavefront's weights
// (3 KB per tap and group) come from L2 and are its largest stream: 64 bytes per clock and compute unit with NT = 1 at the full
// matrix rate, 32 with 2.  They are requested up to three taps ahead (two with NT = 4).
//
// What bounds it is that the reads of a wavefront and its products take turns: 256 -> 256 at 8 x 14x14 spends 28 % of its cycles in
// products, 35 % in vector memory and 27 % in LDS, and takes their sum, with eight wavefronts on a compute unit as with
// sixteen.  So the reads of the next 32 pixels and of the weights to come stand between the six products of these (behind
// them in one go: 21.5 us where this takes 20.4; 64 -> 64 at 32 x 56x56 54.9 / 52.4, 128 -> 128 at 4 x 28x28 14.9 / 14.2).
//
// The blocks of an XCD that share weights run through them side by side, so every line would be waited for once by all of
// them, with no more in flight than one of them asks for.  At its start each block reads a word of each line of a share of
// them: 256 -> 256 at 8 x 14x14 in a pass over ResNet50 21.6 / 20.1 us, its strided products 42.7 / 37.8.
struct X3Shape { int NT, NI, WM, WN, WK, rows, NP; size_t lds; double cost; };
struct X3Args {
  LdsArgs p;
  int WM;
  unsigned shares;  // blocks of an XCD that read the same weights
};

// acc += a wavefront's share (groups g0, g0 + gstep, ...) for one row tile and pixel (n, i, j) of each lane, on the fp32
// matrix instructions (kernels_f32_x3.h: where the pieces gave no finite sum).  As above, what lies outside the image is 0.
__device__ __forceinline__ void x3_contract_f32(const LdsArgs& a, const LdsClass& c, unsigned n, int i, int j, bool valid,
                                                const uint4* wl, int g0, int gstep, floatx16& acc) {
  const int half = threadIdx.x >> 5 & 1;
#pragma unroll 1
  for (int t = 0; t < c.nr * c.nc; ++t) {
    const unsigned rc = c.rows >> (8 * (t / c.nc)), cc = c.cols >> (8 * (t % c.nc));
    const int h = a.SI * i + (int)(rc & 15) - 1, x = a.SI * j + (int)(cc & 15) - 1;
    const bool in = valid && h >= 0 && h < a.XH && x >= 0 && x < a.XW;
    const float* const xp = in ? a.X + ((size_t)n * a.Kdim + 8 * half) * a.XHW + (size_t)(h * a.XRW + x) * a.XS : a.X;
    const uint4* const w = wl + (size_t)((rc >> 4 & 15) * a.KS + (cc >> 4 & 15)) * a.tap_stride;
#pragma unroll 1
    for (int g = g0; g < a.KG; g += gstep) {
      uint4 p[3];
      float wv[8], xv[8];
#pragma unroll
      for (int e = 0; e < 3; ++e) p[e] = w[(size_t)g * 192 + e * 64];
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = in ? xp[(size_t)(g * 16 + e) * a.XHW] : 0.f;  // (Kdim % 16 == 0)
      join3(p, wv);
      acc = mfma_f32(wv, xv, acc);
    }
  }
}

template <int NT, int TAPS, int NI>
__device__ __forceinline__ void conv_x3_body(const X3Args& xa, const LdsClass& c, char* lds, int tile0, unsigned q0,
                                             unsigned share) {
  const LdsArgs& a = xa.p;
  const int tid = threadIdx.x, lane = tid & 63, T = blockDim.x, waves = T >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
  const int col = lane & 31, half = lane >> 5;
  const int WM = xa.WM, WN = a.WN, WK = a.WK, wm = wave % WM, wr = wave / WM, wn = wr % WN, wk = wr / WN;
  const int XH1 = a.XH + 1, RW = a.RW, KG = a.KG, NP = a.NP;
  const unsigned PHW = (unsigned)(c.PH * c.PW);
  const unsigned n0 = q0 / PHW;
  const int vr0 = (int)n0 * XH1 + a.SI * (int)((q0 - n0 * PHW) / (unsigned)c.PW);
  const int G8 = 2 * WK, PL = NP * 16, PS = G8 * PL, BS = 3 * PS;  // bytes of a group, a piece and a chunk
  const int tile = tile0 + wm;
  const bool live = tile * 32 < a.Mdim;  // uniform per wavefront

  // staging: item i of a thread is a group of eight channels of one position
  const __amdgpu_buffer_rsrc_t rx = rsrc_of(a.X, a.x_bytes);
  unsigned voff[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int u = tid + i * T, g8 = u / NP, pos = u - g8 * NP;
    const unsigned v = virtual_offset(pos, vr0, a.rows, a.rRW, a.rXH1, a.N, a.XH, a.XW, a.XRW, a.XS, (unsigned)a.Kdim * a.XHW);
    voff[i] = g8 < G8 && v != kOutside ? v + (unsigned)(g8 * 8) * a.XHW * 4u : kOutside;
  }
  float xr[NI][8];
  auto fetch = [&](int i, int ch, int j0, int j1) __attribute__((always_inline)) {
    const unsigned k0 = (unsigned)(ch * 16 * WK);
    unsigned vo = voff[i];
    if ((ch + 1) * WK > KG) vo = k0 + (unsigned)((tid + i * T) / NP * 8) < (unsigned)a.Kdim ? vo : kOutside;  // uniform: a short chunk
#pragma unroll
    for (int j = j0; j < j1; ++j)
      xr[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, vo, (k0 + j) * a.XHW * 4u, 0));
  };
  auto put = [&](int i, int buf) __attribute__((always_inline)) {
    uint4 p[3];
    split3(xr[i], p);
    const int u = tid + i * T;
    if (u < G8 * NP) {
      char* const d = lds + buf * BS + u * 16;
      *reinterpret_cast<uint4*>(d) = p[0];
      *reinterpret_cast<uint4*>(d + PS) = p[1];
      *reinterpret_cast<uint4*>(d + 2 * PS) = p[2];
    }
  };

  // the pixels of the wavefront: position of tap (0, 0) in LDS
  unsigned qn[NT];
  int qi[NT], qj[NT];
  bool qv[NT];
  const char* bl[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const unsigned q = q0 + (wn * NT + n) * 32 + col;
    qv[n] = q < c.npix;
    const unsigned qc = qv[n] ? q : c.npix - 1;
    qn[n] = qc / PHW;
    const int qp = (int)(qc - qn[n] * PHW);
    qi[n] = qp / c.PW;
    qj[n] = qp - qi[n] * c.PW;
    bl[n] = lds + (2 * wk + half) * PL + (((int)qn[n] * XH1 + a.SI * qi[n] - vr0) * RW + a.SI * qj[n]) * 16;
  }
  unsigned woff[TAPS];  // tap t: offset of its weight copy, and of its shift in LDS (uniform)
  int boff[TAPS];
#pragma unroll
  for (int t = 0; t < TAPS; ++t) {
    const int ri = t / c.nc, ci = t - ri * c.nc;
    const unsigned rc = c.rows >> (8 * ri), cc = c.cols >> (8 * ci);
    woff[t] = ((rc >> 4 & 15) * (unsigned)a.KS + (cc >> 4 & 15)) * a.tap_stride;
    boff[t] = ((int)(rc & 15) * RW + (int)(cc & 15)) * 16;
  }
  constexpr int RING = TAPS == 9 ? 3 : TAPS;  // taps whose weights are in registers (9 of 9: 3 % slower), a divisor of TAPS
  constexpr int AHEAD = RING == 3 && NT == 4 ? 2 : RING;  // (NT = 4 takes all registers: 64 -> 64 at 32 x 56x56 49 us, 3 ahead 54 to 57)
  const uint4* const wl = reinterpret_cast<const uint4*>(a.Wp) + (size_t)min(tile, (a.Mdim - 1) / 32) * KG * 192 + lane;
  uint4 A[RING][3];
  auto ldA = [&](int t, int ch, int p) __attribute__((always_inline)) {
    A[t % RING][p] = wl[woff[t] + (unsigned)min(ch * WK + wk, KG - 1) * 192u + p * 64u];
  };
  floatx16 acc[NT], acs[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[n][r] = acs[n][r] = 0.f;
  uint4 xb[2][3];  // pixel operands of a step (tap, group of 32 pixels), and of the next
  auto rdX = [&](int step, int buf, int p) __attribute__((always_inline)) {
    xb[step & 1][p] = *reinterpret_cast<const uint4*>(bl[step % NT] + boff[step / NT] + buf * BS + p * PS);
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (loads to registers stay in flight)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
#pragma unroll
  for (int i = 0; i < NI; ++i) fetch(i, 0, 0, 8);
#pragma unroll
  for (int t = 0; t < AHEAD; ++t)
#pragma unroll
    for (int p = 0; p < 3; ++p) ldA(t, 0, p);
  constexpr int NW = 2;
  uint32_t warm[NW];
  {  // the block's share of its row tiles' weights, one word of each line of 128 bytes
    const unsigned per = (unsigned)min(WM, a.Mdim / 32 - tile0) * KG * 24u, lines = per * TAPS;
    const char* const w0 = reinterpret_cast<const char*>(a.Wp) + (size_t)tile0 * KG * 3072;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const unsigned l = (k * xa.shares + share) * T + tid;
      warm[k] = 0;
      if (l < lines) {
        const unsigned t = l / per;
        const unsigned rc = c.rows >> (8 * (t / c.nc)), cc = c.cols >> (8 * (t % c.nc));
        const size_t tap = ((rc >> 4 & 15) * (unsigned)a.KS + (cc >> 4 & 15)) * a.tap_stride;
        warm[k] = *reinterpret_cast<const uint32_t*>(w0 + tap * 16 + (size_t)(l - t * per) * 128);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) put(i, 0);
  barrier();
  const int nchunk = (KG + WK - 1) / WK;
  constexpr int PER = (NI + TAPS - 1) / TAPS;  // items requested per tap
  auto chunk = [&](int ch, auto more_c) __attribute__((always_inline)) {
    constexpr bool more = decltype(more_c)::value;
    const int buf = ch & 1;
    if (more || ch * WK + wk < KG) {  // uniform per wavefront; only the last chunk can be short
#pragma unroll
      for (int p = 0; p < 3; ++p) rdX(0, buf, p);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < TAPS * NT; ++s) {
        const int t = s / NT, n = s % NT;
        const uint4(&w)[3] = A[t % RING];
        const uint4(&x)[3] = xb[s & 1];
        auto weights = [&](int p) __attribute__((always_inline)) {
          if (t + AHEAD < TAPS) ldA(t + AHEAD, ch, p);
          else if constexpr (more) ldA(t + AHEAD - TAPS, ch + 1, p);
        };
        auto beside = [&](int k) __attribute__((always_inline)) {  // behind the k-th product
          if (k < 3 && s + 1 < TAPS * NT) rdX(s + 1, buf, k);
          if (AHEAD < RING) {
            if (n == 0 && k < 3) weights(2 - k);
          } else if (n == NT - 1) {
            if (k == 0) weights(2);
            if (k == 2) weights(1);
            if (k == 5) weights(0);
          }
          if constexpr (more) {
            if (n == NT - 1 && (k == 3 || k == 4))
#pragma unroll
              for (int i = t * PER; i < (t + 1) * PER; ++i)
                if (i < NI) fetch(i, ch + 1, k == 3 ? 0 : 4, k == 3 ? 4 : 8);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        acs[n] = mfma_bf16(w[2], x[0], acs[n]);
        beside(0);
        acs[n] = mfma_bf16(w[1], x[0], acs[n]);
        beside(1);
        acs[n] = mfma_bf16(w[1], x[1], acs[n]);
        beside(2);
        acc[n] = mfma_bf16(w[0], x[0], acc[n]);
        beside(3);
        acs[n] = mfma_bf16(w[0], x[1], acs[n]);
        beside(4);
        acs[n] = mfma_bf16(w[0], x[2], acs[n]);
        beside(5);
      }
    }
    if constexpr (more) {
#pragma unroll
      for (int i = 0; i < NI; ++i) put(i, buf ^ 1);
      barrier();
    }
  };
  for (int ch = 0; ch + 1 < nchunk; ++ch) chunk(ch, std::true_type{});
  chunk(nchunk - 1, std::false_type{});
#pragma unroll
  for (int k = 0; k < NW; ++k) asm volatile("" ::"v"(warm[k]));  // (their only use)

  const size_t OHW = (size_t)a.OH * a.OW;
  auto row = [&](int r) { return tile * 32 + 8 * (r >> 2) + 4 * half + (r & 3); };
  auto at = [&](int n) {
    return a.Y + (size_t)qn[n] * a.Mdim * OHW + (size_t)(a.SO * qi[n] + c.oy) * a.OW + a.SO * qj[n] + c.ox;
  };
  // the sums of pixel group n that are not finite, over the wavefront's share of the contraction
  auto again = [&](int n, unsigned& sn, int& si, int& sj, bool& in) __attribute__((always_inline)) {
    const unsigned q = q0 + (wn * NT + n) * 32 + col, qc = min(q, c.npix - 1);
    sn = qc / PHW;
    si = (int)((qc - sn * PHW) / (unsigned)c.PW);
    sj = (int)(qc - sn * PHW) - si * c.PW;
    in = q < c.npix;
    floatx16 v = zero16();
    x3_contract_f32(a, c, sn, si, sj, in, wl, wk, WK, v);
    return v;
  };
  if (NT == 4 || WK == 1) {  // (NT = 4 never splits the contraction: x3_shape)
    if (!live) return;
    float bad = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      float* const yq = at(n);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float v = acc[n][r] + acs[n][r];
        bad = fmaf(v, 0.f, bad);
        if (qv[n]) yq[(size_t)row(r) * OHW] = v + (a.bias ? a.bias[row(r)] : 0.f);  // (Mdim % 32 == 0)
      }
    }
    if (any_not_finite(bad)) {  // over what was stored
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
      for (int n = 0; n < NT; ++n) {
        unsigned sn;
        int si, sj;
        bool in;
        const floatx16 v = again(n, sn, si, sj, in);
        float* const yq = a.Y + (size_t)sn * a.Mdim * OHW + (size_t)(a.SO * si + c.oy) * a.OW + a.SO * sj + c.ox;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (in && !finite_f(yq[(size_t)row(r) * OHW])) yq[(size_t)row(r) * OHW] = v[r] + (a.bias ? a.bias[row(r)] : 0.f);
      }
    }
    return;
  }
  float bad = 0.f;
#pragma unroll
  for (int n = 0; n < NT; ++n) bad = add_small(acc[n], acs[n], bad);
  if (any_not_finite(bad)) {
#pragma unroll 1
    for (int n = 0; n < NT; ++n) {
      unsigned sn;
      int si, sj;
      bool in;
      const floatx16 v = again(n, sn, si, sj, in);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        if (n == j) take_not_finite(acc[j], v);
    }
  }
  float* const red = reinterpret_cast<float*>(lds);
  const int rpw = 16 / WK;  // accumulator rows that each of the WK wavefronts finishes
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    __syncthreads();  // the partial tiles overwrite the staged pixels, and then each other
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[n][r];
    __syncthreads();
    for (int rr = 0; rr < rpw; ++rr) {
      const int r = wk * rpw + rr;
      float v = 0.f;
      for (int k = 0; k < WK; k += 2)  // fixed order
        v += red[(((k * WN + wn) * WM + wm) * 16 + r) * 64 + lane] + red[((((k + 1) * WN + wn) * WM + wm) * 16 + r) * 64 + lane];
      if (!qv[n] || !live) continue;
      at(n)[(size_t)row(r) * OHW] = v + (a.bias ? a.bias[row(r)] : 0.f);
    }
  }
}

// ALL: one class reached by all nine taps; else the class decides (1, 2 or 4 taps, or none: zeros)
template <int NT, bool ALL, int NI>
__global__ __launch_bounds__(512, 2) void conv_x3_f32_kernel(X3Args xa) {
  extern __shared__ __attribute__((aligned(16))) char xlds[];
  const LdsArgs& a = xa.p;
  const LdsClass& c = a.cls[blockIdx.z];
  const unsigned id = xcd_grouped(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  // the row tiles of one pixel block share an L2, or the pixel blocks of one row tile (the larger operand)
  const unsigned d = a.CH ? gridDim.y : gridDim.x, hi = id / d, lo = id - hi * d;
  const int tile0 = __builtin_amdgcn_readfirstlane((int)(a.CH ? lo : hi)) * xa.WM;
  const unsigned q0 = __builtin_amdgcn_readfirstlane(a.CH ? hi : lo) * (unsigned)(32 * NT * a.WN);
  if (q0 >= c.npix) return;  // uniform: a smaller parity class
  const unsigned share = (a.CH ? hi : lo) % xa.shares;
  if constexpr (ALL) {
    conv_x3_body<NT, 9, NI>(xa, c, xlds, tile0, q0, share);
  } else {
    const int nt = c.nr * c.nc;
    if (nt == 4) conv_x3_body<NT, 4, NI>(xa, c, xlds, tile0, q0, share);
    else if (nt == 2) conv_x3_body<NT, 2, NI>(xa, c, xlds, tile0, q0, share);
    else if (nt == 1) conv_x3_body<NT, 1, NI>(xa, c, xlds, tile0, q0, share);
    else {
      const unsigned PHW = (unsigned)(c.PH * c.PW), P = 32 * NT * a.WN;
      for (unsigned i = threadIdx.x; i < P * 32u * xa.WM; i += blockDim.x) {
        const unsigned q = q0 + i % P, m = tile0 * 32 + i / P;
        if (q >= c.npix || m >= (unsigned)a.Mdim) continue;
        const unsigned n = q / PHW, p = q - n * PHW, r = p / (unsigned)c.PW;
        a.Y[((size_t)n * a.Mdim + m) * a.OH * a.OW + (size_t)(a.SO * r + c.oy) * a.OW + a.SO * (p - r * c.PW) + c.ox] = 0.f;
      }
    }
  }
}
constexpr size_t kX3Lds = 156 * 1024;

bool x3_shape(const LdsArgs& a, int ncls, int NT, int WM, int WN, int WK, X3Shape& p) {
  const int waves = WM * WN * WK, P = 32 * NT * WN;
  if (waves > 8 || waves < 2 || (WK > 1 && (WK > a.KG || NT == 4)) || WM > a.Mdim / 32) return false;
  p.NT = NT; p.WM = WM; p.WN = WN; p.WK = WK;
  p.rows = 0;
  for (int i = 0; i < ncls; ++i) p.rows = std::max(p.rows, tile_rows(P, a.cls[i].PH, a.cls[i].PW, a.SI, a.XH));
  p.NP = (p.rows * a.RW + 15) & ~15;
  p.NI = cdiv(2 * WK * p.NP, 64 * waves);
  p.lds = std::max((size_t)2 * 96 * WK * p.NP, WK > 1 ? (size_t)waves * 4096 : (size_t)0);
  return p.NI <= 4 && p.lds <= kX3Lds;
}

template <int NT, int NI>
void launch_x3(hipStream_t st, const char* name, const X3Args& a, const X3Shape& p, dim3 grid, bool all) {
  const dim3 block(64 * p.WM * p.WN * p.WK);
  if (all) KLAUNCH_NAMED(name, (conv_x3_f32_kernel<NT, true, NI>), grid, block, p.lds, st, a);
  else KLAUNCH_NAMED(name, (conv_x3_f32_kernel<NT, false, NI>), grid, block, p.lds, st, a);
}
template <int NT>
void launch_x3(hipStream_t st, const char* name, const X3Args& a, const X3Shape& p, dim3 grid, bool all) {
  switch (p.NI) {
    case 1: launch_x3<NT, 1>(st, name, a, p, grid, all); break;
    case 2: launch_x3<NT, 2>(st, name, a, p, grid, all); break;
    case 3: launch_x3<NT, 3>(st, name, a, p, grid, all); break;
    default: launch_x3<NT, 4>(st, name, a, p, grid, all); break;
  }
}
void run_x3(hipStream_t st, const char* name, const LdsArgs& sizes, int ncls, const X3Shape& p, const float* Wp, const float* X,
            float* Y, const float* bias) {
  X3Args a;
  a.p = sizes;
  a.p.Wp = reinterpret_cast<const float4*>(Wp);
  a.p.X = X; a.p.Y = Y; a.p.bias = bias;
  a.p.KG = cdiv(sizes.Kdim, 16);
  a.p.tap_stride = (unsigned)(x3_pack_floats(sizes.Mdim, sizes.Kdim) / 4);
  a.p.WN = p.WN; a.p.WK = p.WK; a.p.rows = p.rows; a.p.NP = p.NP;
  a.WM = p.WM;
  unsigned most = 0;
  for (int i = 0; i < ncls; ++i) most = std::max(most, a.p.cls[i].npix);
  // (6 bytes a weight)
  a.p.CH = (size_t)sizes.Mdim * sizes.KS * sizes.KS * 3 < (size_t)sizes.N * sizes.XH * sizes.XW * 2;
  const dim3 grid((unsigned)cdiv(most, 32 * p.NT * p.WN), (unsigned)cdiv(sizes.Mdim / 32, p.WM), (unsigned)ncls);
  // (grid.x * grid.y / 8: the blocks of an XCD)
  const unsigned here = std::max(1u, grid.x * grid.y / 8);
  a.shares = std::max(1u, std::min(grid.x, a.p.CH ? here / grid.y : here));
  const bool all = ncls == 1 && a.p.cls[0].nr * a.p.cls[0].nc == 9;
  if (p.NT == 1) launch_x3<1>(st, name, a, p, grid, all);
  else if (p.NT == 2) launch_x3<2>(st, name, a, p, grid, all);
  else launch_x3<4>(st, name, a, p, grid, all);
}

// The block shape: enough shares of the contraction for two wavefronts per SIMD, up to four row tiles per block (more pixels
// instead only where there are fewer), and more pixels per wavefront where there is plenty of work; of the shapes that fit, the
// nearest.
// Measured at ResNet50's layers (us, fp32 matrix instructions / best shape / this one's neighbours): 64 -> 64 at 32 x 56x56 104 /
// 52 (4 pixel groups) / 57 (2) / 57 (1); 128 -> 128 at 8 x 28x28 32.5 / 19.8 (2 shares, 4 row tiles) / 20.1 (2 row tiles); 256 ->
// 256 at 8 x 14x14 33.2 / 20.4 (4 shares) / 21.1 (2); 512 -> 512 at 8 x 7x7 36.8 / 22.6 (8 shares) / 24.0 (4).
bool search_x3(const LdsArgs& sizes, int ncls, X3Shape& best) {
  LdsArgs a = sizes;
  a.KG = cdiv(sizes.Kdim, 16);
  const int mt = sizes.Mdim / 32;
  long tiles = 0;
  for (int i = 0; i < ncls; ++i) tiles += sizes.cls[i].nr * sizes.cls[i].nc ? (long)cdiv(sizes.cls[i].npix, 32) * mt : 0;
  const bool all = ncls == 1 && sizes.cls[0].nr * sizes.cls[0].nc == 9;
  int wk = 1;
  while (wk < 8 && wk * tiles < (all && a.KG >= 16 * wk ? 2000 : 1200) && wk * 2 <= std::max(1, a.KG / 2)) wk *= 2;
  const int wm = std::min(mt, std::max(1, std::min(4, 8 / wk)));
  // Four row tiles: every wavefront reads weights of its own, so two groups of pixels share each read where that takes fewer rounds
  // of blocks.  Four wavefronts with one group run three to a compute unit, eight wavefronts one; a round with two groups
  // takes 1.1 times a round with one, beside two shares of the contraction 1.4 to 1.5 times.  us, one group / two: 128 -> 128 at
  // 32 x 28x28 (two rounds, one) 57.7 / 49; 256 -> 256 at 32 x 14x14, two shares, 58.7 / 50.2; 64 -> 256 at 13 x 36x36 (two
  // rounds each, the second of the 264 blocks of two groups nearly empty) 38.5 / 51.4; 128 -> 128 at 16 x 28x28 (one each) 32 / 44.
  const bool one = sizes.KS == 1 && ncls == 1;
  auto rounds = [&](int NT) {  // of the whole chip (three times 256, full to a hundredth: the next size has a second round)
    const int wn = wk == 1 ? NT : 1;
    const long blocks = (long)cdiv(sizes.cls[0].npix, 32 * NT * wn) * cdiv(mt, 4);
    return cdiv(blocks, wk * wn == 1 ? 760 : 256);
  };
  const bool two = all && wm == 4 && wk * tiles >= 3000 && rounds(1) > (wk == 1 ? 1.1 : 1.5) * rounds(2);
  const int nt = all && tiles >= 6000 ? 4 : two || (tiles >= 3000 && one) ? 2 : 1;
  const int wn = wk == 1 && (wm < 4 || (all && nt == 2) || (!all && sizes.KS == 3)) ? 8 / wm : 1;
  best.cost = 1e30;
  for (int NT = 1; NT <= 4; NT *= 2)
    for (int WM = 1; WM <= 8; ++WM)
      for (int WN = 1; WN <= 8; WN *= 2)
        for (int WK = 1; WK <= 8; WK *= 2) {
          X3Shape p;
          if (!x3_shape(a, ncls, NT, WM, WN, WK, p)) continue;
          p.cost = 3 * std::fabs(std::log2((double)WK / wk)) + 2 * std::fabs(std::log2((double)NT / nt)) +
                   std::fabs(std::log2((double)WM / wm)) + 1.1 * std::fabs(std::log2((double)WN / wn));
          if (p.cost < best.cost) best = p;
        }
  return best.cost < 1e30;
}
// The sizes that this product takes; other channel counts leave its tiles partly empty and stay with the kernels above.
bool plan_x3(bool dgrad, int N, int Kdim, int Mdim, int H, int W, int KS, int S, LdsArgs& a, int& ncls, X3Shape& p) {
  if (Kdim % 16 || Mdim % 32 || !product_sizes(dgrad, N, Kdim, Mdim, H, W, KS, S, a, ncls)) return false;
  if ((x3_pack_floats(Mdim, Kdim) / 4) * KS * KS >= kOutside) return false;
  static thread_local std::map<std::array<int, 9>, X3Shape> seen;  // (the choice depends on the sizes alone)
  const std::array<int, 9> key = {dgrad, N, Kdim, Mdim, H, W, KS, S, 0};
  auto it = seen.find(key);
  if (it == seen.end()) {
    X3Shape q;
    search_x3(a, ncls, q);
    if (seen.size() >= 1024) seen.clear();
    it = seen.emplace(key, q).first;
  }
  p = it->second;
  return p.cost < 1e30;
}
}  // namespace

bool conv_x3_takes(bool dgrad, int N, int Kdim, int Mdim, int H, int W, int KS, int S) {
  LdsArgs a;
  X3Shape p;
  int ncls;
  return plan_x3(dgrad, N, Kdim, Mdim, H, W, KS, S, a, ncls, p);
}
bool conv_x3_product(hipStream_t st, const char* name, bool dgrad, const float* Wp, const float* X, float* Y,
                     const float* bias, int N, int Kdim, int Mdim, int H, int W, int KS, int S) {
  LdsArgs a;
  X3Shape p;
  int ncls;
  if (!plan_x3(dgrad, N, Kdim, Mdim, H, W, KS, S, a, ncls, p)) return false;
  run_x3(st, name, a, ncls, p, Wp, X, Y, bias);
  return true;
}

// ------------------------------------------------------------------ weight gradient
namespace {

struct LdsWgArgs {
  const float* g;   // [N][Cout][Ho][Wo]
  const float* x;   // [N][Cin][H][W], or every XS-th row and column of a larger one
  float* part;      // [chunk][Cout][Cin][KS*KS]
  int N, Cin, Cout, H, W, Ho, Wo, S, XS, XRW;
  unsigned XHW, x_bytes, g_bytes;
  int rows, RW, NP, PT, per, nstage, nbuf, flush;
  unsigned rRW, rH1, rWo;
  unsigned npix;
};

constexpr int kFlush = 8 * 16 * 64;  // words: one 32 x 32 tile of eight wavefronts

// Strided convolutions, and rows of 128 columns and more (the others: kernels_f32_conv_wg.hip).
// Block of eight wavefronts, one per compute unit: a 32 x 32 tile of (cout, cin), all taps (1x1: 64 x 64), over a run of
// stages of PT consecutive output pixels, whatever samples they lie in.  A stage copies g [32][PT] and the virtual rows of x
// under it to LDS with coalesced loads (lanes along the pixels: a load per lane and channel row would touch 64 cache
// lines instead of 2 to 4) while the stage before is multiplied; the products read one word of g and one of x per
// tap for a pair of pixels.  Wavefront w takes the w-th eighth of every stage's pixels; every `flush` stages the eight
// tiles are added through LDS into totals, two rows of the tile in registers of each wavefront, which leave as whole rows
// of the partial.  Pitches are 2 modulo 64: the 32 channel rows and the two neighbouring pixels of a pair hit 64 different
// banks.
template <int KS>
__global__ __launch_bounds__(512) void conv_lds_wgrad_f32_kernel(LdsWgArgs w) {
  constexpr int KK = KS * KS, TI = KS == 1 ? 2 : 1, TJ = TI, NA = KK * TI * TJ;  // 32 x 32 tiles of (cout, cin)
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
  const int PT = w.PT, PG = round_up64(PT) + 2, PL = w.NP * 64 + 2, RW = w.RW, H1 = w.H + 1, HWo = w.Ho * w.Wo;
  // a stage: g [32*TI][PG], x [32*TJ][PL], [PT] position of an output pixel's tap (0, 0)
  const int XO = 32 * TI * PG, TO = XO + 32 * TJ * PL, bufsz = TO + PT;
  const unsigned tiles_ci = (unsigned)(w.Cin + 32 * TJ - 1) / (32 * TJ);
  const unsigned tiles = tiles_ci * (unsigned)((w.Cout + 32 * TI - 1) / (32 * TI));
  const unsigned id = xcd_grouped(blockIdx.x, gridDim.x);
  const int chunk = (int)(id / tiles), tile = (int)(id % tiles);
  const int ci_base = (tile % (int)tiles_ci) * 32 * TJ, co_base = (tile / (int)tiles_ci) * 32 * TI;
  const __amdgpu_buffer_rsrc_t rx = rsrc_of(w.x, w.x_bytes), rg = rsrc_of(w.g, w.g_bytes);
  floatx16 acc[NA];
#pragma unroll
  for (int t = 0; t < NA; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
  float tot[NA][2] = {};
  int left = w.flush;
  const int s_begin = chunk * w.per, s_end = min(s_begin + w.per, w.nstage);
  auto stage = [&](int s, float* buf) __attribute__((always_inline)) {
    const unsigned q0 = (unsigned)s * PT;
    const unsigned n0 = q0 / (unsigned)HWo;
    const int vr0 = (int)n0 * H1 + w.S * (int)((q0 - n0 * (unsigned)HWo) / (unsigned)w.Wo);
    for (int p0 = 0; p0 < PT; p0 += 64) {  // a pixel past the last one: zeros (its x words then do not matter)
      const unsigned q = q0 + p0 + lane, qc = min(q, w.npix - 1), n = qc / (unsigned)HWo;
      const int p = (int)(qc - n * (unsigned)HWo);
      const unsigned voff = (q < w.npix && p0 + lane < PT) ? (n * (unsigned)(w.Cout * HWo) + (unsigned)p) * 4u : kOutside;
#pragma unroll
      for (int k = 0; k < 4 * TI; ++k) {
        const int c = wave + 8 * k;
        copy_to_lds(rg, buf + c * PG + p0, voff, (unsigned)min(co_base + c, w.Cout - 1) * (unsigned)HWo * 4u);
      }
      if (wave == 0 && p0 + lane < PT) {
        const int i = w.rWo ? (int)__umulhi((unsigned)p, w.rWo) : p, j = p - i * w.Wo;
        reinterpret_cast<int*>(buf + TO)[p0 + lane] = ((int)n * H1 + w.S * i - vr0) * RW + w.S * j;
      }
    }
    for (int i = 0; i < w.NP; ++i) {
      const unsigned voff = virtual_offset(i * 64 + lane, vr0, w.rows, w.rRW, w.rH1, w.N, w.H, w.W, w.XRW, w.XS,
                                           (unsigned)w.Cin * w.XHW);
#pragma unroll
      for (int k = 0; k < 4 * TJ; ++k) {
        const int c = wave + 8 * k;
        copy_to_lds(rx, buf + XO + c * PL + i * 64, voff, (unsigned)min(ci_base + c, w.Cin - 1) * w.XHW * 4u);
      }
    }
  };
  stage(s_begin, lds);
  __syncthreads();  // (waits for the copies)
  for (int s = s_begin; s < s_end; ++s) {
    const float* buf = lds + (w.nbuf == 2 ? ((s - s_begin) & 1) * bufsz : 0);
    if (w.nbuf == 2 && s + 1 < s_end) stage(s + 1, lds + ((s + 1 - s_begin) & 1) * bufsz);
    const int p0 = wave * (PT / 8) + half;
    const float* ga = buf + row * PG + p0;
    const int* ta = reinterpret_cast<const int*>(buf + TO) + p0;
    const float* xa = buf + XO + row * PL;
    float av[2][TI], b[2][KK * TJ];
    const int ks = PT / 16;  // pairs of pixels per wavefront: even
    int pos = ta[0];         // one pair ahead of its use
    auto ld = [&](int k, float (&a)[TI], float (&bb)[KK * TJ]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TI; ++i) a[i] = ga[2 * k + i * 32 * PG];
      const float* xb = xa + pos;
      pos = ta[2 * min(k + 1, ks - 1)];
#pragma unroll
      for (int t = 0; t < KK * TJ; ++t) bb[t] = KS == 1 ? xb[RW + 1 + t * 32 * PL] : xb[(t / 3) * RW + t % 3];
    };
    auto mma = [&](const float (&a)[TI], const float (&bb)[KK * TJ]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int t = 0; t < KK * TJ; ++t)
          acc[i * KK * TJ + t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], bb[t], acc[i * KK * TJ + t], 0, 0, 0);
    };
    ld(0, av[0], b[0]);
    // Operands one pair ahead of the products.  The scheduler, left alone, moves the reads of a pair behind the
    // products that should cover them; and a conditional last read costs register copies that wait for it.
    for (int k = 0; k < ks; k += 2) {
      ld(k + 1, av[1], b[1]);
      __builtin_amdgcn_sched_barrier(0);
      mma(av[0], b[0]);
      __builtin_amdgcn_sched_barrier(0);
      ld(min(k + 2, ks - 1), av[0], b[0]);  // (the last one is not used)
      __builtin_amdgcn_sched_barrier(0);
      mma(av[1], b[1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // the sums of the stages since the last time, from the accumulators of eight wavefronts to `tot`; taps go through two
    // scratch areas in turn, [8 wavefronts][8 pairs of rows][64 lanes] each
    if (--left == 0 || s + 1 == s_end) {  // uniform
      left = w.flush;
      float2* const own = reinterpret_cast<float2*>(lds + (buf - lds));  // the stage just multiplied
      float2* const past = reinterpret_cast<float2*>(lds + w.nbuf * bufsz);
      float2* const f0 = bufsz >= kFlush ? own : past;
      float2* const f1 = bufsz >= 2 * kFlush ? own + kFlush / 2 : bufsz >= kFlush ? past : past + kFlush / 2;
      auto give = [&](int t) __attribute__((always_inline)) {
        float2* const f = (t & 1 ? f1 : f0) + wave * 512 + lane;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          f[r * 64] = make_float2(acc[t][2 * r], acc[t][2 * r + 1]);
          acc[t][2 * r] = acc[t][2 * r + 1] = 0.f;
        }
      };
      give(0);
#pragma unroll
      for (int t = 0; t < NA; ++t) {
        __syncthreads();
        const float2* const f = (t & 1 ? f1 : f0) + wave * 64 + lane;
        float2 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = f[k * 512];
        if (t + 1 < NA) give(t + 1);
        tot[t][0] = (float)(tot[t][0] + ((((double)v[0].x + v[1].x) + ((double)v[2].x + v[3].x)) +
                                         (((double)v[4].x + v[5].x) + ((double)v[6].x + v[7].x))));
        tot[t][1] = (float)(tot[t][1] + ((((double)v[0].y + v[1].y) + ((double)v[2].y + v[3].y)) +
                                         (((double)v[4].y + v[5].y) + ((double)v[6].y + v[7].y))));
      }
      __syncthreads();
    }
    if (w.nbuf == 1 && s + 1 < s_end) {
      stage(s + 1, lds);
      __syncthreads();
    }
  }
  // [32*TI co][32*TJ ci][KK] of the tile, then rows of 32*TJ*KK floats
  constexpr int RO = 32 * TJ * KK;
  float* so = lds;
#pragma unroll
  for (int t = 0; t < NA; ++t) {
    const int ti = t / (KK * TJ), tj = KS == 1 ? t % TJ : 0, tap = KS == 1 ? 0 : t;
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
      const int r = 2 * wave + rr, co = ti * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
      so[co * RO + (tj * 32 + row) * KK + tap] = tot[t][rr];
    }
  }
  __syncthreads();
  const int nci = min(32 * TJ, w.Cin - ci_base) * KK, nco = min(32 * TI, w.Cout - co_base);
  float* out = w.part + (((size_t)chunk * w.Cout + co_base) * w.Cin + ci_base) * KK;
  for (int co = wave; co < nco; co += 8)
    for (int i = lane; i < nci; i += 64) out[(size_t)co * w.Cin * KK + i] = so[co * RO + i];
}

// Most pixels that a wavefront adds up in one 32-bit accumulator before a flush: a sum's rounding error grows with the root
// of its chain of additions, so the chain must not grow with the micro-batch.  As long as the direct kernel's, and at most
// 128.  Relative error of dW against 64 bits, direct kernel / one chain per block / now: 512 -> 512 at 32 x 7x7 1.34e-7,
// 1.67e-7, 1.24e-7; 256 -> 256 at 8 x 14x14 1.19e-7, 1.30e-7, 1.02e-7, at 64 x 28x28 2.9e-7, 6.9e-7, 2.1e-7.  A flush takes
// about 4 us, the time of its LDS traffic; more and shorter blocks instead, with more partials, took longer: backward of the
// first layer 214 us before, 236 with chains of 64 that way, 223 with flushes.
int chain_limit(int N, int Cin, int Cout, int HWo) { return std::min(128, conv_mfma_wgrad_chain(N, Cin, Cout, HWo)); }

struct LdsWgPick {
  int PT = 0, per, chunks, rows, NP, nbuf, chain;
  long npix;
  size_t buf, lds;  // bytes of a stage's buffer and of a block
  // stages between two flushes of a run of `run` stages: equal shares, none of more than `chain` pixels a wavefront
  int flush(int run) const { return cdiv(run, cdiv(std::min((long)run * PT, npix), 8 * chain)); }
};

LdsWgPick search_wgrad(int N, int Cin, int Cout, int H, int W, int KS, int S) {
  LdsWgPick best;
  const int pad = KS / 2, Ho = (H + 2 * pad - KS) / S + 1, Wo = (W + 2 * pad - KS) / S + 1;
  if (!copies_reach(N, Cin, H, W) || !copies_reach(N, Cout, Ho, Wo)) return best;
  if (KS == 1) { H = Ho; W = Wo; S = 1; }  // from here on: the rows and columns that are staged
  const long npix = (long)N * Ho * Wo, tw = KS == 1 ? 64 : 32, tiles = (long)cdiv(Cin, tw) * cdiv(Cout, tw);
  if ((size_t)N * (H + 2) * (H + 1) >= ((size_t)1 << 32) || (size_t)Ho * Wo * Wo >= ((size_t)1 << 32)) return best;  // reciprocals
  double cost = 1e30;
  for (int PT = 32; PT <= 128; PT *= 2) {
    LdsWgPick p;
    p.PT = PT;
    p.chain = chain_limit(N, Cin, Cout, Ho * Wo);
    p.npix = npix;
    p.rows = tile_rows(PT, Ho, Wo, S, H);
    p.NP = cdiv(p.rows * (W + 2), 64);
    p.buf = ((size_t)tw * (round_up64(PT) + 2 + p.NP * 64 + 2) + PT) * 4;
    const size_t beside = p.buf >= 8 * kFlush ? 0 : p.buf >= 4 * kFlush ? 4 * kFlush : 8 * kFlush;  // scratch of the flushes
    p.nbuf = 2 * p.buf + beside <= kWgradLds ? 2 : 1;
    p.lds = std::max(p.nbuf * p.buf + beside, (size_t)tw * tw * KS * KS * 4);
    if (p.lds > kWgradLds) continue;
    const int nstage = cdiv(npix, PT);
    for (int per = 1; per <= nstage; per = per < 8 ? per + 1 : per + per / 4) {
      const int chunks = cdiv(nstage, per);
      if (chunks * tiles > 8192 && per < nstage) continue;
      const double mfma = PT / 8 * (KS == 1 ? 4 : 9) * 64.0, bytes = tw * 256.0 * (p.NP + cdiv(PT, 64));
      const double stage = 2000 + bytes / 20;
      const double one = p.nbuf == 2 ? std::max(mfma, stage) + bytes / 40 + 800 : mfma + stage;
      const int run = cdiv(nstage, chunks), flushes = cdiv(run, p.flush(run));  // the last one is the block's end
      const double c = std::ceil(chunks * tiles / 256.0) * (run * one + stage + 3000 + KS * KS * (1000 * flushes - 500)) +
                       (double)chunks * tiles * KS * KS * tw * tw * 8 / 1500;  // writing and reducing the partials
      if (c < cost) {
        cost = c;
        p.per = cdiv(nstage, chunks);
        p.chunks = cdiv(nstage, p.per);
        best = p;
      }
    }
  }
  return best;
}

bool pick_wgrad(int N, int Cin, int Cout, int H, int W, int KS, int S, int cap, LdsWgPick& p) {
  static thread_local std::map<std::array<int, 7>, LdsWgPick> seen;
  const std::array<int, 7> key = {N, Cin, Cout, H, W, KS, S};
  auto it = seen.find(key);
  if (it == seen.end()) {
    if (seen.size() >= 1024) seen.clear();
    it = seen.emplace(key, search_wgrad(N, Cin, Cout, H, W, KS, S)).first;
  }
  p = it->second;
  if (p.PT > 0 && p.chunks > cap) {
    const int nstage = cdiv((long)N * ((H + 2 * (KS / 2) - KS) / S + 1) * ((W + 2 * (KS / 2) - KS) / S + 1), p.PT);
    p.per = cdiv(nstage, cap);
    p.chunks = cdiv(nstage, p.per);
  }
  return p.PT > 0;
}

}  // namespace

int conv_lds_wgrad_parts(int N, int Cin, int Cout, int H, int W, int KS, int S, int cap) {
  LdsWgPick p;
  return pick_wgrad(N, Cin, Cout, H, W, KS, S, cap, p) ? p.chunks : 0;
}

void conv_lds_wgrad(hipStream_t st, const char* name, const float* g, const float* x, float* part, int N, int Cin, int Cout,
                    int H, int W, int KS, int S, int cap) {
  LdsWgPick p;
  if (!pick_wgrad(N, Cin, Cout, H, W, KS, S, cap, p)) return;
  LdsWgArgs w;
  w.g = g; w.x = x; w.part = part;
  w.N = N; w.Cin = Cin; w.Cout = Cout; w.H = H; w.W = W; w.S = S;
  w.Ho = (H + 2 * (KS / 2) - KS) / S + 1;
  w.Wo = (W + 2 * (KS / 2) - KS) / S + 1;
  w.XS = 1; w.XRW = W; w.XHW = (unsigned)(H * W);
  if (KS == 1 && S > 1) { w.H = w.Ho; w.W = w.Wo; w.S = 1; w.XS = S; }
  w.x_bytes = (unsigned)N * Cin * w.XHW * 4u;
  w.g_bytes = (unsigned)N * Cout * w.Ho * w.Wo * 4u;
  w.npix = (unsigned)N * w.Ho * w.Wo;
  w.rRW = reciprocal(w.W + 2); w.rH1 = reciprocal(w.H + 1); w.rWo = reciprocal(w.Wo);
  w.rows = p.rows; w.RW = w.W + 2; w.NP = p.NP; w.PT = p.PT; w.per = p.per; w.nbuf = p.nbuf;
  w.flush = p.flush(p.per);
  w.nstage = cdiv(w.npix, p.PT);
  const int tw = KS == 1 ? 64 : 32;
  const dim3 grid((unsigned)(p.chunks * cdiv(Cin, tw) * cdiv(Cout, tw)));
  if (KS == 3) KLAUNCH_NAMED(name, (conv_lds_wgrad_f32_kernel<3>), grid, dim3(512), p.lds, st, w);
  else KLAUNCH_NAMED(name, (conv_lds_wgrad_f32_kernel<1>), grid, dim3(512), p.lds, st, w);
}

// The kernels of this file may use more than the default 64 KiB of dynamic LDS: allowed once per stage, for its device, always
// up to the same sizes.  (Set per launch to that launch's size, it was state shared with the launches of other threads.)
template <int NT, int NI>
static hipError_t x3_allow() {
  if (hipError_t e = hipFuncSetAttribute((const void*)conv_x3_f32_kernel<NT, true, NI>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kX3Lds)) return e;
  return hipFuncSetAttribute((const void*)conv_x3_f32_kernel<NT, false, NI>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kX3Lds);
}
template <int NT>
static hipError_t x3_allow() {
  if (hipError_t e = x3_allow<NT, 1>()) return e;
  if (hipError_t e = x3_allow<NT, 2>()) return e;
  if (hipError_t e = x3_allow<NT, 3>()) return e;
  return x3_allow<NT, 4>();
}
hipError_t conv_lds_allow() {
  const std::pair<const void*, size_t> kernels[] = {
      {(const void*)conv_lds_f32_kernel<1, false>, kProductLds}, {(const void*)conv_lds_f32_kernel<1, true>, kProductLds},
      {(const void*)conv_lds_f32_kernel<2, false>, kProductLds}, {(const void*)conv_lds_f32_kernel<2, true>, kProductLds},
      {(const void*)conv_lds_wgrad_f32_kernel<1>, kWgradLds},    {(const void*)conv_lds_wgrad_f32_kernel<3>, kWgradLds}};
  for (const auto& k : kernels)
    if (hipError_t e = hipFuncSetAttribute(k.first, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second)) return e;
  if (hipError_t e = conv_x3_wgrad_allow()) return e;
  if (hipError_t e = x3_allow<1>()) return e;
  if (hipError_t e = x3_allow<2>()) return e;
  return x3_allow<4>();
}

}  // namespace ast

// The choices above, for tests that name one.  what: 0 forward, 1 input gradient, 2 weight gradient of a conv with
// these sizes (H, W: its input); 3: a weight gradient with the partials of a stage that has to fit the static workspace.  0:
// other kernels run (conv_x3_f32_kernel, conv_wgrad_x3_f32_kernel, the direct ones).  1: staged; out = {row tiles, pixel groups, shares of the
// contraction, classes of result pixels, 0, 0}, or for a weight gradient {pixels per stage, stages per block, partials,
// buffers, stages per flush, scratch areas of a flush inside the stage's buffer}.
extern "C" int ast_conv_lds_choice(int what, int N, int Cin, int Cout, int H, int W, int KS, int S, int out[6]) {
  using namespace ast;
  if (what >= 2) {
    const int cap = what == 2 ? INT_MAX : conv_mfma_wgrad_compact_parts(N, Cin, Cout, H, W, KS, S);
    LdsWgPick p;
    if (conv_x3_wgrad_parts(N, Cin, Cout, H, W, KS, S, cap) || !pick_wgrad(N, Cin, Cout, H, W, KS, S, cap, p)) return 0;
    out[0] = p.PT; out[1] = p.per; out[2] = p.chunks; out[3] = p.nbuf;
    out[4] = p.flush(p.per);
    out[5] = p.buf >= 8 * kFlush ? 2 : p.buf >= 4 * kFlush ? 1 : 0;
    return 1;
  }
  LdsArgs a;
  LdsPick p;
  int ncls;
  const int Kdim = what ? Cout : Cin, Mdim = what ? Cin : Cout;
  if (conv_x3_takes(what == 1, N, Kdim, Mdim, H, W, KS, S) || !plan_product(what == 1, N, Kdim, Mdim, H, W, KS, S, a, ncls, p)) return 0;
  out[0] = p.MT; out[1] = p.WN; out[2] = p.WK; out[3] = ncls;
  out[4] = out[5] = 0;
  return 1;
}

// The same for the products on the bf16 matrix cores; out = {pixel groups per wavefront, row tiles, pixel groups, shares of
// the contraction, items per thread, classes}.
extern "C" int ast_conv_x3_choice(int dgrad, int N, int Cin, int Cout, int H, int W, int KS, int S, int out[6]) {
  using namespace ast;
  LdsArgs a;
  X3Shape p;
  int ncls;
  if (!plan_x3(dgrad != 0, N, dgrad ? Cout : Cin, dgrad ? Cin : Cout, H, W, KS, S, a, ncls, p)) return 0;
  out[0] = p.NT; out[1] = p.WM; out[2] = p.WN; out[3] = p.WK; out[4] = p.NI; out[5] = ncls;
  return 1;
}
