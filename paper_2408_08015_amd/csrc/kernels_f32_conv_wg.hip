// Weight gradient of 3x3 convolutions of stride 1 on the bf16 matrix cores with split operands (kernels_f32_x3.h).
#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <map>
#include "device_utils.h"
#include "kernels.h"
#include "kernels_f32_x3.h"
#include "prof.h"

namespace ast {
namespace {

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

struct WgX3Args {
  const float* g;  // [N][Cout][H][W]
  const float* x;  // [N][Cin][H][W]
  float* part;     // [chunk][Cout][Cin][9]
  int Cin, Cout, H, W, rows;
  unsigned HW;
  size_t g_words, x_words;
  int C8, R, XP, GP, per, nstage;
  unsigned rH1;  // ceil(2^32 / (H + 1))
};

constexpr size_t kWgX3Lds = 156 * 1024;
constexpr int kWaves = 12, kThreads = kWaves * 64, kShares = kWaves / 3;
constexpr size_t kSumsLds = (size_t)kWaves * 3 * 1024 * 4;

// acc += tap (dy, dx) of one 32 x 32 tile over share sh of the stages [s0, s1), in steps of 16 columns, on the fp32 matrix
// instructions (kernels_f32_x3.h: where the pieces gave no finite sum).  x outside the image is 0.
template <int kSteps>
__device__ __forceinline__ void wgx3_contract_f32(const WgX3Args& w, int co, int ci, int dy, int dx, int sh, int s0, int s1,
                                                  floatx16& acc) {
  const int half = threadIdx.x >> 5 & 1, RC = w.R * w.C8;
  co += threadIdx.x & 31;
  ci += threadIdx.x & 31;
#pragma unroll 1
  for (int s = s0; s < s1; ++s)
#pragma unroll 1
    for (int j = 0; j < kSteps; ++j) {
      const int k0 = 2 * (sh + j * kShares), k = k0 + half;
      if (k0 >= RC) break;  // uniform
      const int lr = k / w.C8, c = (k - lr * w.C8) * 8, vr = s * w.R + lr, n = vr / (w.H + 1), i = vr - n * (w.H + 1);
      const int h = i + dy - 1;
      const bool row = k < RC && vr < w.rows && i < w.H, xrow = row && h >= 0 && h < w.H && ci < w.Cin;
      const float* const gp = w.g + ((size_t)n * w.Cout + co) * w.HW + (size_t)i * w.W;
      const float* const xp = w.x + ((size_t)n * w.Cin + ci) * w.HW + (size_t)(xrow ? h : 0) * w.W;
      float g[8], x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int cx = c + e + dx - 1;
        g[e] = row && co < w.Cout && c + e < w.W ? gp[c + e] : 0.f;
        x[e] = xrow && c + e < w.W && cx >= 0 && cx < w.W ? xp[cx] : 0.f;  // (no term past the row's end)
      }
      acc = mfma_f32(g, x, acc);
    }
}

// eight values of a row from column `col` on, zeros past its end; VL: words that divide W
template <int VL>
__device__ __forceinline__ void load8(__amdgpu_buffer_rsrc_t r, unsigned voff, int col, int W, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; e += VL) {
    const unsigned o = col + e < W ? voff + (unsigned)e * 4u : kOutside;
    if constexpr (VL == 4) {
      const auto q = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
      v[e] = q.x; v[e + 1] = q.y; v[e + 2] = q.z; v[e + 3] = q.w;
    } else if constexpr (VL == 2) {
      const auto q = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
      v[e] = q.x; v[e + 1] = q.y;
    } else {
      v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
    }
  }
}

// The samples' rows stand in one column of virtual rows, with a row of zeros behind each sample, and a row is C8 chunks of
// eight columns of which at least the last column is zero.  In that order a tap is a shift of x by whole rows and by one
// column, the zeros are the padding, and a chunk is a lane's share of a matrix instruction.
//
// Block of twelve wavefronts, one per compute unit: 32 x 32 of (cout, cin), all nine taps, over a run of stages of R rows (at
// most CH chunks).  A wavefront has the three taps of one row and a quarter of the stage's steps of 16 columns: the sums of
// all nine taps, each with its small products, would leave one wavefront per SIMD.  (One sum per tap, to which a step's six
// products are added when they are complete, took 69 us below: the additions cost as much as the products, and a large
// product that meets a smaller sum cuts it downwards (kernels_f32_x3.h), so the error of the step grew five times.)  A thread reads a chunk of g or x
// (CH 16: up to two), a stage ahead, splits it and writes its three pieces to LDS while the stage before is multiplied: g to
// the other of two buffers, x to a ring of 2R + 2 rows, so that no row is split twice.  A third of the wavefronts does that
// before its products and the others behind them, so that a SIMD's matrix core is not idle meanwhile.  Chunk pitches are
// odd: 16 lanes' reads hit 64 different banks.  Shifts by one column are made of the words read and of one neighbouring word
// on each side.
//
// Against the fp32 matrix instructions (kernels_f32_conv_lds.hip), us and relative error against 64 bits with x behind a
// ReLU: 64 -> 64 at 32 x 56x56 115 -> 66, 1.4e-7 -> 9.0e-8; 8 x 56x56 36 -> 25; 128 -> 128 at 8 x 28x28 38 -> 24; 256 -> 256
// at 8 x 14x14 38 -> 24; 512 -> 512 at 8 x 7x7 34 -> 25, 8.1e-8 -> 5.3e-8; 13 x 45x45 35 -> 27; 32 -> 32 at 16 x 112x112
// 60 -> 38.  A sixth of the first one's products is padding; the matrix cores' own rate is 25 us.
template <int CH, int VL>
__global__ __launch_bounds__(kThreads) void conv_wgrad_x3_f32_kernel(WgX3Args w) {
  constexpr int kSteps = CH / 2 / kShares;  // of 16 columns, of a wavefront in a stage
  constexpr int kItems = (64 * CH + kThreads - 1) / kThreads;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), dy = wave % 3, sh = wave / 3;
  const int C8 = w.C8, R = w.R, RC = R * C8, NS = 2 * R + 2, XP = w.XP, GP = w.GP, H1 = w.H + 1;
  const int gsz = 96 * GP, xsz = NS * 96 * XP;  // 16-byte words
  uint4* const gl = reinterpret_cast<uint4*>(lds);
  const unsigned tiles_ci = (unsigned)(w.Cin + 31) / 32u, tiles = tiles_ci * ((unsigned)(w.Cout + 31) / 32u);
  const unsigned id = xcd_grouped(blockIdx.x, gridDim.x);
  const int chunk = (int)(id / tiles), tile = (int)(id % tiles);
  const int ci_base = (tile % (int)tiles_ci) * 32, co_base = (tile / (int)tiles_ci) * 32;
  const int s_begin = chunk * w.per, s_end = min(s_begin + w.per, w.nstage), r0 = s_begin * R;
  const __amdgpu_buffer_rsrc_t rg = rsrc_words(w.g, w.g_words), rx = rsrc_words(w.x, w.x_words);

  for (int i = tid; i < 2 * gsz + 1 + xsz; i += kThreads) gl[i] = uint4{0, 0, 0, 0};
  __syncthreads();

  // the thread's chunks of a stage: 32 channels of g, from a multiple of 64 on 32 channels of x
  const int G64 = (32 * RC + 63) & ~63;
  int vr[kItems], col[kItems], at[kItems];  // the next virtual row to read, its first column, where the next pieces go
  unsigned cw[kItems];
  bool is_x[kItems], has[kItems], in_c[kItems];  // the first one uniform
  float v[kItems][8];
  auto load = [&](int i, int r) __attribute__((always_inline)) {
    const int n = (int)__umulhi((unsigned)r, w.rH1), h = r - n * H1;  // (a row above the first one: dropped)
    const unsigned o = ((unsigned)(n * (is_x[i] ? w.Cin : w.Cout)) * w.HW + (unsigned)(h * w.W) + cw[i]) * 4u;
    load8<VL>(is_x[i] ? rx : rg, o, in_c[i] && (unsigned)r < (unsigned)w.rows && h < w.H ? col[i] : w.W, w.W, v[i]);
  };
  auto put = [&](int i, int to) __attribute__((always_inline)) {
    uint4 p[3];
    split3(v[i], p);
    const int pitch = 32 * (is_x[i] ? XP : GP);
    if (has[i]) {
#pragma unroll
      for (int j = 0; j < 3; ++j) gl[to + j * pitch] = p[j];
    }
  };
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    is_x[i] = wave * 64 + i * kThreads >= G64;
    const int it = tid + i * kThreads - (is_x[i] ? G64 : 0), c = it / RC, k = it - c * RC, lr = k / C8, ch = k - lr * C8;
    const int cc = (is_x[i] ? ci_base : co_base) + c;
    has[i] = c < 32;
    in_c[i] = has[i] && cc < (is_x[i] ? w.Cin : w.Cout);
    col[i] = ch * 8;
    cw[i] = (unsigned)cc * w.HW + (unsigned)(ch * 8);
    vr[i] = r0 + lr + (is_x[i] ? 1 : 0);  // of x the rows that the stage before has not
    at[i] = is_x[i] ? 2 * gsz + 1 + (2 + lr) % NS * 96 * XP + c * XP + ch : c * GP + k;
    if (is_x[i])
      for (int q = 0; q + lr < 2; q += R) {  // the two rows of x in front
        load(i, r0 - 1 + q + lr);
        put(i, 2 * gsz + 1 + (q + lr) * 96 * XP + c * XP + ch);
      }
  }
  auto load_stage = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      load(i, vr[i]);
      vr[i] += R;
    }
  };
  auto put_stage = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      put(i, at[i]);
      if (is_x[i]) {  // uniform
        at[i] += R * 96 * XP;
        at[i] -= at[i] > 2 * gsz + xsz ? xsz : 0;
      } else {
        at[i] += at[i] >= gsz ? -gsz : gsz;
      }
    }
  };
  load_stage();
  put_stage();
  if (s_begin + 1 < s_end) load_stage();

  int xo[kSteps], xr[kSteps];
#pragma unroll
  for (int j = 0; j < kSteps; ++j) {  // (a chunk past the last one: zeros of g)
    const int kx = min(2 * (sh + j * kShares) + half, RC - 1);
    xr[j] = kx / C8;
    xo[j] = 2 * gsz + 1 + row * XP + kx - xr[j] * C8;  // (the word in front is the padding left of the first row)
  }
  floatx16 acc[3], acs[3];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = acs[t][r] = 0.f;

  int base = dy;  // the ring's row of the tap at the stage's first row
  for (int s = s_begin; s < s_end; ++s) {
    const int b = (s - s_begin) & 1;
    __syncthreads();
    if (wave < 4 && s + 1 < s_end) {  // uniform
      put_stage();
      if (s + 2 < s_end) load_stage();
    }
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
      if (2 * (sh + j * kShares) >= RC) break;  // uniform
      uint4 a[3], m[3];
      uint32_t lo[3], hi[3];
      const uint4* const ga = gl + b * gsz + row * GP + 2 * (sh + j * kShares) + half;
      int sl = base + xr[j];
      sl -= sl >= NS ? NS : 0;
      const uint4* const xs = gl + sl * 96 * XP + xo[j];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        a[i] = ga[i * 32 * GP];
        m[i] = xs[i * 32 * XP];
        lo[i] = reinterpret_cast<const uint32_t*>(xs + i * 32 * XP)[-1];
        hi[i] = reinterpret_cast<const uint32_t*>(xs + i * 32 * XP)[4];
      }
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        uint4 f[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          auto join = [](uint32_t h, uint32_t l) { return __builtin_amdgcn_alignbit(h, l, 16); };
          f[i] = dx == 1 ? m[i]
               : dx == 0 ? uint4{join(m[i].x, lo[i]), join(m[i].y, m[i].x), join(m[i].z, m[i].y), join(m[i].w, m[i].z)}
                         : uint4{join(m[i].y, m[i].x), join(m[i].z, m[i].y), join(m[i].w, m[i].z), join(hi[i], m[i].w)};
        }
        acs[dx] = mfma_bf16(a[2], f[0], acs[dx]);
        acc[dx] = mfma_bf16(a[0], f[0], acc[dx]);
        acs[dx] = mfma_bf16(a[0], f[2], acs[dx]);
        acs[dx] = mfma_bf16(a[1], f[1], acs[dx]);
        acs[dx] = mfma_bf16(a[1], f[0], acs[dx]);
        acs[dx] = mfma_bf16(a[0], f[1], acs[dx]);
      }
    }
    if (wave >= 4 && s + 1 < s_end) {  // uniform
      put_stage();
      if (s + 2 < s_end) load_stage();
    }
    base += R;
    base -= base >= NS ? NS : 0;
  }

  float bad = 0.f;
#pragma unroll
  for (int t = 0; t < 3; ++t) bad = add_small(acc[t], acs[t], bad);
  if (any_not_finite(bad)) {
#pragma unroll 1
    for (int t = 0; t < 3; ++t) {
      floatx16 again = zero16();
      wgx3_contract_f32<kSteps>(w, co_base, ci_base, dy, t, sh, s_begin, s_end, again);
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (t == j) take_not_finite(acc[j], again);
    }
  }
  // the sums of the four wavefronts of a tap, added in 64 bits; then [32 co][32 ci][9], whole rows of which leave
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) lds[((sh * 9 + dy * 3 + t) * 16 + r) * 64 + lane] = acc[t][r];
  __syncthreads();
  float tot[9 * 1024 / kThreads];
#pragma unroll
  for (int i = 0; i < 9 * 1024 / kThreads; ++i) {
    const float* const f = lds + tid + i * kThreads;
    double d = 0.0;
#pragma unroll
    for (int q = 0; q < kShares; q += 2) d += (double)f[q * 9216] + f[(q + 1) * 9216];
    tot[i] = (float)d;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 9 * 1024 / kThreads; ++i) {
    const int e = tid + i * kThreads, t = e >> 10, r = e >> 6 & 15;
    lds[(8 * (r >> 2) + 4 * half + (r & 3)) * 288 + row * 9 + t] = tot[i];
  }
  __syncthreads();
  const int nci = min(32, w.Cin - ci_base) * 9, nco = min(32, w.Cout - co_base);
  float* out = w.part + (((size_t)chunk * w.Cout + co_base) * w.Cin + ci_base) * 9;
  for (int co = wave; co < nco; co += kWaves)
    for (int i = lane; i < nci; i += 64) out[(size_t)co * w.Cin * 9 + i] = lds[co * 288 + i];
}

struct WgX3Pick {
  int R = 0, CH, C8, XP, GP, per, chunks, nstage;
  size_t lds;
};

// Rows shorter than 64 columns: CH 8.  With 16 the second chunk of a thread does not fit the registers (8 x 56x56 27 us
// against 25, 512 -> 512 at 8 x 7x7 32 against 25); longer rows need it.
// Cycles: a stage's matrix instructions; a block's first rows, its sums and the partials cost as much as some stages, so a
// block gets as many as leave no compute unit idle, at most 32 steps.
WgX3Pick search_wgx3(int CH, int N, int Cin, int Cout, int H, int W) {
  WgX3Pick p;
  if ((size_t)N * std::max(Cin, Cout) * H * W * 4 > kOutside - 64 || ((size_t)N + 1) * (H + 1) * (H + 1) >= ((size_t)1 << 31)) return p;  // (the reciprocal)
  p.C8 = (W + 8) / 8;
  p.CH = CH;
  const int R = std::min(CH / p.C8, N * (H + 1));
  if (R < 1) return p;
  p.XP = (p.C8 + 1) | 1;
  p.GP = (R * p.C8 + 1) | 1;
  p.lds = std::max((size_t)(2 * 96 * p.GP + 1 + (2 * R + 2) * 96 * p.XP) * 16, kSumsLds);
  if (p.lds > kWgX3Lds) return p;
  p.R = R;
  p.nstage = cdiv((long)N * (H + 1), R);
  const long tiles = (long)cdiv(Cin, 32) * cdiv(Cout, 32);
  double cost = 1e30;
  for (int per = 1; per <= std::min(p.nstage, 256 / CH); ++per) {
    const int chunks = cdiv(p.nstage, per), run = cdiv(p.nstage, chunks);
    const double c = std::ceil(chunks * tiles / 256.0) * (run * (CH == 8 ? 4600.0 : 8000) + 14000) + (double)chunks * tiles * 36864 * 2 / 2000;
    if (c < cost) {
      cost = c;
      p.per = run;
      p.chunks = cdiv(p.nstage, run);
    }
  }
  return p;
}

bool pick_wgx3(int N, int Cin, int Cout, int H, int W, int KS, int S, int cap, WgX3Pick& p) {
  if (KS != 3 || S != 1) return false;
  static thread_local std::map<std::array<int, 5>, WgX3Pick> seen;  // (the choice depends on the sizes alone)
  const std::array<int, 5> key = {N, Cin, Cout, H, W};
  auto it = seen.find(key);
  if (it == seen.end()) {
    if (seen.size() >= 1024) seen.clear();
    it = seen.emplace(key, search_wgx3(W < 64 ? 8 : 16, N, Cin, Cout, H, W)).first;
  }
  p = it->second;
  // (fewer partials would make the chains longer than they are measured for; the staged kernel adds up in between)
  return p.R > 0 && p.chunks <= cap;
}

}  // namespace

int conv_x3_wgrad_parts(int N, int Cin, int Cout, int H, int W, int KS, int S, int cap) {
  WgX3Pick p;
  return pick_wgx3(N, Cin, Cout, H, W, KS, S, cap, p) ? p.chunks : 0;
}

bool conv_x3_wgrad(hipStream_t st, const char* name, const float* g, const float* x, float* part, int N, int Cin, int Cout,
                   int H, int W, int KS, int S, int cap) {
  WgX3Pick p;
  if (!pick_wgx3(N, Cin, Cout, H, W, KS, S, cap, p)) return false;
  WgX3Args w;
  w.g = g; w.x = x; w.part = part;
  w.Cin = Cin; w.Cout = Cout; w.H = H; w.W = W;
  w.rows = N * (H + 1);
  w.HW = (unsigned)(H * W);
  w.g_words = (size_t)N * Cout * w.HW;
  w.x_words = (size_t)N * Cin * w.HW;
  w.rH1 = (unsigned)((((uint64_t)1 << 32) + H) / (H + 1));
  w.C8 = p.C8; w.R = p.R; w.XP = p.XP; w.GP = p.GP; w.per = p.per; w.nstage = p.nstage;
  const dim3 grid((unsigned)(p.chunks * cdiv(Cin, 32) * cdiv(Cout, 32)));
  auto run = [&](auto k4, auto k2, auto k1) {
    if (W % 4 == 0) KLAUNCH_NAMED(name, k4, grid, dim3(kThreads), p.lds, st, w);
    else if (W % 2 == 0) KLAUNCH_NAMED(name, k2, grid, dim3(kThreads), p.lds, st, w);
    else KLAUNCH_NAMED(name, k1, grid, dim3(kThreads), p.lds, st, w);
  };
  if (p.CH == 8) run(conv_wgrad_x3_f32_kernel<8, 4>, conv_wgrad_x3_f32_kernel<8, 2>, conv_wgrad_x3_f32_kernel<8, 1>);
  else run(conv_wgrad_x3_f32_kernel<16, 4>, conv_wgrad_x3_f32_kernel<16, 2>, conv_wgrad_x3_f32_kernel<16, 1>);
  return true;
}

hipError_t conv_x3_wgrad_allow() {
  for (const void* k : {(const void*)conv_wgrad_x3_f32_kernel<8, 1>, (const void*)conv_wgrad_x3_f32_kernel<8, 2>,
                        (const void*)conv_wgrad_x3_f32_kernel<8, 4>, (const void*)conv_wgrad_x3_f32_kernel<16, 1>,
                        (const void*)conv_wgrad_x3_f32_kernel<16, 2>, (const void*)conv_wgrad_x3_f32_kernel<16, 4>})
    if (hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWgX3Lds)) return e;
  return hipSuccess;
}

}  // namespace ast

// The choice above, for tests: out = {rows per stage, chunks of eight columns per row, stages per block, partials}.  0:
// another kernel runs.
extern "C" int ast_conv_wgrad_x3_choice(int N, int Cin, int Cout, int H, int W, int KS, int S, int out[4]) {
  using namespace ast;
  WgX3Pick p;
  if (!pick_wgx3(N, Cin, Cout, H, W, KS, S, INT_MAX, p)) return 0;
  out[0] = p.R; out[1] = p.C8; out[2] = p.per; out[3] = p.chunks;
  return 1;
}
