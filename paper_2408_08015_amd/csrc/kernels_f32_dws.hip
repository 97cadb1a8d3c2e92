// BatchNorm -> activation -> depthwise K x K -> BatchNorm -> activation (the middle of an inverted-residual block) in ONE
// launch per direction, for channels that fit the LDS of a compute unit.
//
// Every operator of that run works on one channel at a time, so a block takes one channel of the whole micro-batch: it
// reads the channel once, keeps the activated (forward) or differentiated (backward) planes zero-padded in LDS, and finishes
// both BatchNorms' statistics with block sums instead of partials in memory.  Forward: x (the first BatchNorm's input) in,
// y (the convolution's output, kept for the backward) and z (the second activation's output) out.  Backward: g = dz, y, x in,
// dx out; dW, dgamma and dbeta of both BatchNorms are added into G by the one block that owns the channel.  Results wait for
// the sums in registers, or where those of a 1024-thread block (128) do not hold them, in scratch: in the build 14 of the 90
// backward forms spill, most of them 5x5 (32 values, Q = 1 / 2 / 4: 88, 43 and 55 registers; stride 2 21 to 55), 3x3 of 32 values up to 13.
//
// Bound by memory where channels are large (3 and 4 passes over a tensor, where the launches that it replaces make 5 and 9), by
// one chain of load, sum, multiply, sum, store where they are small, and for 5x5 backward by that scratch: 240 channels of 32 x
// 30x30 read 121 MB and write 68 where the operands are 83 and 28, and take 47 us where those bytes are 22 and the multiply-adds 9.
// In the stages, us per launch, against the launches that it replaces (forward / backward):
//   384 channels of 8 x 14x14   7.3 / 7.8     14.6 / 21      (before: statistics, convolution, normalisation; sums, convolution,
//   960 of 8 x 7x7              6.9 / 7.0     15 / 22         input gradient of the first BatchNorm)
//   192 of 32 x 28x28           18.1 / 23.7   30 / 50        58 and 77 MB
//   144 of 8 x 56x56            16.3 / 22.5   26 / 36
//   240 of 32 x 30x30, 5x5      30 / 47       52 / 76
// (dws_faster: where the one launch is not taken.)
#include <algorithm>
#include <climits>

#include "bn_common.h"
#include "device_utils.h"
#include "kernels.h"
#include "prof.h"

namespace ast {

namespace {

constexpr int kLds = 160 * 1024 - 9 * 1024;  // dynamic part of a compute unit's LDS: all but the sums

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
// index / d without a branch; exact for index * d < 2^32 (indices stay below 2^16 here, and no divisor is larger)
struct Div {
  unsigned m, one;
};
inline Div div_by(int d) { return d <= 1 ? Div{0u, ~0u} : Div{(unsigned)((1ull << 32) / (unsigned)d) + 1u, 0u}; }
__device__ __forceinline__ int fdiv(int i, const Div& d) { return (int)(__umulhi((unsigned)i, d.m) + ((unsigned)i & d.one)); }

// ReLU and ReLU6 without a branch per value.  hi: 6, or for ReLU a NaN, which a minimum passes over and no comparison reaches.
__device__ __forceinline__ float clamp_of(int act) { return act == ACT_RELU6 ? 6.f : __builtin_nanf(""); }
template <bool SW> __device__ __forceinline__ float act_value(float v, float hi) {
  if (SW) return v * sigmoid_f(v);
  return fminf(fmaxf(v, 0.f), hi);
}
template <bool SW> __device__ __forceinline__ void act_both(float v, float hi, float& val, float& slope) {
  if (SW) {
    const float s = sigmoid_f(v);
    val = v * s;
    slope = s + val * (1.f - s);
  } else {
    val = fminf(fmaxf(v, 0.f), hi);
    slope = v > 0.f && !(v >= hi) ? 1.f : 0.f;
  }
}
// the value is in its register from here on: a load of it is not moved behind a wait for something else
__device__ __forceinline__ void have(float v) { asm volatile("" ::"s"(v)); }

// Threads work on strips of Q neighbouring results of a row, and rows in LDS start at multiples of Q words, so that the middle
// of a window is read as one word of Q (4: planes of a multiple of four columns; 2: of an even number; else 1).  With
// single words (28x28 planes, 192 channels of 32 samples: 22 us forward, 34 backward) a launch waited for LDS and for the
// write path.
typedef float floatx2 __attribute__((ext_vector_type(2)));
template <int Q> struct Vec { typedef float T __attribute__((ext_vector_type(Q))); };
template <> struct Vec<1> { typedef float T; };
__device__ __forceinline__ float entry(float v, int) { return v; }
__device__ __forceinline__ float entry(floatx2 v, int j) { return v[j]; }
__device__ __forceinline__ float entry(floatx4 v, int j) { return v[j]; }
// v[at .. at + Q) = p[0 .. Q), and back
template <int Q, int N> __device__ __forceinline__ void read_vec(const float* __restrict__ p, float (&v)[N], int at) {
  const typename Vec<Q>::T t = *reinterpret_cast<const typename Vec<Q>::T*>(p);
#pragma unroll
  for (int j = 0; j < Q; ++j) v[at + j] = entry(t, j);
}
template <int Q, int N> __device__ __forceinline__ void write_vec(float* __restrict__ p, const float (&v)[N], int at) {
  if constexpr (Q == 1) {
    *p = v[at];
  } else {
    typename Vec<Q>::T t;
#pragma unroll
    for (int j = 0; j < Q; ++j) t[j] = v[at + j];
    *reinterpret_cast<typename Vec<Q>::T*>(p) = t;
  }
}

// The planes of one channel in LDS: rows of RS floats, at least `pad` zeros between rows (right of one row, left of the next)
// and `pad` zero rows between planes.
struct Padded {
  int H, W, RS, PS, lead, words4;  // words4: 16-byte words of the whole copy
  Div mHW, mW;
};
inline Padded padded(int N, int H, int W, int pad, int Q) {
  Padded p;
  p.H = H; p.W = W;
  p.RS = cdiv(W + pad, Q) * Q;
  p.PS = (H + pad) * p.RS;
  p.lead = pad * p.RS + cdiv(pad, Q) * Q;
  p.mHW = div_by(H * W);
  p.mW = div_by(W);
  return p;
}
// A thread's work: one strip of columns of one band of rows of one plane.
struct Items {
  int cols, bands, rows, n;  // strips per row, bands per plane, rows per band; items in all
  Div mcols, mbands;
};
// as many bands as there are threads for
inline Items items_of(int N, int H, int cols, int T) {
  Items it{};
  for (int b = 1; b <= H && (long)N * cols * b <= T; ++b) {
    const int rows = cdiv(H, b);
    if (cdiv(H, rows) == b) it = {cols, b, rows, N * cols * b, div_by(cols), div_by(b)};
  }
  return it;
}

struct Geom {
  int N, C, H, W, Ho, Wo;
  Div mHW;  // of the convolution's input planes
  double inv, inv_o;     // 1 / values of a channel, in front of and behind the convolution
  float unb, unb_o;      // values / (values - 1), of the running variance
  Padded p;
  Items it;
};

// Words of a thread's V values: LV consecutive ones, word k of thread t at t + k * T of the channel's planes.  Q == 1: planes
// may be of any size; else they are multiples of four values.  Past the end the last word again (no branch around a load).
template <int Q> constexpr int kLoad = Q == 1 ? 1 : 4;
template <int Q, int T, int V>
__device__ __forceinline__ void load_channel(const float* __restrict__ src, size_t sample, int E, int HW, const Div& mHW,
                                             float (&v)[V]) {
  constexpr int LV = kLoad<Q>;
#pragma unroll
  for (int k = 0; k < V / LV; ++k) {
    const int i = min(LV * (int)(threadIdx.x + k * T), E - LV), n = fdiv(i, mHW);
    read_vec<LV>(src + n * sample + (i - __mul24(n, HW)), v, LV * k);
  }
}
// value k of the thread is one of the channel's
template <int Q, int T> __device__ __forceinline__ bool holds(int k, int E) {
  constexpr int LV = kLoad<Q>;
  return LV * (int)(threadIdx.x + k / LV * T) < E;
}
// the same values into the padded copy
template <int Q, int T, int V>
__device__ __forceinline__ void store_padded(float* __restrict__ sh, const Padded& p, int E, const float (&v)[V]) {
  constexpr int LV = kLoad<Q>;
  const int HW = p.H * p.W;
#pragma unroll
  for (int k = 0; k < V; k += Q) {  // a strip lies in one row
    const int i = LV * (threadIdx.x + k / LV * T) + k % LV;
    if (i < E) {
      const int n = fdiv(i, p.mHW), e = i - __mul24(n, HW), r = fdiv(e, p.mW);
      write_vec<Q>(sh + p.lead + __mul24(n, p.PS) + __mul24(r, p.RS) + (e - __mul24(r, p.W)), v, k);
    }
  }
}

// v of the lane 16 (32) further: the sums of the two halves of the wavefront (of two rows of 16) swap places in the VALU
__device__ __forceinline__ double swap_add32(double a, double b) {  // lanes 0-31: a of both halves; 32-63: b of both
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double swap_add16(double v) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// f(AT) + .. + f(AT + N - 1) as a tree: the rounding of a chain of 32 additions is 2 to 3 times that of the separate launches, whose
// threads add up 16 values in pairs
template <int N, int AT = 0, typename F> __device__ __forceinline__ float tree_sum(F f) {
  if constexpr (N == 1) return f(AT);
  else return tree_sum<N / 2, AT>(f) + tree_sum<N - N / 2, AT + N / 2>(f);
}
// Both sums over the block, in 64 bits and a fixed order, the same in every thread; red: 2 * T / 64 words of their own.  The
// halves of a wavefront take a sum each, and so do they over the block's wavefronts: an eighth of the 64-bit additions of two
// sums one after the other in every lane.
template <int T>
__device__ __forceinline__ void block_sums(float f1, float f2, double* red, double& d1, double& d2) {
  constexpr int NW = T / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double v = swap_add16(row16_sum(swap_add32((double)f1, (double)f2)));
  if ((lane & 31) == 0) red[(lane >> 5) * NW + w] = v;
  __syncthreads();
  const double r = row16_sum((lane & 31) < NW ? red[(lane >> 5) * NW + (lane & 15)] : 0.0);
  d1 = lane_value(r, 0);
  d2 = lane_value(r, 32);
}

// The strip of Q columns of a band of rows that a thread works on (one: a block has a thread for each), and its results so
// far: V / Q rows of them in registers at most.
struct Strip {
  int n, col, r0, rows;  // rows of the band that there are
};
template <int Q> __device__ __forceinline__ Strip strip_of(const Geom& g) {
  const int i = min((int)threadIdx.x, g.it.n - 1), q = fdiv(i, g.it.mcols), n = fdiv(q, g.it.mbands);
  Strip s;
  s.n = n;
  s.col = (i - __mul24(q, g.it.cols)) * Q;
  s.r0 = __mul24(q - __mul24(n, g.it.bands), g.it.rows);
  s.rows = (int)threadIdx.x < g.it.n ? min(g.it.rows, g.Ho - s.r0) : 0;
  return s;
}

// f(row of the band, live, window) for every row of outputs of the strip: window(u, v, j) is the operand of tap (u, v) of
// output j, from the padded copy.  R rows of results from one batch of reads (a step of one row waits out the latency of
// LDS at every row).  Past the end of a band `live` is false and the window is of other rows.
template <int K, int S, int Q, int V> constexpr int kRows = (S == 2 || (K == 5 && Q == 4)) && V / Q > 2 ? 2 : V / Q > 4 ? 4 : V / Q;
template <int K, int S, int Q, int V, typename F>
__device__ __forceinline__ void each_window(const float* __restrict__ sh, const Geom& g, const Strip& st, F f) {
  constexpr int P = K / 2, R = kRows<K, S, Q, V>, NR = (R - 1) * S + K, NC = (Q - 1) * S + K, RIGHT = K - S - P;
  const float* p = sh + g.p.lead + __mul24(st.n, g.p.PS) + __mul24(st.r0 * S - P, g.p.RS) + st.col * S;
  float win[NR][NC];
  auto row = [&](const float* s, float (&w)[NC]) {
#pragma unroll
    for (int b = 0; b < P; ++b) w[b] = s[b - P];
#pragma unroll
    for (int b = 0; b < S; ++b) read_vec<Q>(s + b * Q, w, P + b * Q);
#pragma unroll
    for (int b = 0; b < RIGHT; ++b) w[P + Q * S + b] = s[Q * S + b];
  };
#pragma unroll
  for (int a = 0; a < K - S; ++a) row(p + a * g.p.RS, win[a]);
  p += (K - S) * g.p.RS;
#pragma unroll
  for (int r = 0; r < V / Q; r += R) {
    if (r < g.it.rows) {
#pragma unroll
      for (int a = 0; a < R * S; ++a) row(p + a * g.p.RS, win[K - S + a]);
      p += R * S * g.p.RS;
#pragma unroll
      for (int k = 0; k < R; ++k)
        f(r + k, r + k < st.rows, [&](int u, int v, int j) { return win[k * S + u][j * S + v]; });
#pragma unroll
      for (int a = 0; a < K - S; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) win[a][b] = win[a + R * S][b];
    }
  }
}

// What a BatchNorm's statistics make of a channel.  inv: 1 / count.
struct Coef {
  float mean, istd, scale, shift, var;
};
__device__ __forceinline__ Coef coefficients(double s1, double s2, double inv, float gamma, float beta, float eps) {
  const double mean = s1 * inv;
  double var = s2 * inv - mean * mean;
  if (var < 0) var = 0;
  // 1 / sqrt by the hardware's estimate and two Newton steps: the division and the root of the general routine are 0.3 us of
  // dependent instructions here
  const double v = var + (double)eps;
  double r;
  if (v > 1e-200 && v < 1e200) {
    r = __builtin_amdgcn_rsq(v);
    r = r * fma(-0.5 * v * r, r, 1.5);
    r = r * fma(-0.5 * v * r, r, 1.5);
  } else {
    r = 1.0 / sqrt(v);
  }
  const double sc = (double)gamma * r;
  return {(float)mean, (float)r, (float)sc, (float)((double)beta - mean * sc), (float)var};
}
// by one thread, at the end of the kernel; rmean, rvar: the running values before
__device__ __forceinline__ void record(const DwsBn& b, int c, int C, const Coef& k, float unb, float rmean, float rvar) {
  b.stat[c] = k.mean;
  b.stat[C + c] = k.istd;
  b.ss[c] = k.scale;
  b.ss[C + c] = k.shift;
  b.running[c] = rmean + 0.1f * (k.mean - rmean);
  b.running[C + c] = rvar + 0.1f * (k.var * unb - rvar);
}

struct FwdArgs {
  const float* x;
  const float* w;
  float* y;
  float* z;
  DwsBn b1, b2;
};

template <int K, int S, bool SW, int Q, int T, int V>
__global__ __launch_bounds__(T) void dws_fwd_kernel(FwdArgs a, Geom g) {
  extern __shared__ __align__(16) float sh[];
  __shared__ double red[4 * (T / 64)];
  const int c = blockIdx.x, HW = g.H * g.W, E = g.N * HW, HWo = g.Ho * g.Wo;
  const size_t sample = (size_t)g.C * HW;
  const float hi1 = clamp_of(a.b1.act), hi2 = clamp_of(a.b2.act);
  float v[V];
  load_channel<Q, T, V>(a.x + (size_t)c * HW, sample, E, HW, g.p.mHW, v);
  // every word of the channel's parameters is requested here, not behind the barrier where it is used
  float wk[K * K];
#pragma unroll
  for (int t = 0; t < K * K; ++t) wk[t] = a.w[(size_t)c * (K * K) + t];
  const float gamma1 = a.b1.gamma[c], beta1 = a.b1.beta[c], gamma2 = a.b2.gamma[c], beta2 = a.b2.beta[c];
  have(gamma1); have(beta1); have(gamma2); have(beta2);
  const float rm1 = a.b1.running[c], rv1 = a.b1.running[g.C + c], rm2 = a.b2.running[c], rv2 = a.b2.running[g.C + c];
  for (int i = threadIdx.x; i < g.p.words4; i += T) reinterpret_cast<float4*>(sh)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < V; ++k)
    if (!holds<Q, T>(k, E)) v[k] = 0.f;
  double d1, d2;  // (the barrier in it is behind the zeros)
  block_sums<T>(tree_sum<V>([&](int k) { return v[k]; }), tree_sum<V>([&](int k) { return v[k] * v[k]; }), red, d1, d2);
  const Coef k1 = coefficients(d1, d2, g.inv, gamma1, beta1, a.b1.eps);
#pragma unroll
  for (int k = 0; k < V; ++k) v[k] = act_value<SW>(v[k] * k1.scale + k1.shift, hi1);
  store_padded<Q, T, V>(sh, g.p, E, v);
  __syncthreads();

  auto conv = [&](auto win, float (&o)[Q]) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      o[j] = 0.f;
#pragma unroll
      for (int u = 0; u < K; ++u)
#pragma unroll
        for (int q = 0; q < K; ++q) o[j] += wk[u * K + q] * win(u, q, j);
    }
  };
  constexpr int RM = V / Q;
  const Strip st = strip_of<Q>(g);
  float o[RM][Q] = {};
  each_window<K, S, Q, V>(sh, g, st, [&](int r, bool live, auto win) {
    conv(win, o[r]);
#pragma unroll
    for (int j = 0; j < Q; ++j) o[r][j] = live ? o[r][j] : 0.f;
  });
  block_sums<T>(tree_sum<V>([&](int k) { return o[k / Q][k % Q]; }),
                tree_sum<V>([&](int k) { return o[k / Q][k % Q] * o[k / Q][k % Q]; }), red + 2 * (T / 64), d1, d2);
  const Coef k2 = coefficients(d1, d2, g.inv_o, gamma2, beta2, a.b2.eps);
  const size_t at = ((size_t)st.n * g.C + c) * HWo + __mul24(st.r0, g.Wo) + st.col;
#pragma unroll
  for (int r = 0; r < RM; ++r) {
    if (r < st.rows) {
      float z[Q];
#pragma unroll
      for (int j = 0; j < Q; ++j) z[j] = act_value<SW>(o[r][j] * k2.scale + k2.shift, hi2);
      write_vec<Q>(a.y + at + r * g.Wo, o[r], 0);
      write_vec<Q>(a.z + at + r * g.Wo, z, 0);
    }
  }
  if (threadIdx.x == 0) {
    record(a.b1, c, g.C, k1, g.unb, rm1, rv1);
    record(a.b2, c, g.C, k2, g.unb_o, rm2, rv2);
  }
}

struct BwdArgs {
  const float* g;   // gradient of z
  const float* y;
  const float* x;
  const float* w;
  float* dx;        // may be NULL
  float* Gw;
  DwsBn b1, b2;
  float *Gg1, *Gb1, *Gg2, *Gb2;
};

// stride 2: the row (column) of the backward's window that tap u joins, and the parity of the pixel it joins it with
constexpr int dws_parity(int K, int u) { return (u + K / 2) & 1; }
constexpr int dws_tap(int K, int u) { return (dws_parity(K, u) + K / 2 - u) / 2 + (K == 3 ? 0 : 1); }

// f(row of the band, live, window) for every row of the strip of Q pixels (stride 2: Q quads of 2 x 2) of dx: window(u, v, j) is
// the entry of the padded gradient that tap (u, v) joins to strip entry j.
template <int K, int S, int Q, int V> constexpr int kGradRows = K == 5 && Q == 4 ? 1 : V / Q > 2 ? (Q == 1 ? 4 : 2) : V / Q;
template <int K, int S, int Q, int V, typename F>
__device__ __forceinline__ void each_gradient(const float* __restrict__ sh, const Geom& g, const Strip& st, F f) {
  constexpr int G = S == 1 ? K : (K + 1) / 2;            // window rows
  constexpr int UP = S == 1 ? K / 2 : (K == 3 ? 0 : 1);  // ... of them above the item's own row
  constexpr int R = V / Q < kGradRows<K, S, Q, V> ? V / Q : kGradRows<K, S, Q, V>;
  constexpr int NR = R + G - 1, NC = Q + G - 1, RIGHT = G - 1 - UP;
  const float* p = sh + g.p.lead + __mul24(st.n, g.p.PS) + __mul24(st.r0 - UP, g.p.RS) + st.col;
  auto row = [&](const float* s, float (&w)[NC]) {
#pragma unroll
    for (int b = 0; b < UP; ++b) w[b] = s[b - UP];
    read_vec<Q>(s, w, UP);
#pragma unroll
    for (int b = 0; b < RIGHT; ++b) w[UP + Q + b] = s[Q + b];
  };
  float win[NR][NC];
#pragma unroll
  for (int a = 0; a < G - 1; ++a) row(p + a * g.p.RS, win[a]);
  p += (G - 1) * g.p.RS;
#pragma unroll
  for (int r = 0; r < V / Q; r += R) {
    if (r < g.it.rows) {
#pragma unroll
      for (int a = 0; a < R; ++a) row(p + a * g.p.RS, win[G - 1 + a]);
      p += R * g.p.RS;
#pragma unroll
      for (int k = 0; k < R; ++k)
        f(r + k, r + k < st.rows, [&](int u, int v, int j) {
          return S == 1 ? win[k + K - 1 - u][j + K - 1 - v] : win[k + dws_tap(K, u)][j + dws_tap(K, v)];
        });
#pragma unroll
      for (int a = 0; a < G - 1; ++a)
#pragma unroll
        for (int b = 0; b < NC; ++b) win[a][b] = win[a + R][b];
    }
  }
}

template <int K, int S, bool SW, int Q, int T, int V>
__global__ __launch_bounds__(T) void dws_bwd_kernel(BwdArgs a, Geom g) {
  extern __shared__ __align__(16) float sh[];
  // a strip's row of x: Q pixels, or for stride 2 the 2 x 2Q pixels of its quads, 2Q of the upper row first
  constexpr int KK = K * K, NR = T / 16, RM = V / Q, XN = S * S * Q;
  __shared__ double red[4 * (T / 64)];
  __shared__ float wsum[NR * KK];
  const int c = blockIdx.x, HW = g.H * g.W, HWo = g.Ho * g.Wo, Eo = g.N * HWo;
  const size_t sample_o = (size_t)g.C * HWo;
  const float hi1 = clamp_of(a.b1.act), hi2 = clamp_of(a.b2.act);
  const Strip st = strip_of<Q>(g);
  const size_t at = ((size_t)st.n * g.C + c) * HW + __mul24(st.r0, g.W) * S + st.col * S;
  float xs[RM][XN];
  float mean1, istd1, sc1, sf1, gamma1, gb1, gg1, gw, wk[KK];

  // x as the strips need it, held to the end (past the end of a band or a plane: some row or column of it, not used).
  // Requested with y and g, or, where that would spill (more) registers, as soon as theirs are free.
  constexpr bool LATE = V >= 16 && (K == 5 || (V == 32 && Q < 4));
  auto load_x = [&] {
    const int last = max(st.rows, 1) - 1;
#pragma unroll
    for (int r = 0; r < RM; ++r) {
#pragma unroll
      for (int b = 0; b < S; ++b) {
        const float* const p = a.x + at + min(min(r, last) * S + b, g.H - 1 - st.r0 * S) * g.W;
        if (S == 2 && Q == 1) {
          xs[r][2 * b] = p[0];
          xs[r][2 * b + 1] = p[2 * st.col + 1 < g.W ? 1 : 0];
        } else {
#pragma unroll
          for (int q = 0; q < S; ++q) read_vec<Q>(p + q * Q, xs[r], (b * S + q) * Q);
        }
      }
    }
  };

  // the second BatchNorm's backward, in registers, into the padded copy
  {
    float gm[V], xh[V];
    load_channel<Q, T, V>(a.y + (size_t)c * HWo, sample_o, Eo, HWo, g.p.mHW, xh);
    load_channel<Q, T, V>(a.g + (size_t)c * HWo, sample_o, Eo, HWo, g.p.mHW, gm);
    if (!LATE) load_x();
    // every word of the channel's parameters is requested here, not where it is used (no other block adds to these sums)
    const float mean2 = a.b2.stat[c], istd2 = a.b2.stat[g.C + c], sc2 = a.b2.ss[c], sf2 = a.b2.ss[g.C + c];
    const float gamma2 = a.b2.gamma[c], gb2 = a.Gb2[c], gg2 = a.Gg2[c];
    mean1 = a.b1.stat[c]; istd1 = a.b1.stat[g.C + c]; sc1 = a.b1.ss[c]; sf1 = a.b1.ss[g.C + c];
    gamma1 = a.b1.gamma[c]; gb1 = a.Gb1[c]; gg1 = a.Gg1[c];
    gw = threadIdx.x < KK ? a.Gw[(size_t)c * KK + threadIdx.x] : 0.f;
#pragma unroll
    for (int t = 0; t < KK; ++t) wk[t] = a.w[(size_t)c * KK + t];
    have(mean1); have(istd1); have(sc1); have(sf1); have(mean2); have(istd2); have(sc2); have(sf2); have(gamma1); have(gamma2);
    for (int i = threadIdx.x; i < g.p.words4; i += T) reinterpret_cast<float4*>(sh)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      float val, slope;
      act_both<SW>(xh[k] * sc2 + sf2, hi2, val, slope);
      gm[k] = holds<Q, T>(k, Eo) ? gm[k] * slope : 0.f;
      xh[k] = holds<Q, T>(k, Eo) ? (xh[k] - mean2) * istd2 : 0.f;
    }
    double d1, d2;
    block_sums<T>(tree_sum<V>([&](int k) { return gm[k]; }), tree_sum<V>([&](int k) { return gm[k] * xh[k]; }), red, d1, d2);
    if (threadIdx.x == 0) {
      a.Gb2[c] = gb2 + (float)d1;
      a.Gg2[c] = gg2 + (float)d2;
    }
    // (m1 by itself off a rounded product loses the same part of m1 in every value: the next BatchNorm's sums, in which the
    // values cancel, came out 3 to 5 times as far off as with the term of xh added to it first)
    const float k2 = gamma2 * istd2, m1 = (float)(d1 * g.inv_o), m2 = (float)(d2 * g.inv_o);
#pragma unroll
    for (int k = 0; k < V; ++k) gm[k] = k2 * (gm[k] - fmaf(xh[k], m2, m1));
    store_padded<Q, T, V>(sh, g.p, Eo, gm);
  }
  if (LATE) load_x();
  __syncthreads();

  // input gradient of the convolution in front of the first activation, the weight gradient's sums, and those of the first
  // BatchNorm
  // The sums: a tree over all values where they are all held at once; for 5x5, which has no registers for that, trees over the
  // rows of a batch, added up (planes of 28x28, forward and backward: 3x3 4 % less time by the first, 5x5 9 % by the second)
  constexpr bool AT_END = K == 3;
  constexpr int R = kGradRows<K, S, Q, V>;
  float d[RM][XN], acc[KK], s1 = 0.f, s2 = 0.f, t1 = 0.f, t2 = 0.f;
  if (AT_END) {
#pragma unroll
    for (int k = 0; k < RM * XN; ++k) d[k / XN][k % XN] = 0.f;
  }
#pragma unroll
  for (int t = 0; t < KK; ++t) acc[t] = 0.f;
  // the pixel of strip entry j that tap (u, v) joins
  auto pixel = [](int u, int v, int j) { return S == 1 ? j : dws_parity(K, u) * 2 * Q + 2 * j + dws_parity(K, v); };
  // (stride 2, odd planes: the quads of the last row and column reach past them)
  auto outside = [&](int r, int k) { return S == 2 && Q == 1 && (2 * (st.r0 + r) + k / 2 >= g.H || 2 * st.col + k % 2 >= g.W); };
  each_gradient<K, S, Q, V>(sh, g, st, [&](int r, bool live, auto win) {
    float xt[XN], sl[XN], o[XN];
#pragma unroll
    for (int k = 0; k < XN; ++k) {
      act_both<SW>(xs[r][k] * sc1 + sf1, hi1, xt[k], sl[k]);
      if (!live || outside(r, k)) xt[k] = sl[k] = 0.f;
      o[k] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < K; ++u)
#pragma unroll
      for (int q = 0; q < K; ++q)
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          const float w = win(u, q, j);
          o[pixel(u, q, j)] += wk[u * K + q] * w;
          acc[u * K + q] += xt[pixel(u, q, j)] * w;
        }
#pragma unroll
    for (int k = 0; k < XN; ++k) d[r][k] = o[k] * sl[k];
    if (!AT_END) {
      const float a1 = tree_sum<XN>([&](int k) { return d[r][k]; });
      const float a2 = tree_sum<XN>([&](int k) { return d[r][k] * ((xs[r][k] - mean1) * istd1); });
      t1 = r % R ? t1 + a1 : a1;
      t2 = r % R ? t2 + a2 : a2;
      if (r % R == R - 1) {
        s1 += t1;
        s2 += t2;
      }
    }
  });
#pragma unroll
  for (int t = 0; t < KK; ++t) acc[t] = row16_sum(acc[t]);
  if ((threadIdx.x & 15) == 0) {
#pragma unroll
    for (int t = 0; t < KK; ++t) wsum[(threadIdx.x >> 4) * KK + t] = acc[t];
  }
  if (AT_END) {
    s1 = tree_sum<RM * XN>([&](int k) { return d[k / XN][k % XN]; });
    s2 = tree_sum<RM * XN>([&](int k) { return d[k / XN][k % XN] * ((xs[k / XN][k % XN] - mean1) * istd1); });
  }
  double d1, d2;
  block_sums<T>(s1, s2, red + 2 * (T / 64), d1, d2);
  if (a.dx) {
    const float k1 = gamma1 * istd1, m1 = (float)(d1 * g.inv), m2 = (float)(d2 * g.inv);
    float* const dp = a.dx + at;
#pragma unroll
    for (int r = 0; r < RM; ++r) {
      if (r < st.rows) {
#pragma unroll
        for (int k = 0; k < XN; ++k) d[r][k] = k1 * (d[r][k] - fmaf((xs[r][k] - mean1) * istd1, m2, m1));
#pragma unroll
        for (int b = 0; b < S * S; ++b) {
          float* const p = dp + (r * S + b / S) * g.W + b % S * Q;
          if (S == 1 || Q > 1) write_vec<Q>(p, d[r], b * Q);
          else if (!outside(r, b)) *p = d[r][b];
        }
      }
    }
  }
  if (threadIdx.x < KK) {
    double s = 0.0;
#pragma unroll 16
    for (int r = 0; r < NR; ++r) s += (double)wsum[r * KK + threadIdx.x];
    a.Gw[(size_t)c * KK + threadIdx.x] = gw + (float)s;
  }
  if (threadIdx.x == 64) {
    a.Gb1[c] = gb1 + (float)d1;
    a.Gg1[c] = gg1 + (float)d2;
  }
}

struct Pick {
  int T = 0, V = 0, Q = 1;
  size_t lds = 0;
  Geom g{};
};
// The smallest block of a pass that has a thread for every strip and registers for its rows; T = 0: a channel is too large.
Pick pick(bool bwd, int K, int N, int C, int H, int W, int S) {
  const int Ho = (H - 1) / S + 1, Wo = (W - 1) / S + 1;
  const int h = bwd ? Ho : H, w = bwd ? Wo : W, pad = bwd && S == 2 ? 1 : K / 2;
  const long E = (long)N * H * W, Eo = (long)N * Ho * Wo, held = (long)N * h * w;
  Pick p;
  if (E > 32768) return p;
  // strips: whole ones in every row, words of planes aligned, and (stride 2) no quad that reaches past the last row or column:
  // single ones check for that, wider strips would write the row behind a plane
  const bool even = H == S * Ho && W == S * Wo && (Ho * Wo) % 4 == 0 && (H * W) % 4 == 0;
  p.Q = even && Wo % 4 == 0 ? 4 : even && Wo % 2 == 0 ? 2 : 1;
  p.g = {N, C, H, W, Ho, Wo, div_by(H * W), 1.0 / (double)E, 1.0 / (double)Eo, (float)(E > 1 ? (double)E / (E - 1) : 1.0),
         (float)(Eo > 1 ? (double)Eo / (Eo - 1) : 1.0), padded(N, h, w, pad, p.Q), {}};
  constexpr int blocks[][2] = {{256, 4}, {512, 4}, {512, 8}, {1024, 8}, {1024, 16}, {1024, 32}};
  for (const auto& b : blocks) {
    if (bwd && S == 2 && b[1] > 8) break;  // (four pixels of x to an output)
    if (held > (long)b[0] * b[1]) continue;
    p.g.it = items_of(N, Ho, Wo / p.Q, b[0]);
    if (p.g.it.n <= 0 || p.g.it.n > b[0] || p.g.it.rows * p.Q > b[1]) continue;
    // rows behind the last that are read and not used: those that a shorter last band does not have, and of a last batch
    const long slack = (p.g.it.bands * p.g.it.rows - Ho + 3) * (bwd ? 1 : S);
    p.g.p.words4 = cdiv(N * (long)p.g.p.PS + p.g.p.lead + slack * p.g.p.RS, 4);
    p.lds = (size_t)p.g.p.words4 * 16;
    if (p.lds > (size_t)kLds) break;
    p.T = b[0];
    p.V = b[1];
    break;
  }
  return p;
}

// every kernel of (K, SW), by stride, strip and block
#define DWS_BLOCKS(S, Q, KERNEL) \
  f(S, Q, 256, 4, KERNEL<K, S, SW, Q, 256, 4>); \
  f(S, Q, 512, 4, KERNEL<K, S, SW, Q, 512, 4>); \
  f(S, Q, 512, 8, KERNEL<K, S, SW, Q, 512, 8>); \
  f(S, Q, 1024, 8, KERNEL<K, S, SW, Q, 1024, 8>);
#define DWS_LARGE(S, Q, KERNEL) \
  f(S, Q, 1024, 16, KERNEL<K, S, SW, Q, 1024, 16>); \
  f(S, Q, 1024, 32, KERNEL<K, S, SW, Q, 1024, 32>);
template <int K, bool SW, typename F>
void each_fwd(F f) {
  DWS_BLOCKS(1, 1, dws_fwd_kernel) DWS_BLOCKS(1, 2, dws_fwd_kernel) DWS_BLOCKS(1, 4, dws_fwd_kernel)
  DWS_LARGE(1, 1, dws_fwd_kernel) DWS_LARGE(1, 2, dws_fwd_kernel) DWS_LARGE(1, 4, dws_fwd_kernel)
  DWS_BLOCKS(2, 1, dws_fwd_kernel) DWS_BLOCKS(2, 2, dws_fwd_kernel) DWS_BLOCKS(2, 4, dws_fwd_kernel)
  DWS_LARGE(2, 1, dws_fwd_kernel) DWS_LARGE(2, 2, dws_fwd_kernel) DWS_LARGE(2, 4, dws_fwd_kernel)
}
template <int K, bool SW, typename F>
void each_bwd(F f) {
  DWS_BLOCKS(1, 1, dws_bwd_kernel) DWS_BLOCKS(1, 2, dws_bwd_kernel) DWS_BLOCKS(1, 4, dws_bwd_kernel)
  DWS_LARGE(1, 1, dws_bwd_kernel) DWS_LARGE(1, 2, dws_bwd_kernel) DWS_LARGE(1, 4, dws_bwd_kernel)
  DWS_BLOCKS(2, 1, dws_bwd_kernel) DWS_BLOCKS(2, 2, dws_bwd_kernel) DWS_BLOCKS(2, 4, dws_bwd_kernel)
}
#undef DWS_BLOCKS
#undef DWS_LARGE
template <typename F> void each_fwd_kernel(F f) {
  each_fwd<3, false>([&](auto... a) { f(3, false, a...); });
  each_fwd<3, true>([&](auto... a) { f(3, true, a...); });
  each_fwd<5, true>([&](auto... a) { f(5, true, a...); });
}
template <typename F> void each_bwd_kernel(F f) {
  each_bwd<3, false>([&](auto... a) { f(3, false, a...); });
  each_bwd<3, true>([&](auto... a) { f(3, true, a...); });
  each_bwd<5, true>([&](auto... a) { f(5, true, a...); });
}

}  // namespace

bool dws_supported(int K, int N, int C, int H, int W, int S, int act1, int act2) {
  const bool sw = act1 == ACT_SWISH;
  auto relu = [](int act) { return act == ACT_RELU || act == ACT_RELU6; };
  if (sw ? act2 != ACT_SWISH : !relu(act1) || !relu(act2)) return false;
  if (!(K == 3 || (K == 5 && sw)) || (S != 1 && S != 2)) return false;
  return pick(false, K, N, C, H, W, S).T && pick(true, K, N, C, H, W, S).T;
}

// Blocks of up to 16 values a thread are always the faster form (936 sizes: 1.05 times and more).  Those of 32, one to a compute
// unit, take a round of t = 14 us + their rows' time, filled or not, and spill registers in the 5x5 backward; the separate
// launches cost 27 us more at their start (20 where they read words of 16 bytes and these blocks single ones) and more for every
// value.  us of both directions, one launch / separate: 5x5, 31x31 x 27: 8 channels 72 / 44, 240 channels 109 / 149, 272
// 175 / 160; 3x3 with ReLU6 there: 8 channels 46 / 37, 96 57 / 67.  Fitted to 2048 sizes of such blocks, of which 206 are faster
// apart, down to 0.6; by this rule a call takes 0.14 % more than by the faster form of each.
bool dws_faster(int K, int N, int C, int H, int W, int S, int act) {
  const Pick p = pick(false, K, N, C, H, W, S);
  if (p.V < 32 || (S == 2 && p.Q > 1)) return true;
  const int kind = K == 5 ? 2 : act == ACT_SWISH ? 1 : 0;  // of ReLU, swish, 5x5:
  constexpr double row1[] = {0.9, 0.9, 1.6}, row[] = {0.4, 0.62, 0.95}, row2[] = {1.0, 1.0, 1.9};  // us per value in a strip's column
  constexpr double gain[] = {24, 28, 32}, gain2[] = {10, 12, 22};  // us per 256 channels of 10000 values
  const double t = 14 + p.g.it.rows * p.Q * (S == 2 ? row2 : p.Q == 1 ? row1 : row)[kind];
  const double apart = p.Q == 1 && H * W % 4 == 0 ? 20 : 27;
  return apart + (S == 2 ? gain2 : gain)[kind] * ((double)N * H * W / 1e4) * C / 256 >= cdiv(C, 256) * t;
}

hipError_t dws_allow(int K, int N, int C, int H, int W, int S, int act) {
  hipError_t e = hipSuccess;
  for (const bool bwd : {false, true}) {
    const Pick p = pick(bwd, K, N, C, H, W, S);
    auto allow = [&](int k, bool s, int S_, int Q, int T, int V, auto kern) {
      if (e == hipSuccess && p.lds > 48 * 1024 && k == K && s == (act == ACT_SWISH) && S_ == S && Q == p.Q && T == p.T && V == p.V)
        e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    };
    if (bwd) each_bwd_kernel(allow);
    else each_fwd_kernel(allow);
  }
  return e;
}

void dws_fwd_f32(hipStream_t st, const float* x, const float* w, float* y, float* z, const DwsBn& b1, const DwsBn& b2, int K,
                 int N, int C, int H, int W, int S) {
  const Pick p = pick(false, K, N, C, H, W, S);
  const FwdArgs a{x, w, y, z, b1, b2};
  const bool sw = b1.act == ACT_SWISH;
  each_fwd_kernel([&](int k, bool s, int S_, int Q, int T, int V, auto kern) {
    if (k == K && s == sw && S_ == S && Q == p.Q && T == p.T && V == p.V)
      KLAUNCH_NAMED("dws_fwd_kernel", kern, dim3(C), dim3(T), p.lds, st, a, p.g);
  });
}

void dws_bwd_f32(hipStream_t st, const float* gz, const float* y, const float* x, const float* w, float* dx, float* Gw,
                 float* Gg1, float* Gb1, float* Gg2, float* Gb2, const DwsBn& b1, const DwsBn& b2, int K, int N, int C, int H,
                 int W, int S) {
  const Pick p = pick(true, K, N, C, H, W, S);
  const BwdArgs a{gz, y, x, w, dx, Gw, b1, b2, Gg1, Gb1, Gg2, Gb2};
  const bool sw = b1.act == ACT_SWISH;
  each_bwd_kernel([&](int k, bool s, int S_, int Q, int T, int V, auto kern) {
    if (k == K && s == sw && S_ == S && Q == p.Q && T == p.T && V == p.V)
      KLAUNCH_NAMED("dws_bwd_kernel", kern, dim3(C), dim3(T), p.lds, st, a, p.g);
  });
}

}  // namespace ast

// The choice above, for tests that name one: strip, threads and values per thread of the forward (bwd: backward) block.
// 0: the run has no such launch; 1: it has one that the separate launches are faster than; 2: it runs so.
extern "C" int ast_dws_choice(int bwd, int K, int N, int C, int H, int W, int S, int act, int out[3]) {
  using namespace ast;
  if (!dws_supported(K, N, C, H, W, S, act, act)) return 0;
  const Pick p = pick(bwd != 0, K, N, C, H, W, S);
  out[0] = p.Q; out[1] = p.T; out[2] = p.V;
  return dws_faster(K, N, C, H, W, S, act) ? 2 : 1;
}
