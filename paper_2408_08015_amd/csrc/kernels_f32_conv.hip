// fp32 NCHW depthwise 3x3 convolution.
//
// The first kernels stage whole (n, c) planes (they are contiguous) with a zero halo in LDS; the
// backward kernel produces the input gradient and the nine weight-gradient sums of each plane from
// one read of g and x.  The ones behind them keep a window of rows in registers and take most shapes.
#include <algorithm>
#include "bn_common.h"
#include "device_utils.h"
#include "kernels.h"
#include "prof.h"

namespace ast {

static inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
static inline int conv_out(int H, int k, int stride, int pad) { return (H + 2 * pad - k) / stride + 1; }

// ============================================================== depthwise 3x3 (pad 1, stride 1 or 2)
struct DwGeom {
  int C, H, W, Ho, Wo, stride, ppb, NC;
};

// planes per block: about 4096 input elements per block, a power of two in [1, 16]
// planes per block of the LDS kernels: a power of two up to 16 with about 4096 elements per
// block, but fewer while that leaves under 1024 blocks (small tensors are latency-bound: more,
// shorter blocks, and one wavefront per plane in the BatchNorm prologues)
static int dw_ppb(int H, int W, long NC) {
  int p = 4096 / (H * W);
  int r = 1;
  while (r * 2 <= p && r < 16 && NC / (r * 2) >= 1024) r *= 2;
  return r;
}

// Zero `count` floats of LDS (all 256 threads), then barrier.
__device__ __forceinline__ void dw_zero(float* dst, int count) {
  for (int i = threadIdx.x; i < count; i += 256) dst[i] = 0.f;
  __syncthreads();
}
// Copy one h x w plane into an LDS plane of (h+2) x (w+2) (halo already zero) with the tpp
// threads of the plane's group (t = index in the group).  Four loads are issued before
// the first LDS write so the memory latency is paid once per four elements, not per element.
// With act >= 0 every element is first mapped to act(v*sc + sf): the plane is the input of a
// BatchNorm(+activation) whose output is never written out.
// `pre` (w % 4 == 0 only): the first four words of this thread, requested earlier with
// dw_stage_preload so that their latency overlaps the kernel's prologue.
struct DwPre { float4 v[4]; };
struct DwPreS { float v[4]; };  // the same for widths that are not multiples of four (4-byte words)
__device__ __forceinline__ void dw_stage_preload_s(DwPreS& pre, const float* __restrict__ src, int ne, int t, int tpp) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int e = t + u * tpp;
    pre.v[u] = e < ne ? src[e] : 0.f;
  }
}
__device__ __forceinline__ void dw_stage_preload(DwPre& pre, const float* __restrict__ src, int h, int w, int t,
                                                 int tpp) {
  const int nq = (h * w) >> 2;
  const float4* s4 = reinterpret_cast<const float4*>(src);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int q = t + u * tpp;
    pre.v[u] = q < nq ? s4[q] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}
__device__ __forceinline__ void dw_stage_plane(float* dst, const float* __restrict__ src, int h, int w, int t,
                                               int tpp, float sc = 1.f, float sf = 0.f, int act = -1,
                                               const DwPre* pre = nullptr, const DwPreS* pres = nullptr) {
  const int pw = w + 2;
  if ((w & 3) == 0) {
    const int nq = (h * w) >> 2, qpr = w >> 2;
    const float4* s4 = reinterpret_cast<const float4*>(src);
    for (int q0 = t; q0 < nq; q0 += 4 * tpp) {
      float4 v[4];
      if (pre && q0 == t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = pre->v[u];
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          int q = q0 + u * tpp;
          v[u] = q < nq ? s4[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        int q = q0 + u * tpp;
        if (q < nq) {
          int i = q / qpr, j = (q - i * qpr) * 4;
          float* d = dst + (i + 1) * pw + j + 1;
          if (act >= 0) {
            v[u].x = apply_act(v[u].x * sc + sf, act); v[u].y = apply_act(v[u].y * sc + sf, act);
            v[u].z = apply_act(v[u].z * sc + sf, act); v[u].w = apply_act(v[u].w * sc + sf, act);
          }
          d[0] = v[u].x; d[1] = v[u].y; d[2] = v[u].z; d[3] = v[u].w;
        }
      }
    }
  } else {
    const int ne = h * w;
    for (int e0 = t; e0 < ne; e0 += 4 * tpp) {
      float v[4];
      if (pres && e0 == t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = pres->v[u];
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          int e = e0 + u * tpp;
          v[u] = e < ne ? src[e] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        int e = e0 + u * tpp;
        if (e < ne) {
          int i = e / w, j = e - i * w;
          dst[(i + 1) * pw + j + 1] = act >= 0 ? apply_act(v[u] * sc + sf, act) : v[u];
        }
      }
    }
  }
}

__global__ __launch_bounds__(256) void dw3x3_fwd_f32_kernel(const float* __restrict__ x,
                                                            const float* __restrict__ w,
                                                            float* __restrict__ y, DwGeom gm, DwBnIn bi, DwBnOut bo) {
  extern __shared__ float sm[];
  const int PW = gm.W + 2, PSZ = (gm.H + 2) * PW;
  float* sx = sm;
  float* sw = sm + gm.ppb * PSZ;   // [ppb][9]
  float* scoef = sw + gm.ppb * 9;  // [ppb][2] scale, shift of the input BatchNorm
  double* sred = reinterpret_cast<double*>(sm + ((gm.ppb * (PSZ + 11) + 1) & ~1));  // [4 waves][2]
  const int plane0 = blockIdx.x * gm.ppb;
  const int np = min(gm.ppb, gm.NC - plane0);
  const int tpp = 256 / gm.ppb;
  const int pl = threadIdx.x / tpp, t = threadIdx.x - pl * tpp;
  const bool live = pl < np;
  // the first words of the plane are requested before the prologue and the LDS clear
  const bool vecw = (gm.W & 3) == 0;
  DwPre pre;
  DwPreS pres;
  if (live && vecw) dw_stage_preload(pre, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H, gm.W, t, tpp);
  if (live && !vecw) dw_stage_preload_s(pres, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H * gm.W, t, tpp);
  if (bi.on) {  // finish the statistics of each plane's channel: one wavefront per plane
    for (int q = threadIdx.x >> 6; q < np; q += 4) {
      const int plane = plane0 + q, c = plane % gm.C;
      double s1, s2;
      bn_add_partials(bi.ws, c, bi.P, s1, s2);
      if ((threadIdx.x & 63) == 0)  // the sample-0 plane of a channel records its statistics
        bn_coefficients(s1, s2, bi.count, bi.gamma[c], bi.beta[c], bi.eps, c, gm.C, plane < gm.C, bi.stat, bi.ss,
                        bi.running, scoef[2 * q], scoef[2 * q + 1]);
    }
  }
  dw_zero(sx, gm.ppb * PSZ);  // ends with a barrier: the coefficients are visible
  if (live) {
    if (bi.on)
      dw_stage_plane(sx + pl * PSZ, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H, gm.W, t, tpp, scoef[2 * pl],
                     scoef[2 * pl + 1], bi.act, vecw ? &pre : nullptr, vecw ? nullptr : &pres);
    else
      dw_stage_plane(sx + pl * PSZ, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H, gm.W, t, tpp, 1.f, 0.f, -1,
                     vecw ? &pre : nullptr, vecw ? nullptr : &pres);
  }
  for (int i = threadIdx.x; i < np * 9; i += 256) sw[i] = w[((plane0 + i / 9) % gm.C) * 9 + i % 9];
  __syncthreads();
  float s1 = 0.f, s2 = 0.f;
  if (live) {
    const float* wc = sw + pl * 9;
    const float w0 = wc[0], w1 = wc[1], w2 = wc[2], w3 = wc[3], w4 = wc[4], w5 = wc[5], w6 = wc[6], w7 = wc[7], w8 = wc[8];
    const float* sp = sx + pl * PSZ;
    float* yp = y + (size_t)(plane0 + pl) * gm.Ho * gm.Wo;
    const int s = gm.stride;
    for (int o = t; o < gm.Ho * gm.Wo; o += tpp) {
      int i = o / gm.Wo, j = o - i * gm.Wo;
      const float* b = sp + (i * s) * PW + j * s;
      float acc = w0 * b[0] + w1 * b[1] + w2 * b[2];
      acc += w3 * b[PW] + w4 * b[PW + 1] + w5 * b[PW + 2];
      acc += w6 * b[2 * PW] + w7 * b[2 * PW + 1] + w8 * b[2 * PW + 2];
      yp[o] = acc;
      s1 += acc;
      s2 += acc * acc;
    }
  }
  if (!bo.on) return;  // uniform
  // per-plane (sum, sum of squares) of the output for the BatchNorm that follows: fp32 per
  // thread, fp64 across the tpp threads of the plane (tpp is a power of two >= 16)
  double d1 = (double)s1, d2 = (double)s2;
  const int span = tpp < 64 ? tpp : 64;
  d1 = row16_sum(d1);
  d2 = row16_sum(d2);
  for (int o = 16; o < span; o <<= 1) {  // across the rows of 16 lanes of a wider plane group
    d1 += __shfl_xor(d1, o, 64);
    d2 += __shfl_xor(d2, o, 64);
  }
  const int plane = plane0 + pl;
  const int N = gm.NC / gm.C;
  double* out = bo.ws + ((size_t)(plane % gm.C) * N + plane / gm.C) * 2;
  if (tpp <= 64) {
    if (live && t == 0) {
      out[0] = d1;
      out[1] = d2;
    }
  } else {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
      sred[2 * wave] = d1;
      sred[2 * wave + 1] = d2;
    }
    __syncthreads();
    if (live && t == 0) {
      const int w0i = threadIdx.x >> 6, nw = tpp >> 6;
      double a = 0.0, b = 0.0;
      for (int q = 0; q < nw; ++q) {
        a += sred[2 * (w0i + q)];
        b += sred[2 * (w0i + q) + 1];
      }
      out[0] = a;
      out[1] = b;
    }
  }
}

// BatchNorm backward folded into the load of the conv's upstream gradient (see DwBwdFuse)
struct DwBnBwd {
  float k, m1, m2, mean, istd, sc, sf;
  int act;
};
__device__ __forceinline__ float dw_bn_dx(float g, float y, const DwBnBwd& b) {
  return b.k * (g * act_mask(y * b.sc + b.sf, b.act) - b.m1 - (y - b.mean) * b.istd * b.m2);
}
// whole wavefront: finish the backward sums of channel c; with `record` lane 0 adds dbeta, dgamma
__device__ __forceinline__ DwBnBwd dw_bn_bwd_coef(const DwBwdFuse& f, int c, int C, bool record) {
  double s1, s2;
  bn_add_partials(f.ws_out, c, f.P_out, s1, s2);
  DwBnBwd b;
  b.mean = f.ystat[c]; b.istd = f.ystat[C + c]; b.sc = f.yss[c]; b.sf = f.yss[C + c];
  b.k = f.ygamma[c] * b.istd;
  b.m1 = (float)(s1 / f.ycount);
  b.m2 = (float)(s2 / f.ycount);
  b.act = f.yact;
  if (record && (threadIdx.x & 63) == 0) {
    f.Gbeta[c] += (float)s1;
    f.Ggamma[c] += (float)s2;
  }
  return b;
}

// Input gradient (if dx) and the nine weight-gradient sums of every plane:
//   dx[i][j] = sum_{u,v} w[u][v] g[(i+1-u)/s][(j+1-v)/s]   (terms with a non-integer index drop)
//   part[plane][u*3+v] = sum_{i,j} g[i][j] x[i*s-1+u][j*s-1+v]
__global__ __launch_bounds__(256) void dw3x3_bwd_f32_kernel(const float* __restrict__ g,
                                                            const float* __restrict__ x,
                                                            const float* __restrict__ w,
                                                            float* __restrict__ dx, float* __restrict__ part,
                                                            DwGeom gm, DwBwdFuse f) {
  extern __shared__ float sm[];
  const int PW = gm.W + 2, PSZ = (gm.H + 2) * PW;
  const int GW = gm.Wo + 2, GSZ = (gm.Ho + 2) * GW;
  float* sx = sm;
  float* sg = sx + gm.ppb * PSZ;
  float* sw = sg + gm.ppb * GSZ;   // [ppb][9]
  float* sred = sw + gm.ppb * 9;   // [4 waves][11]
  float* scoef = sred + 44;        // [ppb][3]: k, m1, m2 of the BatchNorm behind the conv
  const int plane0 = blockIdx.x * gm.ppb;
  const int np = min(gm.ppb, gm.NC - plane0);
  const int tpp = 256 / gm.ppb;
  const int pl = threadIdx.x / tpp, t = threadIdx.x - pl * tpp;
  const bool live = pl < np;
  // Widths that are not multiples of four (the usual case here): a thread's first four words of
  // x, g (and y) are requested before the prologue and the LDS clear; the thread that stages
  // element e also computes dx[e], so x is not read again for the sums of the BatchNorm in front.
  const bool vecw = (gm.W & 3) == 0, vecg = (gm.Wo & 3) == 0;
  DwPreS xpre{}, gpre{}, ypre{};
  if (live && !vecw) dw_stage_preload_s(xpre, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H * gm.W, t, tpp);
  if (live && (f.y || !vecg)) {
    dw_stage_preload_s(gpre, g + (size_t)(plane0 + pl) * gm.Ho * gm.Wo, gm.Ho * gm.Wo, t, tpp);
    if (f.y) dw_stage_preload_s(ypre, f.y + (size_t)(plane0 + pl) * gm.Ho * gm.Wo, gm.Ho * gm.Wo, t, tpp);
  }
  if (f.y) {  // one wavefront per plane finishes the sums of the BatchNorm behind the conv
    for (int q = threadIdx.x >> 6; q < np; q += 4) {
      const DwBnBwd b = dw_bn_bwd_coef(f, (plane0 + q) % gm.C, gm.C, plane0 + q < gm.C);
      if ((threadIdx.x & 63) == 0) {
        scoef[3 * q] = b.k;
        scoef[3 * q + 1] = b.m1;
        scoef[3 * q + 2] = b.m2;
      }
    }
  }
  dw_zero(sx, gm.ppb * (PSZ + GSZ));  // sx and sg are adjacent; ends with a barrier
  const int ch = (plane0 + (live ? pl : 0)) % gm.C;
  if (live) {
    if (f.xss)  // x is the input of a BatchNorm(+activation) whose output the convolution saw
      dw_stage_plane(sx + pl * PSZ, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H, gm.W, t, tpp, f.xss[ch],
                     f.xss[gm.C + ch], f.xact, nullptr, vecw ? nullptr : &xpre);
    else
      dw_stage_plane(sx + pl * PSZ, x + (size_t)(plane0 + pl) * gm.H * gm.W, gm.H, gm.W, t, tpp, 1.f, 0.f, -1, nullptr,
                     vecw ? nullptr : &xpre);
    if (f.y) {  // the conv's upstream gradient = input gradient of the BatchNorm behind it
      DwBnBwd b;
      b.k = scoef[3 * pl]; b.m1 = scoef[3 * pl + 1]; b.m2 = scoef[3 * pl + 2];
      b.mean = f.ystat[ch]; b.istd = f.ystat[gm.C + ch]; b.sc = f.yss[ch]; b.sf = f.yss[gm.C + ch]; b.act = f.yact;
      const float* gsrc = g + (size_t)(plane0 + pl) * gm.Ho * gm.Wo;
      const float* ysrc = f.y + (size_t)(plane0 + pl) * gm.Ho * gm.Wo;
      float* dst = sg + pl * GSZ;
      const int ne = gm.Ho * gm.Wo;
      for (int e0 = t; e0 < ne; e0 += 4 * tpp) {
        float gv[4], yv[4];
        if (e0 == t) {
#pragma unroll
          for (int u = 0; u < 4; ++u) { gv[u] = gpre.v[u]; yv[u] = ypre.v[u]; }
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * tpp;
            gv[u] = e < ne ? gsrc[e] : 0.f;
            yv[u] = e < ne ? ysrc[e] : 0.f;
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = e0 + u * tpp;
          if (e < ne) {
            const int i = e / gm.Wo, jj = e - i * gm.Wo;
            dst[(i + 1) * GW + jj + 1] = dw_bn_dx(gv[u], yv[u], b);
          }
        }
      }
    } else {
      dw_stage_plane(sg + pl * GSZ, g + (size_t)(plane0 + pl) * gm.Ho * gm.Wo, gm.Ho, gm.Wo, t, tpp, 1.f, 0.f, -1, nullptr,
                     vecg ? nullptr : &gpre);
    }
  }
  for (int i = threadIdx.x; i < np * 9; i += 256) sw[i] = w[((plane0 + i / 9) % gm.C) * 9 + i % 9];
  __syncthreads();
  const int s = gm.stride;
  float acc[11];  // nine weight-gradient sums, then the two sums of the BatchNorm in front
#pragma unroll
  for (int k = 0; k < 11; ++k) acc[k] = 0.f;
  if (live) {
    const float* wc = sw + pl * 9;
    const float* gp = sg + pl * GSZ;
    const float* xp = sx + pl * PSZ;
    if (dx) {
      float* dp = dx + (size_t)(plane0 + pl) * gm.H * gm.W;
      const float* xraw = x + (size_t)(plane0 + pl) * gm.H * gm.W;
      const float mean1 = f.ws_in ? f.xstat[ch] : 0.f, istd1 = f.ws_in ? f.xstat[gm.C + ch] : 0.f;
      auto dx_at = [&](int e, float raw) {
        int i = e / gm.W, j = e - i * gm.W;
        float v = 0.f;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          int a = i + 1 - u;
          if (s == 2 && (a & 1)) continue;
          int io = s == 2 ? (a >> 1) : a;  // in [-1, Ho]: the halo holds zeros
#pragma unroll
          for (int v3 = 0; v3 < 3; ++v3) {
            int bb = j + 1 - v3;
            if (s == 2 && (bb & 1)) continue;
            int jo = s == 2 ? (bb >> 1) : bb;
            v += wc[u * 3 + v3] * gp[(io + 1) * GW + jo + 1];
          }
        }
        dp[e] = v;
        if (f.ws_in) {  // backward sums of the BatchNorm in front: g' = dx*act'(.), g'*xhat
          const float gmk = v * act_mask(xp[(i + 1) * PW + j + 1], f.xact);
          acc[9] += gmk;
          acc[10] += gmk * ((raw - mean1) * istd1);
        }
      };
      const int ne = gm.H * gm.W;
      int e = t;
      if (!vecw) {  // the first four elements of this thread: x is still in registers
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (t + u * tpp < ne) dx_at(t + u * tpp, xpre.v[u]);
        }
        e = t + 4 * tpp;
      }
      for (; e < ne; e += tpp) dx_at(e, f.ws_in ? xraw[e] : 0.f);
    }
    for (int o = t; o < gm.Ho * gm.Wo; o += tpp) {
      int i = o / gm.Wo, j = o - i * gm.Wo;
      float gv = gp[(i + 1) * GW + j + 1];
      const float* b = xp + (i * s) * PW + j * s;
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v3 = 0; v3 < 3; ++v3) acc[u * 3 + v3] += gv * b[u * PW + v3];
    }
  }
  // reduce the sums over the tpp threads of each plane (tpp is a power of two >= 16)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int span = tpp < 64 ? tpp : 64;
#pragma unroll
  for (int k = 0; k < 11; ++k) {
    acc[k] = row16_sum(acc[k]);
    for (int o = 16; o < span; o <<= 1) acc[k] += __shfl_xor(acc[k], o, 64);  // across rows of 16 lanes
  }
  const int N = gm.NC / gm.C;
  double* bws = f.ws_in ? f.ws_in + ((size_t)ch * N + (plane0 + pl) / gm.C) * 2 : nullptr;
  if (tpp <= 64) {
    if (live && t == 0) {
#pragma unroll
      for (int k = 0; k < 9; ++k) part[(size_t)(plane0 + pl) * 9 + k] = acc[k];
      if (bws) {
        bws[0] = (double)acc[9];
        bws[1] = (double)acc[10];
      }
    }
  } else {
    if (lane == 0)
#pragma unroll
      for (int k = 0; k < 11; ++k) sred[wave * 11 + k] = acc[k];
    __syncthreads();
    if (live && t == 0) {
      const int w0 = threadIdx.x >> 6, nw = tpp >> 6;
      float v[11];
      for (int k = 0; k < 11; ++k) {
        v[k] = 0.f;
        for (int q = 0; q < nw; ++q) v[k] += sred[(w0 + q) * 11 + k];
      }
      for (int k = 0; k < 9; ++k) part[(size_t)(plane0 + pl) * 9 + k] = v[k];
      if (bws) {
        bws[0] = (double)v[9];
        bws[1] = (double)v[10];
      }
    }
  }
}

// ============================================================== depthwise, register windows
// Kernels without LDS for widths that are a multiple of the strip width VW (4, 2 or 1 pixels:
// 16-, 8- or 4-byte accesses) with at most 64 strips per row: one wavefront per (n, c) plane
// (or per band of rows of a plane).  Lane (s = l % SW, rg = l / SW) owns the VW-pixel column
// strip s (SW = W/VW strips per row) of the rows of row group rg and slides a three-row
// register window down them; the columns left and right of a strip come from the neighbouring
// lanes, zeros at the image border.  Rows travel as raw words (zeros where not readable), some
// steps ahead, and are only transformed when they enter the window, so a load is not waited
// for before the rows ahead of it are used up.  Sums stay in registers and are reduced over
// the wavefront at the end.
template <int VW> struct DwVec { float e[VW]; };
template <int VW>
__device__ __forceinline__ DwVec<VW> dw_zero_vec() {
  DwVec<VW> r;
#pragma unroll
  for (int j = 0; j < VW; ++j) r.e[j] = 0.f;
  return r;
}
template <int VW>
__device__ __forceinline__ DwVec<VW> dw_ldv(const float* __restrict__ p) {
  DwVec<VW> r;
  if constexpr (VW == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    r.e[0] = t.x; r.e[1] = t.y; r.e[2] = t.z; r.e[3] = t.w;
  } else if constexpr (VW == 2) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    r.e[0] = t.x; r.e[1] = t.y;
  } else {
    r.e[0] = *p;
  }
  return r;
}
template <int VW>
__device__ __forceinline__ void dw_stv(float* __restrict__ p, const DwVec<VW>& v) {
  if constexpr (VW == 4) *reinterpret_cast<float4*>(p) = make_float4(v.e[0], v.e[1], v.e[2], v.e[3]);
  else if constexpr (VW == 2) *reinterpret_cast<float2*>(p) = make_float2(v.e[0], v.e[1]);
  else *p = v.e[0];
}
template <int VW>
__device__ __forceinline__ DwVec<VW> dw_norm(DwVec<VW> v, float sc, float sf, int act) {
#pragma unroll
  for (int j = 0; j < VW; ++j) v.e[j] = apply_act(v.e[j] * sc + sf, act);
  return v;
}
// a row of the window: v[0] = the column left of the strip, v[1..VW] = the strip, v[VW+1] = the
// column right of it
template <int VW> struct DwRow { float v[VW + 2]; };
template <int VW>
__device__ __forceinline__ DwRow<VW> dw_make_row(const DwVec<VW>& c, int s, int SW) {
  DwRow<VW> r;
  const float left = lane_up1(c.e[VW - 1]), right = lane_down1(c.e[0]);
  r.v[0] = s == 0 ? 0.f : left;
#pragma unroll
  for (int j = 0; j < VW; ++j) r.v[j + 1] = c.e[j];
  r.v[VW + 1] = s == SW - 1 ? 0.f : right;
  return r;
}

// Stride-1 backward: per row a lane issues one load of g, of x (and of y with a BatchNorm behind)
// and one store of dx.  D = rows requested ahead of the window.
template <int VW, int D>
__global__ __launch_bounds__(256) void dw3x3_bwd_s1_f32_kernel(const float* __restrict__ g,
                                                               const float* __restrict__ x,
                                                               const float* __restrict__ w, float* __restrict__ dx,
                                                               float* __restrict__ part, int NC, int C, int H,
                                                               int W, int RPG, DwBands bd, DwBwdFuse f) {
  typedef DwVec<VW> Vec;
  typedef DwRow<VW> Row;
  const int lane = threadIdx.x & 63;
  const int pb = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (pb >= NC * bd.bands) return;  // whole wavefront
  const int plane = pb / bd.bands, band = pb - plane * bd.bands;
  const int b0 = band * bd.rpb, b1 = min(b0 + bd.rpb, H);  // this wavefront's rows of the plane
  const int ch = plane % C;
  const int pidx = (plane / C) * bd.bands + band, nparts = (NC / C) * bd.bands;  // partial index, partials per channel
  const int SW = W / VW;
  const int rg = lane / SW, s = lane - rg * SW;
  const int r0 = b0 + rg * RPG;
  const int r1 = min(r0 + RPG, b1);  // lanes past the last group: r0 >= b1, no rows
  const float* gp = g + (size_t)plane * H * W + VW * s;
  const float* xp = x + (size_t)plane * H * W + VW * s;
  const float* yp = f.y ? f.y + (size_t)plane * H * W + VW * s : nullptr;
  float* dp = dx ? dx + (size_t)plane * H * W + VW * s : nullptr;
  float wk[9];
  const float* wc = w + (size_t)ch * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) wk[k] = wc[k];
  DwBnBwd yb{};
  // a row is readable by this lane if it lies in the image and the lane has rows at all
  const bool has = r0 < b1;
  auto rowok = [&](int row, bool ok) -> bool { return ok && has && row >= 0 && row < H; };
  struct Pend { Vec g, y, x; };
  auto load_row = [&](int row, bool ok) -> Pend {
    Pend q;
    q.g = q.y = q.x = dw_zero_vec<VW>();
    if (rowok(row, ok)) {
      q.g = dw_ldv<VW>(gp + (size_t)row * W);
      if (f.y) q.y = dw_ldv<VW>(yp + (size_t)row * W);
      q.x = dw_ldv<VW>(xp + (size_t)row * W);
    }
    return q;
  };
  auto use_g = [&](const Pend& q, bool valid) -> Vec {
    Vec gv = q.g;
    if (f.y && valid) {  // input gradient of the BatchNorm behind the conv
#pragma unroll
      for (int j = 0; j < VW; ++j) gv.e[j] = dw_bn_dx(gv.e[j], q.y.e[j], yb);
    }
    return gv;
  };
  // with xss the convolution's input was act(x*scale + shift) (a BatchNorm whose output is not
  // kept); the padding around it stays zero
  const float xsc = f.xss ? f.xss[ch] : 1.f, xsf = f.xss ? f.xss[C + ch] : 0.f;
  const float mean1 = f.ws_in ? f.xstat[ch] : 0.f, istd1 = f.ws_in ? f.xstat[C + ch] : 0.f;
  auto use_x = [&](const Pend& q, bool valid) -> Vec {
    return (f.xss && valid) ? dw_norm<VW>(q.x, xsc, xsf, f.xact) : q.x;
  };
  // the first rows are requested before the BatchNorm sums are finished
  const Pend pm = load_row(r0 - 1, true), pc = load_row(r0, true);
  Pend pn[D];
  pn[0] = load_row(r0 + 1, true);
#pragma unroll
  for (int d = 1; d < D; ++d) pn[d] = load_row(r0 + 1 + d, r0 + 1 + d <= r1);
  if (f.y) yb = dw_bn_bwd_coef(f, ch, C, plane < C && band == 0);
  Row gm = dw_make_row<VW>(use_g(pm, rowok(r0 - 1, true)), s, SW);
  Row gc = dw_make_row<VW>(use_g(pc, rowok(r0, true)), s, SW);
  Row xm = dw_make_row<VW>(use_x(pm, rowok(r0 - 1, true)), s, SW);
  Row xc = dw_make_row<VW>(use_x(pc, rowok(r0, true)), s, SW);
  Vec xcr = pc.x;
  float acc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.f;
  float bs1 = 0.f, bs2 = 0.f;
  for (int i = 0; i < RPG; ++i) {  // uniform trip count: the lane exchanges need every lane
    const int a = r0 + i;
    // past its last row a lane must not see the next group's rows as its own window
    const bool v1 = rowok(a + 1, a + 1 <= r1);
    const Row gq = dw_make_row<VW>(use_g(pn[0], v1), s, SW), xq = dw_make_row<VW>(use_x(pn[0], v1), s, SW);
    const Vec xqr = pn[0].x;
#pragma unroll
    for (int d = 0; d + 1 < D; ++d) pn[d] = pn[d + 1];
    pn[D - 1] = load_row(a + 1 + D, a + 1 + D <= r1);
    if (a < r1) {
      if (dp) {
        Vec o;
#pragma unroll
        for (int j = 0; j < VW; ++j) {
          float v = 0.f;
#pragma unroll
          for (int q = 0; q < 3; ++q) {  // dx[a][b] = sum_{u,q} w[u][q] g[a-u+1][b-q+1]
            v += wk[0 * 3 + q] * gq.v[j + 2 - q];
            v += wk[1 * 3 + q] * gc.v[j + 2 - q];
            v += wk[2 * 3 + q] * gm.v[j + 2 - q];
          }
          o.e[j] = v;
        }
        dw_stv<VW>(dp + (size_t)a * W, o);
        if (f.ws_in) {  // backward sums of the BatchNorm in front: g' = dx*act'(.), g'*xhat
#pragma unroll
          for (int j = 0; j < VW; ++j) {
            const float gmk = o.e[j] * act_mask(xc.v[j + 1], f.xact);
            bs1 += gmk;
            bs2 += gmk * ((xcr.e[j] - mean1) * istd1);
          }
        }
      }
#pragma unroll
      for (int j = 0; j < VW; ++j) {  // dW[u][q] += g[a][b] x[a+u-1][b+q-1]
        const float gv = gc.v[j + 1];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          acc[0 * 3 + q] += gv * xm.v[j + q];
          acc[1 * 3 + q] += gv * xc.v[j + q];
          acc[2 * 3 + q] += gv * xq.v[j + q];
        }
      }
    }
    gm = gc; gc = gq;
    xm = xc; xc = xq;
    xcr = xqr;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = wave_sum(acc[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 9; ++k) part[((size_t)pidx * C + ch) * 9 + k] = acc[k];
  if (f.ws_in) {
    const double d1 = wave_sum_d((double)bs1), d2 = wave_sum_d((double)bs2);
    if (lane == 0) {
      double* o = f.ws_in + ((size_t)ch * nparts + pidx) * 2;
      o[0] = d1;
      o[1] = d2;
    }
  }
}

// Stride-2 counterpart (VW = 4 or 2, H even): lane (s, rg) owns input columns VW*s .. VW*s+VW-1
// = output columns (VW/2)*s .., and per step one output row i = two input rows 2i, 2i+1.
// y[i][j] = sum_{u,q} w[u][q] x[2i+u-1][2j+q-1], so an even input row/column meets only the
// centre tap and an odd one the two outer taps of the neighbouring outputs.
template <int VW> struct DwG2 { float v[VW / 2 + 1]; };  // the strip's output columns and the one right of them
template <int VW> struct DwX2 { float v[VW + 1]; };      // the input column left of the strip, then the strip
template <int VW>
__device__ __forceinline__ DwG2<VW> dw_make_g2(const DwVec<VW / 2>& c, int s, int SW) {
  DwG2<VW> r;
  const float right = lane_down1(c.e[0]);
#pragma unroll
  for (int j = 0; j < VW / 2; ++j) r.v[j] = c.e[j];
  r.v[VW / 2] = s == SW - 1 ? 0.f : right;
  return r;
}
template <int VW>
__device__ __forceinline__ DwX2<VW> dw_make_x2(const DwVec<VW>& c, int s) {
  DwX2<VW> r;
  const float left = lane_up1(c.e[VW - 1]);
  r.v[0] = s == 0 ? 0.f : left;
#pragma unroll
  for (int j = 0; j < VW; ++j) r.v[j + 1] = c.e[j];
  return r;
}
// one input row of dx from the output-gradient rows that reach it through kernel rows wa / wb:
// an even input column c meets the centre tap of output column c/2, an odd one the outer taps
// of output columns (c-1)/2 and (c+1)/2
template <int VW>
__device__ __forceinline__ DwVec<VW> dw_dx_row2(const float* wa, const DwG2<VW>& ga, const float* wb,
                                                const DwG2<VW>& gb, bool two) {
  DwVec<VW> o;
#pragma unroll
  for (int c = 0; c < VW; ++c) {
    if (c % 2 == 0) o.e[c] = wa[1] * ga.v[c / 2];
    else o.e[c] = wa[0] * ga.v[(c + 1) / 2] + wa[2] * ga.v[(c - 1) / 2];
  }
  if (two) {
#pragma unroll
    for (int c = 0; c < VW; ++c) {
      if (c % 2 == 0) o.e[c] += wb[1] * gb.v[c / 2];
      else o.e[c] += wb[0] * gb.v[(c + 1) / 2] + wb[2] * gb.v[(c - 1) / 2];
    }
  }
  return o;
}
template <int VW>
__global__ __launch_bounds__(256) void dw3x3_bwd_s2_f32_kernel(const float* __restrict__ g,
                                                               const float* __restrict__ x,
                                                               const float* __restrict__ w, float* __restrict__ dx,
                                                               float* __restrict__ part, int NC, int C, int H,
                                                               int W, int RPG, DwBands bd, DwBwdFuse f) {
  constexpr int VG = VW / 2;  // output columns per lane
  typedef DwVec<VW> Vec;
  typedef DwVec<VG> VecG;
  const int lane = threadIdx.x & 63;
  const int pb = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (pb >= NC * bd.bands) return;  // whole wavefront
  const int plane = pb / bd.bands, band = pb - plane * bd.bands;
  const int ch = plane % C;
  const int pidx = (plane / C) * bd.bands + band, nparts = (NC / C) * bd.bands;  // partial index, partials per channel
  const int SW = W / VW, Ho = H >> 1, Wo = W >> 1;
  const int b0 = band * bd.rpb, b1 = min(b0 + bd.rpb, Ho);  // this wavefront's output rows
  const int rg = lane / SW, s = lane - rg * SW;
  const int r0 = b0 + rg * RPG;       // output rows [r0, r1)
  const int r1 = min(r0 + RPG, b1);
  const bool has = r0 < b1;
  const float* gp = g + (size_t)plane * Ho * Wo + VG * s;
  const float* yp = f.y ? f.y + (size_t)plane * Ho * Wo + VG * s : nullptr;
  const float* xp = x + (size_t)plane * H * W + VW * s;
  float* dp = dx ? dx + (size_t)plane * H * W + VW * s : nullptr;
  float wk[9];
  const float* wc = w + (size_t)ch * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) wk[k] = wc[k];
  DwBnBwd yb{};
  const float xsc = f.xss ? f.xss[ch] : 1.f, xsf = f.xss ? f.xss[C + ch] : 0.f;
  const float mean1 = f.ws_in ? f.xstat[ch] : 0.f, istd1 = f.ws_in ? f.xstat[C + ch] : 0.f;
  auto xok = [&](int row, bool ok) -> bool { return ok && has && row >= 0 && row < H; };
  auto gok = [&](int row, bool ok) -> bool { return ok && has && row >= 0 && row < Ho; };
  // the words of a step: input rows 2i, 2i+1, gradient row i+1
  struct Pend { Vec x0, x1; VecG g, y; };
  auto load_step = [&](int i, bool ok) -> Pend {
    Pend q;
    q.x0 = q.x1 = dw_zero_vec<VW>();
    q.g = q.y = dw_zero_vec<VG>();
    if (xok(2 * i, ok)) q.x0 = dw_ldv<VW>(xp + (size_t)(2 * i) * W);
    if (xok(2 * i + 1, ok)) q.x1 = dw_ldv<VW>(xp + (size_t)(2 * i + 1) * W);
    if (gok(i + 1, ok)) {
      q.g = dw_ldv<VG>(gp + (size_t)(i + 1) * Wo);
      if (f.y) q.y = dw_ldv<VG>(yp + (size_t)(i + 1) * Wo);
    }
    return q;
  };
  auto use_g = [&](VecG gv, const VecG& yv, bool valid) -> VecG {
    if (f.y && valid) {  // input gradient of the BatchNorm behind the conv
#pragma unroll
      for (int j = 0; j < VG; ++j) gv.e[j] = dw_bn_dx(gv.e[j], yv.e[j], yb);
    }
    return gv;
  };
  // with xss: the BatchNorm(+activation) output the convolution saw; the padding stays zero
  auto use_x = [&](const Vec& raw, bool valid) -> Vec {
    return (f.xss && valid) ? dw_norm<VW>(raw, xsc, xsf, f.xact) : raw;
  };
  // the first rows are requested before the BatchNorm sums are finished
  Vec xm_raw = dw_zero_vec<VW>();
  VecG gc_raw = dw_zero_vec<VG>(), yc_raw = dw_zero_vec<VG>();
  if (xok(2 * r0 - 1, true)) xm_raw = dw_ldv<VW>(xp + (size_t)(2 * r0 - 1) * W);
  if (gok(r0, true)) {
    gc_raw = dw_ldv<VG>(gp + (size_t)r0 * Wo);
    if (f.y) yc_raw = dw_ldv<VG>(yp + (size_t)r0 * Wo);
  }
  Pend p1 = load_step(r0, true), p2 = load_step(r0 + 1, r0 + 1 < r1);
  if (f.y) yb = dw_bn_bwd_coef(f, ch, C, plane < C && band == 0);
  DwX2<VW> xm = dw_make_x2<VW>(use_x(xm_raw, xok(2 * r0 - 1, true)), s);
  DwG2<VW> gc = dw_make_g2<VW>(use_g(gc_raw, yc_raw, gok(r0, true)), s, SW);
  float acc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.f;
  float bs1 = 0.f, bs2 = 0.f;
  for (int it = 0; it < RPG; ++it) {  // uniform trip count: the lane exchanges need every lane
    const int i = r0 + it;
    const bool ok = it == 0 || i < r1;  // a lane must not see the next group's rows as its own
    const DwX2<VW> x0 = dw_make_x2<VW>(use_x(p1.x0, xok(2 * i, ok)), s);
    const DwX2<VW> x1 = dw_make_x2<VW>(use_x(p1.x1, xok(2 * i + 1, ok)), s);
    const Vec x0r = p1.x0, x1r = p1.x1;
    const DwG2<VW> gq = dw_make_g2<VW>(use_g(p1.g, p1.y, gok(i + 1, ok)), s, SW);
    p1 = p2;
    p2 = load_step(i + 2, i + 2 < r1);
    if (i < r1) {
      if (dp) {
        // input row 2i: centre kernel row of output row i; row 2i+1: kernel row 0 of output
        // row i+1 and kernel row 2 of output row i
        const Vec d0 = dw_dx_row2<VW>(wk + 3, gc, wk + 3, gc, false);
        const Vec d1 = dw_dx_row2<VW>(wk + 0, gq, wk + 6, gc, true);
        dw_stv<VW>(dp + (size_t)(2 * i) * W, d0);
        dw_stv<VW>(dp + (size_t)(2 * i + 1) * W, d1);
        if (f.ws_in) {  // backward sums of the BatchNorm in front: g' = dx*act'(.), g'*xhat
#pragma unroll
          for (int j = 0; j < VW; ++j) {
            const float g0 = d0.e[j] * act_mask(x0.v[j + 1], f.xact), g1 = d1.e[j] * act_mask(x1.v[j + 1], f.xact);
            bs1 += g0 + g1;
            bs2 += g0 * ((x0r.e[j] - mean1) * istd1) + g1 * ((x1r.e[j] - mean1) * istd1);
          }
        }
      }
#pragma unroll
      for (int j = 0; j < VG; ++j) {  // dW[u][q] += g[i][j'] x[2i+u-1][2j'+q-1]
        const float gv = gc.v[j];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          acc[0 * 3 + q] += gv * xm.v[2 * j + q];
          acc[1 * 3 + q] += gv * x0.v[2 * j + q];
          acc[2 * 3 + q] += gv * x1.v[2 * j + q];
        }
      }
    }
    xm = x1;
    gc = gq;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = wave_sum(acc[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 9; ++k) part[((size_t)pidx * C + ch) * 9 + k] = acc[k];
  if (f.ws_in) {
    const double d1 = wave_sum_d((double)bs1), d2 = wave_sum_d((double)bs2);
    if (lane == 0) {
      double* o = f.ws_in + ((size_t)ch * nparts + pidx) * 2;
      o[0] = d1;
      o[1] = d2;
    }
  }
}

// Forward, the same lane layout: one load and one store per lane and row (stride 2: two loads,
// one half-width store); with a BatchNorm in front rows are normalised when they enter the
// window (padding stays zero).
template <int VW, int D>  // D = rows requested ahead of the window
__global__ __launch_bounds__(256) void dw3x3_fwd_s1_f32_kernel(const float* __restrict__ x,
                                                               const float* __restrict__ w, float* __restrict__ y,
                                                               int NC, int C, int H, int W, int RPG, DwBands bd,
                                                               DwBnIn bi, DwBnOut bo) {
  typedef DwVec<VW> Vec;
  typedef DwRow<VW> Row;
  const int lane = threadIdx.x & 63;
  const int pb = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (pb >= NC * bd.bands) return;  // whole wavefront
  const int plane = pb / bd.bands, band = pb - plane * bd.bands;
  const int b0 = band * bd.rpb, b1 = min(b0 + bd.rpb, H);  // this wavefront's rows of the plane
  const int ch = plane % C;
  const int pidx = (plane / C) * bd.bands + band, nparts = (NC / C) * bd.bands;  // partial index, partials per channel
  const int SW = W / VW;
  const int rg = lane / SW, s = lane - rg * SW;
  const int r0 = b0 + rg * RPG;
  const int r1 = min(r0 + RPG, b1);  // lanes past the last group: r0 >= b1, no rows
  const bool has = r0 < b1;
  const float* xp = x + (size_t)plane * H * W + VW * s;
  float* yp = y + (size_t)plane * H * W + VW * s;
  float wk[9];
  const float* wc = w + (size_t)ch * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) wk[k] = wc[k];
  auto rowok = [&](int row, bool ok) -> bool { return ok && has && row >= 0 && row < H; };
  auto load_row = [&](int row, bool ok) -> Vec {
    Vec v = dw_zero_vec<VW>();
    if (rowok(row, ok)) v = dw_ldv<VW>(xp + (size_t)row * W);
    return v;
  };
  // the first rows are requested before the statistics of the BatchNorm in front are finished
  const Vec pm = load_row(r0 - 1, true), pc = load_row(r0, true);
  Vec pn[D];
  pn[0] = load_row(r0 + 1, true);
#pragma unroll
  for (int d = 1; d < D; ++d) pn[d] = load_row(r0 + 1 + d, r0 + 1 + d <= r1);
  float sc = 1.f, sf = 0.f;
  if (bi.on) {  // every lane computes the same coefficients; lane 0 of a sample-0 plane records them
    double s1, s2;
    bn_add_partials(bi.ws, ch, bi.P, s1, s2);
    bn_coefficients(s1, s2, bi.count, bi.gamma[ch], bi.beta[ch], bi.eps, ch, C, plane < C && band == 0 && lane == 0,
                    bi.stat, bi.ss, bi.running, sc, sf);
  }
  auto use_x = [&](const Vec& raw, bool valid) -> Vec {
    return (bi.on && valid) ? dw_norm<VW>(raw, sc, sf, bi.act) : raw;
  };
  Row xm = dw_make_row<VW>(use_x(pm, rowok(r0 - 1, true)), s, SW);
  Row xc = dw_make_row<VW>(use_x(pc, rowok(r0, true)), s, SW);
  float t1 = 0.f, t2 = 0.f;
  for (int i = 0; i < RPG; ++i) {  // uniform trip count: the lane exchanges need every lane
    const int a = r0 + i;
    // past its last row a lane must not see the next group's rows as its own window
    const Row xq = dw_make_row<VW>(use_x(pn[0], rowok(a + 1, a + 1 <= r1)), s, SW);
#pragma unroll
    for (int d = 0; d + 1 < D; ++d) pn[d] = pn[d + 1];
    pn[D - 1] = load_row(a + 1 + D, a + 1 + D <= r1);
    if (a < r1) {
      Vec o;
#pragma unroll
      for (int j = 0; j < VW; ++j) {  // y[a][b] = sum_{u,q} w[u][q] x[a+u-1][b+q-1]
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          v += wk[0 * 3 + q] * xm.v[j + q];
          v += wk[1 * 3 + q] * xc.v[j + q];
          v += wk[2 * 3 + q] * xq.v[j + q];
        }
        o.e[j] = v;
        t1 += v;
        t2 += v * v;
      }
      dw_stv<VW>(yp + (size_t)a * W, o);
    }
    xm = xc;
    xc = xq;
  }
  if (bo.on) {  // (sum, sum of squares) of this wavefront's rows for the BatchNorm behind
    const double d1 = wave_sum_d((double)t1), d2 = wave_sum_d((double)t2);
    if (lane == 0) {
      double* o = bo.ws + ((size_t)ch * nparts + pidx) * 2;
      o[0] = d1;
      o[1] = d2;
    }
  }
}

// stride 2 (VW = 4 or 2, H even): per step one output row i = input rows 2i, 2i+1 (row 2i-1 is
// carried over)
template <int VW>
__global__ __launch_bounds__(256) void dw3x3_fwd_s2_f32_kernel(const float* __restrict__ x,
                                                               const float* __restrict__ w, float* __restrict__ y,
                                                               int NC, int C, int H, int W, int RPG, DwBands bd,
                                                               DwBnIn bi, DwBnOut bo) {
  constexpr int VG = VW / 2;  // output columns per lane
  typedef DwVec<VW> Vec;
  const int lane = threadIdx.x & 63;
  const int pb = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (pb >= NC * bd.bands) return;  // whole wavefront
  const int plane = pb / bd.bands, band = pb - plane * bd.bands;
  const int ch = plane % C;
  const int pidx = (plane / C) * bd.bands + band, nparts = (NC / C) * bd.bands;  // partial index, partials per channel
  const int SW = W / VW, Ho = H >> 1, Wo = W >> 1;
  const int b0 = band * bd.rpb, b1 = min(b0 + bd.rpb, Ho);  // this wavefront's output rows
  const int rg = lane / SW, s = lane - rg * SW;
  const int r0 = b0 + rg * RPG;  // output rows [r0, r1)
  const int r1 = min(r0 + RPG, b1);
  const bool has = r0 < b1;
  const float* xp = x + (size_t)plane * H * W + VW * s;
  float* yp = y + (size_t)plane * Ho * Wo + VG * s;
  float wk[9];
  const float* wc = w + (size_t)ch * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) wk[k] = wc[k];
  auto rowok = [&](int row, bool ok) -> bool { return ok && has && row >= 0 && row < H; };
  auto load_row = [&](int row, bool ok) -> Vec {
    Vec v = dw_zero_vec<VW>();
    if (rowok(row, ok)) v = dw_ldv<VW>(xp + (size_t)row * W);
    return v;
  };
  const Vec pm = load_row(2 * r0 - 1, true);
  Vec p1a = load_row(2 * r0, true), p1b = load_row(2 * r0 + 1, true);
  Vec p2a = load_row(2 * r0 + 2, r0 + 1 < r1), p2b = load_row(2 * r0 + 3, r0 + 1 < r1);
  float sc = 1.f, sf = 0.f;
  if (bi.on) {
    double s1, s2;
    bn_add_partials(bi.ws, ch, bi.P, s1, s2);
    bn_coefficients(s1, s2, bi.count, bi.gamma[ch], bi.beta[ch], bi.eps, ch, C, plane < C && band == 0 && lane == 0,
                    bi.stat, bi.ss, bi.running, sc, sf);
  }
  auto use_x = [&](const Vec& raw, bool valid) -> Vec {
    return (bi.on && valid) ? dw_norm<VW>(raw, sc, sf, bi.act) : raw;
  };
  DwX2<VW> xm = dw_make_x2<VW>(use_x(pm, rowok(2 * r0 - 1, true)), s);
  float t1 = 0.f, t2 = 0.f;
  for (int it = 0; it < RPG; ++it) {  // uniform trip count: the lane exchanges need every lane
    const int i = r0 + it;
    const bool ok = it == 0 || i < r1;  // a lane must not see the next group's rows as its own
    const DwX2<VW> x0 = dw_make_x2<VW>(use_x(p1a, rowok(2 * i, ok)), s);
    const DwX2<VW> x1 = dw_make_x2<VW>(use_x(p1b, rowok(2 * i + 1, ok)), s);
    p1a = p2a;
    p1b = p2b;
    p2a = load_row(2 * i + 4, i + 2 < r1);
    p2b = load_row(2 * i + 5, i + 2 < r1);
    if (i < r1) {
      DwVec<VG> o;
#pragma unroll
      for (int j = 0; j < VG; ++j) {  // y[i][j'] = sum_{u,q} w[u][q] x[2i+u-1][2j'+q-1]
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          v += wk[0 * 3 + q] * xm.v[2 * j + q];
          v += wk[1 * 3 + q] * x0.v[2 * j + q];
          v += wk[2 * 3 + q] * x1.v[2 * j + q];
        }
        o.e[j] = v;
        t1 += v;
        t2 += v * v;
      }
      dw_stv<VG>(yp + (size_t)i * Wo, o);
    }
    xm = x1;
  }
  if (bo.on) {
    const double d1 = wave_sum_d((double)t1), d2 = wave_sum_d((double)t2);
    if (lane == 0) {
      double* o = bo.ws + ((size_t)ch * nparts + pidx) * 2;
      o[0] = d1;
      o[1] = d2;
    }
  }
}

// G[c][t] += sum_n part[n][c][t]: eight sample lanes per output, fixed butterfly order
__global__ __launch_bounds__(256) void dw3x3_wgrad_final_kernel(const float* __restrict__ part,
                                                                float* __restrict__ G, int N, int C) {
  const int i = blockIdx.x * 32 + (threadIdx.x >> 3), nl = threadIdx.x & 7;
  float s = 0.f;
  if (i < C * 9)
    for (int n = nl; n < N; n += 8) s += part[(size_t)n * C * 9 + i];
  s = group8_sum(s);
  if (nl == 0 && i < C * 9) G[i] += s;
}

// The register-window kernels give a plane to one wavefront, or to several (each a band of
// rows) while there are too few planes to fill the chip; every wavefront leaves its own partial
// sums, so a channel has dw3x3_parts() partials instead of N.
// strip width of the register-window kernels for a shape: the widest of 4, 2, 1 pixels that
// divides W with at most 64 strips per row (stride 2: even H and W); 0 = LDS kernels
static int dw_vw(int H, int W, int stride) {
  if (stride == 2 && (H % 2 || W % 2)) return 0;
  if (stride != 1 && stride != 2) return 0;
  if (W % 4 == 0 && W / 4 <= 64) return 4;
  if (W % 2 == 0 && W / 2 <= 64) return 2;
  if (stride == 1 && W <= 64) return 1;
  return 0;
}
static DwBands dw_bands(int N, int C, int H, int W, int stride) {
  DwBands b{1, stride == 1 ? H : H / 2};
  const int vw = dw_vw(H, W, stride);
  if (!vw) return b;
  const int rows = b.rpb, groups = 64 / (W / vw);
  const long want = (4096 + (long)N * C - 1) / ((long)N * C);  // wavefronts wanted per plane
  const int cap = rows / (2 * groups) > 1 ? rows / (2 * groups) : 1;  // at least two rows per lane group
  int bands = (int)(want < cap ? want : cap);
  if (bands < 1) bands = 1;
  b.rpb = cdiv(rows, bands);
  b.bands = cdiv(rows, b.rpb);
  return b;
}
int dw3x3_parts(int N, int C, int H, int W, int stride) { return N * dw_bands(N, C, H, W, stride).bands; }
// Shapes the depthwise kernels cover: every shape with register windows; otherwise one padded
// plane of x and of g must fit the LDS kernels' 160 KB
bool dw3x3_supported(int H, int W, int stride) {
  if (stride != 1 && stride != 2) return false;
  if (dw_vw(H, W, stride)) return true;
  const long Ho = conv_out(H, 3, stride, 1), Wo = conv_out(W, 3, stride, 1);
  return ((long)(H + 2) * (W + 2) + (Ho + 2) * (Wo + 2) + 64) * 4 <= 150 * 1024;
}

static DwGeom dw_geom(int N, int C, int H, int W, int stride) {
  DwGeom gm;
  gm.C = C; gm.H = H; gm.W = W; gm.stride = stride;
  gm.Ho = conv_out(H, 3, stride, 1); gm.Wo = conv_out(W, 3, stride, 1);
  gm.NC = N * C;
  gm.ppb = dw_ppb(H, W, gm.NC);
  return gm;
}

void dw3x3_fwd_f32(hipStream_t st, const float* x, const float* w, float* y, int N, int C, int H, int W,
                   int stride, const DwBnIn* bn_in, double* stats_out) {
  DwBnIn bi{};
  if (bn_in) bi = *bn_in;
  DwBnOut bo{stats_out, stats_out != nullptr};
  if (const int vw = dw_vw(H, W, stride)) {
    const DwBands bd = dw_bands(N, C, H, W, stride);
    const int groups = 64 / (W / vw);
    const int rpg = cdiv(bd.rpb, groups);
    const dim3 grid(cdiv((long)N * C * bd.bands, 4));
#define DW_FWD(name, kern) KLAUNCH_NAMED(name, kern, grid, dim3(256), 0, st, x, w, y, N * C, C, H, W, rpg, bd, bi, bo)
    if (stride == 2) {
      if (vw == 4) DW_FWD("dw3x3_fwd_s2_f32_kernel<w4>", (dw3x3_fwd_s2_f32_kernel<4>));
      else DW_FWD("dw3x3_fwd_s2_f32_kernel<w2>", (dw3x3_fwd_s2_f32_kernel<2>));
    } else if (rpg <= 4) {  // short row groups: every row of a lane is requested up front
      if (vw == 4) DW_FWD("dw3x3_fwd_s1_f32_kernel<w4,4>", (dw3x3_fwd_s1_f32_kernel<4, 4>));
      else if (vw == 2) DW_FWD("dw3x3_fwd_s1_f32_kernel<w2,4>", (dw3x3_fwd_s1_f32_kernel<2, 4>));
      else DW_FWD("dw3x3_fwd_s1_f32_kernel<w1,4>", (dw3x3_fwd_s1_f32_kernel<1, 4>));
    } else {
      if (vw == 4) DW_FWD("dw3x3_fwd_s1_f32_kernel<w4,2>", (dw3x3_fwd_s1_f32_kernel<4, 2>));
      else if (vw == 2) DW_FWD("dw3x3_fwd_s1_f32_kernel<w2,2>", (dw3x3_fwd_s1_f32_kernel<2, 2>));
      else DW_FWD("dw3x3_fwd_s1_f32_kernel<w1,2>", (dw3x3_fwd_s1_f32_kernel<1, 2>));
    }
#undef DW_FWD
    return;
  }
  DwGeom gm = dw_geom(N, C, H, W, stride);
  // planes, weights, coefficients; then (8-byte aligned) four pairs of doubles
  size_t lds = ((((size_t)gm.ppb * ((H + 2) * (W + 2) + 11)) + 1) & ~(size_t)1) * sizeof(float) + 8 * sizeof(double);
  (void)hipFuncSetAttribute((const void*)dw3x3_fwd_f32_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  KLAUNCH(dw3x3_fwd_f32_kernel, dim3(cdiv(gm.NC, gm.ppb)), dim3(256), lds, st, x, w, y, gm, bi, bo);
}
size_t dw3x3_bwd_f32_ws(int N, int C, int H, int W, int stride) {
  return (size_t)dw3x3_parts(N, C, H, W, stride) * C * 9;
}
void dw3x3_bwd_f32(hipStream_t st, const float* g, const float* x, const float* w, float* dx, float* part,
                   float* G, int N, int C, int H, int W, int stride, const DwBwdFuse* fuse) {
  DwBwdFuse f;
  if (fuse) f = *fuse;
  if (!dx || !f.xss) f.ws_in = nullptr;  // those sums need dx and the normalised input
  if (const int vw = dw_vw(H, W, stride)) {
    const DwBands bd = dw_bands(N, C, H, W, stride);
    const int groups = 64 / (W / vw);
    const int rpg = cdiv(bd.rpb, groups);
    const dim3 grid(cdiv((long)N * C * bd.bands, 4));
#define DW_BWD(name, kern) KLAUNCH_NAMED(name, kern, grid, dim3(256), 0, st, g, x, w, dx, part, N * C, C, H, W, rpg, bd, f)
    // stride 1: two rows ahead; four cost a wavefront of occupancy at 16-byte strips (three tensors
    // per row) and measured slower there; narrow strips have the registers for it
    if (stride == 1) {
      if (vw == 4) DW_BWD("dw3x3_bwd_s1_f32_kernel<w4>", (dw3x3_bwd_s1_f32_kernel<4, 2>));
      else if (vw == 2) DW_BWD("dw3x3_bwd_s1_f32_kernel<w2>", (dw3x3_bwd_s1_f32_kernel<2, 4>));
      else DW_BWD("dw3x3_bwd_s1_f32_kernel<w1>", (dw3x3_bwd_s1_f32_kernel<1, 4>));
    } else {
      if (vw == 4) DW_BWD("dw3x3_bwd_s2_f32_kernel<w4>", (dw3x3_bwd_s2_f32_kernel<4>));
      else DW_BWD("dw3x3_bwd_s2_f32_kernel<w2>", (dw3x3_bwd_s2_f32_kernel<2>));
    }
#undef DW_BWD
    if (G) KLAUNCH(dw3x3_wgrad_final_kernel, dim3(cdiv(C * 9, 32)), dim3(256), 0, st, part, G, N * bd.bands, C);
    return;
  }
  DwGeom gm = dw_geom(N, C, H, W, stride);
  size_t lds =
      ((size_t)gm.ppb * ((H + 2) * (W + 2) + (gm.Ho + 2) * (gm.Wo + 2) + 9 + 3) + 44) * sizeof(float);
  (void)hipFuncSetAttribute((const void*)dw3x3_bwd_f32_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  KLAUNCH(dw3x3_bwd_f32_kernel, dim3(cdiv(gm.NC, gm.ppb)), dim3(256), lds, st, g, x, w, dx, part, gm, f);
  if (G) KLAUNCH(dw3x3_wgrad_final_kernel, dim3(cdiv(C * 9, 32)), dim3(256), 0, st, part, G, N, C);
}

}  // namespace ast
