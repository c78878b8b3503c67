// fp32 pipeline of the verify-token pass (fp32 weights and cache) for gfx950, on the fp32 matrix
// cores (v_mfma_f32_16x16x4_f32: exact products of fp32 operands, fp32 sums). Per layer:
//
//   q/k/v projection, RMSNorm scale and rotary in its epilogue      -> q, k_self, v_self
//   attention (k_attn_f32 -> k_merge_mx, or k_attn_short_f32; kvprm_attn.hip)
//   output projection + residual (x += .., sums of squares, u = x * gamma_ffn)
//   gate/up projection + SwiGLU (RMSNorm scale)
//   down projection + residual (x += .., sums of squares, u = x * gamma_attn of the next layer)
//
// RMSNorm is applied as a per-candidate scale after the product: W (x gamma r) = r W (x gamma).
// The rotation is evaluated in fp64 (angles and products). Every reduction has a fixed order.
//
// Matrix-core operand layout (lane l, c = l / 16, n = l % 16): A holds row n, B column n, both
// reduction slot c; D holds rows 4c .. 4c+3 of column n. A 16-byte load gives a lane four
// consecutive inputs 4c .. 4c+3 of a 16-input block, which four products then contract one
// element at a time: any assignment of inputs to slots works if A and B use the same one, so both
// operands are read straight from row-major memory.
#include <math.h>
#include <string.h>

#include "kvprm_internal.h"
#include "kvprm_mx_common.h"

namespace kvprm {

// ------------------------------------------------------------------------------- init

// x_b = e_v, u = e_v * gamma_attn(0), the sums of squares per 16-row tile (one block each) and
// the rotary table (cos, sin in fp64) of position L_b.
__global__ __launch_bounds__(256) void k_init32(float *x, float *u, float *ss, const float *ev,
                                                const float *gamma0, int B, int H,
                                                const int32_t *lengths, float theta, int d,
                                                double *rope) {
  const int r0 = blockIdx.x * 16;
  for (int idx = threadIdx.x; idx < 16 * B; idx += 256) {
    const int r = r0 + (idx & 15), b = idx >> 4;
    const float v = ev[r];
    x[(size_t)b * H + r] = v;
    u[(size_t)b * H + r] = v * gamma0[r];
  }
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) sq += ev[r0 + i] * ev[r0 + i];
  if (threadIdx.x < B) ss[(size_t)blockIdx.x * B + threadIdx.x] = sq;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < B * (d / 2); e += gridDim.x * 256) {
    const int b = e / (d / 2), i = e - b * (d / 2);
    const double inv = pow((double)theta, (-2.0 * (double)i) / (double)d);
    double sn, cs;
    sincos((double)lengths[b] * inv, &sn, &cs);
    rope[2 * e] = cs;
    rope[2 * e + 1] = sn;
  }
}

// ------------------------------------------------------------------------------- projections

enum { F32_RESID = 1, F32_SWIGLU = 2, F32_ROPE = 3 };

struct F32Args {
  const float *w[3];  // row-major weight segments [rows_i][K], stacked rows
  int seg_rows[3];
  int nseg;
  int K;
  const float *in;  // [B][K]
  int B, H, F;
  float *x, *ss;       // residual stream and its sums of squares [H / 16][B]
  float eps;
  const float *gamma;  // gain of the next RMSNorm (RESID; null after the last layer)
  float *u;            // x * gamma (RESID)
  float *h;            // SwiGLU output [B][F]
  float *q, *ks, *vs;  // ROPE outputs
  const double *rope;
  int nq, nkv, d;
};

// A block owns MT row tiles (RESID one; SWIGLU the gate and the up tile; ROPE the two halves of a
// head's rotary pairs) over the whole input, for 16 NG candidates (grid y: further ones); its
// WPB waves split the input in blocks of 16, and their sums are added in LDS in wave order. At
// the small shapes this path serves, a launch is all latency: fusing the element-wise step and
// spreading one row tile over eight waves takes the place of one thread per row and separate
// kernels (two-layer shape H = 256, 4 candidates: 22 launches, 23-53 us per projection, 490 us a
// call, before; 14 launches and 63 us now).
template <int MT, int NG, int WPB, int EPI>
__global__ __launch_bounds__(64 * WPB) void k_gemv32(F32Args a) {
  constexpr int NC = 16 * NG, P = 64 * WPB / NC;  // candidates, threads per candidate (RMSNorm)
  constexpr int U = NG >= 4 ? 2 : 4;              // input blocks in flight
  constexpr bool RMS = EPI != F32_RESID;
  static_assert(P >= 1 && NG <= WPB, "one wave per candidate group in the epilogue");
  __shared__ floatx4 red_s[WPB][MT][NG][64];
  __shared__ float part_s[P][NC], inv_s[NC];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n = lane & 15, c = lane >> 4;
  const int B = a.B, K = a.K, b0 = blockIdx.y * NC;
  int tile[MT];
  tile[0] = blockIdx.x;
  if (EPI == F32_SWIGLU) tile[MT - 1] = blockIdx.x + a.F / 16;
  if (EPI == F32_ROPE) {
    const int half = a.d / 32;
    tile[0] = (blockIdx.x / half) * (a.d / 16) + blockIdx.x % half;
    tile[MT - 1] = tile[0] + half;
  }
  const float *wp[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    int seg = 0, base = 0;
    while (seg < a.nseg - 1 && tile[m] * 16 >= base + a.seg_rows[seg]) base += a.seg_rows[seg++];
    wp[m] = a.w[seg] + (size_t)(tile[m] * 16 - base + n) * K + 4 * c;
  }
  const float *up[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g)  // absent candidates repeat the last one (their columns are discarded)
    up[g] = a.in + (size_t)min(b0 + 16 * g + n, B - 1) * K + 4 * c;
  float sq = 0.f;  // this thread's share of its candidate's sum of squares
  if (RMS) {
    const int b = min(b0 + (int)threadIdx.x % NC, B - 1);
    for (int i = threadIdx.x / NC; i < a.H / 16; i += P) sq += a.ss[(size_t)i * B + b];
  }
  // what the epilogue reads besides (wave g: rows 4c .. 4c+3 of candidate n of group g), loaded now
  // so that no memory round trip is left for the end
  const int b = b0 + 16 * wave + n;
  const bool ok = wave < NG && b < B;
  const int bc = ok ? b : B - 1;
  const int r0 = tile[0] * 16 + 4 * c;
  floatx4 xv = {0.f, 0.f, 0.f, 0.f}, gm = xv;
  double rope[4][2];
  if (wave < NG && EPI == F32_RESID) {
    xv = *(const floatx4 *)(a.x + (size_t)bc * a.H + r0);
    if (a.gamma) gm = *(const f32x4u *)(a.gamma + r0);
  }
  if (wave < NG && EPI == F32_ROPE) {
    const double *rp = a.rope + ((size_t)bc * (a.d / 2) + r0 % a.d) * 2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      rope[i][0] = rp[2 * i];
      rope[i][1] = rp[2 * i + 1];
    }
  }
  floatx4 acc[MT][NG];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[m][g] = floatx4{0.f, 0.f, 0.f, 0.f};
  // this wave's input blocks [k0, k1), U at a time (wave-uniform bounds)
  const int nkb = K >> 4, per = (nkb + WPB - 1) / WPB;
  const int k0 = min(nkb, wave * per), k1 = min(nkb, k0 + per);
  f32x4u wa[U][MT], ua[U][NG], wb[U][MT], ub[U][NG];
  auto load = [&](int kb, f32x4u(&w)[U][MT], f32x4u(&u)[U][NG]) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (kb + i >= k1) break;
      const size_t k = (size_t)(kb + i) * 16;
#pragma unroll
      for (int m = 0; m < MT; ++m) w[i][m] = *(const f32x4u *)(wp[m] + k);
#pragma unroll
      for (int g = 0; g < NG; ++g) u[i][g] = *(const f32x4u *)(up[g] + k);
    }
  };
  auto mma = [&](int kb, const f32x4u(&w)[U][MT], const f32x4u(&u)[U][NG]) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (kb + i >= k1) break;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int g = 0; g < NG; ++g) acc[m][g] = mfma4(w[i][m][e], u[i][g][e], acc[m][g]);
    }
  };
  if (k0 < k1) {
    load(k0, wa, ua);
    for (int kb = k0; kb < k1; kb += 2 * U) {
      load(kb + U, wb, ub);
      mma(kb, wa, ua);
      load(kb + 2 * U, wa, ua);
      mma(kb + U, wb, ub);
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int g = 0; g < NG; ++g) red_s[wave][m][g][lane] = acc[m][g];
  if (RMS) part_s[threadIdx.x / NC][threadIdx.x % NC] = sq;
  __syncthreads();
  if (RMS) {
    if (threadIdx.x < NC) {
      float s = 0.f;
#pragma unroll
      for (int p = 0; p < P; ++p) s += part_s[p][threadIdx.x];
      inv_s[threadIdx.x] = 1.0f / sqrtf(s / (float)a.H + a.eps);
    }
    __syncthreads();
  }
  if (wave >= NG) return;
  // wave g: the outputs of candidate group g, rows 4c .. 4c+3 of column n
  floatx4 y[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    y[m] = red_s[0][m][wave][lane];
#pragma unroll
    for (int w = 1; w < WPB; ++w) {
      const floatx4 v = red_s[w][m][wave][lane];
#pragma unroll
      for (int i = 0; i < 4; ++i) y[m][i] += v[i];
    }
  }
  if (EPI == F32_RESID) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      xv[i] += y[0][i];
      s += xv[i] * xv[i];
    }
    s = column_sum(s);  // the tile's 16 rows
    if (!ok) return;
    *(floatx4 *)(a.x + (size_t)b * a.H + r0) = xv;
    if (a.gamma) {
#pragma unroll
      for (int i = 0; i < 4; ++i) gm[i] *= xv[i];
      *(floatx4 *)(a.u + (size_t)b * a.H + r0) = gm;
    }
    if (c == 0) a.ss[(size_t)tile[0] * B + b] = s;
    return;
  }
  if (!ok) return;
  const float inv = inv_s[16 * wave + n];
  if (EPI == F32_SWIGLU) {
    floatx4 hv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float gv = y[0][i] * inv, uv = y[MT - 1][i] * inv;
      hv[i] = gv / (1.0f + expf(-gv)) * uv;
    }
    *(floatx4 *)(a.h + (size_t)b * a.F + r0) = hv;
  } else {
    const int d = a.d, head = tile[0] / (d / 16);
    const bool rot = head < a.nq + a.nkv;
    float *dst = head < a.nq ? a.q + ((size_t)b * a.nq + head) * d
                 : rot       ? a.ks + ((size_t)b * a.nkv + head - a.nq) * d
                             : a.vs + ((size_t)b * a.nkv + head - a.nq - a.nkv) * d;
    floatx4 o1, o2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float y1 = y[0][i] * inv, y2 = y[MT - 1][i] * inv;
      const double cs = rope[i][0], sn = rope[i][1];
      o1[i] = rot ? (float)((double)y1 * cs - (double)y2 * sn) : y1;
      o2[i] = rot ? (float)((double)y2 * cs + (double)y1 * sn) : y2;
    }
    dst += r0 - head * d;  // the lane's first dimension (first half)
    *(floatx4 *)dst = o1;
    *(floatx4 *)(dst + d / 2) = o2;
  }
}

template <int MT, int EPI>
static hipError_t launch_gemv32(const F32Args &a, int blocks, hipStream_t s) {
  constexpr int WPB = 8;
  if (a.B <= 16)
    hipLaunchKernelGGL((k_gemv32<MT, 1, WPB, EPI>), dim3(blocks), dim3(64 * WPB), 0, s, a);
  else if (a.B <= 32)
    hipLaunchKernelGGL((k_gemv32<MT, 2, WPB, EPI>), dim3(blocks), dim3(64 * WPB), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemv32<MT, 4, WPB, EPI>), dim3(blocks, (a.B + 63) / 64), dim3(64 * WPB),
                       0, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------- sequencing

hipError_t launch_init_f32(const Dims &dm, const Plan &p, const Workspace &w, const void *ev,
                           const void *gamma0, const int32_t *lengths, hipStream_t s) {
  hipLaunchKernelGGL(k_init32, dim3(dm.H / 16), dim3(256), 0, s, w.x, w.u, w.ss,
                     (const float *)ev, (const float *)gamma0, p.B, dm.H, lengths, dm.theta, dm.d,
                     w.rope64);
  return hipGetLastError();
}

static F32Args f32_args(const Dims &dm, const Plan &p, const Workspace &w, const float *in, int K) {
  F32Args a;
  memset(&a, 0, sizeof a);
  a.in = in;
  a.K = K;
  a.B = p.B;
  a.H = dm.H;
  a.F = dm.F;
  a.x = w.x;
  a.ss = w.ss;
  a.eps = dm.eps;
  a.u = w.u;
  a.h = w.hffn;
  a.q = w.q;
  a.ks = w.kself;
  a.vs = w.vself;
  a.rope = w.rope64;
  a.nq = dm.nq;
  a.nkv = dm.nkv;
  a.d = dm.d;
  return a;
}

hipError_t launch_qkv_f32(const Dims &dm, const Plan &p, const Workspace &w, const void *wq,
                          const void *wk, const void *wv, hipStream_t s) {
  F32Args a = f32_args(dm, p, w, w.u, dm.H);
  a.w[0] = (const float *)wq;
  a.w[1] = (const float *)wk;
  a.w[2] = (const float *)wv;
  a.seg_rows[0] = dm.nq * dm.d;
  a.seg_rows[1] = a.seg_rows[2] = dm.nkv * dm.d;
  a.nseg = 3;
  return launch_gemv32<2, F32_ROPE>(a, (dm.nq + 2 * dm.nkv) * (dm.d / 32), s);
}

hipError_t launch_gateup_f32(const Dims &dm, const Plan &p, const Workspace &w, const void *wg,
                             const void *wu, hipStream_t s) {
  F32Args a = f32_args(dm, p, w, w.u, dm.H);
  a.w[0] = (const float *)wg;
  a.w[1] = (const float *)wu;
  a.seg_rows[0] = a.seg_rows[1] = dm.F;
  a.nseg = 2;
  return launch_gemv32<2, F32_SWIGLU>(a, dm.F / 16, s);
}

hipError_t launch_resid_f32(const Dims &dm, const Plan &p, const Workspace &w, const void *wt,
                            const float *in, int K, const void *gamma, hipStream_t s) {
  F32Args a = f32_args(dm, p, w, in, K);
  a.w[0] = (const float *)wt;
  a.seg_rows[0] = dm.H;
  a.nseg = 1;
  a.gamma = (const float *)gamma;
  return launch_gemv32<1, F32_RESID>(a, dm.H / 16, s);
}

}  // namespace kvprm
