// Small stages: timestep conditioning (sinusoidal features -> 2-layer MLP -> adaLN-single
// projection), and the fp32 <-> bf16 casts at the ends of the residual stream.
//
// The conditioning touches B rows only (B is 1 or 2), so its three linears are
// matrix-vector products bound by reading the weights once: one wavefront per output
// feature, 16-byte weight loads, fp32 accumulation, wave reduction.
#include "ddit_common.hpp"

namespace {

struct TArgs { int B; float t[64]; };

// e[b, i] = cos(t_b f_i), e[b, 128+i] = sin(t_b f_i), f_i = 10000^(-i/128).
// Evaluated in fp64: t reaches 1000 rad, where fast fp32 sin/cos lose accuracy.
__global__ void k_timestep_features(TArgs a, float *__restrict__ e) {
  const int b = blockIdx.x, i = threadIdx.x;  // 128 threads
  const double f = exp(-log(10000.0) * (double)i / 128.0);
  const double arg = (double)a.t[b] * f;
  e[b * 256 + i] = (float)cos(arg);
  e[b * 256 + 128 + i] = (float)sin(arg);
}

// out[b, o] = sum_i act(in[b, i]) W[o, i] + bias[o];  act = SiLU if silu_in.
__global__ __launch_bounds__(256) void k_rowvec_linear(const float *__restrict__ in, const bf16_t *__restrict__ W,
                                                       const bf16_t *__restrict__ bias, int n_out, int n_in,
                                                       int silu_in, float *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int o = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int b = blockIdx.y;
  if (o >= n_out) return;
  const bf16_t *w = W + (int64_t)o * n_in;
  const float *x = in + (int64_t)b * n_in;
  float acc = 0.f;
  for (int i = lane * 8; i < n_in; i += 64 * 8) {
    const bf16x8 wv = *reinterpret_cast<const bf16x8 *>(w + i);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float xv = x[i + e];
      if (silu_in) xv = xv / (1.0f + __expf(-xv));
      acc += xv * (float)wv[e];
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) out[(int64_t)b * n_out + o] = acc + (bias ? (float)bias[o] : 0.f);
}

__global__ void k_bf16_to_f32(const bf16_t *__restrict__ in, float *__restrict__ out, int64_t n8) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n8) return;
  const bf16x8 v = reinterpret_cast<const bf16x8 *>(in)[i];
  float4 a, b;
  a.x = (float)v[0]; a.y = (float)v[1]; a.z = (float)v[2]; a.w = (float)v[3];
  b.x = (float)v[4]; b.y = (float)v[5]; b.z = (float)v[6]; b.w = (float)v[7];
  reinterpret_cast<float4 *>(out)[2 * i] = a;
  reinterpret_cast<float4 *>(out)[2 * i + 1] = b;
}

__global__ void k_f32_to_bf16(const float *__restrict__ in, bf16_t *__restrict__ out, int64_t n8) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n8) return;
  const float4 a = reinterpret_cast<const float4 *>(in)[2 * i];
  const float4 b = reinterpret_cast<const float4 *>(in)[2 * i + 1];
  bf16x8 v;
  v[0] = (bf16_t)a.x; v[1] = (bf16_t)a.y; v[2] = (bf16_t)a.z; v[3] = (bf16_t)a.w;
  v[4] = (bf16_t)b.x; v[5] = (bf16_t)b.y; v[6] = (bf16_t)b.z; v[7] = (bf16_t)b.w;
  reinterpret_cast<bf16x8 *>(out)[i] = v;
}

// x[n, :] + gate_b * sum of the pending parts' row n: rounded to bf16 into out (TO_BF16), or back into x
template <bool TO_BF16>
__global__ void k_add_pending(float *__restrict__ x, ddit::PendingSum pend, bf16_t *__restrict__ out, int64_t n4,
                              int d4, int64_t tokens_per_sample) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const int64_t row = i / d4;
  float4 part[ddit::MAX_PENDING_PARTS];
#pragma unroll
  for (int q = 0; q < ddit::MAX_PENDING_PARTS; ++q)   // all loads before the first use; a part too many reads the last one again
    part[q] = reinterpret_cast<const float4 *>(pend.part + (q < pend.parts ? q : pend.parts - 1) * pend.part_stride)[i];
  float4 a = part[0];
#pragma unroll
  for (int q = 1; q < ddit::MAX_PENDING_PARTS; ++q)
    if (q < pend.parts) { a.x += part[q].x; a.y += part[q].y; a.z += part[q].z; a.w += part[q].w; }
  const float4 g = ddit::pending_gate(pend, row / tokens_per_sample, (int)(i - row * d4));
  const float4 v = ddit::add_gated(reinterpret_cast<const float4 *>(x)[i], g, a);
  if constexpr (TO_BF16) {
    bf16x4 o;
    o[0] = (bf16_t)v.x; o[1] = (bf16_t)v.y; o[2] = (bf16_t)v.z; o[3] = (bf16_t)v.w;
    reinterpret_cast<bf16x4 *>(out)[i] = o;
  } else {
    reinterpret_cast<float4 *>(x)[i] = v;
  }
}

}  // namespace

namespace ddit {

int launch_cast_sum_to_bf16(const float *x, const PendingSum &pending, void *out, int64_t N, int64_t tokens_per_sample, int D,
                            hipStream_t s) {
  const int64_t n4 = N * (D / 4);
  if (n4 == 0) return 0;
  hipLaunchKernelGGL(k_add_pending<true>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, const_cast<float *>(x), pending,
                     reinterpret_cast<bf16_t *>(out), n4, D / 4, tokens_per_sample);
  return hip_fail(hipGetLastError(), "cast launch");
}

int launch_add_pending(float *x, const PendingSum &pending, int64_t N, int64_t tokens_per_sample, int D, hipStream_t s) {
  const int64_t n4 = N * (D / 4);
  if (n4 == 0) return 0;
  hipLaunchKernelGGL(k_add_pending<false>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, x, pending, nullptr, n4, D / 4,
                     tokens_per_sample);
  return hip_fail(hipGetLastError(), "pending sum launch");
}

int launch_cast_bf16_to_f32(const void *in, float *out, int64_t n, hipStream_t s) {
  const int64_t n8 = n / 8;  // callers guarantee n % 8 == 0
  if (n8 == 0) return 0;
  hipLaunchKernelGGL(k_bf16_to_f32, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const bf16_t *>(in), out, n8);
  return hip_fail(hipGetLastError(), "cast launch");
}

int launch_cast_f32_to_bf16(const float *in, void *out, int64_t n, hipStream_t s) {
  const int64_t n8 = n / 8;
  if (n8 == 0) return 0;
  hipLaunchKernelGGL(k_f32_to_bf16, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s, in,
                     reinterpret_cast<bf16_t *>(out), n8);
  return hip_fail(hipGetLastError(), "cast launch");
}

int launch_timestep_conditioning(const CondArgs &c, const void *w_t1, const void *b_t1, const void *w_t2,
                                 const void *b_t2, const void *w_ada, const void *b_ada, const float *temb_in,
                                 float *c6_out, float *scratch, hipStream_t s) {
  const int B = c.B, D = c.D;
  const float *temb = temb_in;
  if (!temb) {
    TArgs ta;
    ta.B = B;
    for (int i = 0; i < 64; ++i) ta.t[i] = i < B ? c.t[i] : 0.f;
    float *feat = scratch;            // [B,256]
    float *hid = scratch + B * 256;   // [B,D]
    float *tout = hid + B * D;        // [B,D]
    hipLaunchKernelGGL(k_timestep_features, dim3(B), dim3(128), 0, s, ta, feat);
    hipLaunchKernelGGL(k_rowvec_linear, dim3((D + 3) / 4, B), dim3(256), 0, s, feat,
                       reinterpret_cast<const bf16_t *>(w_t1), reinterpret_cast<const bf16_t *>(b_t1), D, 256, 0, hid);
    hipLaunchKernelGGL(k_rowvec_linear, dim3((D + 3) / 4, B), dim3(256), 0, s, hid,
                       reinterpret_cast<const bf16_t *>(w_t2), reinterpret_cast<const bf16_t *>(b_t2), D, D, 1, tout);
    temb = tout;
  }
  hipLaunchKernelGGL(k_rowvec_linear, dim3((6 * D + 3) / 4, B), dim3(256), 0, s, temb,
                     reinterpret_cast<const bf16_t *>(w_ada), reinterpret_cast<const bf16_t *>(b_ada), 6 * D, D, 1,
                     c6_out);
  return hip_fail(hipGetLastError(), "timestep conditioning launch");
}

}  // namespace ddit
