// Fused adaLN-single modulation + LayerNorm:  out = bf16( LN(x) * (1 + scale_b) + shift_b ).
//
// LN is taken over the hidden axis without affine parameters and with the biased
// variance; (shift_b, scale_b) are two rows of the per-layer table plus the sample's
// conditioning vector.  The stage is HBM-bound (reads 4 B, writes 2 B per element), so
// the kernel keeps a token row of a wavefront entirely in registers: one pass over
// HBM, 16-byte loads, 8-byte stores, mean and variance by two wave reductions (the
// variance from the deviations, not from E[x^2]).
#include "ddit_common.hpp"

namespace {

// CHUNKS = float4 chunks per lane; D <= 256*CHUNKS.  A wavefront takes ROWS (1 or 2) consecutive token
// rows.  The sample's (1 + scale) and shift vectors, four vectors of D floats to read against one row of x,
// are formed once per workgroup and kept in LDS: read per row, or per wavefront, that traffic through the
// CU's vector cache costs as much time as the HBM side.  Rows of another sample than the workgroup's first
// row (the last rows of a sample, tiny shapes) read theirs from memory.
// PARTS > 0: a residual update that came as so many partial sums is added to the row first, and the row written back.
// Their number is known to the compiler so that all of a row's loads are in flight at once: in a loop over the parts each
// addition waited for its load, some fifteen memory latencies one after the other (kernel trace, 1152 features: 200 rows in
// three parts 10.4 -> 7.1 us, 2304 rows in two 12.4 -> 11.7; a layer of 64 tokens 92.7 -> 90.2 us, 200 89.8 -> 87.5).  Above 1280
// features that takes 136 to 256 registers, and so few rows leave them free: a block of 64 tokens and 1536 features 187.8 -> 183.8
// us, 2048 246.0 -> 240.1, 4096 461.3 -> 452.1; of 400 to 1200 tokens within 0.7 % either way.
template <int CHUNKS, int ROWS, bool STREAM, int PARTS>
__global__ __launch_bounds__(256) void k_modulated_layernorm(float *__restrict__ x,
                                                             const float *__restrict__ tab,
                                                             const float *__restrict__ c6, int which, int64_t N,
                                                             int64_t tokens_per_sample, int D, float eps,
                                                             bf16_t *__restrict__ out, ddit::PendingSum pend, ddit::Prefetch ahead) {
  if (blockIdx.y) {
    ddit::prefetch_share<256>(ahead);
    return;
  }
  extern __shared__ __attribute__((aligned(16))) float4 mod[];   // [2 (+ 1)][nchunk]: 1 + scale, shift (, gate of the pending update)
  const int lane = threadIdx.x & 63;
  const int64_t wg_row0 = (int64_t)blockIdx.x * (4 * ROWS);
  const int64_t row0 = wg_row0 + (threadIdx.x >> 6) * ROWS;
  const int nchunk = D >> 2;
  const float4 *t_shift = reinterpret_cast<const float4 *>(tab + (int64_t)(3 * which) * D);
  const float4 *t_scale = reinterpret_cast<const float4 *>(tab + (int64_t)(3 * which + 1) * D);
  auto modulation = [&](int64_t b, int c, float4 &sc1, float4 &sh) {
    const float4 *c_shift = reinterpret_cast<const float4 *>(c6 + b * 6 * (int64_t)D + (int64_t)(3 * which) * D);
    const float4 *c_scale = reinterpret_cast<const float4 *>(c6 + b * 6 * (int64_t)D + (int64_t)(3 * which + 1) * D);
    const float4 ts = t_shift[c], tc = t_scale[c], cs = c_shift[c], cc = c_scale[c];
    sh = make_float4(ts.x + cs.x, ts.y + cs.y, ts.z + cs.z, ts.w + cs.w);
    sc1 = make_float4(1.f + (tc.x + cc.x), 1.f + (tc.y + cc.y), 1.f + (tc.z + cc.z), 1.f + (tc.w + cc.w));
  };
  // the first row's loads are issued before the modulation vectors are fetched
  float4 v[CHUNKS];
  auto load_row = [&](int64_t row) {
    const floatx4 *xr = reinterpret_cast<const floatx4 *>(x + row * (int64_t)D);
#pragma unroll
    for (int j = 0; j < CHUNKS; ++j) {
      const int c = lane + 64 * j;
      v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (c < nchunk) {
        const floatx4 t = STREAM ? __builtin_nontemporal_load(xr + c) : xr[c];
        v[j] = make_float4(t[0], t[1], t[2], t[3]);
      }
    }
  };
  if (row0 < N) load_row(row0);
  constexpr bool SUM = PARTS > 0;
  float4 part[SUM ? PARTS : 1][CHUNKS];   // the row's pending update, before its gate
  if constexpr (SUM) {
    static_assert(ROWS == 1, "one row per wavefront");
    const int64_t row = row0 < N ? row0 : N - 1;
#pragma unroll
    for (int q = 0; q < PARTS; ++q)
#pragma unroll
      for (int j = 0; j < CHUNKS; ++j) {
        const int c = lane + 64 * j < nchunk ? lane + 64 * j : nchunk - 1;   // past the row: what is there, not used
        part[q][j] = reinterpret_cast<const float4 *>(pend.part + q * pend.part_stride + row * (int64_t)D)[c];
      }
  }
  const int64_t b_wg = wg_row0 / tokens_per_sample;
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    modulation(b_wg, c, mod[c], mod[nchunk + c]);
    if constexpr (SUM) mod[2 * nchunk + c] = ddit::pending_gate(pend, b_wg, c);
  }
  __syncthreads();
  if (row0 >= N) return;
  const int64_t row_end = row0 + ROWS < N ? row0 + ROWS : N;
  const int64_t wg_sample_end = (b_wg + 1) * tokens_per_sample;
#pragma unroll 1
  for (int64_t row = row0; row < row_end; ++row) {
    const bool here = row < wg_sample_end;
    if constexpr (SUM) {
      floatx4 *xw = reinterpret_cast<floatx4 *>(x + row * (int64_t)D);
#pragma unroll
      for (int j = 0; j < CHUNKS; ++j) {
        const int c = lane + 64 * j;
        if (c < nchunk) {
          const float4 g = here ? mod[2 * nchunk + c] : ddit::pending_gate(pend, row / tokens_per_sample, c);
          float4 a = part[0][j];
#pragma unroll
          for (int q = 1; q < PARTS; ++q) { a.x += part[q][j].x; a.y += part[q][j].y; a.z += part[q][j].z; a.w += part[q][j].w; }
          v[j] = ddit::add_gated(v[j], g, a);
          xw[c] = floatx4{v[j].x, v[j].y, v[j].z, v[j].w};
        }
      }
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < CHUNKS; ++j) s += (v[j].x + v[j].y) + (v[j].z + v[j].w);   // chunks past D hold zeros
    const float mean = wave_sum(s) / (float)D;
    float ss = 0.f;
    float4 dv[CHUNKS];
#pragma unroll
    for (int j = 0; j < CHUNKS; ++j) {
      dv[j] = make_float4(v[j].x - mean, v[j].y - mean, v[j].z - mean, v[j].w - mean);
      if (lane + 64 * j < nchunk) ss += (dv[j].x * dv[j].x + dv[j].y * dv[j].y) + (dv[j].z * dv[j].z + dv[j].w * dv[j].w);
    }
    // the next row is on its way while this one is reduced and written
    if (ROWS > 1 && row + 1 < row_end) load_row(row + 1);
    const float rstd = rsqrtf(wave_sum(ss) / (float)D + eps);
    bf16x4 *orow = reinterpret_cast<bf16x4 *>(out + row * (int64_t)D);
#pragma unroll
    for (int j = 0; j < CHUNKS; ++j) {
      const int c = lane + 64 * j;
      if (c < nchunk) {
        float4 sc1, sh;
        if (here) { sc1 = mod[c]; sh = mod[nchunk + c]; }
        else modulation(row / tokens_per_sample, c, sc1, sh);
        bf16x4 o;
        o[0] = (bf16_t)(dv[j].x * rstd * sc1.x + sh.x);
        o[1] = (bf16_t)(dv[j].y * rstd * sc1.y + sh.y);
        o[2] = (bf16_t)(dv[j].z * rstd * sc1.z + sh.z);
        o[3] = (bf16_t)(dv[j].w * rstd * sc1.w + sh.w);
        __builtin_nontemporal_store(o, orow + c);
      }
    }
  }
}

}  // namespace

namespace ddit {

template <int CHUNKS, int ROWS, bool STREAM, int PARTS>
void launch_ln(float *x, const float *tab, const float *c6, int which, int64_t N, int64_t tps, int D, float eps,
               bf16_t *o, const PendingSum &pend, const Prefetch &ahead, hipStream_t s) {
  const unsigned lds = (PARTS > 0 ? 3u : 2u) * (unsigned)D * 4u;   // at most 48 KB
  const unsigned blocks = (unsigned)((N + 4 * ROWS - 1) / (4 * ROWS));
  hipLaunchKernelGGL((k_modulated_layernorm<CHUNKS, ROWS, STREAM, PARTS>), dim3(blocks, prefetch_rows(ahead, blocks)), dim3(256),
                     lds, s, x, tab, c6, which, N, tps, D, eps, o, pend, ahead);
}
template <int CHUNKS>
void launch_ln(float *x, const float *tab, const float *c6, int which, int64_t N, int64_t tps, int D, float eps,
               bf16_t *o, const PendingSum *pend, const Prefetch &ahead, hipStream_t s) {
  // A wavefront with a second row hides its latency behind the first one's reductions; below 8192 rows there are
  // not four wavefronts per SIMD and the second row only makes the launch longer.  D = 1152, 1 / 2 rows: 256 rows
  // 3.5 / 4.8 us, 2304 rows 5.6 / 6.2 us, 12960 rows 19.6 / 19.8 us, 48600 rows 53.1 / 50.1 us (6.7 TB/s).
  // Wider rows fill the registers by themselves, and a second one takes away wavefronts (D = 2048, 1 / 2 rows: 12960 rows
  // 28.5 / 29.8 us, 48600 92.3 / 94.4; D = 4096: 12960 55.8 / 71.9, 48600 196 / 231).
  // A stream too large for the memory-side cache is read past the L2, which keeps other launches' weights, and past
  // that cache, which keeps what is read again (plain / streaming: 20000 rows of 1280, 26 M elements, 31.6 / 26.6 us;
  // 12960 of 2048, 27 M, 33.9 / 28.5; 108000 of 256, 28 M, 40.8 / 36.2; 20000 of 1152, 23 M, 25.1 / 24.5).
  constexpr int ROWS = CHUNKS <= 5 ? 2 : 1;
  const PendingSum none = {0, nullptr, 0, nullptr, nullptr, 0};
  if (pend && pend->parts == 2) launch_ln<CHUNKS, 1, false, 2>(x, tab, c6, which, N, tps, D, eps, o, *pend, ahead, s);
  else if (pend && pend->parts == 3) launch_ln<CHUNKS, 1, false, 3>(x, tab, c6, which, N, tps, D, eps, o, *pend, ahead, s);
  else if (N < 8192) launch_ln<CHUNKS, 1, false, 0>(x, tab, c6, which, N, tps, D, eps, o, none, ahead, s);
  else if (N * (int64_t)D <= (int64_t)24 << 20) launch_ln<CHUNKS, ROWS, false, 0>(x, tab, c6, which, N, tps, D, eps, o, none, ahead, s);
  else launch_ln<CHUNKS, ROWS, true, 0>(x, tab, c6, which, N, tps, D, eps, o, none, ahead, s);
}

int launch_modulated_layernorm(float *x, const float *ada_table, const float *c6, int which, int64_t N,
                               int64_t tokens_per_sample, int D, float eps, void *out, hipStream_t s,
                               const PendingSum *pending, const Prefetch &ahead) {
  if (N == 0) return 0;
  if (pending && (pending->parts < 0 || pending->parts > MAX_PENDING_PARTS || pending->parts == 1)) {
    set_error("modulated_layernorm: a pending update in %d parts", pending->parts);
    return -2;
  }
  bf16_t *o = reinterpret_cast<bf16_t *>(out);
  if (D <= 256 * 2) launch_ln<2>(x, ada_table, c6, which, N, tokens_per_sample, D, eps, o, pending, ahead, s);
  else if (D <= 256 * 5) launch_ln<5>(x, ada_table, c6, which, N, tokens_per_sample, D, eps, o, pending, ahead, s);
  else if (D <= 256 * 8) launch_ln<8>(x, ada_table, c6, which, N, tokens_per_sample, D, eps, o, pending, ahead, s);
  else if (D <= 256 * 16) launch_ln<16>(x, ada_table, c6, which, N, tokens_per_sample, D, eps, o, pending, ahead, s);
  else {
    set_error("D=%d: hidden size above 4096 is not supported by the LayerNorm kernel", D);
    return -2;
  }
  return hip_fail(hipGetLastError(), "modulated_layernorm launch");
}

}  // namespace ddit
