// Temporal self-attention: for every (sample, location, head) the T frames attend to each other,
//   O = softmax(Q K^T / sqrt(dh)) V  over T <= 32 rows that lie a whole frame (S tokens) apart.
//
// The arithmetic is tiny (4 T A flop per token against 8 A bytes); what matters is how memory is
// touched: a (location, head) sequence is T pieces of 2 dh bytes, S rows apart.  A workgroup
// therefore takes FOUR neighbouring heads of one location, so that every row contributes one
// contiguous piece of 8 dh bytes per operand, fetched as 16-byte chunks, and the four workgroups
// of a location (16 heads) are dealt to the same XCD so that cache lines straddling two head
// groups are served from its L2.
//
// Short sequences are packed: a workgroup takes P neighbouring locations, R = P * T <= 32 rows (location-major), and
// the scores between different locations are masked.  LDS holds the R rows and no padding, so three workgroups of
// T = 30 fit a CU (1620 locations, 16 heads: 101 -> 95 us = 4.7 TB/s of q, k, v and O, bound by memory with rows
// in pieces of 576 bytes; 3600 locations, 4 heads: 62 -> 52 us).
//
// Each wavefront then owns one head.  R <= 32 fits a single 32x32 matrix-core tile:
// S^T = K Q^T (keys x queries; a lane owns one query, so the softmax is a register reduction
// plus one lane exchange), P^T rounded to bf16 is the second operand of O^T = V^T P^T as it
// stands, with V^T gathered from LDS in the key order the accumulator registers enumerate.
// The head dim is padded with zeros in registers only.  O is staged in LDS (over Q, which is
// dead by then) and written out as 16-byte chunks of whole rows.
#include "ddit_common.hpp"
#include <algorithm>

namespace {

constexpr int HG = 4;      // heads per workgroup, one per wavefront
constexpr int TP = 32;     // rows of the matrix-core tile

struct TemporalParams {
  const bf16_t *q, *k, *v;
  bf16_t *o;
  float *lse;
  int64_t ld_q, ld_kv, ld_o;
  int B, T, S, H;
  int n_hg;            // head groups per location
  int P, R;            // locations per workgroup; rows R = P * T
  int n_packs;         // workgroups a sample's locations take (a pack never holds two samples' locations)
  float inv_T;         // r / T = (int)((r + 0.5) * inv_T) for r < 32
  float scale_log2;    // log2(e) / sqrt(dh)
  float scale;         // 1 / sqrt(dh)
  // optional treatment of q and k on their way in (OPTS form of the kernel):
  const bf16_t *g_q, *g_k;   // per-head RMS-norm scales [dh], or null
  const float2 *rope;        // (cos, sin) of frame t, pair i at [t * dh/2 + i], or null
  float norm_eps;
  ddit::Prefetch ahead;
};

template <int DH>
struct TCfg {
  static constexpr int DCH = DH / 8;                 // 16-byte chunks per head row
  static constexpr int RCH = HG * DCH;               // chunks per LDS row (four heads)
  static constexpr int PITCH = RCH * 16 + 16;        // +16 B: 16 consecutive rows hit 16 different bank groups
  static constexpr int KS = (DH + 15) / 16;          // k-steps of Q K^T
  static constexpr int DT = (DH + 31) / 32;          // 32-row tiles of V^T
  static_assert((PITCH / 16) % 2 == 1, "odd pitch in 16-byte units keeps the reads conflict-free");
};

__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// OPTS: q and k are RMS-normalised per head and rotated by their frame's angles after they have
// landed in LDS (every sequence is loaded exactly once here, so this costs no memory traffic):
// one thread per (operand, row, head), two passes over its d_h elements, fp32 arithmetic,
// one rounding back to bf16.  Scales and the (cos, sin) rows of the T frames, 9 KB that all workgroups share, are read
// from cache into registers ahead of their use: a copy in LDS beside the operands let only two workgroups of T = 30
// onto a CU (T = 30, LDS / registers: 1620 locations, 16 heads 166 / 122 us; 3600, 4 heads 99 / 73; read where they are
// used, without the lead: 149 and 82, and short clips 5 % longer).
// PACK: more than one location per workgroup.
template <int DH, bool OPTS, bool PACK>
__global__ __launch_bounds__(256, 3) void k_temporal_attn(TemporalParams p) {
  using C = TCfg<DH>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // Q, K, V: R rows each
  if (blockIdx.y) {
    ddit::prefetch_share<256>(p.ahead);
    return;
  }
  const int R = p.R, MAT = R * C::PITCH;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lh = lane >> 5;

  // block -> (location, head group): the head groups of a location are 8 blocks apart (same XCD)
  const int xcd = blockIdx.x & 7;
  const int rest = blockIdx.x >> 3;
  const int hg = rest % p.n_hg;
  const int64_t pack = (int64_t)(rest / p.n_hg) * 8 + xcd;
  if (pack >= (int64_t)p.B * p.n_packs) return;
  const int b = (int)(pack / p.n_packs), s0 = (int)(pack - (int64_t)b * p.n_packs) * p.P;   // first location
  const int h0 = hg * HG;
  const int nh = p.H - h0 < HG ? p.H - h0 : HG;               // heads of this group that exist
  const int64_t tok0 = (int64_t)b * p.T * p.S + s0;           // token of row 0
  const int n_loc = p.S - s0 < p.P ? p.S - s0 : p.P;          // locations of this pack that exist
  const int rows = n_loc * p.T;
  auto loc_of = [&](int r) { return PACK ? (int)(((float)r + 0.5f) * p.inv_T) : 0; };
  auto row_token = [&](int r) {                               // row r = (location r / T, frame r % T)
    const int j = loc_of(r);
    return tok0 + j + (int64_t)(r - j * p.T) * p.S;
  };

  // OPTS: (operand, row, head) of this thread's treatment (R <= 32 and four heads: at most 256); its angles are on
  // their way before the operands
  const int t_hh = tid & 3, t_r = (tid >> 2) % TP, t_mat = tid / (4 * TP);
  const bool treats = OPTS && t_mat < 2 && t_r < rows && t_hh < nh;
  float4 ang[OPTS ? DH / 4 : 1];    // two (cos, sin) pairs each
  if constexpr (OPTS) {
    if (treats && p.rope) {
      const float4 *cs = reinterpret_cast<const float4 *>(p.rope) + (t_r - loc_of(t_r) * p.T) * (DH / 4);
#pragma unroll
      for (int c = 0; c < DH / 4; ++c) ang[c] = cs[c];
    }
  }

  // ---- operands -> LDS: the chunks of the existing locations and heads, zeros in the other rows.
  // All of a thread's loads are issued before the first one is used.
  {
    constexpr int NCH = (3 * TP * C::RCH + 255) / 256;
    uint4 val[NCH];
    int dst[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      dst[i] = -1;
      if (256 * i >= 3 * R * C::RCH) continue;
      const int m = tid + 256 * i;
      const int rr = m / C::RCH, ch = m - rr * C::RCH;           // rr = operand * R + row
      const int mat = (rr >= R) + (rr >= 2 * R);
      const int r = rr - mat * R;
      if (rr < 3 * R) dst[i] = rr * C::PITCH + ch * 16;
      val[i] = make_uint4(0u, 0u, 0u, 0u);
      if (rr < 3 * R && r < rows && ch < nh * C::DCH) {
        const int64_t tok = row_token(r);
        const bf16_t *src = mat == 0 ? p.q + tok * p.ld_q : (mat == 1 ? p.k + tok * p.ld_kv : p.v + tok * p.ld_kv);
        val[i] = *reinterpret_cast<const uint4 *>(src + h0 * DH + ch * 8);
      }
    }
#pragma unroll
    for (int i = 0; i < NCH; ++i)
      if (dst[i] >= 0) *reinterpret_cast<uint4 *>(smem + dst[i]) = val[i];
  }
  if constexpr (OPTS) {
    bf16x8 gain[C::DCH];   // in the registers that the operands have left
    if (treats && p.g_q) {
      const bf16x8 *g = reinterpret_cast<const bf16x8 *>(t_mat == 0 ? p.g_q : p.g_k);
#pragma unroll
      for (int c = 0; c < C::DCH; ++c) gain[c] = g[c];
    }
    wg_barrier();
    if (treats) {
      unsigned char *row = smem + t_mat * MAT + t_r * C::PITCH + t_hh * (DH * 2);
      float rinv = 1.0f;
      if (p.g_q) {
        float ss = 0.f;
#pragma unroll
        for (int c = 0; c < C::DCH; ++c) {
          const bf16x8 v = *reinterpret_cast<const bf16x8 *>(row + c * 16);
#pragma unroll
          for (int e = 0; e < 8; ++e) ss += (float)v[e] * (float)v[e];
        }
        rinv = rsqrtf(ss * (1.0f / DH) + p.norm_eps);
      }
#pragma unroll
      for (int c = 0; c < C::DCH; ++c) {
        bf16x8 v = *reinterpret_cast<const bf16x8 *>(row + c * 16);
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = (float)v[e] * rinv;
        if (p.g_q) {
#pragma unroll
          for (int e = 0; e < 8; ++e) f[e] *= (float)gain[c][e];
        }
        if (p.rope) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float4 a = ang[c * 2 + j];
            const float x0 = f[4 * j], x1 = f[4 * j + 1], x2 = f[4 * j + 2], x3 = f[4 * j + 3];
            f[4 * j] = x0 * a.x - x1 * a.y;
            f[4 * j + 1] = x1 * a.x + x0 * a.y;
            f[4 * j + 2] = x2 * a.z - x3 * a.w;
            f[4 * j + 3] = x3 * a.z + x2 * a.w;
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (bf16_t)f[e];
        *reinterpret_cast<bf16x8 *>(row + c * 16) = v;
      }
    }
  }
  wg_barrier();

  const int h = h0 + wave;
  floatx16 oacc[C::DT];
  float m_q = 0.f, l_q = 1.f;
  if (wave < nh) {
    // ---- S^T = K Q^T: lane holds key/query l32, d = 16 ks + 8 lh .. +7 (zeros past DH; rows >= R clamp)
    const int row = l32 < R ? l32 : R - 1;
    const unsigned char *qrow = smem + row * C::PITCH + wave * (DH * 2);
    const unsigned char *krow = qrow + MAT;
    const int first = loc_of(row) * p.T;      // the keys of this lane's query: first .. first + T - 1
    floatx16 sc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      const int c = 2 * ks + lh;
      bf16x8 qf, kf;
#pragma unroll
      for (int e = 0; e < 8; ++e) { qf[e] = (bf16_t)0.f; kf[e] = (bf16_t)0.f; }
      if (c < C::DCH) {
        qf = *reinterpret_cast<const bf16x8 *>(qrow + c * 16);
        kf = *reinterpret_cast<const bf16x8 *>(krow + c * 16);
      }
      sc = mfma32(kf, qf, sc);
    }
    // register r of this lane: key 8 (r >> 2) + 4 lh + (r & 3), query l32
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = 8 * (r >> 2) + 4 * lh + (r & 3);
      if (PACK ? (unsigned)(key - first) >= (unsigned)p.T : key >= p.T) sc[r] = -INFINITY;
      mx = fmaxf(mx, sc[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mb = mx * p.scale_log2;
    bf16x8 pf[2];
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bf16_t pb = (bf16_t)__builtin_amdgcn_exp2f(sc[r] * p.scale_log2 - mb);
      pf[r >> 3][r & 7] = pb;
      psum += (float)pb;      // the sum of what the matrix core will use
    }
    psum += __shfl_xor(psum, 32, 64);
    m_q = mx;
    l_q = psum;

    // ---- O^T = V^T P^T: first operand V^T[d = 32 dt + l32][key]; contraction index (kc, lh, j)
    // stands for key 16 kc + 8 (j >> 2) + 4 lh + (j & 3), the order of the accumulator registers
    const unsigned char *vcol = smem + 2 * MAT + wave * (DH * 2);
    auto pv = [&](floatx16 (&acc)[C::DT], int key0, int key1) {   // keys key0 .. key1 - 1
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt) {
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
        const int d = 32 * dt + l32;
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
          bf16x8 vf;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int key = 16 * kc + 8 * (j >> 2) + 4 * lh + (j & 3);
            uint16_t bits = 0;
            if (d < DH && key >= key0 && key < key1) bits = *reinterpret_cast<const uint16_t *>(vcol + key * C::PITCH + d * 2);
            vf[j] = __builtin_bit_cast(bf16_t, bits);
          }
          acc[dt] = mfma32(vf, pf[kc], acc[dt]);
        }
      }
    };
    pv(oacc, 0, R);
    if constexpr (PACK) {
      // A probability of zero times another location's infinity or NaN is a NaN that does not belong here: where a
      // result is not finite, the locations are multiplied one by one.
      bool finite = true;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) finite = finite && __builtin_fabsf(oacc[dt][e]) < INFINITY;
      if (__builtin_amdgcn_ballot_w64(!finite) != 0) {
#pragma unroll 1
        for (int j = 0; j < p.P; ++j) {
          floatx16 one[C::DT];
          pv(one, j * p.T, (j + 1) * p.T);
          if (first == j * p.T) {
#pragma unroll
            for (int dt = 0; dt < C::DT; ++dt) oacc[dt] = one[dt];
          }
        }
      }
    }
  }
  wg_barrier();   // every wavefront is done with Q: its place takes O

  if (wave < nh && l32 < rows) {
    // register r of tile dt: d = 32 dt + 8 (r >> 2) + 4 lh + (r & 3), query l32
    const float inv = 1.0f / l_q;
    unsigned char *orow = smem + l32 * C::PITCH + wave * (DH * 2);
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d0 = 32 * dt + 8 * g + 4 * lh;
        if (d0 < DH) {
          bf16x4 ov;
#pragma unroll
          for (int e = 0; e < 4; ++e) ov[e] = (bf16_t)(oacc[dt][4 * g + e] * inv);
          *reinterpret_cast<bf16x4 *>(orow + d0 * 2) = ov;
        }
      }
    if (p.lse && lh == 0) p.lse[row_token(l32) * p.H + h] = m_q * p.scale + __logf(l_q);
  }
  wg_barrier();
  {
    const int row_ch = nh * C::DCH;   // chunks of a row that hold existing heads
#pragma unroll 4
    for (int m = tid; m < rows * row_ch; m += 256) {
      const int r = m / row_ch, ch = m - r * row_ch;
      const uint4 val = *reinterpret_cast<const uint4 *>(smem + r * C::PITCH + ch * 16);
      *reinterpret_cast<uint4 *>(p.o + row_token(r) * p.ld_o + h0 * DH + ch * 8) = val;
    }
  }
}

template <int DH>
int launch_t(const TemporalParams &p, hipStream_t s) {
  const bool opts = p.g_q != nullptr || p.rope != nullptr;
  const int64_t packs = (int64_t)p.B * p.n_packs;
  const int64_t blocks = ((packs + 7) / 8) * p.n_hg * 8;
  if (blocks > 0x7fffffff) { ddit::set_error("temporal attention: too many workgroups"); return -2; }
  const dim3 grid((unsigned)blocks, ddit::prefetch_rows(p.ahead, blocks));
  const unsigned lds = 3u * p.R * TCfg<DH>::PITCH;
  if (opts) {
    if (p.P > 1) hipLaunchKernelGGL((k_temporal_attn<DH, true, true>), grid, dim3(256), lds, s, p);
    else hipLaunchKernelGGL((k_temporal_attn<DH, true, false>), grid, dim3(256), lds, s, p);
  } else {
    if (p.P > 1) hipLaunchKernelGGL((k_temporal_attn<DH, false, true>), grid, dim3(256), lds, s, p);
    else hipLaunchKernelGGL((k_temporal_attn<DH, false, false>), grid, dim3(256), lds, s, p);
  }
  return ddit::hip_fail(hipGetLastError(), "temporal attention launch");
}

}  // namespace

namespace ddit {

int temporal_attn_max_T() { return TP; }

int launch_temporal_attn(const void *q, const void *k, const void *v, void *o, float *lse, int64_t ld_q,
                         int64_t ld_kv, int64_t ld_o, int B, int T, int S, int H, int dh, const void *g_q,
                         const void *g_k, float norm_eps, const float *rope_table, const Prefetch &prefetch, hipStream_t s) {
  if (B == 0 || S == 0 || T == 0) return 0;
  if (T > TP) { set_error("temporal attention kernel: T=%d exceeds %d", T, TP); return -2; }
  TemporalParams p;
  p.q = reinterpret_cast<const bf16_t *>(q);
  p.k = reinterpret_cast<const bf16_t *>(k);
  p.v = reinterpret_cast<const bf16_t *>(v);
  p.o = reinterpret_cast<bf16_t *>(o);
  p.lse = lse;
  p.ld_q = ld_q; p.ld_kv = ld_kv; p.ld_o = ld_o;
  p.B = B; p.T = T; p.S = S; p.H = H;
  p.n_hg = (H + HG - 1) / HG;
  // Up to ten frames: as many locations as the tile holds.  One location per workgroup leaves most of the tile, of the
  // threads and (options) of the rows treated idle, and four times the workgroups; microseconds, one / packed:
  // 3680 tokens, T = 4: 24.8 / 12.9 (q/k treated: 34.1 / 13.6), 7360, T = 8: 29.4 / 20.7, 4050, T = 10: 16.4 / 15.0.
  // Above that a single location already keeps the loads coming, and more workgroups fit a CU: 2304, T = 16:
  // 10.2 / 11.9, 12960, T = 16: 33.3 / 35.4; T = 13: 21.9 / 20.0, treated 27.3 / 30.7.
  // But never fewer workgroups than CUs for it: where that many packs are not to be had, the power of two below (1, what
  // is taken / as many as the tile holds): 16 heads, T = 2, 144 locations 9.1, 9.1 / 10.6, 405 locations 15.0, 9.4 / 10.7;
  // 4 heads, T = 2, 144 locations 8.6, 8.6 / 10.5, 405 8.4, 8.4 / 10.6, T = 4, 920 11.9, 9.6 / 10.9, T = 8, 144 9.4,
  // 9.4 / 10.6.
  p.P = 1;
  if (T <= 10) {
    const int most = std::min(TP / T, S);
    const int64_t per_cu = (int64_t)B * S * p.n_hg / device_cus();
    if (per_cu >= most) p.P = most;
    else while (2 * p.P <= per_cu) p.P *= 2;
  }
  p.R = p.P * T;
  p.n_packs = (S + p.P - 1) / p.P;
  p.inv_T = 1.0f / (float)T;
  p.scale = 1.0f / sqrtf((float)dh);
  p.scale_log2 = p.scale * 1.4426950408889634f;
  p.g_q = reinterpret_cast<const bf16_t *>(g_q);
  p.g_k = reinterpret_cast<const bf16_t *>(g_k);
  p.rope = reinterpret_cast<const float2 *>(rope_table);
  p.norm_eps = norm_eps;
  p.ahead = prefetch;
  if (dh == 72) return launch_t<72>(p, s);
  if (dh == 64) return launch_t<64>(p, s);
  set_error("dh=%d: supported head dims are 64 and 72", dh);
  return -2;
}

}  // namespace ddit
