// bf16 Linear  out = u W^T + b  on the CDNA4 matrix cores, with fused epilogues.
//
// u is [N,k] tokens x in-features, W is [n,k]: both operands have the contraction axis
// contiguous, which is exactly what v_mfma_f32_32x32x16_bf16 wants in its registers
// (8 consecutive k per lane), so tiles go global -> LDS -> registers as 16-byte pieces
// with no transposition anywhere.
//
// Tiling.  A workgroup of WGM x WGN (x WGK) wavefronts owns a BM x BN tile of the output (BM tokens,
// BN out-features); a wavefront owns TM x TN MFMA tiles of 32x32 with fp32 accumulators in
// registers.  The MFMA is issued with W as its first operand and u as its second, so a lane
// ends up holding, for one token, 4 consecutive out-features per accumulator group.
// The main configuration is 192 x 384 with eight wavefronts (2 x 4, each 96 x 96): the
// accumulators fill half of the compute unit's register file and a tile does 128 flop per byte
// fetched (384 divides the model's widths 1152, 3456 and 4608).  Small tiles also run eight
// wavefronts, two per SIMD, so that one's LDS reads run under the other's MFMAs: WGK = 2 gives
// each half of every k-step to a different set of wavefronts, whose partial sums meet in LDS once
// per tile.
//
// Operand path.  k is walked in steps of 64, i.e. whole 128-byte cache lines of every operand row:
// a row piece of 64 bytes (32 of k) costs the path from L2 into the CU as much as a whole line does
// (measured with a load-only loop over the tiles of 192 x 384, all CUs busy: 58 bytes per ns and CU
// with 64-byte pieces, 96 with 128-byte ones), and that path is what the k loop waits for.  Tiles go
// global -> LDS with 16-byte buffer loads: no staging registers, no ds_write; the resource descriptor
// carries the tile's base and what is left of the matrix, so rows past the end are not fetched, and a
// lane needs one offset per operand for the whole kernel.  The loads of NS k-steps are in flight in
// NS LDS stages; the stream of k-steps runs on into the workgroup's next tile, so a tile's epilogue
// runs while the first operands of the next one arrive.  Completion is tracked with the
// vector-memory counter, which retires in order: before the barrier of k-step i each wavefront waits
// until only its loads of later k-steps are outstanding, so past the barrier stage i+1 is complete.
// A wave-wide load places lane l's piece at LDS base + 16 l, i.e. 8 consecutive 128-byte rows.  The
// LDS of this chip has 64 banks (256 B per clock): 16-byte chunk c of row r is stored at slot
// c ^ ((r >> 1) & 7), so the 16 lanes that a ds_read_b128 serves per clock (16 consecutive rows, same
// chunk) touch 16 different 16-byte bank groups.  Since the load instruction fixes where each lane's
// piece lands, the swizzle is applied to the GLOBAL address each lane fetches from.  A k tail (k not a
// multiple of 64) is zero-filled by pointing the lanes past the end of the row past the end of the
// buffer.
//
// Tile order.  Persistent workgroups; see tile_sequence_index.
//
// Epilogue.  Each wavefront stages its accumulators, 32 token rows at a time, through a part of the
// last k-step's LDS stage that is its own (no barrier between the pieces), so that global memory is
// written in row pieces of 64 bytes and more, 16 bytes per lane: bf16 store; GELU(tanh form) + bf16
// store; gated residual update of the fp32 stream (x += gate_b * (acc + bias)), optionally
// also storing bf16(x).
#include "ddit_common.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

constexpr int BK = 64;         // k per pipeline step (bf16 elements)
constexpr int ROW = 128;       // bytes per LDS row
constexpr int BIAS_SLOTS = 4;  // tiles whose bias may be in LDS at once (see GemmCfg::MIN_STEPS)

struct GemmParams {
  const bf16_t *u; int64_t ld_u;
  const bf16_t *W;
  const bf16_t *bias;
  int64_t N; int n; int k;
  bf16_t *out; int64_t ld_out;
  float *resid;
  const float *gate_tab;
  const float *gate_c6; int64_t gate_c6_stride;
  int64_t tokens_per_sample;
  int tiles_m; int tiles_n; int group_w; int total_tiles; int rounds;
  int split_steps; int split_tiles; int64_t split_stride;   // partial sums (EPI 3): k-steps and output tiles of one part, floats between parts
  int plain;   // row strides below 2^26 elements: a row group's offsets fit 32 bits
  unsigned tok0;   // tokens of the linear before this launch's first (a linear in two launches)
};

// A grouped launch: one token matrix u against G weight matrices of the same shape [group_n, k], each
// with its own bias and its own output (the text k|v projections of all layers of a step).  To the
// tile loop it is one problem with G * group_n out-features; a tile lies inside one group
// (group_n is a multiple of the tile's columns), whose pointers it takes from this table.
constexpr int MAX_GROUPS = 128;
struct GroupTable {
  int group_n;
  const bf16_t *W[MAX_GROUPS];
  const bf16_t *bias[MAX_GROUPS];
  bf16_t *out[MAX_GROUPS];
};
struct NoGroups {};

__device__ __forceinline__ float gelu_tanh_f(float u) {
  // 0.5 u (1 + tanh(z)) == u / (1 + exp(-2 z)),  z = sqrt(2/pi) (u + 0.044715 u^3)
  const float kA = -2.0f * 0.7978845608028654f * 1.4426950408889634f;  // -2 sqrt(2/pi) log2(e)
  const float t = u * u;
  const float z2 = u * (kA + (kA * 0.044715f) * t);                    // -2 z log2(e)
  return u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z2));
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() would also wait for the
// epilogue's global stores of the previous tile to be acknowledged; nothing in this kernel
// communicates through global memory inside a workgroup.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 16-byte LDS reads that the compiler does not see as LDS reads.  It guards every LDS read it
// knows of with a wait for ALL outstanding vector-memory operations (it cannot tell the
// direct-to-LDS loads from stores), which in the epilogues would make each read wait for the round
// trip of the stores issued just before it.  The epilogues read only what the same wavefront has
// staged (LDS operations of a wavefront complete in order), so no vector-memory wait is needed there.
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned lds_offset(const void *p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ void lds_read2_b128(uintx4 (&v)[2], unsigned a0, unsigned a1) {
  asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1])
               : "v"(a0), "v"(a1)
               : "memory");
}
// four 32x32 fp32 row pieces: 8 rows of PITCH bytes further each
template <int STEP>
__device__ __forceinline__ void lds_read4_b128(uintx4 (&v)[4], unsigned a) {
  asm volatile(
      "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%5\n\tds_read_b128 %2, %4 offset:%6\n\t"
      "ds_read_b128 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
      : "v"(a), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP)
      : "memory");
}
// a lane's four fragments of 32 operand rows (see k_gemm_few)
__device__ __forceinline__ void lds_read_frags(uintx4 (&v)[4], unsigned a0, unsigned a1, unsigned a2, unsigned a3) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
               : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
               : "memory");
}
// the tile's bias for this lane: 4 consecutive features (8 bytes) at each of four 8-feature steps
__device__ __forceinline__ void lds_read4_b64(uint2 (&v)[4], unsigned a) {
  asm volatile(
      "ds_read_b64 %0, %4\n\tds_read_b64 %1, %4 offset:16\n\tds_read_b64 %2, %4 offset:32\n\t"
      "ds_read_b64 %3, %4 offset:48\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
      : "v"(a)
      : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "the counter has 6 bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// scheduling-group masks of __builtin_amdgcn_sched_group_barrier
#define SG_MFMA 0x008
#define SG_VMEM_RD 0x020
#define SG_DS_RD 0x100

// Issue order for one sub-step: NM MFMAs with NS instructions of class OTHER spread between them.
template <int OTHER, int I, int NM, int NS>
__device__ __forceinline__ void sched_interleave() {
  if constexpr (I < NM) {
    __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
    constexpr int cnt = (I < NS % NM ? 1 : 0) + NS / NM;
    if constexpr (cnt > 0) __builtin_amdgcn_sched_group_barrier(OTHER, cnt, 0);
    sched_interleave<OTHER, I + 1, NM, NS>();
  }
}

// Order of the output tiles.  Tiles are enumerated in groups of `group_w` out-feature tiles and,
// inside a group, token-panel major; that sequence is cut into 8 contiguous parts, one per XCD
// (workgroups are dealt round-robin to the XCDs, each with its own L2), and in every round the
// workgroups of an XCD take the next consecutive tiles of its part.  An XCD therefore works for
// many rounds on the same few W tiles (they stay in its L2) while it streams token panels of u,
// each of which is shared by the group_w workgroups next to each other.
__device__ __forceinline__ int tile_sequence_index(const GemmParams &p, int round) {
  const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3, per = gridDim.x >> 3;
  const int q8 = p.total_tiles >> 3, r8 = p.total_tiles & 7;
  const int cnt = q8 + (xcd < r8 ? 1 : 0);
  const int idx = round * per + loc;
  if (idx >= cnt) return -1;
  return xcd * q8 + (xcd < r8 ? xcd : r8) + idx;
}
__device__ __forceinline__ void decode_tile(const GemmParams &p, int L, int &tile_m, int &tile_n) {
  const int gsz = p.tiles_m * p.group_w;
  int g = L / gsz;
  const int full = p.tiles_n / p.group_w;
  int bw = p.group_w;
  if (g >= full) { g = full; bw = p.tiles_n - full * p.group_w; }
  const int r = L - g * gsz;
  tile_m = r / bw;
  tile_n = g * p.group_w + (r - tile_m * bw);
}

template <int WGM, int WGN, int WGK, int TM, int TN, int NS>
struct GemmCfg {
  static constexpr int NW = WGM * WGN * WGK;                 // wavefronts per workgroup
  static constexpr int NT = 64 * NW;
  static constexpr int BM = WGM * TM * 32;
  static constexpr int BN = WGN * TN * 32;
  static constexpr int STAGE = (BM + BN) * ROW;
  static constexpr int NJU = BM / 8 / NW, NJW = BN / 8 / NW; // wave-wide loads (8 rows each) per wavefront and k-step
  static constexpr int NJ = NJU + NJW;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "the rows of both operands divide over the wavefronts");
  static_assert(NW % 2 == 0, "a wavefront's loads share one swizzle");
  static_assert(WGK == 1 || (WGK == 2 && TM * TN > 0), "at most two k halves");
  static constexpr int SUBS = 4 / WGK;                       // MFMA groups of 16 k per wavefront and k-step
  // WGK = 2: each wavefront gives the accumulators it does not write out to its partner through LDS
  static constexpr int XCH_TILES = WGK == 2 ? WGM * WGN * TM * TN : 0;
  static constexpr int XCH_PER_STAGE = STAGE / 4096;
  // The stages of a tile's last DEFER k-steps are used by its epilogue; their refill waits until it is done.
  static constexpr int FW = TN * 32;                         // a wavefront's out-features
  static constexpr int PITCH_F32 = 32 * 4 + 16;              // staged row pitches: 32 features fp32,
  static constexpr int bf16_pitch(int na) { return na * 64 + 16; }   // na * 32 features bf16
  static constexpr int EPI_WAVE = 32 * (PITCH_F32 > bf16_pitch(TN) || WGK == 2 ? PITCH_F32 : bf16_pitch(TN));
  static constexpr int XCH_STAGES = WGK == 2 ? (XCH_TILES + XCH_PER_STAGE - 1) / XCH_PER_STAGE : 0;
  static constexpr int EPI_STAGES = (NW + STAGE / EPI_WAVE - 1) / (STAGE / EPI_WAVE);
  static constexpr int DEFER = XCH_STAGES > EPI_STAGES ? XCH_STAGES : EPI_STAGES;
  static_assert(DEFER < NS, "at least one stage keeps prefetching under the epilogue");
  // A tile takes at least this many k-steps (missing ones are zero-filled), so that the load stream is
  // never more than BIAS_SLOTS - 1 tiles ahead of the tile being multiplied.
  static constexpr int MIN_STEPS = (NS + BIAS_SLOTS - 2) / (BIAS_SLOTS - 1) > DEFER ? (NS + BIAS_SLOTS - 2) / (BIAS_SLOTS - 1) : DEFER;
  static constexpr int BIAS_BYTES = BIAS_SLOTS * BN * 2;
  static constexpr int SMEM = NS * STAGE + BIAS_BYTES;
  // Residual update: a wavefront writes OWN MFMA tiles; where their rows of x fit the registers beside the
  // accumulators they are fetched when the tile begins, else a few at a time under the epilogue.
  static constexpr int OWN = (TM * TN + WGK - 1) / WGK;
  static constexpr bool X_EARLY = TM * TN <= 4 && NW <= 8;
  // ... or, of a tile's first X_AHEAD and where the wavefront is all inside, when the last k-steps begin (as many as fit without
  // spills): the epilogue began with waiting for them.  With whole wavefronts at a problem's edge (gemm_epilogue) steps of 12960 and 7360 tokens
  // 36.3 -> 35.8 and 25.5 -> 25.3 ms, 108000 with 4 heads 199.9 -> 199.4, 48600 as before.
  static constexpr int X_AHEAD = X_EARLY ? 0 : NW > 8 ? 2 : TM * TN <= 6 ? 3 : TM * TN <= 8 ? 2 : 1;
  static constexpr int X_DEPTH = NW > 8 ? 2 : 3;             // tiles whose rows are in flight under the epilogue
  static constexpr int X_ROWS = X_EARLY ? OWN : X_AHEAD;
  static_assert(BN / 8 <= 64, "one wavefront fetches the tile's bias");
  static_assert((NS - 1) * NJ < 64 && NS >= 2, "pipeline depth");
};

// the same pointer in every lane, said so that the compiler believes it (a resource it thinks might differ between
// lanes costs a loop around every load)
__device__ __forceinline__ void *uniform_ptr(const void *q) {
  const uint64_t v = (uint64_t)q;
  const uint64_t lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
  const uint64_t hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
  return (void *)(hi << 32 | lo);
}

// One output tile as the epilogue sees it.
struct TileOut {
  int64_t row0; int col0;      // first token, first out-feature
  bf16_t *out; int shift;      // output of the tile's problem; its first out-feature
  float *part;                 // partial sums: where this part's fp32 rows go
  unsigned smp0;               // sample of the wavefront's first token ...
  bool one_sample;             // ... and of all of its tokens
};

// The sample a token belongs to (token counts stay below 2^30).
__device__ __forceinline__ unsigned sample_of(const GemmParams &p, int64_t tok) {
  return p.tokens_per_sample > 0x7fffffff ? 0u : ((unsigned)tok + p.tok0) / (unsigned)p.tokens_per_sample;
}

// Rows of the residual stream and gate vectors of a wavefront's tiles, fetched before they are needed: lane l of a
// group of 8 rows holds four features of row l / 8.
template <int TILES, int TN>
struct XRows {
  float4 x[TILES][4];
  float4 gate[TN];
};

// gate vector of a sample at this lane's features (f4 .. f4 + 3) of the MFMA column that starts at feature col
__device__ __forceinline__ float4 gate_vector(const GemmParams &p, unsigned smp, int f) {
  float4 g = make_float4(1.f, 1.f, 1.f, 1.f);
  if (p.gate_tab) {
    if (f > p.n - 4) f = p.n - 4;                 // past the edge: what is there, not used
    g = *reinterpret_cast<const float4 *>(p.gate_tab + f);
    if (p.gate_c6) {
      const float4 c = *reinterpret_cast<const float4 *>(p.gate_c6 + (int64_t)smp * p.gate_c6_stride + f);
      g.x += c.x; g.y += c.y; g.z += c.z; g.w += c.w;
    }
  }
  return g;
}

// Writes out the MFMA tiles T0 .. T1-1 of this wavefront (tile t = b * TN + a covers the wavefront's token
// rows 32 b .. 32 b + 31 and out-features 32 a .. 32 a + 31; acc[a][b][4g+e] = C[token l32][feature
// 8g + 4 lh + e] of it, bias inside).  `stg`: this wavefront's staging bytes (LDS offset); nothing here
// synchronises with other wavefronts.
// FULL: the whole tile lies inside the problem and (residual update) inside one sample: straight-line code.
// EPI: 0 bf16, 1 GELU + bf16, 2 residual update, 3 partial sums, 4 residual update with streaming stores of the stream
constexpr bool is_residual(int epi) { return epi == 2 || epi == 4; }

template <class C, int TM, int TN, int EPI, int T0, int T1, bool FULL>
__device__ __forceinline__ void gemm_epilogue_as(floatx16 (&acc)[TN][TM], unsigned stg, unsigned char *stg_ptr,
                                              const GemmParams &p, const TileOut &to, int lane, int wm, int wn, unsigned smp0,
                                                 bool one_sample, const XRows<C::X_ROWS, TN> &early) {
  const int l32 = lane & 31, lh = lane >> 5;
  const int64_t row_w = to.row0 + wm * (TM * 32);   // the wavefront's first token and out-feature
  const int col_w = to.col0 + wn * (TN * 32);
  if constexpr (EPI < 2) {
    // rows of AG * 64 bytes: the whole width of the wavefront where it owns all of it, else one MFMA tile
    constexpr int AG = (T0 == 0 && T1 == TM * TN) ? TN : 1;
    constexpr int PITCH = C::bf16_pitch(AG), CPR = AG * 4, ITERS = AG * 2;
    unsigned char *const o0 = reinterpret_cast<unsigned char *>(uniform_ptr(to.out + row_w * p.ld_out + (col_w - to.shift)));
#pragma unroll
    for (int t = T0; t < T1; t += AG) {
      const int b = t / TN, a0 = t - b * TN;
      asm volatile("" : "+v"(lane));   // nothing of a piece's index arithmetic is kept in registers for the next
      // bias is inside; (+ GELU), round to bf16, stage
#pragma unroll
      for (int a = 0; a < AG; ++a)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float v = acc[a0 + a][b][4 * g + e];
            if (EPI == 1) v = gelu_tanh_f(v);
            o[e] = (bf16_t)v;
          }
          *reinterpret_cast<bf16x4 *>(stg_ptr + l32 * PITCH + (a * 32 + 8 * g + 4 * lh) * 2) = o;
        }
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");   // the reads below are not visible as LDS reads: keep them after the writes
#pragma unroll
      for (int i0 = 0; i0 < ITERS; i0 += 2) {
        uintx4 piece[2];
        unsigned la[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int idx = lane + 64 * (i0 + j), rl = idx / CPR, c = idx - rl * CPR;
          la[j] = stg + rl * PITCH + c * 16;
        }
        lds_read2_b128(piece, la[0], la[1]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int idx = lane + 64 * (i0 + j), rl = idx / CPR, c = idx - rl * CPR;
          const int64_t tok = row_w + b * 32 + rl;
          const int f = col_w + a0 * 32 + c * 8;
          // streaming store: the output is not read again by this launch, and a plain store would push
          // the operand lines that other workgroups still re-read out of the L2
          if (FULL) {
            const unsigned place = ((unsigned)rl * (unsigned)p.ld_out + (unsigned)(c * 8)) * 2u;
            __builtin_nontemporal_store(piece[j], reinterpret_cast<uintx4 *>(o0 + ((int64_t)(b * 32) * p.ld_out + a0 * 32) * 2 + place));
          } else if (tok < p.N && f < p.n) {
            __builtin_nontemporal_store(piece[j], reinterpret_cast<uintx4 *>(to.out + tok * p.ld_out + (f - to.shift)));
          }
        }
      }
    }
  } else {
    // Gated residual update.  One MFMA tile at a time is staged as it is; on the way out a lane holds four
    // consecutive features of a row (8 lanes a row of 128 bytes, 8 rows per instruction), so the
    // stream is read and written in whole lines.  The reads of x run DEPTH tiles ahead of their use: memory
    // requests complete in order, loads and stores alike, so a tile's loads are issued BEFORE the stores of
    // the tiles processed while they are in flight, and waiting for them never waits for a store.
    // Partial sums (EPI 3) leave the same way, fp32 rows as they are, with no stream to read.
    constexpr bool EARLY = is_residual(EPI) && C::X_EARLY;
    constexpr int DEPTH = EPI == 3 ? 1 : EARLY ? T1 - T0 : !FULL ? 1 : T1 - T0 < C::X_DEPTH ? T1 - T0 : C::X_DEPTH;
    int r8 = lane >> 3, f4 = (lane & 7) * 4;
    // this wavefront's corner of the stream and of its bf16 copy, and this lane's place in a group of 8 rows
    unsigned char *const x0 = reinterpret_cast<unsigned char *>(uniform_ptr((EPI == 3 ? to.part : p.resid) + row_w * p.n + col_w));
    unsigned char *const o0 = reinterpret_cast<unsigned char *>(uniform_ptr(p.out + (p.out ? row_w * p.ld_out + col_w : 0)));
    const unsigned lane_x = (unsigned)(r8 * p.n + f4) * 4u, lane_o = ((unsigned)r8 * (unsigned)p.ld_out + f4) * 2u;
    float4 xr[DEPTH][4];
    auto issue_x = [&](int t, int slot) {
      const int b = t / TN, a = t - b * TN;
      if constexpr (!FULL) asm volatile("" : "+v"(r8), "+v"(f4));   // nothing of a tile's index arithmetic is kept for the next
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const floatx4 *src;
        if constexpr (FULL) {
          src = reinterpret_cast<const floatx4 *>(x0 + ((int64_t)(b * 32 + 8 * i) * p.n + a * 32) * 4 + lane_x);
        } else {   // lanes past the edge read what is there and do not use it
          int64_t tok = row_w + b * 32 + 8 * i + r8;
          int f = col_w + a * 32 + f4;
          if (tok > p.N - 1) tok = p.N - 1;
          if (f > p.n - 4) f = p.n - 4;
          src = reinterpret_cast<const floatx4 *>(p.resid + tok * p.n + f);
        }
        const floatx4 v = *src;
        xr[slot][i] = make_float4(v[0], v[1], v[2], v[3]);
      }
    };
    float4 gate[TN];
    if constexpr (EARLY) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) xr[d][i] = early.x[d][i];
#pragma unroll
      for (int a = 0; a < TN; ++a) gate[a] = early.gate[a];
    } else if constexpr (FULL && is_residual(EPI)) {
      static_assert(C::X_AHEAD <= DEPTH, "");
#pragma unroll
      for (int d = 0; d < C::X_AHEAD; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) xr[d][i] = early.x[d][i];
#pragma unroll
      for (int d = C::X_AHEAD; d < DEPTH; ++d) issue_x(T0 + d, d);
#pragma unroll
      for (int a = 0; a < TN; ++a) gate[a] = gate_vector(p, smp0, col_w + a * 32 + f4);
    }
#pragma unroll
    for (int t = T0; t < T1; ++t) {
      const int b = t / TN, a = t - b * TN, slot = (t - T0) % DEPTH;
      if constexpr (!FULL && !EARLY && is_residual(EPI)) issue_x(t, slot);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[a][b][4 * g + e];
        *reinterpret_cast<floatx4 *>(stg_ptr + l32 * C::PITCH_F32 + (8 * g + 4 * lh) * 4) = v;
      }
      asm volatile("" ::: "memory");
      uintx4 piece[4];
      lds_read4_b128<8 * C::PITCH_F32>(piece, stg + r8 * C::PITCH_F32 + f4 * 4);
      auto update = [&](int i, float4 g) {
        floatx4 r;
        r[0] = xr[slot][i].x + g.x * __uint_as_float(piece[i][0]);
        r[1] = xr[slot][i].y + g.y * __uint_as_float(piece[i][1]);
        r[2] = xr[slot][i].z + g.z * __uint_as_float(piece[i][2]);
        r[3] = xr[slot][i].w + g.w * __uint_as_float(piece[i][3]);
        return r;
      };
      auto copy_of = [](floatx4 r) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16_t)r[e];
        return o;
      };
      if constexpr (EPI == 3) {
        // the next launch reads them: plain stores
        if constexpr (!FULL) asm volatile("" : "+v"(r8), "+v"(f4));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t tok = row_w + b * 32 + 8 * i + r8;
          const int f = col_w + a * 32 + f4;
          if constexpr (FULL)
            *reinterpret_cast<uintx4 *>(x0 + ((int64_t)(b * 32 + 8 * i) * p.n + a * 32) * 4 + lane_x) = piece[i];
          else if (tok < p.N && f < p.n)
            *reinterpret_cast<uintx4 *>(to.part + tok * p.n + f) = piece[i];
        }
      } else if constexpr (FULL) {
        floatx4 r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          r[i] = update(i, gate[a]);
          floatx4 *const dst = reinterpret_cast<floatx4 *>(x0 + ((int64_t)(b * 32 + 8 * i) * p.n + a * 32) * 4 + lane_x);
          // the two stores are two kernels: in one, as a choice at run time, the compiler makes both of them plain
          if constexpr (EPI == 4) __builtin_nontemporal_store(r[i], dst);
          else *dst = r[i];
        }
        if (p.out) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            __builtin_nontemporal_store(copy_of(r[i]), reinterpret_cast<bf16x4 *>(o0 + ((int64_t)(b * 32 + 8 * i) * p.ld_out + a * 32) * 2 + lane_o));
        }
      } else {
        float4 g0 = make_float4(1.f, 1.f, 1.f, 1.f);
        if (one_sample) g0 = EARLY ? gate[a] : gate_vector(p, smp0, col_w + a * 32 + f4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t tok = row_w + b * 32 + 8 * i + r8;
          const int f = col_w + a * 32 + f4;
          if (tok < p.N && f < p.n) {
            const floatx4 r = update(i, one_sample ? g0 : gate_vector(p, sample_of(p, tok), f));
            *reinterpret_cast<floatx4 *>(p.resid + tok * p.n + f) = r;
            if (p.out) __builtin_nontemporal_store(copy_of(r), reinterpret_cast<bf16x4 *>(p.out + tok * p.ld_out + f));
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (FULL && !EARLY && is_residual(EPI)) {
        if (t + DEPTH < T1) issue_x(t + DEPTH, slot);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

template <class C, int TM, int TN, int EPI, int T0, int T1>
__device__ __forceinline__ void gemm_epilogue(floatx16 (&acc)[TN][TM], unsigned stg, unsigned char *stg_ptr,
                                              const GemmParams &p, const TileOut &to, int lane, int wm, int wn,
                                              const XRows<C::X_ROWS, TN> &early) {
  // What lies inside is asked of the wavefront's own rows and columns, not of the tile's: where 256 columns end at 1152 of 1280 half of the
  // wavefronts have nothing to write and the others all of theirs, and a launch of one round lasts as long as its slowest tile.
  const int64_t row_w = to.row0 + wm * (TM * 32);
  const int col_w = to.col0 + wn * (TN * 32);
  if (row_w >= p.N || col_w >= p.n) return;
  const bool inside = p.plain && row_w + TM * 32 <= p.N && col_w + TN * 32 <= p.n;
  const unsigned smp0 = to.smp0;
  const bool one_sample = to.one_sample;
  if (inside && one_sample)
    gemm_epilogue_as<C, TM, TN, EPI, T0, T1, true>(acc, stg, stg_ptr, p, to, lane, wm, wn, smp0, one_sample, early);
  else
    gemm_epilogue_as<C, TM, TN, EPI, T0, T1, false>(acc, stg, stg_ptr, p, to, lane, wm, wn, smp0, one_sample, early);
}

typedef __attribute__((address_space(3))) void *lds_ptr_t;
typedef __attribute__((address_space(1))) const void *gbl_ptr_t;

template <int WGM, int WGN, int WGK, int TM, int TN, int NS, int EPI, bool DRAIN, class GT>
__device__ __forceinline__ void gemm_tiles(GemmParams p, GT gt) {
  using C = GemmCfg<WGM, WGN, WGK, TM, TN, NS>;
  constexpr bool GROUPED = !std::is_same<GT, NoGroups>::value;
  static_assert(!GROUPED || EPI < 2, "grouped launches write bf16 outputs");
  constexpr int BM = C::BM, BN = C::BN, STAGE = C::STAGE, NW = C::NW, NJ = C::NJ, NJU = C::NJU, SUBS = C::SUBS;
  constexpr int NFRAG = TM + TN, NMFMA = TM * TN, DEFER = C::DEFER;
  // a k-step's loads are issued in two parts: after the barrier that frees their stage, and under the
  // next k-step's first MFMAs
  constexpr int LA = (NJ + 1) / 2;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char *const smem_bias = smem + NS * STAGE;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = WGK == 2 ? wave / (WGM * WGN) : 0;
  const int wt = wave - wk * (WGM * WGN);
  const int wm = wt / WGN, wn = wt - wm * WGN;
  const int l32 = lane & 31, lh = lane >> 5;
  // k-steps of a tile: all of k, or (partial sums) one part of it
  const int nk_all = EPI == 3 ? p.split_steps : (p.k + BK - 1) / BK;
  const int nk = nk_all > C::MIN_STEPS ? nk_all : C::MIN_STEPS;

  // fragment reads: row (tile*32 + l32) of 128 B, chunk 2 sub + lh at slot chunk ^ ((row >> 1) & 7)
  const int frag_u = (wm * (TM * 32) + l32) * ROW;
  const int frag_w = BM * ROW + (wn * (TN * 32) + l32) * ROW;
  int coff[SUBS];
#pragma unroll
  for (int s = 0; s < SUBS; ++s) coff[s] = ((2 * (wk * SUBS + s) + lh) ^ ((l32 >> 1) & 7)) << 4;
  // loads: this wave's j-th instruction covers tile rows 8 (wave + NW j) .. + 7 of the token rows (j < NJU) or of
  // the W rows; this lane: row lane/8 of the eight, slot lane%8
  const int ld_row = wave * 8 + (lane >> 3);
  const int ld_chunk = (lane & 7) ^ ((ld_row >> 1) & 7);          // the global 16-byte chunk that lands in this slot
  const unsigned voff_u = (unsigned)ld_row * (unsigned)p.ld_u * 2u + ld_chunk * 16;
  const unsigned voff_w = (unsigned)ld_row * (unsigned)p.k * 2u + ld_chunk * 16;
  const unsigned bias_lds = lds_offset(smem_bias) + (wn * (TN * 32) + 4 * lh) * 2;

  // ---- the load stream: k-steps of this workgroup's tiles, one after the other, stage by stage.  Past the
  // last tile it goes on with resources of length zero (nothing is fetched), so the loops need no branches
  // and the counts of outstanding loads stay the same.
  int ld_round = 0, ld_k = 0;           // the next k-step to fetch
  const bf16_t *ld_u = p.u, *ld_W = p.W;   // operands of its tile: first row ...
  int ld_k0 = 0, ld_kend = p.k;         // partial sums: first k-step and end of its part of k
  int64_t tot_u = 0, tot_w = 0;         // ... and bytes from there to the matrix's last element (below 2^32)
  const int64_t du = (int64_t)p.ld_u * (NW * 16), dw = (int64_t)p.k * (NW * 16);   // bytes between a wave's loads

  // Start of a tile's operand stream: its place, and its bias (one wavefront fetches it, ahead of everything
  // else, so it has landed when k-step 0 has).
  auto ld_tile = [&](int tile) {
    if (tile < 0) { tot_u = tot_w = 0; return; }
    int part = 0;
    if constexpr (EPI == 3) {
      part = tile / p.split_tiles;
      tile -= part * p.split_tiles;
      ld_k0 = part * p.split_steps;
      ld_kend = ld_k0 * BK + p.split_steps * BK < p.k ? ld_k0 * BK + p.split_steps * BK : p.k;
    }
    int tm, tn;
    decode_tile(p, tile, tm, tn);
    const int64_t row0 = (int64_t)tm * BM;
    int f0 = tn * BN, n_all = p.n;
    const bf16_t *bias = p.bias;
    ld_W = p.W;
    if constexpr (GROUPED) {
      const int g = f0 / gt.group_n;
      ld_W = gt.W[g]; bias = gt.bias[g];
      f0 -= g * gt.group_n; n_all = gt.group_n;
    }
    ld_u = p.u + row0 * p.ld_u;
    ld_W += (int64_t)f0 * p.k;
    tot_u = ((p.N - row0 - 1) * p.ld_u + p.k) * 2;
    tot_w = (int64_t)(n_all - f0) * p.k * 2;
    if (bias && wave == 0 && lane < BN / 8) {
      int f = f0 + lane * 8;
      if (f > n_all - 8) f = n_all - 8;         // overhanging features: a valid address, never stored
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)(bias + f), (lds_ptr_t)(smem_bias + (ld_round % BIAS_SLOTS) * (BN * 2)), 16, 0, 0);
    }
  };
  // This lane's offsets of the stream's k-step; past the row's end: past every buffer, which fetches nothing and
  // writes zeros.  k is in the lane's offset because that is what a buffer's length is checked against: whether the
  // scalar offset counts there too is described both ways, and with a length of zero the difference would wrap.
  unsigned ld_vu, ld_vw;
  auto ld_offsets = [&]() {
    const unsigned k0 = (unsigned)__builtin_amdgcn_readfirstlane((ld_k0 + ld_k) * (BK * 2));   // bytes
    const bool in = (ld_k0 + ld_k) * BK + ld_chunk * 8 < ld_kend;
    ld_vu = in ? voff_u + k0 : 0xfffffff0u;
    ld_vw = in ? voff_w + k0 : 0xfffffff0u;
  };
  // loads J0 .. J1-1 of the current k-step of the stream into stage ST; each instruction has a resource that
  // starts at its eight rows
  auto ld_issue = [&](auto j0_tag, auto j1_tag, int st) {
    constexpr int J0 = decltype(j0_tag)::value, J1 = decltype(j1_tag)::value;
#pragma unroll
    for (int j = J0; j < J1; ++j) {
      const bool is_u = j < NJU;
      const int64_t off = is_u ? du * j : dw * (j - NJU), left = (is_u ? tot_u : tot_w) - off;
      const unsigned lim = (unsigned)left & ~(unsigned)(left >> 63);
      const unsigned char *base = reinterpret_cast<const unsigned char *>(is_u ? ld_u : ld_W) + off;
      __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(base), 0, __builtin_amdgcn_readfirstlane((int)lim), 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(smem + st * STAGE + (wave + NW * j) * 1024), 16, is_u ? ld_vu : ld_vw, 0, 0, 0);
    }
  };
  auto ld_advance = [&]() {
    if (++ld_k == nk) {
      ld_k = 0;
      ++ld_round;
      ld_tile(ld_round < p.rounds ? tile_sequence_index(p, ld_round) : -1);
    }
    ld_offsets();
  };
  using J_0 = std::integral_constant<int, 0>;
  using J_A = std::integral_constant<int, LA>;
  using J_N = std::integral_constant<int, NJ>;

#define DL_READ_FRAGS(BUF, ST, S)                                                                  \
  do {                                                                                             \
    const unsigned char *sb_ = smem + (ST) * STAGE + coff[S];                                      \
    _Pragma("unroll") for (int b = 0; b < TM; ++b)                                                 \
        uf[BUF][b] = *reinterpret_cast<const bf16x8 *>(sb_ + frag_u + b * 32 * ROW);               \
    _Pragma("unroll") for (int a = 0; a < TN; ++a)                                                 \
        wf[BUF][a] = *reinterpret_cast<const bf16x8 *>(sb_ + frag_w + a * 32 * ROW);               \
  } while (0)

#define DL_MFMAS(BUF)                                                                              \
  do {                                                                                             \
    _Pragma("unroll") for (int a = 0; a < TN; ++a)                                                 \
        _Pragma("unroll") for (int b = 0; b < TM; ++b)                                             \
            acc[a][b] = mfma32(wf[BUF][a], uf[BUF][b], acc[a][b]);                                 \
  } while (0)

  int tile = tile_sequence_index(p, 0);
  if (tile < 0) return;
  ld_tile(tile);
  ld_offsets();
  // the first NS k-steps, less the second part of the last one (the first k-step of the loop issues that)
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s + 1 < NS) {
      ld_issue(J_0{}, J_N{}, s);
      ld_advance();
    } else {
      ld_issue(J_0{}, J_A{}, s);
    }
  }
  wait_vmcnt<(NS - 2) * NJ + LA>();   // k-step 0 (and the bias) has landed
  lds_barrier();

  int st = 0;                 // stage of the k-step being multiplied
  for (int round = 0;; ++round) {
    int tile_m, tile_n, part = 0;
    if constexpr (EPI == 3) { part = tile / p.split_tiles; tile -= part * p.split_tiles; }
    decode_tile(p, tile, tile_m, tile_n);
    TileOut to;
    to.part = EPI == 3 ? p.resid + part * p.split_stride : nullptr;
    to.row0 = (int64_t)tile_m * BM; to.col0 = tile_n * BN; to.out = p.out; to.shift = 0;
    to.smp0 = 0; to.one_sample = true;
    XRows<C::X_ROWS, TN> early;
    if constexpr (is_residual(EPI)) {
      if (p.gate_tab && p.gate_c6) {
        const int64_t first = to.row0 + wm * (TM * 32), end = first + TM * 32;   // the wavefront's rows; past the last token: that one
        to.smp0 = sample_of(p, first < p.N ? first : p.N - 1);
        to.one_sample = to.smp0 == sample_of(p, (end < p.N ? end : p.N) - 1);
      }
      if constexpr (C::X_EARLY) {
        // this wavefront's rows of x and gates, behind the loads in flight: they have arrived long before the epilogue
        const int64_t row_w = to.row0 + wm * (TM * 32) + (lane >> 3);
        const int col_w = to.col0 + wn * (TN * 32) + (lane & 7) * 4;
#pragma unroll
        for (int d = 0; d < C::OWN; ++d) {
          int t = wk * C::OWN + d;
          if (t > NMFMA - 1) t = NMFMA - 1;
          const int b = t / TN, a = t - b * TN;
          int f = col_w + a * 32;
          if (f > p.n - 4) f = p.n - 4;            // lanes past the edge read what is there and do not use it
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            int64_t tok = row_w + b * 32 + 8 * i;
            if (tok > p.N - 1) tok = p.N - 1;
            const floatx4 v = *reinterpret_cast<const floatx4 *>(p.resid + tok * p.n + f);
            early.x[d][i] = make_float4(v[0], v[1], v[2], v[3]);
          }
        }
#pragma unroll
        for (int a = 0; a < TN; ++a) early.gate[a] = gate_vector(p, to.smp0, col_w + a * 32);
      }
    }
    // the accumulators start from the bias (those of the first k half)
    floatx16 acc[TN][TM];
    {
      const bf16_t *bias = p.bias;
      if constexpr (GROUPED) {
        const int g = to.col0 / gt.group_n;
        bias = gt.bias[g]; to.out = gt.out[g]; to.shift = g * gt.group_n;
      }
#pragma unroll
      for (int a = 0; a < TN; ++a) {
        uint2 bq[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) bq[g] = make_uint2(0u, 0u);
        if (bias && wk == 0 && part == 0) lds_read4_b64(bq, bias_lds + (round % BIAS_SLOTS) * (BN * 2) + a * 64);
#pragma unroll
        for (int b = 0; b < TM; ++b)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            acc[a][b][4 * g + 0] = __uint_as_float(bq[g].x << 16);
            acc[a][b][4 * g + 1] = __uint_as_float(bq[g].x & 0xffff0000u);
            acc[a][b][4 * g + 2] = __uint_as_float(bq[g].y << 16);
            acc[a][b][4 * g + 3] = __uint_as_float(bq[g].y & 0xffff0000u);
          }
      }
    }
    bf16x8 uf[2][TM], wf[2][TN];
    DL_READ_FRAGS(0, st, 0);
    // One k-step.  TAIL = -1: in the middle of the tile; TAIL = i: the i-th of the last ones, whose stage is not filled
    // again (see tail_steps), `last`: the very last.  Each group of MFMAs issues one MFMA first, then the LDS reads of the NEXT
    // group's fragments, then the rest: the wait that the compiler places before the first MFMA (it always
    // waits for every LDS read issued so far) then covers only reads issued a whole group earlier.
    auto k_step = [&](auto tail_tag, auto last_tag) {
      constexpr int TAIL = decltype(tail_tag)::value;
      constexpr bool LAST = decltype(last_tag)::value;
      const int st_next = st + 1 == NS ? 0 : st + 1, st_prev = st == 0 ? NS - 1 : st - 1;
#pragma unroll
      for (int s = 0; s < SUBS; ++s) {
        if (s + 1 < SUBS) {
          DL_READ_FRAGS((s + 1) & 1, st, s + 1);
          if (s == 0 && TAIL <= 0) ld_issue(J_A{}, J_N{}, st_prev);
          DL_MFMAS(s & 1);
          __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
          __builtin_amdgcn_sched_group_barrier(SG_DS_RD, NFRAG, 0);
          if (s == 0 && TAIL <= 0) sched_interleave<SG_VMEM_RD, 0, NMFMA - 1, NJ - LA>();
          else __builtin_amdgcn_sched_group_barrier(SG_MFMA, NMFMA - 1, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (s == 0 && TAIL <= 0) ld_advance();
        } else {
          // every fragment of this k-step is in registers (or on its way): past the barrier its stage is free,
          // and the next k-step's stage is complete
          if constexpr (NS - 2 - TAIL >= 0) wait_vmcnt<(NS - 2 - (TAIL > 0 ? TAIL : 0)) * NJ>();
          lds_barrier();
          if (!LAST) DL_READ_FRAGS((s + 1) & 1, st_next, 0);
          if (TAIL < 0) ld_issue(J_0{}, J_A{}, st);
          DL_MFMAS(s & 1);
          if (!LAST) {
            __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
            __builtin_amdgcn_sched_group_barrier(SG_DS_RD, NFRAG, 0);
            if (TAIL < 0) sched_interleave<SG_VMEM_RD, 0, NMFMA - 1, LA>();
            else __builtin_amdgcn_sched_group_barrier(SG_MFMA, NMFMA - 1, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      st = st_next;
    };
    // The last k-steps of a tile, which fill no stage: DEFER, whose stages the epilogue uses.  Of a workgroup's last tile they
    // are all that the ring holds, as behind it there is nothing to fetch: loads of length zero cost as much as others to
    // issue.  DRAIN: where the ring is long and the contraction fills it (launch_one); with three or four stages it gave
    // nothing, and of the large tiles the compiler would keep the accumulators twice.  It is worth little: a step of 28 blocks
    // without / with, ms: 16 tokens 4.56 / 4.57, 64 4.80 / 4.77, 128 4.85 / 4.87, 320 5.45 / 5.44, 512 6.02 / 6.00, 1200 7.77 / 7.70, 2304
    // 10.14 / 10.14; 4 of the 16 heads 200 tokens 4.62 / 4.64, 1200 6.66 / 6.62, 2304 8.09 / 8.01.
    auto tail_steps = [&](auto n_tag) {
      constexpr int N = decltype(n_tag)::value;
      static_assert(N <= 8, "k_step calls");
#define DL_TAIL(I) if constexpr (N > I) k_step(std::integral_constant<int, I>{}, std::integral_constant<bool, I == N - 1>{})
      DL_TAIL(0); DL_TAIL(1); DL_TAIL(2); DL_TAIL(3); DL_TAIL(4); DL_TAIL(5); DL_TAIL(6); DL_TAIL(7);
#undef DL_TAIL
    };
    const bool last_tile = DRAIN && nk >= NS && (round + 1 >= p.rounds || tile_sequence_index(p, round + 1) < 0);
    const int full = nk - (last_tile ? NS : DEFER);
    for (int kt = 0; kt < full; ++kt) k_step(std::integral_constant<int, -1>{}, std::false_type{});
    if constexpr (is_residual(EPI) && C::X_AHEAD > 0) {
      const int64_t row_w = to.row0 + wm * (TM * 32);
      const int col_w = to.col0 + wn * (TN * 32);
      if (p.plain && row_w + TM * 32 <= p.N && col_w + TN * 32 <= p.n) {
        const unsigned char *const x0 = reinterpret_cast<const unsigned char *>(uniform_ptr(p.resid + row_w * p.n + col_w));
        const unsigned lane_x = (unsigned)((lane >> 3) * p.n + (lane & 7) * 4) * 4u;
#pragma unroll
        for (int d = 0; d < C::X_AHEAD; ++d)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const floatx4 v = *reinterpret_cast<const floatx4 *>(x0 + ((int64_t)(d / TN * 32 + 8 * i) * p.n + d % TN * 32) * 4 + lane_x);
            early.x[d][i] = make_float4(v[0], v[1], v[2], v[3]);
          }
      }
      asm volatile("" ::: "memory");
    }
    if (last_tile) tail_steps(std::integral_constant<int, DRAIN ? NS : DEFER>{});
    else tail_steps(std::integral_constant<int, DEFER>{});

    // the i-th slice of EACH bytes inside the stages of the last DEFER k-steps
    auto slice = [&](int i, int each) {
      const int per = STAGE / each, d = i / per;
      int s = st - DEFER + d;
      if (s < 0) s += NS;
      return s * STAGE + (i - d * per) * each;
    };
    if constexpr (WGK == 1) {
      const int at = slice(wave, C::EPI_WAVE);
      gemm_epilogue<C, TM, TN, EPI, 0, NMFMA>(acc, lds_offset(smem) + at, smem + at, p, to, lane, wm, wn, early);
    } else {
      // Partial sums meet: of its tiles a wavefront of the first k half keeps the first part and gives the rest to
      // its partner, and the other way round.
      constexpr int H = (NMFMA + 1) / 2;
      auto meet = [&](auto keep0_tag, auto keep1_tag) {
        constexpr int K0 = decltype(keep0_tag)::value, K1 = decltype(keep1_tag)::value;
#pragma unroll
        for (int t = 0; t < NMFMA; ++t)
          if (t < K0 || t >= K1) {
            unsigned char *at = smem + slice(wt * NMFMA + t, 4096) + lane * 16;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              floatx4 v;
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = acc[t % TN][t / TN][4 * g + e];
              *reinterpret_cast<floatx4 *>(at + g * 1024) = v;
            }
          }
        lds_barrier();
#pragma unroll
        for (int t = K0; t < K1; ++t) {
          uintx4 v[4];
          lds_read4_b128<1024>(v, lds_offset(smem) + slice(wt * NMFMA + t, 4096) + lane * 16);
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t % TN][t / TN][4 * g + e] += __uint_as_float(v[g][e]);
        }
        lds_barrier();   // the same bytes take the staged rows
        const int at = slice(wave, C::EPI_WAVE);
        if constexpr (K0 < K1)
          gemm_epilogue<C, TM, TN, EPI, K0, K1>(acc, lds_offset(smem) + at, smem + at, p, to, lane, wm, wn, early);
      };
      if (wk == 0) meet(std::integral_constant<int, 0>{}, std::integral_constant<int, H>{});
      else meet(std::integral_constant<int, H>{}, std::integral_constant<int, NMFMA>{});
    }
    tile = round + 1 < p.rounds ? tile_sequence_index(p, round + 1) : -1;
    if (tile < 0) break;
    lds_barrier();   // every wavefront is done with the stages it staged in: refill them
#pragma unroll
    for (int d = 0; d < DEFER; ++d) {
      int s = st - DEFER + d;
      if (s < 0) s += NS;
      if (d + 1 < DEFER) {
        ld_issue(J_0{}, J_N{}, s);
        ld_advance();
      } else {
        ld_issue(J_0{}, J_A{}, s);
      }
    }
  }
  wait_vmcnt<0>();   // no load may still write to the LDS when the workgroup leaves it
#undef DL_READ_FRAGS
#undef DL_MFMAS
}

template <int WGM, int WGN, int WGK, int TM, int TN, int NS, int EPI, bool DRAIN, class GT>
__global__ __launch_bounds__(WGM *WGN *WGK * 64, 2) void k_gemm_bf16(GemmParams p, GT gt) {
  gemm_tiles<WGM, WGN, WGK, TM, TN, NS, EPI, DRAIN, GT>(p, gt);
}
// 192 x 192 on twelve wavefronts, three a SIMD, each with 96 x 32 of it: eight could not share its 36 MFMA tiles evenly.
template <int EPI>
__global__ __launch_bounds__(768, 3) void k_gemm_twelve(GemmParams p) {
  gemm_tiles<2, 6, 1, 3, 1, 3, EPI, false, NoGroups>(p, NoGroups());
}

// ---------------------------------------------------------------------------------------------
// Few tokens: output tiles of 32 x 32, 64 x 32 or 64 x 64, the k-steps dealt out to the wavefronts.
//
// What bounds such a launch is the path into a CU (105 bytes per ns when the lines are in the L2) and the time around it, not
// the matrix cores: a 64 x 64 tile with k = 1152 fetches 295 KB through it, and at 64 tokens 18 of 256 CUs do all of the work.
// A 32 x 32 tile fetches half of that, on four times as many CUs.  Every wavefront owns the whole tile for k-steps w, w + NW, ... and
// a ring of NS stages of its own, so nothing synchronises until the partial tiles meet in LDS once, and with k = 1152
// nearly all of a tile's operands are asked for before the first byte is waited for.
// Launches in a step's state, us with an event pair's 3.5, best of the other tiles / this: 1152 x 1152, 64 tokens 11.8 / 8.6, with the
// residual update and the bf16 copy 13.1 / 9.2; 192 tokens 11.2 / 8.6; 448 (64 x 32) 11.2 / 10.5; 3456 x 1152, 64 tokens 13.0 / 9.5; 256 x 256, 256
// tokens 7.6 / 6.6, residual 10.3 / 7.0; 1152 x 4608, 128 tokens 29.4 / 17.4, 768 (64 x 64) 30.2 / 27.7.  A step of 28 blocks of 1152
// features, ms: 16 tokens 4.58 / 3.36, 64 4.77 / 3.72, 200 4.98 / 4.45, 256 5.12 / 4.77, 512 6.00 / 5.81; 4 heads 64 4.35 / 3.43.
// ---------------------------------------------------------------------------------------------
template <int TM_, int TN_, int NW_, int NS_>
struct FewCfg {
  static constexpr int TM = TM_, TN = TN_, NW = NW_, NS = NS_;   // MFMA tiles of 32 x 32; wavefronts; stages of each
  static constexpr int BM = 32 * TM, BN = 32 * TN;
  static constexpr int STAGE = (BM + BN) * ROW, LU = BM / 8, LOADS = (BM + BN) / 8;   // wave-wide loads of a k-step
  static constexpr int EG = NW >= 8 && TM * TN > 1 ? 2 : 1;      // groups of 256 threads that write out
  static constexpr int UNITS = TM * TN / EG;                     // MFMA tiles that a group writes out
  static constexpr int SMEM = NW * NS * STAGE;
  static_assert(TM * TN * 4096 <= STAGE, "a partial tile lies in a stage");
  static_assert(TM * TN % EG == 0 && EG * 256 <= NW * 64 && NS <= 3 && 2 * LOADS < 64 && SMEM <= 160 * 1024, "");
};

template <class C, int EPI>
__global__ __launch_bounds__(64 * C::NW, (C::NW + 3) / 4) void k_gemm_few(GemmParams p) {
  constexpr int TM = C::TM, TN = C::TN, NW = C::NW, UNITS = C::UNITS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  // tiles in runs per XCD, the token tiles of one set of columns next to each other (they share W)
  const int xcd = blockIdx.x & 7, q8 = p.total_tiles >> 3, r8 = p.total_tiles & 7;
  int tile = blockIdx.x >> 3;
  if (tile >= q8 + (xcd < r8 ? 1 : 0)) return;
  tile += xcd * q8 + (xcd < r8 ? xcd : r8);
  int part = 0, k0 = 0, kend = p.k;
  if constexpr (EPI == 3) {
    part = tile / p.split_tiles;
    tile -= part * p.split_tiles;
    k0 = part * p.split_steps;
    kend = (k0 + p.split_steps) * BK < p.k ? (k0 + p.split_steps) * BK : p.k;
  }
  const int tile_n = tile / p.tiles_m, tile_m = tile - tile_n * p.tiles_m;
  const int row0 = tile_m * C::BM, col0 = tile_n * C::BN;
  const int steps = (kend - k0 * BK + BK - 1) / BK;      // k-steps of the tile
  const int ring = p.rounds;                             // stages of a wavefront

  // A thread of the first EG * 256 writes four features of one token of UNITS MFMA tiles.  What it needs besides the sums is asked for
  // ahead of the operands: loads complete in order, so the waits below count the operands alone.
  const int group = tid >> 8, r = (tid >> 3) & 31;
  float4 x[UNITS], gate[UNITS];
  uint2 bias[UNITS];
  auto place = [&](int i, int64_t &tok, int &f) {
    const int u = group + C::EG * i, b = u / TN, a = u - b * TN;
    tok = row0 + 32 * b + r;
    f = col0 + 32 * a + (tid & 7) * 4;
    return group < C::EG && tok < p.N && f < p.n;
  };
#pragma unroll
  for (int i = 0; i < UNITS; ++i) {
    int64_t tok; int f;
    x[i] = make_float4(0.f, 0.f, 0.f, 0.f); gate[i] = make_float4(1.f, 1.f, 1.f, 1.f); bias[i] = make_uint2(0u, 0u);
    if (place(i, tok, f)) {
      if (p.bias && part == 0) bias[i] = *reinterpret_cast<const uint2 *>(p.bias + f);
      if constexpr (is_residual(EPI)) {
        x[i] = *reinterpret_cast<const float4 *>(p.resid + tok * p.n + f);
        gate[i] = gate_vector(p, p.gate_tab && p.gate_c6 ? sample_of(p, tok) : 0, f);
      }
    }
  }
  asm volatile("" ::: "memory");

  // Loads as in the large kernel: 8 rows of 128 bytes each, chunk c of row r at slot c ^ ((r >> 1) & 7); rows past the operands and
  // the k tail are zeros by the buffers' lengths.
  const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(
      uniform_ptr(p.u + (int64_t)row0 * p.ld_u), 0,
      __builtin_amdgcn_readfirstlane((int)(unsigned)(((p.N - row0 - 1) * p.ld_u + p.k) * 2)), 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      uniform_ptr(p.W + (int64_t)col0 * p.k), 0, __builtin_amdgcn_readfirstlane((int)(unsigned)((int64_t)(p.n - col0) * p.k * 2)), 0x00020000);
  const int chunk0 = (lane & 7) ^ (lane >> 4);           // of rows 8 j + lane / 8, j even; j odd: chunk0 ^ 4
  const unsigned row_u = (unsigned)(lane >> 3) * (unsigned)p.ld_u * 2u, row_w = (unsigned)(lane >> 3) * (unsigned)p.k * 2u;
  unsigned char *const mem = smem + wave * (ring * C::STAGE);
  auto issue = [&](int t, int st) {
    const int at = (k0 + wave + t * NW) * BK;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int kk = at + (chunk0 ^ (4 * o)) * 8;
      const bool in = kk < kend;
      const unsigned ou = in ? row_u + (unsigned)kk * 2u : 0u, ow = in ? row_w + (unsigned)kk * 2u : 0u;
#pragma unroll
      for (int j = o; j < C::LOADS; j += 2) {
        const bool is_u = j < C::LU;
        const unsigned to = is_u ? ou + (unsigned)(j * 16) * (unsigned)p.ld_u : ow + (unsigned)((j - C::LU) * 16) * (unsigned)p.k;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(is_u ? ru : rw, (lds_ptr_t)(mem + st * C::STAGE + j * 1024), 16, in ? to : 0xfffffff0u, 0, 0, 0);
      }
    }
  };
  const int mine_steps = (steps - wave + NW - 1) / NW;   // of this wavefront; none where k is short
  for (int t = 0; t < ring; ++t)
    if (t < mine_steps) issue(t, t);

  floatx16 acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
  unsigned frag[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) frag[s] = lds_offset(mem) + l32 * ROW + (((2 * s + lh) ^ ((l32 >> 1) & 7)) << 4);
  int st = 0;
  for (int t = 0; t < mine_steps; ++t) {
    const int behind = mine_steps - 1 - t < ring - 1 ? mine_steps - 1 - t : ring - 1;   // k-steps asked for after this one
    if (behind >= 2) wait_vmcnt<2 * C::LOADS>();
    else if (behind == 1) wait_vmcnt<C::LOADS>();
    else wait_vmcnt<0>();
    uintx4 fr[TM + TN][4];   // rows of 32 tokens, then of 32 features
#pragma unroll
    for (int i = 0; i < TM + TN; ++i) lds_read_frags(fr[i], frag[0] + st * C::STAGE + i * 32 * ROW, frag[1] + st * C::STAGE + i * 32 * ROW,
                                                     frag[2] + st * C::STAGE + i * 32 * ROW, frag[3] + st * C::STAGE + i * 32 * ROW);
    if (t + ring < mine_steps) issue(t + ring, st);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
          acc[a][b] = mfma32(__builtin_bit_cast(bf16x8, fr[TM + a][s]), __builtin_bit_cast(bf16x8, fr[b][s]), acc[a][b]);
    st = st + 1 == ring ? 0 : st + 1;
  }
  // The partial tiles meet: every wavefront's lies where its first stage was, 16-byte pieces of a row swizzled like the operands'.
  if (mine_steps > 0) {
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
      for (int b = 0; b < TM; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          floatx4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[a][b][4 * g + e];
          *reinterpret_cast<floatx4 *>(mem + (b * TN + a) * 4096 + l32 * ROW + (((2 * g + lh) ^ ((l32 >> 1) & 7)) << 4)) = v;
        }
  }
  lds_barrier();
  auto rounded = [](float4 v) { bf16x4 o; o[0] = (bf16_t)v.x; o[1] = (bf16_t)v.y; o[2] = (bf16_t)v.z; o[3] = (bf16_t)v.w; return o; };
#pragma unroll
  for (int i = 0; i < UNITS; ++i) {
    int64_t tok; int f;
    if (!place(i, tok, f)) continue;
    float4 sum = make_float4(__uint_as_float(bias[i].x << 16), __uint_as_float(bias[i].x & 0xffff0000u), __uint_as_float(bias[i].y << 16),
                             __uint_as_float(bias[i].y & 0xffff0000u));
    const unsigned char *const from = smem + (group + C::EG * i) * 4096 + r * ROW + (((tid & 7) ^ ((r >> 1) & 7)) << 4);
#pragma unroll
    for (int w = 0; w < NW; ++w)
      if (w < steps) {
        const floatx4 v = *reinterpret_cast<const floatx4 *>(from + w * (ring * C::STAGE));
        sum.x += v[0]; sum.y += v[1]; sum.z += v[2]; sum.w += v[3];
      }
    if constexpr (EPI < 2) {
      if (EPI == 1) sum = make_float4(gelu_tanh_f(sum.x), gelu_tanh_f(sum.y), gelu_tanh_f(sum.z), gelu_tanh_f(sum.w));
      *reinterpret_cast<bf16x4 *>(p.out + tok * p.ld_out + f) = rounded(sum);
    } else if constexpr (EPI == 3) {
      *reinterpret_cast<float4 *>(p.resid + part * p.split_stride + tok * p.n + f) = sum;
    } else {
      const float4 v = make_float4(x[i].x + gate[i].x * sum.x, x[i].y + gate[i].y * sum.y, x[i].z + gate[i].z * sum.z, x[i].w + gate[i].w * sum.w);
      *reinterpret_cast<float4 *>(p.resid + tok * p.n + f) = v;
      if (p.out) *reinterpret_cast<bf16x4 *>(p.out + tok * p.ld_out + f) = rounded(v);
    }
  }
}

template <class C, int EPI>
int launch_few(const GemmParams &p0, hipStream_t s) {
  GemmParams p = p0;
  const int nk = EPI == 3 ? p.split_steps : (p.k + BK - 1) / BK;
  p.tiles_m = (int)((p.N + C::BM - 1) / C::BM);
  p.tiles_n = (p.n + C::BN - 1) / C::BN;
  p.total_tiles = p.split_tiles = p.tiles_m * p.tiles_n;
  if (EPI == 3) p.total_tiles *= ((p.k + BK - 1) / BK + p.split_steps - 1) / p.split_steps;
  p.rounds = std::min(C::NS, (nk + C::NW - 1) / C::NW);   // no more stages than a wavefront has k-steps: the LDS holds further workgroups
  static bool attr_set = false;  // benign race: the attribute is idempotent
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_few<C, EPI>), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
    if (e != hipSuccess) return ddit::hip_fail(e, "gemm hipFuncSetAttribute");
    attr_set = true;
  }
  hipLaunchKernelGGL((k_gemm_few<C, EPI>), dim3((unsigned)((p.total_tiles + 7) & ~7)), dim3(64 * C::NW), C::NW * p.rounds * C::STAGE, s, p);
  return ddit::hip_fail(hipGetLastError(), "gemm launch");
}

using Few32 = FewCfg<1, 1, 6, 3>;
using Few64x32 = FewCfg<2, 1, 6, 2>;
using Few64 = FewCfg<2, 2, 8, 1>;

// Which of those forms a linear takes (0: none): the smallest tile whose grid, `parts` times as large with partial sums of `steps`
// k-steps, finds room on the chip at once, which for short contractions is several workgroups a CU; beyond that the tiles of several
// rounds fetch more than the larger ones (1152 x 1152, 32 x 32: 224 tokens, 252 tiles, 8.6 us, 256 tokens, 288 tiles, 11.3; 768 x 256:
// 640 tokens, 480 tiles, 7.0 against 8.8).  64 x 64 only for long contractions: with 18 k-steps it is as fast as the other kernel's 64 x 64
// (12.4 / 12.5 us), with 32 up to 6 % slower, with 72 7-9 % faster, with 128 8 %.  Over 600 linears of 16 to 1624 tokens
// (profiles/gemm_few_tokens_sweep.txt) the launcher takes 0.3 % more time than the best of all forms; the 443 that take these are 0.78 times the best
// other tile's time on average, 1.03 at worst.
constexpr int FEW_LONG_STEPS = 47;
template <class C>
bool few_fits(int64_t N, int n, int steps, int parts, int cus) {
  const int smem = C::NW * std::min(C::NS, (steps + C::NW - 1) / C::NW) * C::STAGE;
  return (N + C::BM - 1) / C::BM * ((n + C::BN - 1) / C::BN) * parts <= (int64_t)cus * (160 * 1024 / smem);
}
int few_form(int64_t N, int n, int64_t ld_u, int k, int parts, int steps, int cus) {
  if (ld_u >= 1 << 24 || k >= 1 << 24) return 0;
  if (few_fits<Few32>(N, n, steps, parts, cus)) return 1;
  if (few_fits<Few64x32>(N, n, steps, parts, cus)) return 2;
  return steps >= FEW_LONG_STEPS && few_fits<Few64>(N, n, steps, parts, cus) ? 3 : 0;
}

template <int EPI>
int launch_few_form(int form, const GemmParams &p, hipStream_t s) {
  return form == 1 ? launch_few<Few32, EPI>(p, s) : form == 2 ? launch_few<Few64x32, EPI>(p, s) : launch_few<Few64, EPI>(p, s);
}

template <int WGM, int WGN, int WGK, int TM, int TN, int NS, int EPI, bool DRAIN, class GT>
int launch_kernel(const GemmParams &p, int grid, hipStream_t s, const GT &gt) {
  using C = GemmCfg<WGM, WGN, WGK, TM, TN, NS>;
  constexpr bool TWELVE = C::NW == 12;
  auto kernel = [] {
    if constexpr (TWELVE) return &k_gemm_twelve<EPI>;
    else return &k_gemm_bf16<WGM, WGN, WGK, TM, TN, NS, EPI, DRAIN, GT>;
  }();
  static bool attr_set = false;  // benign race: the attribute is idempotent
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
    if (e != hipSuccess) return ddit::hip_fail(e, "gemm hipFuncSetAttribute");
    attr_set = true;
  }
  if constexpr (TWELVE) hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(C::NT), C::SMEM, s, p);
  else hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(C::NT), C::SMEM, s, p, gt);
  return ddit::hip_fail(hipGetLastError(), "gemm launch");
}

template <int WGM, int WGN, int WGK, int TM, int TN, int NS, int EPI, class GT = NoGroups>
int launch_one(const GemmParams &p0, hipStream_t s, const GT &gt = GT()) {
  using C = GemmCfg<WGM, WGN, WGK, TM, TN, NS>;
  static_assert(C::SMEM <= 160 * 1024, "the tile's stages must fit the LDS");
  GemmParams p = p0;
  const int64_t tiles_m = (p.N + C::BM - 1) / C::BM;
  p.tiles_m = (int)tiles_m;
  p.tiles_n = (p.n + C::BN - 1) / C::BN;
  // width of an out-feature group: at most 4 tiles (their W, about 3.5 MB at k = 1152, stays in an XCD's 4 MB L2 next to the token panels
  // streaming through), as even as the tile count allows.  All of them where large tiles are 5 to 8 to a row of no more features
  // than 4 of the largest: the tokens then pass once (steps of 7360 tokens 22.88 -> 22.72 ms, 12960 36.01 -> 35.86, six blocks of 8800
  // 6.36 -> 6.33; 361 linears of 1160 to 1536 features, by count of tiles: 5 0.99 of the time in groups of 4, 6 0.98, 7 0.98, 8 0.98, and 1.00 where
  // 6 or 8 fill 1536).  Wider groups for every tile: 3600 tokens 1.3 % longer, 1600 1 %.
  const int max_w = C::BM >= 192 && C::BN >= 192 && p.tiles_n * C::BN <= 1536 ? p.tiles_n : 4;
  const int n_groups = (p.tiles_n + max_w - 1) / max_w;
  p.group_w = (p.tiles_n + n_groups - 1) / n_groups;
  const int64_t total = tiles_m * p.tiles_n;
  if (total > (int64_t)1 << 30) {
    ddit::set_error("linear: %lld output tiles: too many", (long long)total);
    return -2;
  }
  p.total_tiles = (int)total;
  const int nk = (p.k + BK - 1) / BK;
  if (EPI == 3) {
    p.split_tiles = p.total_tiles;
    p.total_tiles *= (nk + p.split_steps - 1) / p.split_steps;
  }
  p.plain = p.n < (1 << 26) && p.ld_out < (1 << 26);
  // one workgroup per CU (its stages take most of the LDS); a multiple of 8 so that every round gives
  // each XCD a contiguous run of tiles
  int grid = ddit::device_cus() & ~7;
  if (grid < 8) grid = 8;
  if (p.total_tiles <= grid) grid = (p.total_tiles + 7) & ~7;
  p.rounds = ((p.total_tiles + 7) / 8 + grid / 8 - 1) / (grid / 8);
  // A contraction shorter than the ring has no k-steps to drain, and the kernel without them is the shorter one to fetch: a
  // block of hidden size 256, 16 / 64 / 576 tokens, one kernel for both / two, 109.4 / 105.1, 113.4 / 111.7, 124.1 / 123.7 us; 4 heads
  // of 1152 features, 16 tokens 160.2 / 156.8 (a step of 28 blocks, 64 tokens, 4.72 / 4.76 ms, as two kernels take turns; below 192
  // tokens the one without for long contractions too: 64 tokens 4.77 / 4.82, 4 heads 4.32 / 4.39).
  // The residual update is one kernel for both.
  constexpr bool LONG_RING = NS >= 6, EITHER = LONG_RING && !is_residual(EPI);
  if (!EITHER || (EPI == 3 ? p.split_steps : nk) >= NS)
    return launch_kernel<WGM, WGN, WGK, TM, TN, NS, EPI, LONG_RING, GT>(p, grid, s, gt);
  return launch_kernel<WGM, WGN, WGK, TM, TN, NS, EPI, LONG_RING && !EITHER, GT>(p, grid, s, gt);
}

// ---------------------------------------------------------------------------------------------
// Tile choice.  Ten output tiles make up the list that callers can force (ddit_linear_fwd_tile); 320 x 256 and 192 x 192 stand beside it,
// below, and the forms for few tokens above.  Which is fastest depends on how the tile grid divides over
// the CUs far more than on the tile's own efficiency (a 192 x 384 tile does twice the work per byte
// fetched of a 128 x 192 one, but 60 of them leave 196 CUs idle).  The launcher therefore prices every tile
// with a small model of the kernel and takes the cheapest of the list, or one beside it whose price is lower by a margin.  With  tiles = ceil(N / rows) * ceil(n / cols),
// q = ceil(tiles / CUs)  tiles on the busiest CU and  steps = ceil(k / 64),
//     t = (a * steps + e[epilogue]) * q * (1 + s * min(1, tiles / CUs)) + 2.71      [microseconds]
//         (+ f[copy] * min(1, tiles / CUs) for the residual update)
// a: one k-step; e: a tile's epilogue and set-up; s: the clock and memory slow-down of a full chip against a
// single busy CU; f: what the first round's epilogues cost more, when all CUs reach the memory-bound phase
// together; the rest is the launch.  The constants are a least-squares fit (in log time; bench.py --tile-fit) to a sweep
// (bench.py --tile-sweep, kept in profiles/gemm_tile_sweep.txt) of whole layers with every tile forced in turn, so that
// operands, weights and the residual stream are where a step leaves them: hidden 1152 with 16, 8, 4 and 2 heads of 72, 256
// and 2048, 31 token counts from 96 to 98316, twice.  Over that sweep the picks cost 0.5 % more than the best tile
// everywhere, 1.17 times at worst (1.1 % and 1.29 with constants that had been fitted to launches with everything evicted),
// and as much on the token counts that a fit to every other one has not seen.  The residual update that also writes
// bf16(x) has constants of its own: at 12288 tokens, 1152 x 288, the largest tile takes 52.2 us with the copy and 31.6
// without, 256 x 128 39.6 and 35.1.
// Nine are the ones, of fourteen that were swept, that lose least against all fourteen (0.6 % of a layer); 192 x 288 is
// for widths that are multiples of 288 and of nothing wider, the projections of head splits with 2, 6, 10 or 14 heads of
// 72: the grouped text projections need a tile that divides a problem's columns (launch_gemm_grouped).
// ---------------------------------------------------------------------------------------------
struct TileModel {
  int rows, cols, wavefronts, stages;   // stages: depth of the operand ring in LDS
  float a;        // microseconds per k-step of 64
  float e[4];     // epilogue + set-up microseconds: bf16 / GELU / gated residual / gated residual with the bf16 copy
  float s;        // slow-down of a full chip
  float f[2];     // once per launch, residual update without / with the copy
};
constexpr int N_TILES = 10;
constexpr TileModel TILES[N_TILES] = {
    {192, 384, 8, 2, 1.277f, {4.46f, 6.06f, 13.92f, 17.05f}, 0.310f, {1.30f, 17.05f}},
    {256, 256, 8, 2, 1.114f, {4.21f, 5.43f, 12.17f, 15.78f}, 0.340f, {1.94f, 11.88f}},
    {192, 288, 6, 2, 1.192f, {4.27f, 5.97f, 11.16f, 15.29f}, 0.213f, {3.66f, 12.91f}},
    {192, 256, 8, 2, 1.023f, {3.38f, 4.12f, 9.02f, 12.22f}, 0.220f, {2.78f, 8.91f}},
    {256, 128, 8, 3, 0.622f, {2.24f, 2.72f, 6.98f, 8.83f}, 0.370f, {0.13f, 0.00f}},
    {128, 192, 8, 3, 0.542f, {2.04f, 2.56f, 5.51f, 7.77f}, 0.294f, {0.00f, 0.00f}},
    {128, 128, 8, 4, 0.442f, {2.11f, 2.66f, 4.77f, 6.63f}, 0.187f, {0.03f, 0.72f}},
    {64, 192, 8, 4, 0.483f, {1.66f, 1.93f, 3.68f, 5.46f}, 0.056f, {0.82f, 2.20f}},
    {64, 128, 8, 6, 0.364f, {1.42f, 1.92f, 2.78f, 4.25f}, 0.000f, {0.85f, 2.25f}},
    {64, 64, 8, 8, 0.232f, {0.82f, 1.30f, 1.80f, 2.32f}, 0.087f, {0.00f, 2.16f}},
};
// One more, outside the list that callers can force a tile from: 142 flop per byte fetched (192 x 384: 128), ten MFMA tiles a wavefront, 234
// registers.  Its constants are fitted to two sweeps (1164 linears of 500 to 108000 tokens, hidden 1152 with 16 and 4 heads, 2048); taken
// where its price is two hundredths below the best one's it made the sweeps' linears, residual updates of 2048 features among them, 2.7 % of their time shorter, by 8 to 18 % on average where a
// width is 432 to 864, 512 or 2048: fc1 of 12960 tokens 134.5 -> 123.0 us, 48600 448 -> 428, 108000 967 -> 945; 2048 features, 48600
// tokens, q|k|v 974 -> 907.  On a third sweep (256, 512, 768 features, 2 heads of 1152), which the fit has not seen, the same but for
// columns that do not fill a tile (144: 1.03).  Not for residual updates: their widths here are the hidden size, of which 1152 would leave a
// tenth of its columns empty and is never cheapest, and those of short contractions lost (k = 256 1.07 times the other tile's time).
// For the grouped text projections the 300 tokens of a prompt are one row of its tiles (6 % of the
// matrix work on nothing, W through the L2 once) where they are two of 192 rows (22 %, twice): 56 layers of 2304 features, 300
// tokens 125 -> 92 us, 600 203 -> 174, 900 282 -> 262, 1200 and 2400 as before.
// (256 x 192, 384 x 192 and 192 x 128 were swept too: what the model took them for was 0.1 to 0.4 % shorter on average, with one in
// twenty 3 % and more longer.)
constexpr TileModel WIDE_TILE = {320, 256, 8, 2, 1.372f, {3.51f, 5.69f, 0.00f, 0.00f}, 0.255f, {0.00f, 0.00f}};
constexpr float WIDE_BELOW = 0.98f;
constexpr int WIDE_K = 256;
// Over several rounds of a contraction below 1024 the price is too low, a tile being mostly epilogue.  Where it lay 2 to 6.5 hundredths
// below the listed tile's, the linears took 1.00 to 1.18 times that tile's time, and bf16 outputs with k below 512 gained nothing from
// three rounds on (29 linears 0.94-1.07, 1.01 on average; they are bound by writing): 768 x 256, 35058 tokens, 23.3 -> 27.4 us, 74891 43.4 -> 46.3,
// 256 x 256, 101426 tokens, 26.4 -> 29.8; grouped, 56 layers of 512 features with k = 256, 1600 text tokens 35.5 -> 41.8.  Of 193 linears with k = 256 to 768
// 65 are listed tiles by that, 1.03 times as long with this one, and 128 are this tile, 0.97.
constexpr float WIDE_BELOW_SHORT = 0.935f;
constexpr int WIDE_SHORT_K = 1024, WIDE_PLAIN_K = 512;
// In profiles/gemm_forms_sweep.txt, a sweep that the fit has not seen, 67 of 662 linears take it: 0.92 times the listed pick's time on average, 1.05 at worst.
// And 192 x 192, which is one round of the chip up to 8064 tokens of 1152 features, where from 7200 on 192 x 256 leaves a tenth of its
// columns and a quarter of the CUs empty, and in the same place for other widths.  Fitted to a sweep of the same layers with it forced;
// taken where it is one round and its price a hundredth below the best one's: 20 linears of profiles/gemm_forms_sweep.txt, 0.90 of the other tile's
// time on average, 1.05 at worst.  (Over several rounds the model overrates it: steps of 14800 to 56800 tokens 0 to 2 % longer; at equal
// prices, fc1 of 1600 tokens, a step was 0.5 % longer.)  7756 tokens, us with an event pair's 3.5: fc2
// 115.5 -> 86.1, out-projection with the copy 52.8 -> 42.2, without 40.4 -> 32.1, cross-attention q 31.2 -> 26.8; q|k|v of 2440 tokens 33.4 -> 27.6.
// A step of six blocks: 2496 tokens 2.30 -> 2.26 ms, 5440 4.03 -> 3.96, 6848 4.72 -> 4.63, 7360 5.35 -> 4.94; 4 heads 7360 3.78 -> 3.42.
// Wavefronts of 32 x 96 are as fast but spill; four of 96 x 96 take 1.04 times the time.
constexpr TileModel SQUARE_TILE = {192, 192, 12, 3, 0.512f, {3.07f, 2.67f, 6.25f, 8.00f}, 0.703f, {0.00f, 3.88f}};
constexpr float SQUARE_BELOW = 0.99f;
constexpr int WIDE = N_TILES, SQUARE = N_TILES + 1;   // what tile_to_launch calls them
constexpr int RESIDUAL_COPY = 3;   // the model's index of the residual update that also writes bf16(x)
constexpr float LAUNCH_US = 2.71f;
constexpr int CHIP_CUS = 256;
constexpr int FIRST_SMALL_TILE = 4;   // tiles compiled for partial sums and streaming residuals: this one and the smaller ones
// what adding them up later costs: once, a part, a part and million elements; what a split has to gain to be taken
constexpr float PARTIAL_SUM_US = 5.0f, PARTIAL_SUM_US_PER_PART = 1.0f, PARTIAL_SUM_US_PER_M = 0.6f, PARTIAL_MARGIN_US = 1.5f;

float predicted_us(const TileModel &t, int epilogue, int64_t N, int n, int k, int cus) {
  const double tiles = (double)((N + t.rows - 1) / t.rows) * (double)((n + t.cols - 1) / t.cols);
  const double q = std::ceil(tiles / cus);
  const double one = t.a * (double)((k + BK - 1) / BK) + t.e[epilogue];
  const double full = tiles < cus ? tiles / cus : 1.0;
  return (float)(one * q * (1.0 + t.s * full) + (epilogue >= 2 ? t.f[epilogue - 2] * full : 0.0) + LAUNCH_US);
}

float predicted_us(int tile, int epilogue, int64_t N, int n, int k, int cus) {
  return predicted_us(TILES[tile], epilogue, N, n, k, cus);
}

int cheapest_tile(int epilogue, int64_t N, int n, int k, int cus) {
  int best = 0;
  float best_us = predicted_us(0, epilogue, N, n, k, cus);
  for (int t = 1; t < N_TILES; ++t) {
    const float us = predicted_us(t, epilogue, N, n, k, cus);
    if (us < best_us) { best_us = us; best = t; }
  }
  return best;
}

const TileModel &tile_model(int tile) { return tile == WIDE ? WIDE_TILE : tile == SQUARE ? SQUARE_TILE : TILES[tile]; }

// what the 320 x 256 tile's price has to be below, of the best listed one's; `margin` where its price is right
float wide_below(float margin, int epilogue, int64_t N, int n, int k, int cus) {
  const int64_t tiles = (N + WIDE_TILE.rows - 1) / WIDE_TILE.rows * ((n + WIDE_TILE.cols - 1) / WIDE_TILE.cols);
  if (tiles <= cus || k >= WIDE_SHORT_K) return margin;
  return epilogue == 0 && k < WIDE_PLAIN_K && tiles > 2 * cus ? 0.f : WIDE_BELOW_SHORT;
}

// what the launcher takes: cheapest_tile's, or one of the two beside the list
int tile_to_launch(int epilogue, int64_t N, int n, int k, int cus) {
  int tile = cheapest_tile(epilogue, N, n, k, cus);
  const float listed = predicted_us(tile, epilogue, N, n, k, cus);
  float best = listed;
  auto consider = [&](int other, float below) {
    const float t = predicted_us(tile_model(other), epilogue, N, n, k, cus);
    if (t < below * listed && t < best) { tile = other; best = t; }
  };
  if (epilogue < 2 && n >= WIDE_TILE.cols && k >= WIDE_K) consider(WIDE, wide_below(WIDE_BELOW, epilogue, N, n, k, cus));
  if (n >= SQUARE_TILE.cols && (N + SQUARE_TILE.rows - 1) / SQUARE_TILE.rows * ((n + SQUARE_TILE.cols - 1) / SQUARE_TILE.cols) <= cus)
    consider(SQUARE, SQUARE_BELOW);
  return tile;
}

float launch_price(int epilogue, int64_t N, int n, int k, int cus) {
  return predicted_us(tile_model(tile_to_launch(epilogue, N, n, k, cus)), epilogue, N, n, k, cus);
}

template <int WGM, int WGN, int WGK, int TM, int TN, int NS, int EPI>
int launch_checked(int tile, const GemmParams &p, hipStream_t s) {
  using C = GemmCfg<WGM, WGN, WGK, TM, TN, NS>;
  // the model's table and the compiled tile must describe the same thing
  if (TILES[tile].rows != C::BM || TILES[tile].cols != C::BN || TILES[tile].wavefronts != C::NW ||
      TILES[tile].stages != NS) {
    ddit::set_error("linear: tile table entry %d does not match its kernel", tile);
    return -2;
  }
  return launch_one<WGM, WGN, WGK, TM, TN, NS, EPI>(p, s);
}

// How the residual update writes the stream.  The next launches read x again: written plainly a large one is found in the
// 256 MB memory-side cache; one of a few million elements stays there either way, and the launch then ends with writing
// the L2 back; the smallest stay in the L2 itself.  Streaming / plain, microseconds a layer of a step: 600 tokens x 1152
// (0.7 Mi elements) 113.5 / 113.6, 1200 (1.3 Mi) 145.7 / 146.6, 2304 (2.5) 193.0 / 195.1, 3680 (4.0) 253.9 / 257.1, 4600
// (5.1) 301.0 / 301.6, 6000 (6.6) 346.1 / 344.5, 12960 (14.2) 728 / 715, 19000 (20.9) 1131 / 1121, 48600 3518 / 3522;
// x 2048, 2.3 Mi 255.3 / 258.1, 5.5 Mi 427.8 / 427.3, 7.2 Mi 513.4 / 507.7; x 256, 0.9 Mi 76.2 / 75.6, 1.5 Mi 91.7 / 92.2,
// 5.6 Mi 276.0 / 278.3, 14.6 Mi 971 / 962.  Compiled for the tiles that so few elements take.
constexpr int64_t STREAM_WRITES_FROM = (int64_t)5 << 18, PLAIN_WRITES_FROM = (int64_t)6 << 20;

// Two launches for a long contraction (fc2).  Its tiles read the tokens from memory rather than from the L2, the smaller
// tiles more often, but the largest tile may fill the chip a few times and then a small part of it.  Then the tokens of the
// full rounds are one launch of it, and the rest, at most three fifths of a round, another of whichever form suits (few tokens
// included: 16401 tokens 177 / 173 us with the listed tile / 32 x 32, 16600 171.5 / 167.7); where the
// model sees seven hundredths in that, of which it is wont to overstate as much (where it saw 6.4 of them, 1344 x 5376 and 16600
// tokens, it was 230 / 232 us).  The rest may take a tile that sums k in two halves: a prediction's error against 64 bits is
// 0.999-1.000 times that of one launch (16700 to 33600 tokens, six blocks).  Returns the first one's tokens, or 0.  One launch / two,
// microseconds, 1152 x 4608: 16600 tokens 191 / 161, 18000 193 / 172, 20000 206 / 203, 22500 235 / 227, 33500 411 / 331, 36000
// 422 / 362, 42000 429 / 417, 50200 602 / 494, 67000 701 / 639, 70000 704 / 664 (27000, where two thirds of a round are left,
// 274 / 281); 1344 x 5376: 15000 223 / 210, 25500 405 / 363, 67000 975 / 906; 2048 x 8192: 9300 292 / 290,
// 25500 801 / 754.  Contractions of 1152 gain nothing: the model sees up to a sixth, and -4 to +9 hundredths came of it.
// Those prices are of the listed tiles.  Where one launch is of the 320 x 256 tile (bf16 outputs) it is taken instead if its price is 3.5
// hundredths below the two launches': two / one, us, 1024 x 3072: 16674 tokens 102 / 90, 51098 294 / 285; 1536 x 4096: 12371 133 / 119, 38851
// 384 / 373; 2048 x 3072: 10054 119 / 97; 72 linears of 768 to 3072 features 0.82 to 1.00 times the time.  Nearer than that the two are
// faster: 3072 x 3072, 55401 tokens, priced 0.99 of the two, 848 / 901.
constexpr int64_t TWO_LAUNCHES_FROM = 4096;
constexpr int TWO_LAUNCHES_K = 3072;
constexpr float TWO_LAUNCHES_BELOW = 0.93f, ONE_LAUNCH_BELOW = 0.965f;

int64_t tokens_in_front(int epilogue, int64_t N, int n, int k, int cus) {
  if (N < TWO_LAUNCHES_FROM || k < TWO_LAUNCHES_K) return 0;
  const int64_t cols = (n + TILES[0].cols - 1) / TILES[0].cols, round = cus / cols * TILES[0].rows;
  const int64_t rows = (N + TILES[0].rows - 1) / TILES[0].rows;
  const int64_t front = rows * cols / cus * cus / cols * TILES[0].rows;   // whole rows of tiles
  if (front <= 0 || front >= N || (N - front) * 5 > round * 3) return 0;
  auto listed = [&](int64_t tokens) { return predicted_us(cheapest_tile(epilogue, tokens, n, k, cus), epilogue, tokens, n, k, cus); };
  const float first = predicted_us(0, epilogue, front, n, k, cus);
  if (first + listed(N - front) >= TWO_LAUNCHES_BELOW * listed(N)) return 0;
  return launch_price(epilogue, N, n, k, cus) < ONE_LAUNCH_BELOW * (first + launch_price(epilogue, N - front, n, k, cus)) ? 0 : front;
}

int launch_residual_streaming(int tile, const GemmParams &p, hipStream_t s) {
  switch (tile) {
    case 4: return launch_checked<4, 2, 1, 2, 2, 3, 4>(tile, p, s);
    case 5: return launch_checked<4, 2, 1, 1, 3, 3, 4>(tile, p, s);
    case 6: return launch_checked<2, 2, 2, 2, 2, 4, 4>(tile, p, s);
    case 7: return launch_checked<2, 2, 2, 1, 3, 4, 4>(tile, p, s);
    case 8: return launch_checked<2, 2, 2, 1, 2, 6, 4>(tile, p, s);
    default: return launch_checked<2, 2, 2, 1, 1, 8, 4>(tile, p, s);
  }
}

// elements: of the whole residual stream
template <int EPI>
int launch_epi(int tile, const GemmParams &p, int64_t elements, hipStream_t s) {
  if (tile < 0) tile = tile_to_launch(EPI == 2 && p.out ? RESIDUAL_COPY : EPI, p.N, p.n, p.k, ddit::device_cus());
  if (EPI == 2 && tile >= FIRST_SMALL_TILE && tile < N_TILES && elements >= STREAM_WRITES_FROM && elements < PLAIN_WRITES_FROM)
    return launch_residual_streaming(tile, p, s);
  switch (tile) {
    case 0: return launch_checked<2, 4, 1, 3, 3, 2, EPI>(tile, p, s);
    case 1: return launch_checked<2, 4, 1, 4, 2, 2, EPI>(tile, p, s);
    case 2: return launch_checked<2, 3, 1, 3, 3, 2, EPI>(tile, p, s);
    case 3: return launch_checked<2, 4, 1, 3, 2, 2, EPI>(tile, p, s);
    case 4: return launch_checked<4, 2, 1, 2, 2, 3, EPI>(tile, p, s);
    case 5: return launch_checked<4, 2, 1, 1, 3, 3, EPI>(tile, p, s);
    case 6: return launch_checked<2, 2, 2, 2, 2, 4, EPI>(tile, p, s);
    case 7: return launch_checked<2, 2, 2, 1, 3, 4, EPI>(tile, p, s);
    case 8: return launch_checked<2, 2, 2, 1, 2, 6, EPI>(tile, p, s);
    case 9: return launch_checked<2, 2, 2, 1, 1, 8, EPI>(tile, p, s);
    case SQUARE: return launch_one<2, 6, 1, 3, 1, 3, EPI>(p, s);
    case WIDE:
      if constexpr (EPI < 2) return launch_one<2, 4, 1, 5, 2, 2, EPI>(p, s);
  }
  ddit::set_error("linear: no tile %d (there are %d)", tile, N_TILES);
  return -1;
}

}  // namespace

namespace ddit {

int gemm_tile_count() { return N_TILES; }

int gemm_tile_info(int tile, int *rows, int *cols, int *wavefronts, int *wg_per_cu) {
  if (tile < 0 || tile >= N_TILES) return -1;
  *rows = TILES[tile].rows; *cols = TILES[tile].cols;
  *wavefronts = TILES[tile].wavefronts; *wg_per_cu = 1;
  return 0;
}

int gemm_tile_choice(int epilogue, bool copy, int64_t N, int n, int k, int cus, float *us_per_tile) {
  if (epilogue == 2 && copy) epilogue = RESIDUAL_COPY;
  if (cus <= 0) cus = ddit::device_cus();
  if (us_per_tile)
    for (int t = 0; t < N_TILES; ++t) us_per_tile[t] = predicted_us(t, epilogue, N, n, k, cus);
  return cheapest_tile(epilogue, N, n, k, cus);
}

void gemm_form(int epilogue, bool copy, int64_t N, int n, int k, int cus, int *rows, int *cols) {
  if (epilogue == 2 && copy) epilogue = RESIDUAL_COPY;
  if (cus <= 0) cus = device_cus();
  const int few = few_form(N, n, k, k, 1, (k + BK - 1) / BK, cus);
  const TileModel &t = tile_model(tile_to_launch(epilogue, N, n, k, cus));
  *rows = few ? (few == 1 ? 32 : 64) : t.rows;
  *cols = few ? (few == 3 ? 64 : 32) : t.cols;
}

int gemm_few_form(int64_t N, int n, int k, int parts, int cus) {
  return few_form(N, n, k, k, parts, ((k + BK - 1) / BK + parts - 1) / parts, cus > 0 ? cus : device_cus());
}

int64_t gemm_tokens_in_front(int epilogue, bool copy, int64_t N, int n, int k, int cus) {
  return tokens_in_front(epilogue == 2 && copy ? RESIDUAL_COPY : epilogue, N, n, k, cus > 0 ? cus : device_cus());
}

template <int WGM, int WGN, int WGK, int TM, int TN, int NS>
int launch_grouped_tile(const GemmParams &p, const GroupTable &gt, hipStream_t s) {
  return launch_one<WGM, WGN, WGK, TM, TN, NS, 0, GroupTable>(p, s, gt);
}

// The cheapest tile whose columns divide a problem's out-features (a tile must lie inside one problem), or -1.
static int grouped_tile(int64_t N, int n, int k, int G, int cus) {
  const int n_all = G * n;
  int tile = -1;
  float best = 0.f;
  for (int t = 0; t < N_TILES; ++t) {
    if (n % TILES[t].cols) continue;
    const float us = predicted_us(t, 0, N, n_all, k, cus);
    if (tile < 0 || us < best) { tile = t; best = us; }
  }
  return n % WIDE_TILE.cols == 0 && predicted_us(WIDE_TILE, 0, N, n_all, k, cus) < wide_below(1.f, 0, N, n_all, k, cus) * best ? WIDE : tile;
}

static bool can_group(int64_t N, int n, int64_t ld_u, int k, int G) {
  return G >= 2 && G <= MAX_GROUPS && (int64_t)G * n < (int64_t)1 << 30 && (int64_t)n * k < (int64_t)1 << 31 && N * ld_u < (int64_t)1 << 31;
}

void gemm_grouped_form(int64_t N, int n, int k, int G, int cus, int *rows, int *cols) {
  const int tile = can_group(N, n, k, k, G) ? grouped_tile(N, n, k, G, cus > 0 ? cus : device_cus()) : -1;
  *rows = tile < 0 ? 0 : tile_model(tile).rows;
  *cols = tile < 0 ? 0 : tile_model(tile).cols;
}

// One launch for G problems that share u: out[g] = u W[g]^T + bias[g], every W[g] of shape [a.n, a.k].
// Returns 1 (nothing launched) when the shape cannot be grouped: the caller then launches them one by one.
int launch_gemm_grouped(const GemmArgs &a, int G, const void *const *W, const void *const *bias, void *const *out,
                        hipStream_t s) {
  if (a.N == 0 || a.n == 0 || G == 0) return 0;
  const int tile = can_group(a.N, a.n, a.ld_u, a.k, G) ? grouped_tile(a.N, a.n, a.k, G, device_cus()) : -1;
  if (tile < 0) return 1;
  GroupTable gt;
  gt.group_n = a.n;
  for (int g = 0; g < G; ++g) {
    gt.W[g] = reinterpret_cast<const bf16_t *>(W[g]);
    gt.bias[g] = bias ? reinterpret_cast<const bf16_t *>(bias[g]) : nullptr;
    gt.out[g] = reinterpret_cast<bf16_t *>(out[g]);
  }
  GemmParams p{};
  p.u = reinterpret_cast<const bf16_t *>(a.u); p.ld_u = a.ld_u;
  p.W = gt.W[0]; p.bias = gt.bias[0];
  p.N = a.N; p.n = G * a.n; p.k = a.k;
  p.out = gt.out[0]; p.ld_out = a.ld_out;
  p.tokens_per_sample = a.tokens_per_sample > 0 ? a.tokens_per_sample : 1;
  switch (tile) {
    case 0: return launch_grouped_tile<2, 4, 1, 3, 3, 2>(p, gt, s);
    case 1: return launch_grouped_tile<2, 4, 1, 4, 2, 2>(p, gt, s);
    case 2: return launch_grouped_tile<2, 3, 1, 3, 3, 2>(p, gt, s);
    case 3: return launch_grouped_tile<2, 4, 1, 3, 2, 2>(p, gt, s);
    case 4: return launch_grouped_tile<4, 2, 1, 2, 2, 3>(p, gt, s);
    case 5: return launch_grouped_tile<4, 2, 1, 1, 3, 3>(p, gt, s);
    case 6: return launch_grouped_tile<2, 2, 2, 2, 2, 4>(p, gt, s);
    case 7: return launch_grouped_tile<2, 2, 2, 1, 3, 4>(p, gt, s);
    case 8: return launch_grouped_tile<2, 2, 2, 1, 2, 6>(p, gt, s);
    case 9: return launch_grouped_tile<2, 2, 2, 1, 1, 8>(p, gt, s);
    default: return launch_grouped_tile<2, 4, 1, 5, 2, 2>(p, gt, s);   // WIDE_TILE
  }
}

// The residual update in two launches: `parts` partial products over equal parts of k, fp32 [N, n] each, which the
// launch that reads the stream next sums up (launch_modulated_layernorm).  It pays where so few tokens make
// small tiles or idle CUs: the parts are that many more tiles, larger ones with a shorter chain of k-steps each.
// fc2 (1152 x 4608) of 2304 tokens: 216 tiles of 64 x 192 and 72 steps 46 us, two parts of 108 tiles of
// 128 x 192 and 36 steps 33 us, and 7 us more in the LayerNorm; a layer of 16 heads in all, one launch / 2 / 3 parts:
// 200 tokens 102.0 / 97.0 / 95.5 us, 400 106.5 / 103.5 / 103.6, 800 117.0 / 119.5 / 120.8, 1152 144.3 / 142.4 / 138.2,
// 1500 149.8 / 150.8 / 150.6, 1800 180.6 / 175.5 / 177.0, 2048 187.9 / 181.3, 2304 199.8 / 192.5, 2500 202.7 / 198.2,
// 2720 212.6 / 213.4, 2900 to 3500 the same within 0.6 (4 heads alike; 2720 167.8 / 171.2): nothing is split beyond 2.75 M
// elements, 2503 tokens.
// Tiles and parts are priced with the linears' model, the parts side by side being so many more columns, and what the sum
// costs elsewhere is set to these times (standard error 1.5 us, which a split has to gain).
// A third part gains most below 2 M elements, and only there is the room for it small.
// The answer sizes workspaces, so it depends on the shape alone: priced for the whole chip whatever device is current.
int gemm_partial_choice(int64_t N, int n, int k, int max_parts, int *tile_out) {
  const int cus = CHIP_CUS, steps = (k + BK - 1) / BK;
  const int most = N * (int64_t)n <= (int64_t)2 << 20 ? max_parts : N * (int64_t)n <= (int64_t)11 << 18 ? std::min(max_parts, 2) : 0;
  float best = predicted_us(cheapest_tile(2, N, n, k, cus), 2, N, n, k, cus) - PARTIAL_MARGIN_US;
  int chosen = 0;
  for (int parts = 2; parts <= most && parts <= steps; ++parts) {
    const int per = (steps + parts - 1) / parts;
    if ((parts - 1) * per >= steps) continue;   // the last part would be empty (4 k-steps in three parts of two)
    for (int t = FIRST_SMALL_TILE; t < N_TILES; ++t) {
      const int cols = (n + TILES[t].cols - 1) / TILES[t].cols * TILES[t].cols;
      const float us = predicted_us(t, 0, N, parts * cols, per * BK, cus) + PARTIAL_SUM_US +
                       (PARTIAL_SUM_US_PER_PART + PARTIAL_SUM_US_PER_M * (float)(N * n) * 1e-6f) * parts;
      if (us < best) { best = us; chosen = parts; *tile_out = t; }
    }
  }
  return chosen;
}

int launch_partial_tile(int tile, const GemmParams &p, hipStream_t s) {
  switch (tile) {
    case 4: return launch_checked<4, 2, 1, 2, 2, 3, 3>(tile, p, s);
    case 5: return launch_checked<4, 2, 1, 1, 3, 3, 3>(tile, p, s);
    case 6: return launch_checked<2, 2, 2, 2, 2, 4, 3>(tile, p, s);
    case 7: return launch_checked<2, 2, 2, 1, 3, 4, 3>(tile, p, s);
    case 8: return launch_checked<2, 2, 2, 1, 2, 6, 3>(tile, p, s);
    case 9: return launch_checked<2, 2, 2, 1, 1, 8, 3>(tile, p, s);
  }
  set_error("linear: no partial sums with tile %d", tile);
  return -1;
}

int launch_gemm_partial(const GemmArgs &a, int parts, int tile, float *out, int64_t part_stride, hipStream_t s, bool few) {
  if (a.N == 0 || a.n == 0) return 0;
  if ((int64_t)a.n * a.k >= (int64_t)1 << 31 || a.N * a.ld_u >= (int64_t)1 << 31) {
    set_error("linear: n*k = %lld or N*ld_u = %lld exceeds the 31-bit index range", (long long)a.n * a.k, (long long)(a.N * a.ld_u));
    return -2;
  }
  GemmParams p{};
  p.u = reinterpret_cast<const bf16_t *>(a.u); p.ld_u = a.ld_u;
  p.W = reinterpret_cast<const bf16_t *>(a.W);
  p.bias = reinterpret_cast<const bf16_t *>(a.bias);
  p.N = a.N; p.n = a.n; p.k = a.k;
  p.resid = out;
  p.tokens_per_sample = 1;
  const int steps = (a.k + BK - 1) / BK;
  p.split_steps = (steps + parts - 1) / parts;
  // the launch writes ceil(steps / split_steps) parts, and whoever adds them up reads `parts`
  if (parts < 1 || (parts - 1) * p.split_steps >= steps) {
    set_error("linear: k=%d cannot be split into %d parts of whole k-steps of %d", a.k, parts, BK);
    return -2;
  }
  p.split_stride = part_stride;
  if (few) return launch_few_form<3>(few_form(p.N, p.n, p.ld_u, p.k, parts, p.split_steps, device_cus()), p, s);
  return launch_partial_tile(tile, p, s);
}

int launch_gemm(int epilogue, const GemmArgs &a, hipStream_t s) {
  if (a.N == 0 || a.n == 0) return 0;
  if (a.tile >= N_TILES) {
    set_error("linear: no tile %d (there are %d)", a.tile, N_TILES);
    return -1;
  }
  if ((int64_t)a.n * a.k >= (int64_t)1 << 31) {
    set_error("linear: n*k = %lld exceeds the 32-bit weight index range", (long long)a.n * a.k);
    return -2;
  }
  if (a.N * a.ld_u >= (int64_t)1 << 31) {
    set_error("linear: N*ld_u = %lld exceeds the 31-bit activation index range", (long long)(a.N * a.ld_u));
    return -2;
  }
  GemmParams p{};
  p.u = reinterpret_cast<const bf16_t *>(a.u); p.ld_u = a.ld_u;
  p.W = reinterpret_cast<const bf16_t *>(a.W);
  p.bias = reinterpret_cast<const bf16_t *>(a.bias);
  p.N = a.N; p.n = a.n; p.k = a.k;
  p.out = reinterpret_cast<bf16_t *>(a.out); p.ld_out = a.ld_out;
  p.resid = a.resid;
  p.gate_tab = a.gate_tab; p.gate_c6 = a.gate_c6; p.gate_c6_stride = a.gate_c6_stride;
  p.tokens_per_sample = a.tokens_per_sample > 0 ? a.tokens_per_sample : 1;
  if (epilogue < 0 || epilogue > 2) {
    set_error("unknown epilogue %d", epilogue);
    return -1;
  }
  const int64_t elements = p.N * (int64_t)p.n;
  auto launch = [&](int tile, const GemmParams &q) {
    if (const int form = tile < 0 ? few_form(q.N, q.n, q.ld_u, q.k, 1, (q.k + BK - 1) / BK, device_cus()) : 0)
      return epilogue == 0 ? launch_few_form<0>(form, q, s) : epilogue == 1 ? launch_few_form<1>(form, q, s) : launch_few_form<2>(form, q, s);
    return epilogue == 0 ? launch_epi<0>(tile, q, elements, s) : epilogue == 1 ? launch_epi<1>(tile, q, elements, s)
                                                                                : launch_epi<2>(tile, q, elements, s);
  };
  const int64_t front = a.tile < 0 ? gemm_tokens_in_front(epilogue, p.out != nullptr, p.N, p.n, p.k, 0) : 0;
  if (front > 0) {
    GemmParams first = p;
    first.N = front;
    const int rc = launch(0, first);
    if (rc != 0) return rc;
    p.u += front * p.ld_u;
    if (p.out) p.out += front * p.ld_out;
    if (p.resid) p.resid += front * p.n;
    p.N -= front;
    p.tok0 = (unsigned)front;
  }
  return launch(a.tile, p);
}

}  // namespace ddit
