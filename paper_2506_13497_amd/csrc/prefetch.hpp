// Weights and text keys fetched ahead: which launches do it, and which workgroup reads what.  Plain C++, for the host and the device.
#pragma once
#include <stdint.h>

namespace ddit {

// Weights that the launches after this one read.  Further rows of workgroups (blockIdx.y > 0), each as many as the launch's
// own, read them once, in address order, so that they are in the memory-side cache by then.
struct Prefetch {
  const void *p[2];
  unsigned pieces[2];   // of 16 bytes; none: no further row
};

// Whether a launch over N tokens, attention or LayerNorm, which leave the memory idle, fetches `bytes` of the weights of the
// launches after it.  A step reads every weight from memory (2.4 GB of them), and a linear fetches its own in pieces of one
// line from all rows at once, which the memory serves slowly: at 2304 tokens fc1 takes 27.8 us instead of 32.2 once its weights
// are in the memory-side cache, the out-projections 14.8 instead of 18.0, and the launches that fetch them 1-2 us more.  Times
// of a step without / with it, ms, 28 blocks of 1152 features, 16 heads: 64 tokens 5.07 / 4.77, 128 5.02 / 4.88, 192 4.99 / 4.91,
// 256 5.20 / 5.12, 512 6.13 / 6.00, 960 7.24 / 7.02, 1200 8.04 / 7.87, 1920 9.87 / 9.47, 2304 10.69 / 10.35, 3000 11.75 / 11.72;
// 4 heads: 64 4.58 / 4.36, 128 4.58 / 4.39, 1200 6.96 / 6.77, 2304 8.36 / 8.14.  It does not:
// - above 3200 tokens: a layer of 3680 tokens 251.2 / 252.1 us, 5000 294.9 / 295.5;
// - where the last of several rows of 64 tokens, the tiles that few tokens take, holds less than half: its workgroups have
//   little else to do and bring the weights in by themselves (72 tokens 4.70 / 4.77 ms, 136 4.77 / 4.86, 200 4.97 / 5.10, 272
//   5.34 / 5.42, 324 5.40 / 5.46, 392 5.48 / 5.54, 520 6.01 / 6.07, 648 6.23 / 6.28; half full, 96 4.86 / 4.83, 288 5.47 / 5.44;
//   above 768 tokens tiles are larger: 792 6.42 / 6.44, 1032 7.35 / 7.23, 1160 7.81 / 7.79);
// - more than the launch has time for: 24 MB and, from 1000 tokens on, 24 KB a token.  A step of two blocks of 4096 features,
//   16 heads of 64, which fetched 134 MB in a launch: 64 tokens 0.91 / 0.99 ms, 702 1.60 / 1.75; three of 3072, 48 heads: 64 1.15 /
//   1.20, 1200 2.78 / 2.88; of 1536 features, at most 24 MB, 64 tokens 2.07 / 1.96, 702 3.07 / 2.98.
// A caller of single blocks walks over the layers in the same way (28 blocks, 64 tokens 5.41 / 5.12 ms, 2304 11.22 / 10.92); one
// that calls the same block again finds its weights in the cache and pays for the fetch (64 tokens 170 / 176 us a block, 4 heads
// 160 / 163), which nothing in the call tells apart.
// The text's keys and values of a layer, which its few workgroups of cross-attention read at once (16 heads, 64 tokens: 4.2 us of its
// 9.7 wait for them), come with a layer's first launch up to 1024 tokens.  A step without / with it, ms: 16 heads 64 tokens
// 3.72 / 3.69, 128 4.13 / 4.07, 180 4.30 / 4.27, 256 4.77 / 4.75, 512 5.81 / 5.80, 1024 7.07 / 7.05; 4 heads 64 3.44 / 3.37, 256 4.08 / 4.05;
// beyond, 2304 9.78 / 9.83, 3000 11.38 / 11.43.
constexpr int64_t PREFETCH_UP_TO = 3200, PREFETCH_SMALL_TILES_UP_TO = 768, PREFETCH_TEXT_UP_TO = 1024;
constexpr bool prefetch_pays(int64_t N, int64_t bytes) {
  if (N > PREFETCH_UP_TO) return false;
  const int64_t last = N % 64;
  if (N > 64 && N < PREFETCH_SMALL_TILES_UP_TO && last > 0 && last < 32) return false;
  return bytes <= 24000 * (N > 1000 ? N : 1000);
}

// Rows of a grid of `blocks` workgroups: its own, and so many more that none reads over 48 KB (at most 1 + 1563, as no launch
// fetches more than prefetch_pays lets it).
constexpr unsigned prefetch_rows(const Prefetch &f, int64_t blocks) {
  return (unsigned)(1 + ((int64_t)f.pieces[0] + f.pieces[1] + blocks * 3072 - 1) / (blocks * 3072));
}

// What the reader-th of `readers` workgroups reads of n pieces: from .. end-1, nothing if end <= from.
struct PrefetchSpan { unsigned from, end; };
constexpr PrefetchSpan prefetch_span(unsigned n, unsigned readers, unsigned reader) {
  const unsigned share = (n + readers - 1) / readers, from = reader * share;
  return PrefetchSpan{from, from + share < n ? from + share : n};
}
// The piece that a thread's j-th load reads when its workgroup is at piece `at`: past the end the last one again.
constexpr unsigned prefetch_piece(const PrefetchSpan &s, unsigned at, unsigned j, unsigned threads, unsigned thread) {
  return at + j * threads + thread < s.end ? at + j * threads + thread : s.end - 1;
}

}  // namespace ddit
