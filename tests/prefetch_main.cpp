// Reads "pays N bytes" and "span pieces0 pieces1 blocks threads" lines and answers each from csrc/prefetch.hpp: the rule's
// answer, or the rows of the grid, the most 16-byte pieces that a workgroup reads and whether every piece of both arrays is
// read by exactly one workgroup, none twice but an array's last ones of a workgroup, and nothing beyond them.
#include <cstdio>
#include <cstring>
#include <vector>

#include "../paper_2506_13497_amd/csrc/prefetch.hpp"

using namespace ddit;

int main() {
  char what[16];
  while (scanf("%15s", what) == 1) {
    if (!strcmp(what, "pays")) {
      long long N, bytes;
      if (scanf("%lld %lld", &N, &bytes) != 2) return 1;
      printf("%d\n", (int)prefetch_pays(N, bytes));
      continue;
    }
    unsigned pieces[2], blocks, threads;
    if (scanf("%u %u %u %u", &pieces[0], &pieces[1], &blocks, &threads) != 4) return 1;
    const Prefetch f = {{nullptr, nullptr}, {pieces[0], pieces[1]}};
    const unsigned rows = prefetch_rows(f, blocks), readers = blocks * (rows - 1), ahead = 8;
    bool ok = true;
    std::vector<unsigned> of_reader(readers, 0);
    for (int w = 0; w < 2 && readers > 0; ++w) {
      std::vector<unsigned> by(pieces[w], 0);   // the workgroup that read a piece, counted from one
      for (unsigned r = 0; r < readers; ++r) {
        const PrefetchSpan s = prefetch_span(pieces[w], readers, r);
        for (unsigned at = s.from; at < s.end; at += threads * ahead)
          for (unsigned j = 0; j < ahead; ++j)
            for (unsigned t = 0; t < threads; ++t) {
              const unsigned i = prefetch_piece(s, at, j, threads, t);
              if (i >= pieces[w] || (by[i] != 0 && (by[i] != r + 1 || i != s.end - 1))) { ok = false; continue; }
              if (by[i] == 0) ++of_reader[r];
              by[i] = r + 1;
            }
      }
      for (unsigned b : by) ok = ok && b != 0;
    }
    unsigned most = 0;
    for (unsigned n : of_reader) most = n > most ? n : most;
    printf("%u %u %d\n", rows, most, (int)ok);
  }
  return 0;
}
