// The index arithmetic of the gate and up rows' preparation, as the kernel walks it: every
// thread's pieces end, together they are all pieces once, and the rows and columns of the
// first and last are those of the matrix, also beyond 2^32 pieces.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "prep_index.h"

#define CHECK(cond, ...)                                          \
  do {                                                            \
    if (!(cond)) {                                                \
      std::fprintf(stderr, "FAILED %s:%d: %s: ", __FILE__, __LINE__, #cond); \
      std::fprintf(stderr, __VA_ARGS__);                          \
      std::fprintf(stderr, "\n");                                 \
      std::exit(1);                                               \
    }                                                             \
  } while (0)

using namespace dtp;

// Pieces that the thread starting at `g` takes, walked step by step; more than `limit` is no end.
static uint64_t walk(uint64_t g, uint64_t n, unsigned blocks, uint64_t limit, uint64_t* last) {
  uint64_t steps = 0;
  for (; g < n; g = prep_next(g, blocks)) {
    *last = g;
    if (++steps > limit) break;
  }
  return steps;
}

template <int RUN>
static void check_small(int I_pad, int dP) {
  const uint64_t n = prep_pieces(I_pad, dP);
  std::vector<char> seen((size_t)2 * I_pad * (dP / 8));
  CHECK(n == seen.size(), "I_pad=%d dP=%d", I_pad, dP);
  for (uint64_t g = 0; g < n; ++g) {
    const PrepPlace p = prep_place<RUN>(g, dP / (8 * RUN));
    CHECK(p.row < 2u * (unsigned)I_pad && p.col % 8 == 0 && p.col < dP, "piece %llu", (unsigned long long)g);
    char& s = seen[(size_t)p.row * (dP / 8) + p.col / 8];
    CHECK(!s, "piece %llu twice", (unsigned long long)g);
    s = 1;
  }
}

template <int RUN>
static void check_large(int I_pad, int dP) {
  const uint64_t n = prep_pieces(I_pad, dP);
  const unsigned blocks = prep_blocks(n);
  CHECK((double)n == 2.0 * I_pad * dP / 8, "I_pad=%d dP=%d: %llu pieces", I_pad, dP, (unsigned long long)n);
  const uint64_t threads = (uint64_t)blocks * kPrepThreads, most = n / threads + 1;
  CHECK(blocks > 0, "I_pad=%d dP=%d", I_pad, dP);
  uint64_t total = 0, end = 0;
  for (uint64_t t : {prep_first(0, 0), prep_first(blocks / 2, 7), prep_first(blocks - 1, kPrepThreads - 1)}) {
    CHECK(t < threads, "thread %llu", (unsigned long long)t);
    uint64_t last = 0;
    const uint64_t steps = walk(t, n, blocks, most, &last);
    CHECK(steps == (t < n ? (n - t + threads - 1) / threads : 0), "thread %llu: %llu steps", (unsigned long long)t,
          (unsigned long long)steps);
    total += steps;
    end = last > end ? last : end;
  }
  CHECK(total > 0 && end < n, "I_pad=%d dP=%d", I_pad, dP);
  const PrepPlace p = prep_place<RUN>(n - 1, dP / (8 * RUN));
  CHECK(p.row == 2u * (unsigned)I_pad - 1 && p.col == dP - 8, "I_pad=%d dP=%d: last piece at %u, %d", I_pad, dP, p.row,
        p.col);
}

int main() {
  check_small<8>(128, 128);
  check_small<8>(256, 1152);
  check_small<4>(384, 128);
  check_small<4>(128, 1664);
  // around 2^32 pieces, and the largest layer that is accepted
  for (int dP : {16128, 16256, 16384, 16512, 65536}) {
    check_large<8>(1 << 20, dP);
    check_large<4>(1 << 20, dP);
  }
  check_large<8>(262144, 65408);
  check_large<8>(14336, 4096);
  std::printf("index checks passed\n");
  return 0;
}
