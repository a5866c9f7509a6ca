// Index arithmetic of the folded gate and up rows' preparation (affinity.hip), apart from the
// kernel so that a host program can check it at sizes that no test allocates: the pieces of a
// layer can exceed 2^32 (d = 16,384 and I = 2^20 have 2^32 of them in 64 GiB of rows).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

namespace dtp {

constexpr int kPrepThreads = 256;

// 16-byte pieces of 2 I_pad rows of dP columns, and the blocks that walk them.
inline uint64_t prep_pieces(int I_pad, int dP) { return (uint64_t)2 * I_pad * dP / 8; }
inline unsigned prep_blocks(uint64_t pieces) {
  return (unsigned)std::min<uint64_t>((pieces + kPrepThreads - 1) / kPrepThreads, 1u << 20);
}

// A thread's pieces: its global index first, then the next after g.
__host__ __device__ inline uint64_t prep_first(unsigned block, unsigned thread) {
  return (uint64_t)block * kPrepThreads + thread;
}
__host__ __device__ inline uint64_t prep_next(uint64_t g, unsigned blocks) {
  return g + (uint64_t)blocks * kPrepThreads;
}

struct PrepPlace {
  uint32_t row;
  int col;  // the first of its eight
};

// Piece g, in units of 16 rows x RUN pieces, so that RUN consecutive threads read 16 RUN
// contiguous bytes; units_per_row = dP / (8 RUN).
template <int RUN>
__host__ __device__ inline PrepPlace prep_place(uint64_t g, int units_per_row) {
  const uint32_t u = (uint32_t)(g / (16 * RUN)), w = (uint32_t)(g % (16 * RUN));
  return {16 * (u / units_per_row) + w / RUN, 8 * (int)((u % units_per_row) * RUN + w % RUN)};
}

}  // namespace dtp
