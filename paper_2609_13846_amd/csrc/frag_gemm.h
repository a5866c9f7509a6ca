// The bf16 contraction shared by the folding, down-edge and affinity kernels of libdtp.so
// (gfx950): both operands in fragment-major layout, copied into LDS by the buffer unit.
//
// Fragment-major layout of a matrix of R rows (a multiple of 16) x K columns (a multiple of
// 32), K contiguous in the source: the 16 x 32 block (rb, ks) is one 1 KB run,
//   element (row, k) at ((rb * (K / 32) + ks) * 64 + lane) * 8 + k % 8,
//   rb = row / 16, ks = k / 32, lane = (k % 32) / 8 * 16 + row % 16,
// which is lane order of v_mfma_f32_16x16x32_bf16's operands (lane l: row l % 16, columns
// 8 (l / 16) .. + 7).  A fragment is then one contiguous load from memory and one
// conflict-free 16-byte LDS read per lane, with no swizzle and no address arithmetic.
//
// The loop (FragPipe): eight wavefronts, 2 along A x 4 along B, each AF x BF tiles of 16 x 16.
// A stage is 32 columns.  Four LDS slots: stage q + 3 is copied during stage q.  A wavefront
// takes its A fragments in two halves, so that every LDS read is issued half a stage before
// its products: half 1's during half 0's products, the next stage's B and half 0 during
// half 1's.  The one barrier per stage stands between the halves, where neither side of it
// waits for LDS: it says that stage q + 1 has landed for all and that slot (q + 3) % 4, last
// read before half 1 of stage q - 1, may be overwritten.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "tile_mfma.h"

namespace dtp {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// A buffer descriptor: loads past `bytes` return zeros instead of touching memory.
// 0x00020000: the descriptor word that selects 32-bit raw access on gfx9-class GPUs.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frag_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// Offset (in elements) of the 16-byte piece holding (row, k .. k+7) in a fragment-major
// matrix of `ks` stages per row.
__device__ __forceinline__ int64_t frag_offset(int64_t row, int k, int ks) {
  return ((row / 16 * ks + k / 32) * 64 + (k % 32) / 8 * 16 + row % 16) * 8;
}

template <int AF, int BF>
struct FragPipe {
  static constexpr int kAFrags = 2 * AF, kBFrags = 4 * BF, kFrags = kAFrags + kBFrags;
  static constexpr int kARows = 16 * kAFrags, kBRows = 16 * kBFrags;
  static constexpr int kSlot = kFrags * 512;              // bf16 per LDS slot
  static constexpr int kCopies = (kFrags + 7) / 8;        // copies per wavefront and stage, at most
  static constexpr int kFew = kFrags / 8;                 // by the wavefronts with the fewest
  static constexpr int kH0 = (AF + 1) / 2, kH1 = AF - kH0;  // fragments of the two A halves

  int wave, lane, wm, wn;
  bool many;  // this wavefront copies kCopies fragments per stage, not kFew
  __amdgpu_buffer_rsrc_t src[kCopies];
  uint32_t off[kCopies];
  f32x4 acc[AF][BF];
  bf16x8 a0[kH0], a1[kH1 > 0 ? kH1 : 1], b[2][BF];

  // a, b: the block's first A and B row in fragment-major matrices of ks_a and ks_b stages.
  __device__ __forceinline__ FragPipe(const uint16_t* a, int ks_a, const uint16_t* bm, int ks_b) {
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    wm = wave & 1;
    wn = wave >> 1;
    many = wave + 8 * (kCopies - 1) < kFrags;
    const __amdgpu_buffer_rsrc_t ra = frag_rsrc(a, (uint32_t)kAFrags * ks_a * 1024u);
    const __amdgpu_buffer_rsrc_t rb = frag_rsrc(bm, (uint32_t)kBFrags * ks_b * 1024u);
#pragma unroll
    for (int j = 0; j < kCopies; ++j) {
      const int f = wave + 8 * j;
      src[j] = f < kAFrags ? ra : rb;
      off[j] = f < kAFrags ? (uint32_t)f * ks_a * 1024u : (uint32_t)(f - kAFrags) * ks_b * 1024u;
    }
  }

  // Stage q into a slot.
  __device__ __forceinline__ void copy(uint16_t* slot, int q) const {
#pragma unroll
    for (int j = 0; j < kCopies; ++j)
      if (j < kFew || many)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            src[j], (__attribute__((address_space(3))) void*)(slot + (wave + 8 * j) * 512), 16, lane * 16,
            (int)(off[j] + (uint32_t)q * 1024u), 0, 0);
  }

  // Waits until all but the last `stages` stages' copies of this wavefront have landed, then
  // for the block.
  template <int STAGES>
  __device__ __forceinline__ void landed() const {
    if constexpr (kFew == kCopies) {
      __builtin_amdgcn_s_waitcnt(0x0f70 | (STAGES * kCopies));  // vmcnt only
    } else {
      if (many)
        __builtin_amdgcn_s_waitcnt(0x0f70 | (STAGES * kCopies));
      else
        __builtin_amdgcn_s_waitcnt(0x0f70 | (STAGES * kFew));
    }
    static_assert(STAGES * kCopies < 16, "vmcnt field");
    asm volatile("" ::: "memory");  // no LDS access moves across the barrier
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }

  __device__ __forceinline__ bf16x8 frag(const uint16_t* slot, int f) const {
    return *reinterpret_cast<const bf16x8*>(slot + f * 512 + lane * 8);
  }
  __device__ __forceinline__ void read_half0(const uint16_t* slot) {
#pragma unroll
    for (int i = 0; i < kH0; ++i) a0[i] = frag(slot, wm * AF + i);
  }
  __device__ __forceinline__ void read_half1(const uint16_t* slot) {
#pragma unroll
    for (int i = 0; i < kH1; ++i) a1[i] = frag(slot, wm * AF + kH0 + i);
  }
  template <int P>
  __device__ __forceinline__ void read_b(const uint16_t* slot) {
#pragma unroll
    for (int i = 0; i < BF; ++i) b[P][i] = frag(slot, kAFrags + wn * BF + i);
  }

  // Keeps a half stage's order through scheduling: its LDS reads, for the next half, first.
  template <int READS, int MFMAS>
  __device__ __forceinline__ void order() const {
    __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, MFMAS, 0);
    __builtin_amdgcn_sched_barrier(0);
  }

  // Stages 0, 1 and 2 on their way, stage 0's first fragments read.
  __device__ __forceinline__ void begin(uint16_t* s0, uint16_t* s1, uint16_t* s2, int nq) {
    copy(s0, 0);
    copy(s1, min(1, nq - 1));
    copy(s2, min(2, nq - 1));
    landed<2>();
    read_b<0>(s0);
    read_half0(s0);
  }

  // Stage q (P = q % 2) in `cur`, stage q + 1 in `next`, stage q + 3 copied into `fill`.  The
  // copies past the last stage fetch it again, so that the wait counts stay exact.
  template <int P>
  __device__ __forceinline__ void stage(const uint16_t* cur, const uint16_t* next, uint16_t* fill, int q,
                                        int nq) {
    read_half1(cur);
#pragma unroll
    for (int i = 0; i < kH0; ++i)
#pragma unroll
      for (int j = 0; j < BF; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[i], b[P][j], acc[i][j], 0, 0, 0);
    order<kH1, kH0 * BF>();
    landed<1>();
    copy(fill, min(q + 3, nq - 1));
    __builtin_amdgcn_sched_barrier(0);
    read_b<1 - P>(next);
    read_half0(next);
#pragma unroll
    for (int i = 0; i < kH1; ++i)
#pragma unroll
      for (int j = 0; j < BF; ++j)
        acc[kH0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[i], b[P][j], acc[kH0 + i][j], 0, 0, 0);
    order<kH0 + BF, kH1 * BF>();
  }

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < AF; ++i)
#pragma unroll
      for (int j = 0; j < BF; ++j) acc[i][j] = f32x4{};
  }

  // The whole contraction over nq stages.  The copies still in flight at its end are waited
  // for: nothing may land in LDS after the block has given it back.
  __device__ __forceinline__ void contract(uint16_t* s0, uint16_t* s1, uint16_t* s2, uint16_t* s3, int nq) {
    zero();
    begin(s0, s1, s2, nq);
    int q = 0;
    for (; q + 3 < nq; q += 4) {
      stage<0>(s0, s1, s3, q, nq);
      stage<1>(s1, s2, s0, q + 1, nq);
      stage<0>(s2, s3, s1, q + 2, nq);
      stage<1>(s3, s0, s2, q + 3, nq);
    }
    if (q < nq) stage<0>(s0, s1, s3, q, nq);
    if (q + 1 < nq) stage<1>(s1, s2, s0, q + 1, nq);
    if (q + 2 < nq) stage<0>(s2, s3, s1, q + 2, nq);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
  }
};

// Work item of block b among n_a x n_b tiles.  Blocks are dealt to the 8 XCDs round-robin
// and each XCD has its own L2: each takes one contiguous run of an order in bands of `band`
// A tiles, B tile by B tile inside a band, so that the blocks an XCD runs together share
// a few A and B tiles.
__device__ __forceinline__ void frag_work(int blk, int n_a, int n_b, int band, int& ta, int& tb) {
  const int n = n_a * n_b;
  const int x = blk % 8, slot = blk / 8;
  const int j = x * (n / 8) + min(x, n % 8) + slot;
  const int g = j / (band * n_b), r = j % (band * n_b);
  const int gw = min(band, n_a - band * g);
  tb = r / gw;
  ta = band * g + r % gw;
}

}  // namespace dtp
