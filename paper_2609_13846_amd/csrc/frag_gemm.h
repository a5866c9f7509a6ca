// The bf16 contraction shared by the folding, down-edge and affinity kernels of libdtp.so
// (gfx950): both operands in fragment-major layout, copied into LDS by the buffer unit.
//
// Fragment-major layout of a matrix of R rows x K columns (a multiple of 32), K contiguous in
// the source, in tiles of F fragments of 16 rows (R is a multiple of 16 F): the 16 x 32 block
// of fragment f of tile t and stage ks is one 1 KB run,
//   element (row, k) at (((t * (K / 32) + ks) * F + f) * 64 + lane) * 8 + k % 8,
//   t = row / (16 F), f = row / 16 % F, ks = k / 32, lane = (k % 32) / 8 * 16 + row % 16,
// which is lane order of v_mfma_f32_16x16x32_bf16's operands (lane l: row l % 16, columns
// 8 (l / 16) .. + 7).  A fragment is then one conflict-free 16-byte LDS read per lane, with no
// swizzle and no address arithmetic, and what a block needs of a tile at a stage is one run
// of F KB in memory.
//
// The loop (FragPipe): eight wavefronts, 2 along A x 4 along B, each AF x BF tiles of 16 x 16.
// A stage is 32 columns and has an LDS slot, one of four.  A wavefront takes its A fragments in
// two halves, so that every LDS read is issued well before its products: half 1's during half
// 0's products, the next stage's half 0 during half 1's, and each of its B fragments into the
// registers of a column that half 1 has done.  The one barrier per stage stands between the
// halves, where neither side of it waits for LDS: it says that the next stage has landed for
// all, and that this stage's slot, whose last fragments are in registers, may be overwritten.
// So a copy has the time of three stages to land; with two (a slot and a barrier for every other
// stage) the down-edge kernel of the 8B-class shape took 648 us instead of 565.  The copies
// and their scalar work stand beside products (522 us), not between the barrier and the first.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "tile_mfma.h"

namespace dtp {

// A buffer descriptor: loads past `bytes` return zeros instead of touching memory.
// 0x00020000: the descriptor word that selects 32-bit raw access on gfx9-class GPUs.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frag_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// Offset (in elements) of the 16-byte piece holding (row, k .. k+7) in a fragment-major
// matrix of `ks` stages per row, in tiles of F fragments.
template <int F>
__device__ __forceinline__ int64_t frag_offset(uint32_t row, int k, int ks) {
  return (((int64_t)(row / (16 * F)) * ks + k / 32) * F + row / 16 % F) * 512 + ((k % 32) / 8 * 16 + row % 16) * 8;
}

template <int AF, int BF>
struct FragPipe {
  static constexpr int kAFrags = 2 * AF, kBFrags = 4 * BF, kFrags = kAFrags + kBFrags;
  static constexpr int kARows = 16 * kAFrags, kBRows = 16 * kBFrags;
  static constexpr int kSlot = kFrags * 512;  // bf16 per LDS slot
  static constexpr int kCopies = 4;           // fragments per copying wavefront and stage
  static constexpr int kH0 = (AF + 1) / 2, kH1 = AF - kH0;  // fragments of the two A halves
  static_assert(kAFrags % kCopies == 0 && kBFrags % kCopies == 0 && kFrags <= 8 * kCopies, "copies share out");

  // Byte offsets of a stage in the block's A and B tiles.
  struct Source {
    uint32_t a, b;
  };

  int wave, lane, wm, wn;
  bool copies_a;  // the wavefront's share of a stage is of A rows, or else of B rows
  __amdgpu_buffer_rsrc_t src;
  uint32_t first;  // byte offset of its fragments in a stage's run
  f32x4 acc[AF][BF];
  bf16x8 a0[kH0], a1[kH1], b[BF];

  // a, b: the block's first A and B tile, and the bytes that it may read from there on.
  __device__ __forceinline__ FragPipe(const uint16_t* a, uint32_t a_bytes, const uint16_t* bm,
                                      uint32_t b_bytes) {
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    wm = wave & 1;
    wn = wave >> 1;
    copies_a = wave < kAFrags / kCopies;
    src = copies_a ? frag_rsrc(a, a_bytes) : frag_rsrc(bm, b_bytes);
    first = (uint32_t)(kCopies * min(wave, kFrags / kCopies - 1) - (copies_a ? 0 : kAFrags)) * 1024u;
  }

  // A stage into a slot, four fragments per wavefront.  Where eight wavefronts are too many the
  // last copies its neighbour's again: a branch here would keep the products from starting
  // beside the copies.
  __device__ __forceinline__ void copy(uint16_t* slot, Source at) const {
    // Recomputed for each stage: kept over a loop, the addresses of four slots' copies would not
    // fit the scalar registers.
    int w = wave;
    asm("" : "+s"(w) : "s"(at.b));
    w = __builtin_amdgcn_readfirstlane(kFrags == 8 * kCopies ? w : min(w, kFrags / kCopies - 1));
    const uint32_t o = first + (copies_a ? at.a : at.b);
#pragma unroll
    for (int j = 0; j < kCopies; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          src, (__attribute__((address_space(3))) void*)(slot + (kCopies * w + j) * 512), 16, lane * 16,
          __builtin_amdgcn_readfirstlane((int)(o + j * 1024u)), 0, 0);
  }

  // Waits until this wavefront's copies but those of the last STAGES have landed and its LDS
  // reads are done, then for the block.
  template <int STAGES>
  __device__ __forceinline__ void landed() const {
    static_assert(STAGES * kCopies < 16, "vmcnt field");
    asm volatile("" ::: "memory");  // no LDS access moves across the barrier
    __builtin_amdgcn_s_waitcnt(0x0070 | (STAGES * kCopies));  // vmcnt, lgkmcnt(0)
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
  __device__ __forceinline__ void read_b(const uint16_t* slot, int i) {
    b[i] = frag(slot, kAFrags + wn * BF + i);
  }

  // Keeps a half stage's order through scheduling: FIRST LDS reads, then column by column its
  // ROWS products with VALUS vector instructions of an epilogue beside each, LATER reads and
  // one of COPIES copies.
  template <int FIRST, int ROWS, int LATER, int COPIES, int VALUS>
  __device__ __forceinline__ void order() const {
    __builtin_amdgcn_sched_group_barrier(0x100, FIRST, 0);
#pragma unroll
    for (int j = 0; j < BF; ++j) {
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (VALUS > 0) __builtin_amdgcn_sched_group_barrier(0x002, VALUS, 0);
      }
      if (j < COPIES) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      if constexpr (LATER > 0) __builtin_amdgcn_sched_group_barrier(0x100, LATER, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // Half 0 of the stage in `cur`: products of a0 and b, half 1's fragments read.  ZERO starts
  // the accumulators from zero.  `beside` is vector work that touches none of half 0's
  // accumulators, VALUS instructions per product.
  template <bool ZERO, int VALUS, typename F>
  __device__ __forceinline__ void half0(const uint16_t* cur, F&& beside) {
    read_half1(cur);
    beside();
#pragma unroll
    for (int j = 0; j < BF; ++j)
#pragma unroll
      for (int i = 0; i < kH0; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[i], b[j], ZERO ? f32x4{} : acc[i][j], 0, 0, 0);
    order<kH1, kH0, 0, 0, VALUS>();
  }
  template <bool ZERO>
  __device__ __forceinline__ void half0(const uint16_t* cur) {
    half0<ZERO, 0>(cur, [] {});
  }

  // Half 1 of the stage in `cur`: once the next stage has landed for the block, products of a1
  // and b, the fragments of the next stage's half 0 read, each B fragment when its column is
  // done, into the same registers; and the stage four on sent on its way into this one's slot.
  template <bool ZERO, int VALUS, typename F>
  __device__ __forceinline__ void half1(uint16_t* cur, const uint16_t* next, Source at, F&& beside) {
    landed<2>();
    copy(cur, at);
    read_half0(next);
    beside();
#pragma unroll
    for (int j = 0; j < BF; ++j) {
#pragma unroll
      for (int i = 0; i < kH1; ++i)
        acc[kH0 + i][j] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[i], b[j], ZERO ? f32x4{} : acc[kH0 + i][j], 0, 0, 0);
      read_b(next, j);
    }
    order<kH0, kH1, 1, kCopies, VALUS>();
  }
  template <bool ZERO>
  __device__ __forceinline__ void half1(uint16_t* cur, const uint16_t* next, Source at) {
    half1<ZERO, 0>(cur, next, at, [] {});
  }
  // A stage without products.
  __device__ __forceinline__ void skip(uint16_t* cur, const uint16_t* next, Source at) {
    landed<2>();
    copy(cur, at);
    read_next(next);
  }
  __device__ __forceinline__ void read_next(const uint16_t* next) {
    read_half0(next);
#pragma unroll
    for (int j = 0; j < BF; ++j) read_b(next, j);
  }

  // Four stages are on their way: the first has landed, and its first fragments.
  __device__ __forceinline__ void begin(const uint16_t* s0) {
    landed<3>();
    read_next(s0);
  }

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < AF; ++i)
#pragma unroll
      for (int j = 0; j < BF; ++j) acc[i][j] = f32x4{};
  }

  // The whole contraction over nq stages; past the last the copies fetch it again.  Those still
  // in flight at the end are waited for: nothing may land in LDS after the block has given it
  // back.
  __device__ __forceinline__ void contract(uint16_t* s0, uint16_t* s1, uint16_t* s2, uint16_t* s3, int nq) {
    auto at = [&](int q) __attribute__((always_inline)) {
      const uint32_t o = 1024u * (uint32_t)min(q, nq - 1);
      return Source{o * kAFrags, o * kBFrags};
    };
    auto stage = [&](uint16_t* cur, uint16_t* next, int q) __attribute__((always_inline)) {
      const Source later = at(q + 4);
      half0<false>(cur);
      half1<false>(cur, next, later);
    };
    zero();
    copy(s0, at(0));
    copy(s1, at(1));
    copy(s2, at(2));
    copy(s3, at(3));
    begin(s0);
    int q = 0;
    for (; q + 3 < nq; q += 4) {
      stage(s0, s1, q);
      stage(s1, s2, q + 1);
      stage(s2, s3, q + 2);
      stage(s3, s0, q + 3);
    }
    if (q < nq) stage(s0, s1, q);
    if (q + 1 < nq) stage(s1, s2, q + 1);
    if (q + 2 < nq) stage(s2, s3, q + 2);
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

namespace {

// The transpose of a row-major [n_j][n_k] bf16 matrix in fragment-major layout (rows k < 64
// gridDim.x, columns j < 32 ks): element (k, j) = in[j][k], times gamma[j] and rounded to bf16
// with SCALE, zero for k >= n_k or j >= n_j.  64 x 64 tiles through LDS, 16-byte reads along k
// with VEC (n_k and the address allow them) and writes of whole fragments.  HBM-bound: 40 to 49 us
// for 4,096 x 14,336, scaled (106 us with 2-byte accesses).
template <int F, bool SCALE, bool VEC>
__global__ void __launch_bounds__(256)
transpose_fragments_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ gamma, int n_j,
                           int n_k, int ks, uint16_t* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64][64 + 8];
  const int k0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int idx = threadIdx.x + 256 * pass;
    const int r = idx / 8, c = 8 * (idx % 8);
    const int j = j0 + r, k = k0 + c;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (j < n_j && k < n_k) {
      const uint16_t* p = in + (int64_t)j * n_k + k;
      if constexpr (VEC) {
        v = *reinterpret_cast<const u32x4*>(p);
      } else {  // n_k is a multiple of 8 all the same
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (uint32_t)p[2 * e] | ((uint32_t)p[2 * e + 1] << 16);
      }
      if constexpr (SCALE) {
        const float gj = bf16_to_f32(gamma[j]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[e] = (uint32_t)f32_to_bf16(__uint_as_float(v[e] << 16) * gj) |
                 ((uint32_t)f32_to_bf16(__uint_as_float(v[e] & 0xffff0000u) * gj) << 16);
      }
    }
    *reinterpret_cast<u32x4*>(&tile[r][c]) = v;
  }
  __syncthreads();
  // 4 x 2 fragments of 64 pieces: wavefront w writes those of rows 16 w .. + 15
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = 16 * w + lane % 16;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int j = 32 * half + 8 * (lane / 16);
    if (j0 + j >= 32 * ks) continue;
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = (uint32_t)tile[j + 2 * e][k] | ((uint32_t)tile[j + 2 * e + 1][k] << 16);
    *reinterpret_cast<u32x4*>(out + frag_offset<F>(k0 + k, j0 + j, ks)) = o;
  }
}

}  // namespace

}  // namespace dtp
