// First-order head-to-neuron affinity on MI355X (gfx950): Section 3 of the paper,
// "Affinity scores", score FO, accumulated over a stream of calibration tokens.
//
// For token t with residual x (entering the FFN pre-norm), r = sqrt(mean(x^2) + eps),
// gain gamma, neuron k's pre-activations g_k = w^g_k . (gamma x / r) and u_k likewise,
// and head h's normalised piece p_h = gamma (a_h W_o^(h)) / r, the damage is
//   Delta_hk = silu'(g_k) u_k (p_h . w^g_k) + silu(g_k) (p_h . w^u_k)
// and the layer's raw score is A[g, k] = ||w^d_k||^2 sum_t sum_{h in g} Delta_hk^2.
//
// Re-association (exact up to rounding): p_h . w_k = (a_h . F_h[:, k]) / r with the folded
// matrix F_h = W_o^(h) diag(gamma) W^T of shape [dh, I].  So per token
//   Delta_hk = c1_k (a_h . Fg_h[:, k]) + c2_k (a_h . Fu_h[:, k]),
//   c1_k = silu'(g_k) u_k / r,   c2_k = silu(g_k) / r,
// and the whole layer is one long contraction per (token tile, neuron tile): first
// [x] x [gamma W_gate | gamma W_up]^T over d (operating point), then, for every head,
// [a_h] x [Fg_h | Fu_h] over dh, with a register epilogue after each head.
//
// Kernels of the bf16 path:
//   prep_gate_up_fragments_kernel  W' = W diag(gamma), fragment-major
//   transpose_fragments_kernel  W_o^T, fragment-major
//   fold_kernel           F = W' W_o (MFMA)
//   down_norm_*_kernel    n_d[k] = ||w^d_k||^2 (row chunks, then their fixed-order sum)
//   tile_tokens_kernel    1/r per token, [x | a] rewritten fragment-major
//   affinity_bf16_kernel  the fused operating point + per-head damage + token reduction
//   reduce_splits_kernel  deterministic fp64 sum of the per-split partials into A
// Both operands of the fused kernel are fragment-major (frag_gemm.h).  The weights are one
// matrix of 2 I_pad rows, 64 per 32 neurons (their gate rows, then their up rows), and
// Kt = dP + H*dhP columns [W' | F_0 | F_1 | ... | F_{H-1}]; the tokens one of Kt columns [x | a_0 |
// ... | a_{H-1}], rewritten once per slice.  dP is d rounded up to 128 columns and dhP dh to
// whole stages of 32 (past six of them to 128 columns), the columns between them zero.  The fused kernel is one contraction
// over Kt with epilogues at the operating-point and head boundaries.
// The fp32 path (dtype DTP_F32, affinity_f32.hip) runs the same decomposition on fp32 MFMAs.
#include <atomic>
#include <cmath>
#include <vector>

#include "dtp_internal.h"
#include "frag_gemm.h"
#include "prep_index.h"
#include "tile_mfma.h"

namespace dtp {
namespace {

constexpr int kBN = 64;           // neurons per tile of the fp32 path's folded rows
constexpr int kCols = 2 * kBN;    // its rows: 64 gate | 64 up
constexpr int kStage = 32;        // contraction columns per stage of the bf16 kernels
constexpr int kBlockNeurons = 128;     // neurons per block of the fused bf16 kernel
constexpr int kWeightFrags = 2 * kBlockNeurons / 16;  // fragments per tile of weight rows
constexpr int kTokenPad = 192;         // token rows per tile of long slices (choose_launch)
constexpr int kSliceTokens = 1 << 18;  // tokens per internal slice (size of the 1/r buffer)
constexpr int kMaxSplits = 128;        // token splits per launch (size of the partials)
constexpr int kTileTokens = 1 << 15;   // tokens per bf16 slice (size of the tiled token buffer),
constexpr int kSliceSpare = 8;         // and token tiles more for the last slice of a call

template <typename T>
__device__ inline float load_f32(const T* p, int64_t i);
template <>
__device__ inline float load_f32<uint16_t>(const uint16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
template <>
__device__ inline float load_f32<float>(const float* p, int64_t i) { return p[i]; }

// ------------------------------------------------------------------ weight preparation
// out[tile*128 + c][j] (row stride ld) = W[k][j] * gamma[j], k = tile*64 + c%64,
// W = gate for c < 64 else up; rows of padding neurons are zero.
__global__ void prep_gate_up_kernel(const float* __restrict__ w_gate, const float* __restrict__ w_up,
                                    const float* __restrict__ gamma, int I, int d, int n_tiles,
                                    int64_t ld, float* __restrict__ out) {
  const int64_t total = (int64_t)n_tiles * kCols * d;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(idx % d);
    const int64_t rowi = idx / d;
    const int c = (int)(rowi % kCols);
    const int k = (int)(rowi / kCols) * kBN + (c % kBN);
    float v = 0.0f;
    if (k < I) v = (c < kBN ? w_gate : w_up)[(int64_t)k * d + j] * gamma[j];
    out[rowi * ld + j] = v;
  }
}

// The same for the bf16 path: row R of the fragment-major weights is the gate (R % 64 < 32) or
// up row of neuron 32 (R / 64) + R % 32; columns j < dP, zero past d and for padding neurons.
// One thread per 16-byte piece (d is a multiple of 16), placed by prep_place and counted in 64
// bits.  VEC: 16-byte aligned inputs.
template <int RUN, bool VEC>
__global__ void __launch_bounds__(kPrepThreads)
prep_gate_up_fragments_kernel(const uint16_t* __restrict__ w_gate, const uint16_t* __restrict__ w_up,
                              const uint16_t* __restrict__ gamma, int I, int d, int units_per_row,
                              uint64_t n_pieces, int ks, uint16_t* __restrict__ out) {
  for (uint64_t g = prep_first(blockIdx.x, threadIdx.x); g < n_pieces; g = prep_next(g, gridDim.x)) {
    const PrepPlace at = prep_place<RUN>(g, units_per_row);
    const uint32_t row = at.row;
    const int j = at.col;
    const int k = (int)(row / 64) * 32 + (int)(row % 32);
    u32x4 o = {0u, 0u, 0u, 0u};
    if (k < I && j < d) {
      const uint16_t* p = (row % 64 < 32 ? w_gate : w_up) + (int64_t)k * d + j;
      u32x4 v, m;
      if constexpr (VEC) {
        v = *reinterpret_cast<const u32x4*>(p);
        m = *reinterpret_cast<const u32x4*>(gamma + j);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = (uint32_t)p[2 * e] | ((uint32_t)p[2 * e + 1] << 16);
          m[e] = (uint32_t)gamma[j + 2 * e] | ((uint32_t)gamma[j + 2 * e + 1] << 16);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = __uint_as_float(v[e] << 16) * __uint_as_float(m[e] << 16);
        const float hi = __uint_as_float(v[e] & 0xffff0000u) * __uint_as_float(m[e] & 0xffff0000u);
        o[e] = (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
      }
    }
    *reinterpret_cast<u32x4*>(out + frag_offset<kWeightFrags>(row, j, ks)) = o;
  }
}

// F_h[e, m] = sum_j W_o[j][h dh + e] W'[m][j] into column dP + h dhP + e of weight row m.  32 AF
// columns n = h dh + e x 256 weight rows per block; n is the A side, so that a lane's four
// accumulator elements are four consecutive columns of one row, an 8-byte store.
template <int AF>
__global__ void __launch_bounds__(512, 2)
fold_kernel(uint16_t* wcat, const uint16_t* __restrict__ woT, int N, int dh, int dP, int dhP, int ks,
            int n_a, int n_b) {
  using P = FragPipe<AF, 4>;
  __shared__ __attribute__((aligned(16))) uint16_t s0[P::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s1[P::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s2[P::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s3[P::kSlot];
  int ta, tb;
  frag_work(blockIdx.x, n_a, n_b, 4, ta, tb);
  const int nq = dP / kStage;
  P p(woT + (int64_t)ta * P::kARows * dP, (uint32_t)P::kAFrags * nq * 1024u,
      wcat + (int64_t)tb * P::kBRows * ks * kStage, (uint32_t)P::kBFrags * ks * 1024u);
  p.contract(s0, s1, s2, s3, nq);
#pragma unroll
  for (int i = 0; i < AF; ++i) {
    const int n = ta * P::kARows + 16 * (p.wm * AF + i) + 4 * (p.lane >> 4);
    if (n >= N) continue;  // a multiple of 16: whole fragments
    const int k = dP + n / dh * dhP + n % dh;
    const bool last = n % dh / 16 == dh / 16 - 1;  // the fragment that ends its head
    const int head_end = dP + (n / dh + 1) * dhP;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t m = (uint32_t)tb * P::kBRows + 16 * (p.wn * 4 + j) + (p.lane & 15);
      uint2 o;
      o.x = (uint32_t)f32_to_bf16(p.acc[i][j][0]) | ((uint32_t)f32_to_bf16(p.acc[i][j][1]) << 16);
      o.y = (uint32_t)f32_to_bf16(p.acc[i][j][2]) | ((uint32_t)f32_to_bf16(p.acc[i][j][3]) << 16);
      *reinterpret_cast<uint2*>(wcat + frag_offset<kWeightFrags>(m, k, ks) + k % 8) = o;
      if (last)  // the zero columns up to the next head
        for (int z = k + 16; z < head_end; z += 16)
          *reinterpret_cast<uint2*>(wcat + frag_offset<kWeightFrags>(m, z, ks) + z % 8) = make_uint2(0u, 0u);
    }
  }
}

// nd[k] = sum_j w_down[j][k]^2 in two passes: part[c][k] sums the rows of chunk c in row
// order, then the chunks are added in order.  A thread of the first pass takes 8 adjacent
// columns of its chunk, one 16-byte load per row where the rows allow it (VEC), so each
// load carries 8 columns and a thread's rows are in flight together.
template <typename T, bool VEC>
__global__ void __launch_bounds__(256)
down_norm_part_kernel(const T* __restrict__ w_down, int d, int I, int chunk_rows,
                      float* __restrict__ part) {
  const int k0 = 8 * (blockIdx.x * 256 + threadIdx.x);
  const int c = blockIdx.y;
  if (k0 >= I) return;
  const int j1 = min(d, (c + 1) * chunk_rows);
  float s[8] = {};
  if constexpr (VEC) {  // I % 8 == 0 and 16-byte aligned rows
#pragma unroll 4
    for (int j = c * chunk_rows; j < j1; ++j) {
      const T* row = w_down + (int64_t)j * I + k0;
      if constexpr (sizeof(T) == 2) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(row);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = __uint_as_float(v[e] << 16), hi = __uint_as_float(v[e] & 0xffff0000u);
          s[2 * e] = fmaf(lo, lo, s[2 * e]);
          s[2 * e + 1] = fmaf(hi, hi, s[2 * e + 1]);
        }
      } else {
        const float4 a = *reinterpret_cast<const float4*>(row);
        const float4 b = *reinterpret_cast<const float4*>(row + 4);
        const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = fmaf(v[e], v[e], s[e]);
      }
    }
  } else {
    for (int j = c * chunk_rows; j < j1; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (k0 + e < I) {
          const float v = load_f32(w_down, (int64_t)j * I + k0 + e);
          s[e] = fmaf(v, v, s[e]);
        }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (k0 + e < I) part[(int64_t)c * I + k0 + e] = s[e];
}

__global__ void __launch_bounds__(64)
down_norm_sum_kernel(const float* __restrict__ part, int chunks, int I, int I_pad,
                     float* __restrict__ nd) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= I_pad) return;
  double t = 0.0;
  if (k < I) {
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) t += (double)part[(int64_t)c * I + k];
  }
  nd[k] = (float)t;
}

// ------------------------------------------------------------------ per-token scalars
// rinv[t] = 1 / sqrt(mean_j x[t][j]^2 + eps) of fp32 rows; one wavefront per token.
__global__ void __launch_bounds__(256)
rms_kernel(const float* __restrict__ x, int64_t T, int d, float eps, float* __restrict__ rinv) {
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= T) return;  // whole wavefronts exit together
  const float* row = x + t * d;
  float s = 0.0f;
  for (int j = lane; j < d; j += 64) s = fmaf(row[j], row[j], s);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) rinv[t] = 1.0f / sqrtf(s / (float)d + eps);
}

// ------------------------------------------------------------------ token tiling (bf16)
// Each slice of tokens is rewritten once in fragment-major layout, so that every block that
// reads it (one per neuron group) copies whole 1 KB runs.  The head entries of token t are
// multiplied by p_t = pow2_floor(1/r_t), which is exact in bf16, so the per-head
// contractions come out as p_t (a_h . F) and the damage coefficients c1/p_t, c2/p_t that
// multiply them lie within a factor 2 of silu'(g) u and silu(g) (fp16 range, whatever
// the token scale).  One thread moves one 16-byte piece; RUN consecutive threads read
// 16 RUN contiguous bytes of a row.  Rows past the last token and the columns that round
// d and dh up to whole stages (PAD) are zero.
//
// 1/r has no pass of its own: a block takes 16 tokens and a share of their columns, `per` units of
// 8 RUN, and sums the squares of their x rows first (16 threads per row); with x_next the last
// block of each 16 tokens takes 1/r' instead.  With one share per row x comes from HBM once, its
// second reading from the L2; short slices take more shares, so that the blocks fill the chip, and
// read x again in each.  Against a pass for 1/r and one for the tiles: 5,000 tokens of d = 1,040 and
// 12 heads of 80 12.0 us instead of 8.7 + 4.9 and a launch; 32,768 tokens of d = 1,024, 16 heads of
// 128 81 us instead of 65 + 14 (5.0 TB/s); a call of 1,000 of them, ADD, 42 -> 40 us.
__device__ __forceinline__ float pow2_floor(float v) {  // 2^floor(log2 v), v normal and > 0
  return __uint_as_float(__float_as_uint(v) & 0x7f800000u);
}

__device__ __forceinline__ float pow2_fraction(float v) {  // v / pow2_floor(v), in [1, 2)
  return __uint_as_float((__float_as_uint(v) & 0x007fffffu) | 0x3f800000u);
}

__device__ __forceinline__ uint32_t scale_bf16_pair(uint32_t w, float f) {
  // Both halves times a power of two; exact while the results stay normal.
  const float lo = __uint_as_float(w << 16) * f;
  const float hi = __uint_as_float(w & 0xffff0000u) * f;
  return (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u);
}

struct TokenArgs {
  const uint16_t *x, *attn, *x_next;  // x_next may be NULL
  float eps, eps_next;
  int T, T_pad, d, H, dh, dP, dhP;
  uint16_t* xt;
  float *rinv, *rinv_next;  // [T_pad], 0 past the last token
};

template <int F, int RUN, bool PAD>
__global__ void __launch_bounds__(256)
tile_tokens_kernel(TokenArgs p, int units, int per) {
  __shared__ float rs[16];
  const int t0 = 16 * blockIdx.x, HD = p.H * p.dh, ks = (p.dP + p.H * p.dhP) / kStage;
  const int u0 = blockIdx.y * per, u1 = min(u0 + per, units);
  const bool next = u0 >= units;
  if (next || u0 == 0 || 8 * RUN * u1 > p.dP) {  // the head columns need 1/r
    const int r = threadIdx.x / 16, t = t0 + r;
    float lo = 0.0f, hi = 0.0f;
    if (t < p.T) {
      const uint16_t* row = (next ? p.x_next : p.x) + (int64_t)t * p.d;
#pragma unroll 4
      for (int j = 8 * (threadIdx.x % 16); j < p.d; j += 128) {  // d is a multiple of 16
        const u32x4 v = *reinterpret_cast<const u32x4*>(row + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = __uint_as_float(v[e] << 16), b = __uint_as_float(v[e] & 0xffff0000u);
          lo = fmaf(a, a, lo);
          hi = fmaf(b, b, hi);
        }
      }
    }
    float ss = lo + hi;
#pragma unroll
    for (int off = 8; off > 0; off /= 2) ss += __shfl_xor(ss, off, 64);
    const float v = t < p.T ? 1.0f / sqrtf(ss / (float)p.d + (next ? p.eps_next : p.eps)) : 0.0f;
    if (threadIdx.x % 16 == 0) {
      rs[r] = v;
      if (next)
        p.rinv_next[t] = v;
      else if (u0 == 0)
        p.rinv[t] = v;
    }
    if (next) return;
    __syncthreads();
  }
#pragma unroll 4
  for (int i = threadIdx.x; i < (u1 - u0) * 16 * RUN; i += 256) {
    const int w = i % (16 * RUN), t = t0 + w / RUN;
    const int k = 8 * ((u0 + i / (16 * RUN)) * RUN + w % RUN);
    u32x4 v = {0u, 0u, 0u, 0u};
    if (t < p.T) {
      if (k < p.dP) {
        if (!PAD || k < p.d) v = *reinterpret_cast<const u32x4*>(p.x + (int64_t)t * p.d + k);
      } else {
        int col = k - p.dP;
        bool real = true;
        if constexpr (PAD) {
          const int h = col / p.dhP, e = col % p.dhP;
          real = e < p.dh;
          col = h * p.dh + e;
        }
        if (real) {
          v = *reinterpret_cast<const u32x4*>(p.attn + (int64_t)t * HD + col);
          const float f = pow2_floor(rs[w / RUN]);
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = scale_bf16_pair(v[j], f);
        }
      }
    }
    *reinterpret_cast<u32x4*>(p.xt + frag_offset<F>(t, k, ks)) = v;
  }
}

// ------------------------------------------------------------------ fused affinity (bf16)
struct AffinityArgs {
  const uint16_t* xt;     // token rows, fragment-major, padded to whole tiles
  const uint16_t* wcat;   // weight rows, fragment-major
  const float* rinv;      // [padded T], 0 past the last token
  const float* rinv_next; // the same for 1/r' of the residual entering the next layer, or NULL
  const float* nd;        // [I_pad]
  float* partial;         // [splits][G+1][I_pad]: G up rows, then the down statistic
  int ks, nq1, nqh;       // stages per row, of the operating point, per head
  int G, hpg, mtiles, splits, hsplits, I_pad;
  int first;              // splits whose blocks come before those of the others
};

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// The damage coefficients c1/p_t and c2/p_t of an element, rounded to fp16 (11 significant
// bits; the scaled coefficients lie within a factor 2 of silu'(g) u and silu(g)) and packed.
// a and b are first rounded to fp32 (the asm hides the products that made them): otherwise
// the compiler may fuse some products with the conversion (one rounding) and not others
// (two), and a token's coefficients would depend on its row slot.
__device__ __forceinline__ uint32_t pack_coefs(float a, float b) {
  asm("" : "+v"(a), "+v"(b));
  half2_t c;
  c.x = (_Float16)a;
  c.y = (_Float16)b;
  return __builtin_bit_cast(uint32_t, c);
}

// Delta = c1 G + c2 U as two mixed-precision fmas that read the fp16 halves in place.  The
// packed word goes through a scalar before the cast.
__device__ __forceinline__ float damage(uint32_t w, float g, float u) {
  const half2_t c = __builtin_bit_cast(half2_t, w);
  return __builtin_fmaf((float)c.y, u, __builtin_fmaf((float)c.x, g, 0.0f));
}

// A block takes 128 neurons, a token split and a range of KV groups; a tile is 32 AF tokens.
// For each tile it runs the operating point's stages (not for the ADD score, which has no
// use for it), then those of its heads.  A wavefront owns 16 AF tokens x 32 neurons, as
// AF x 4 accumulators (two fragments of gate columns, then the same neurons' up columns), so
// c1/c2 and both damage terms of a (token, neuron) pair sit in the same lane.
//
// The stages of all tiles run through the pipe of frag_gemm.h without a break.  Its four
// slots are compile-time names, and so is each stage's place in its head (NQH stages): the
// operating point takes a multiple of four stages (dP is one of 128 columns), and after
// the heads of a tile empty stages (barrier and copy, no products) fill up the last four.  A
// head's epilogue, three vector instructions per element, runs beside the products of the
// half stage that follows: the rows of half 0 during half 1 of the head's last stage, the
// rows of half 1 during half 0 of the next head's first.  The products of a head's first
// stage start from zero.
//
// Bound by the matrix cores and by the waits between their stages: on the three layer shapes
// measured the MFMAs are busy 50 to 62% of the SIMD cycles, at the 1.7 to 2.1 GHz that the clock holds
// under this load, and a quarter to a third of the wave cycles stand at a wait.  (How much of the
// clock power takes was not separated; MFMAs alone on random operands reach 80 to 82% of the
// nominal rate.)  Launches of 32,768 Qwen3-0.6B-shaped and 16,384 8B-class and Danube3-500M-shaped
// tokens: 1,040 to 1,140, 6,680 to 6,840 and 780 to 880 us, as the clock holds, against 1,210, 7,180 and
// 860 us in the better runs of 256 tokens x 64 neurons per block with the token fragments loaded
// straight into registers, whose head epilogues ran with no products of their own wavefront
// beside them.
template <int AF, bool ADD, bool DOWN, int NQH>
struct AffinityBlock {
  using Pipe = FragPipe<AF, 4>;
  static constexpr int kElems = ADD ? AF * 4 : AF * 8;
  // vector instructions of an epilogue beside each product of a half
  static constexpr int kEpi0 = (3 * Pipe::kH1 * 8 + Pipe::kH0 * 4 - 1) / (Pipe::kH0 * 4);
  static constexpr int kEpi1 = (3 * Pipe::kH0 * 8 + Pipe::kH1 * 4 - 1) / (Pipe::kH1 * 4);

  Pipe f;
  uint32_t cf[kElems];  // FO: packed (c1, c2) per [row fragment][neuron fragment][element]; ADD: row weights
  float colsum[2];
  float* red;           // this wavefront's banks
  uint16_t *s0, *s1, *s2, *s3;
  int hpg, done, group;  // query heads per group; heads done of the current group
  int reps;              // NQH = 0: stages per head over four
  // the next stage to copy: position in the tile's sequence, and the tile's offset
  int pos, tiles_left;
  uint32_t tile_off, tile_bytes;
  int n1, n2, n2p, base2;  // stages of the operating point and of the heads, with fill; first head stage

  // The slot of stage STEP, counted from the tile's start.
  template <int STEP>
  __device__ __forceinline__ uint16_t* stage() const {
    return STEP % 4 == 0 ? s0 : STEP % 4 == 1 ? s1 : STEP % 4 == 2 ? s2 : s3;
  }

  // Byte offsets of the next stage to copy; past the last tile it is fetched again.  All of it
  // is the same for the whole wavefront, which the compiler does not see everywhere.
  __device__ __forceinline__ typename Pipe::Source next_source() {
    const int src = __builtin_amdgcn_readfirstlane(pos < n1 ? pos : base2 + min(pos - n1, n2 - 1));
    const uint32_t at = (uint32_t)src * 1024u;
    const typename Pipe::Source o = {tile_off + at * Pipe::kAFrags, at * Pipe::kBFrags};
    const bool wrap = pos + 1 == n1 + n2p, more = wrap && tiles_left > 1;
    pos = __builtin_amdgcn_readfirstlane(wrap ? 0 : pos + 1);
    tiles_left -= more ? 1 : 0;
    tile_off = __builtin_amdgcn_readfirstlane(tile_off + (more ? tile_bytes : 0u));
    return o;
  }

  template <int FROM, int TO>
  __device__ __forceinline__ void head_epilogue() {
#pragma unroll
    for (int i = FROM; i < TO; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = f.acc[i][j][e], u = f.acc[i][2 + j][e];
          if constexpr (ADD) {  // (1/r)^2 (G^2 + U^2)
            colsum[j] = fmaf(__uint_as_float(cf[i * 4 + e]), fmaf(u, u, g * g), colsum[j]);
          } else {
            const float dl = damage(cf[(i * 2 + j) * 4 + e], g, u);
            colsum[j] = fmaf(dl, dl, colsum[j]);
          }
        }
  }

  // Column sums over the wavefront's rows into a bank: the halves of c0 meet in lanes 0 to 31 and
  // those of c1 in lanes 32 to 63, then the 16-lane rows of each.
  __device__ __forceinline__ void bank(int row, float c0, float c1) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(c0), __float_as_uint(c1), false, false);
    float c = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    c += __uint_as_float(__builtin_amdgcn_ds_swizzle(__float_as_uint(c), 0x401f));  // lane ^ 16
    if ((f.lane & 16) == 0) red[row * 32 + (f.lane & 15) + (f.lane >> 5) * 16] += c;
  }

  __device__ __forceinline__ void head_done() {
    if (++done == hpg) {  // the last query head of its KV group
      bank(group, colsum[0], colsum[1]);
      colsum[0] = colsum[1] = 0.0f;
      done = 0;
      ++group;
    }
  }

  template <int SLOT>
  __device__ __forceinline__ void op_stage() {
    const typename Pipe::Source later = next_source();
    f.template half0<false>(stage<SLOT>());
    f.template half1<false>(stage<SLOT>(), stage<SLOT + 1>(), later);
  }

  template <int SLOT>
  __device__ __forceinline__ void empty_stage() {
    f.skip(stage<SLOT>(), stage<SLOT + 1>(), next_source());
  }

  // Half 1 of stage I of a head, at slot SLOT, and the stages after it.
  template <int SLOT, int I = 0>
  __device__ __forceinline__ void head_rest(typename Pipe::Source later) {
    if constexpr (I == NQH - 1) {
      f.template half1<I == 0, kEpi1>(stage<SLOT>(), stage<SLOT + 1>(), later,
                                      [&]() __attribute__((always_inline)) { head_epilogue<0, Pipe::kH0>(); });
    } else {
      f.template half1<I == 0>(stage<SLOT>(), stage<SLOT + 1>(), later);
      later = next_source();
      f.template half0<false>(stage<SLOT + 1>());
      head_rest<(SLOT + 1) % 4, I + 1>(later);
    }
  }

  // The same for a head of `reps` >= 2 times four stages from slot 0 (NQH = 0).
  __device__ __forceinline__ void long_head_rest(typename Pipe::Source later) {
    f.template half1<true>(s0, s1, later);
    op_stage<1>();
    op_stage<2>();
    op_stage<3>();
    for (int r = 2; r < reps; ++r) {
      op_stage<0>();
      op_stage<1>();
      op_stage<2>();
      op_stage<3>();
    }
    op_stage<0>();
    op_stage<1>();
    op_stage<2>();
    later = next_source();
    f.template half0<false>(s3);
    f.template half1<false, kEpi1>(s3, s0, later, [&]() __attribute__((always_inline)) { head_epilogue<0, Pipe::kH0>(); });
  }

  // A head from half 1 of its first stage to half 0 of the next head's.  `later`: the source
  // that the head's first stage, then the next head's, sends on its way.
  template <int SLOT>
  __device__ __forceinline__ void next_head(typename Pipe::Source& later) {
    if constexpr (NQH == 0)
      long_head_rest(later);
    else
      head_rest<SLOT>(later);
    later = next_source();
    f.template half0<true, kEpi0>(stage<SLOT + NQH>(), [&]() __attribute__((always_inline)) { head_epilogue<Pipe::kH0, AF>(); });
    head_done();
  }

  template <int SLOT>
  __device__ __forceinline__ void last_head(typename Pipe::Source later) {
    if constexpr (NQH == 0)
      long_head_rest(later);
    else
      head_rest<SLOT>(later);
    head_epilogue<Pipe::kH0, AF>();
    head_done();
    constexpr int kNext = (SLOT + NQH) % 4;
    if constexpr (kNext == 1) empty_stage<1>();
    if constexpr (kNext == 1 || kNext == 2) empty_stage<2>();
    if constexpr (kNext != 0) empty_stage<3>();
  }

  // The coefficients change, as far as the compiler can tell, with the head: it would move the
  // conversion of all of them to fp32 out of the loop over heads, and spill.
  __device__ __forceinline__ void hold_coefs(int n) {
    if constexpr (!ADD) {
#pragma unroll
      for (int i = 0; i < kElems; ++i) asm("" : "+v"(cf[i]) : "s"(n));
    }
  }

  // Heads until the next one starts at slot 0 again, not the tile's last.
  static constexpr int kPerRound = NQH % 4 == 0 ? 1 : NQH % 4 == 2 ? 2 : 4;
  template <int SLOT = 0>
  __device__ __forceinline__ void round(int n, typename Pipe::Source& later) {
    hold_coefs(n);
    next_head<SLOT>(later);
    if constexpr ((SLOT + NQH) % 4 != 0) round<(SLOT + NQH) % 4>(n - 1, later);
  }

  // The tile's last heads, kPerRound of them at most, and empty stages back to slot 0.
  template <int SLOT = 0, int LEFT = kPerRound>
  __device__ __forceinline__ void last_round(int n, typename Pipe::Source later) {
    hold_coefs(n);
    if constexpr (LEFT > 1) {
      if (n > 1) {
        next_head<SLOT>(later);
        last_round<(SLOT + NQH) % 4, LEFT - 1>(n - 1, later);
        return;
      }
    }
    last_head<SLOT>(later);
  }

  __device__ __forceinline__ void heads(int n) {
    done = group = 0;
    typename Pipe::Source later = next_source();
    f.template half0<true>(s0);
    for (; n > kPerRound; n -= kPerRound) round(n, later);
    last_round(n, later);
  }

  // Operating point: g, u -> c1 = silu'(g) u / r, c2 = silu(g) / r, stored divided by p_t (the
  // head entries were multiplied by it), and the down statistic (silu(g) u / r')^2 summed.
  __device__ __forceinline__ void operating_point(const float* rv, const float* rv2, int down_row) {
    float ds[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < AF; ++i) {
      const int row = 16 * (f.wm * AF + i) + 4 * (f.lane >> 4);
      const float4 r4 = *reinterpret_cast<const float4*>(rv + row);
      float4 n4 = {};
      if constexpr (DOWN) n4 = *reinterpret_cast<const float4*>(rv2 + row);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float ri = r4[e];
        const float rs = ri > 0.0f ? pow2_fraction(ri) : 0.0f;  // ri / p_t
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float g = f.acc[i][j][e] * ri, u = f.acc[i][2 + j][e] * ri;
          const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-g));
          const float sl = g * sg;  // silu(g); silu'(g) = sg + silu(g) (1 - sg)
          cf[(i * 2 + j) * 4 + e] = pack_coefs((fmaf(-sl, sg, sl) + sg) * u * rs, sl * rs);
          if constexpr (DOWN) {
            const float a = sl * u * n4[e];
            ds[j] = fmaf(a, a, ds[j]);
          }
        }
      }
    }
    if constexpr (DOWN) bank(down_row, ds[0], ds[1]);
  }
};

template <int AF, bool ADD, bool DOWN, int NQH>
__global__ void __launch_bounds__(512, 2)  // two waves per SIMD
affinity_bf16_kernel(AffinityArgs p) {
  using Block = AffinityBlock<AF, ADD, DOWN, NQH>;
  using Pipe = typename Block::Pipe;
  constexpr int kRows = Pipe::kARows;
  constexpr int kRv = (kRows + 63) / 64 * 64;
  // Each slot is an array of its own, so that the compiler can tell the reads of one from the
  // copy into another (one array indexed by the stage makes it wait for the copies).
  __shared__ __attribute__((aligned(16))) uint16_t s0[Pipe::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s1[Pipe::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s2[Pipe::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s3[Pipe::kSlot];
  __shared__ __attribute__((aligned(16))) float rv[ADD ? 4 : kRv];    // 1/r of the tile's rows
  __shared__ __attribute__((aligned(16))) float rv2[DOWN ? kRv : 4];  // 1/r'
  extern __shared__ float banks[];  // [8 wavefronts][rows][32]: the block's KV groups, then the down statistic

  int split, item;
  const int groups = p.I_pad / kBlockNeurons;
  const int items = groups * p.hsplits, first = p.first * items;
  if ((int)blockIdx.x < first) {
    frag_work(blockIdx.x, p.first, items, 4, split, item);
  } else {
    frag_work(blockIdx.x - first, p.splits - p.first, items, 4, split, item);
    split += p.first;
  }
  const int tg = item / p.hsplits, hs = item % p.hsplits;
  const int g0 = hs * p.G / p.hsplits, g1 = (hs + 1) * p.G / p.hsplits;  // KV groups of this block
  const int rows = g1 - g0 + 1;
  for (int i = threadIdx.x; i < 8 * rows * 32; i += 512) banks[i] = 0.0f;

  const int longer = p.mtiles % p.splits;  // splits 0 .. longer - 1 have a tile more
  const int mt_begin = split * (p.mtiles / p.splits) + min(split, longer);
  const int tiles = p.mtiles / p.splits + (split < longer ? 1 : 0);  // >= 1: splits <= mtiles
  {
    const uint32_t tile_bytes = (uint32_t)Pipe::kAFrags * p.ks * 1024u;
    static_assert(Pipe::kBFrags == kWeightFrags, "tiles as laid out");
    Block b{Pipe(p.xt + (int64_t)mt_begin * kRows * p.ks * kStage, (uint32_t)tiles * tile_bytes,
                 p.wcat + (int64_t)tg * Pipe::kBRows * p.ks * kStage, (uint32_t)Pipe::kBFrags * p.ks * 1024u)};
    const int heads = (g1 - g0) * p.hpg;
    b.red = banks + b.f.wave * rows * 32;
    b.s0 = s0;
    b.s1 = s1;
    b.s2 = s2;
    b.s3 = s3;
    b.hpg = p.hpg;
    b.n1 = ADD ? 0 : p.nq1;
    b.reps = p.nqh / 4;
    b.n2 = heads * p.nqh;
    b.n2p = (b.n2 + 3) / 4 * 4;
    b.base2 = p.nq1 + g0 * p.hpg * p.nqh;
    b.pos = 0;
    b.tiles_left = tiles;
    b.tile_off = 0;
    b.tile_bytes = tile_bytes;
    b.colsum[0] = b.colsum[1] = 0.0f;
    b.f.copy(s0, b.next_source());
    b.f.copy(s1, b.next_source());
    b.f.copy(s2, b.next_source());
    b.f.copy(s3, b.next_source());
    b.f.begin(s0);
    for (int mt = 0; mt < tiles; ++mt) {
      const int m0 = (mt_begin + mt) * kRows;
      b.f.zero();
      if constexpr (ADD) {
#pragma unroll
        for (int i = 0; i < AF; ++i) {
          const float4 r4 = *reinterpret_cast<const float4*>(p.rinv + m0 + 16 * (b.f.wm * AF + i) + 4 * (b.f.lane >> 4));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float rs = r4[e] > 0.0f ? pow2_fraction(r4[e]) : 0.0f;
            b.cf[i * 4 + e] = __float_as_uint(rs * rs);
          }
        }
      } else {
        // The previous tile's operating point, the last reader of rv, is at least a head ago.
        if (b.f.wave < kRv / 64) {
          const int at = 64 * b.f.wave;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              frag_rsrc(p.rinv + m0, 4u * kRows), (__attribute__((address_space(3))) void*)(rv + at), 4,
              4 * b.f.lane, 4 * at, 0, 0);
          if constexpr (DOWN)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                frag_rsrc(p.rinv_next + m0, 4u * kRows), (__attribute__((address_space(3))) void*)(rv2 + at), 4,
                4 * b.f.lane, 4 * at, 0, 0);
        }
        for (int s = 0; s < b.n1; s += 4) {
          b.template op_stage<0>();
          b.template op_stage<1>();
          b.template op_stage<2>();
          b.template op_stage<3>();
        }
        b.operating_point(rv, rv2, rows - 1);
      }
      b.heads(heads);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): no copy may land after the LDS is given back
  }
  __syncthreads();

  // Sum the two row waves in a fixed order and scale by ||w^d_k||^2.  The down statistic is
  // the same in every block of a tile: the first range writes it.
  for (int i = threadIdx.x; i < rows * kBlockNeurons; i += 512) {
    const int row = i / kBlockNeurons, nl = i % kBlockNeurons;
    const bool down = row == rows - 1;
    if (down && (!DOWN || hs != 0)) continue;
    const int w = 2 * (nl / 32), k = nl % 32;
    const float sum = banks[(w * rows + row) * 32 + k] + banks[((w + 1) * rows + row) * 32 + k];
    const int n = tg * kBlockNeurons + nl;
    p.partial[((int64_t)split * (p.G + 1) + (down ? p.G : g0 + row)) * p.I_pad + n] =
        down || ADD ? sum : sum * p.nd[n];
  }
}

}  // namespace

// Compute units of the current device, cached per device (atomics: calls on different
// layers may run on several host threads at once).
int device_cus() {
  static std::atomic<int> cus[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

namespace {

// Token rows rounded up to whole tiles.
int64_t pad_tokens(int64_t T, int tile = kTokenPad) { return (T + tile - 1) / tile * tile; }

template <int F>
void launch_tile_tokens(const TokenArgs& p, hipStream_t s) {
  const int Kt = p.dP + p.H * p.dhP, rows = p.T_pad / 16;
  const bool pad = p.dP != p.d || p.dhP != p.dh, wide = Kt % 64 == 0 && !pad;
  // Shares of a row's columns: two blocks per CU, of four units at least.
  const int units = Kt / (wide ? 64 : 32), want = (2 * device_cus() + rows - 1) / rows;
  const int per = std::max((units + want - 1) / want, std::min(units, 4));
  const dim3 grid(rows, (units + per - 1) / per + (p.x_next ? 1 : 0));
  if (wide)
    tile_tokens_kernel<F, 8, false><<<grid, 256, 0, s>>>(p, units, per);
  else if (!pad)
    tile_tokens_kernel<F, 4, false><<<grid, 256, 0, s>>>(p, units, per);
  else
    tile_tokens_kernel<F, 4, true><<<grid, 256, 0, s>>>(p, units, per);
}

void launch_prep_gate_up(const uint16_t* w_gate, const uint16_t* w_up, const uint16_t* gamma, int I, int d,
                         int dP, int I_pad, int ks, uint16_t* out, hipStream_t s) {
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
  const uint64_t n = prep_pieces(I_pad, dP);
  const unsigned grid = prep_blocks(n);
  if (al16(w_gate) && al16(w_up) && al16(gamma))  // dP is a multiple of 128
    prep_gate_up_fragments_kernel<8, true><<<grid, kPrepThreads, 0, s>>>(w_gate, w_up, gamma, I, d, dP / 64, n, ks, out);
  else
    prep_gate_up_fragments_kernel<4, false><<<grid, kPrepThreads, 0, s>>>(w_gate, w_up, gamma, I, d, dP / 32, n, ks, out);
}

// W_o^T in fragments and the fold, in tiles of 256, 128 or 64 columns.  A block runs dP / 32 stages
// whatever its height, one block per CU at a time; a stage takes about 32 : 18 : 12, so the height
// with the fewest rounds of blocks, weighed so, is taken.  Loading a layer of d = 256, I = 1,024, 8
// heads of 64: 21.9 us in tiles of 64 columns and 24.5 in tiles of 256 (16 blocks); of d = 1,040, I =
// 2,810, 12 heads of 80: 66.9, 61.8 (128 columns) and 72.1; of d = 2,048, I = 8,192, 32 heads of 64:
// 193, 152 and 142.
template <int AF>
void launch_fold_tiles(const uint16_t* w_o, int N, int d, int dh, int dP, int dhP, int I_pad, int ks, uint16_t* woT,
                       uint16_t* wcat, hipStream_t s) {
  const int n_a = (N + 32 * AF - 1) / (32 * AF), n_b = I_pad / kBlockNeurons, nq = dP / kStage;
  const dim3 grid((N + 255) / 256 * 4, (nq + 1) / 2);
  if (((uintptr_t)w_o & 15u) == 0)
    transpose_fragments_kernel<2 * AF, false, true><<<grid, 256, 0, s>>>(w_o, nullptr, d, N, nq, woT);
  else
    transpose_fragments_kernel<2 * AF, false, false><<<grid, 256, 0, s>>>(w_o, nullptr, d, N, nq, woT);
  fold_kernel<AF><<<n_a * n_b, 512, 0, s>>>(wcat, woT, N, dh, dP, dhP, ks, n_a, n_b);
}

void launch_fold(const uint16_t* w_o, int N, int d, int dh, int dP, int dhP, int I_pad, int ks, uint16_t* woT,
                 uint16_t* wcat, hipStream_t s) {
  const int64_t cus = device_cus(), n_b = I_pad / kBlockNeurons;
  auto cost = [&](int columns, int64_t stage_cost) {
    return ((N + columns - 1) / columns * n_b + cus - 1) / cus * stage_cost;
  };
  const int64_t high = cost(256, 32), mid = cost(128, 18), low = cost(64, 12);
  (high <= mid && high <= low ? launch_fold_tiles<8> : mid <= low ? launch_fold_tiles<4> : launch_fold_tiles<2>)(
      w_o, N, d, dh, dP, dhP, I_pad, ks, woT, wcat, s);
}

struct LaunchShape {
  int tile = kTokenPad;  // token rows per tile: 192, 128 or 64
  int mtiles = 1, splits = 1, hsplits = 1;
  int64_t cost = -1;
};

// Tile height, token splits and ranges of KV groups of a launch.  A CU runs one block at a time,
// and blocks go to CUs as these become free.  The splits' lengths differ by one tile at most: with
// R blocks per CU, rounded up, of f tiles and as many CUs' worth of them of one more, the launch
// lasts about R f + (longer blocks / CUs, rounded up) tiles and R starts and ends of a block,
// about 12 stages each.  (4,080 tiles
// of a Qwen3-0.6B-shaped slice: 16 tile times in 32 splits, 1,106 us; 128 splits of one or two
// tiles, 22 by this measure, took 1,384.)  Splitting the groups repeats the
// operating point in every range, so it is weighed only where the tiles alone do not give
// each CU two.
//
// A stage of 192, 128 and 64 tokens counts 24 : 19 : 15, about what it takes where a launch has one
// tile per block (one tile of 64 tokens of a Qwen3-0.6B-shaped layer: launches of 30, 25 and 20
// us).  With every CU busy for many tiles the low ones cost less than that, 128 tokens 1.05 to
// 1.09 times as much as 192 per token and 64 1.4 to 1.6 (19 : 24 is 1.19, 15 : 24 1.88), but still more
// than 192, so that the order is the same.
//
// In heads of three, five and six stages a tile of 192 tokens spills registers (FO 129 to 232, ADD
// 18 to 102), in part per tile: most where the block's heads do not end a round of slots, whose
// last heads then leave by a branch.  One head of 192, d = 128, I = 4,096, 30,000 tokens: 490 us in tiles
// of 192 and 203 of 128; two heads of 96 369 and 218, four 354 and 297; 16 of 96 in d = 1,024 537 and
// 524 (16,384 tokens), of 192 742 and 786, and with ADD 318 and 330, 558 and 594.
//
// The costs were fitted to 397 launches of 64 to 65,536 tokens, d = 16 to 4,096, 1 to 65 heads of 16 to
// 256, each timed in tiles of all three heights: the height chosen is within 5% of the fastest in
// all of them and within 2% in 386.  (One cost per number of stages, without the part per tile,
// was up to 2.4 times slower.)  A tie goes to 128.
LaunchShape choose_launch(const AffinityArgs& p, bool add, int T, int64_t max_rows) {
  const int64_t cus = device_cus(), groups = p.I_pad / kBlockNeurons;
  const int n1 = add ? 0 : p.nq1 + 8;  // the operating point's epilogue: about 8 stages
  const bool spills = p.nqh == 3 || p.nqh == 5 || p.nqh == 6;
  const int per_round = p.nqh == 6 ? 2 : 4;  // heads of a round of slots, where it matters
  LaunchShape best;
  auto weigh = [&](int tile, int stage_cost, int mtiles, int s, int hs) {
    const int64_t rounds = (groups * s * hs + cus - 1) / cus;
    const int64_t tiles = rounds * (mtiles / s) + (groups * hs * (mtiles % s) + cus - 1) / cus;
    const int most = (p.G + hs - 1) / hs * p.hpg, least = p.G / hs * p.hpg;  // heads of a block
    int64_t stages = n1 + (most * p.nqh + 3) / 4 * 4;
    if (spills && tile == 192)
      stages += most % per_round || least % per_round ? (add ? 10 : 16) : p.nqh == 3 && !add ? 8 : 0;
    const int64_t cost = (tiles * stages + rounds * 12) * stage_cost;
    if (best.cost < 0 || cost < best.cost) best = {tile, mtiles, s, hs, cost};
  };
  auto weigh_tile = [&](int tile, int stage_cost) {
    if (pad_tokens(T, tile) > max_rows) return;
    const int mtiles = (T + tile - 1) / tile, cap = std::min(mtiles, kMaxSplits);
    for (int s = 1; s <= cap; ++s) weigh(tile, stage_cost, mtiles, s, 1);
    if (groups * mtiles < 2 * cus)
      for (int hs = 2; hs <= p.G; ++hs) weigh(tile, stage_cost, mtiles, cap, hs);
  };
  weigh_tile(128, 19);
  weigh_tile(192, spills && !add ? 25 : 24);
  weigh_tile(64, 15);
  return best;
}

template <int AF, bool ADD, bool DOWN>
void launch_affinity_tiles(AffinityArgs p, const LaunchShape& l, hipStream_t s) {
  p.mtiles = l.mtiles;
  p.splits = l.splits;
  p.hsplits = l.hsplits;
  // Where a CU gets several blocks the longer ones come first, and the others fill what these
  // leave of the CUs: 4,000 tokens of an 8B-class layer 1,871 -> 1,683 us, of one of d = 2,048, I =
  // 6,144 449 -> 343 us.  Otherwise one order for all, which shares more tiles in each L2.
  p.first = (int64_t)p.I_pad / kBlockNeurons * l.splits * l.hsplits > device_cus() ? l.mtiles % l.splits : 0;
  const int rows = (p.G + l.hsplits - 1) / l.hsplits + 1;
  const size_t shm = sizeof(float) * 8 * rows * 32;
  const unsigned grid = (unsigned)(p.I_pad / kBlockNeurons * l.splits * l.hsplits);
  switch (p.nqh) {
#define DTP_AFFINITY(N) \
  case N: affinity_bf16_kernel<AF, ADD, DOWN, N><<<grid, 512, shm, s>>>(p); break;
    DTP_AFFINITY(1)
    DTP_AFFINITY(2)
    DTP_AFFINITY(3)
    DTP_AFFINITY(4)
    DTP_AFFINITY(5)
    DTP_AFFINITY(6)
    default: affinity_bf16_kernel<AF, ADD, DOWN, 0><<<grid, 512, shm, s>>>(p);  // a multiple of four
#undef DTP_AFFINITY
  }
}

template <int AF>
void launch_affinity(const AffinityArgs& p, const LaunchShape& l, bool add, hipStream_t s) {
  if (add)
    launch_affinity_tiles<AF, true, false>(p, l, s);
  else if (p.rinv_next)
    launch_affinity_tiles<AF, false, true>(p, l, s);
  else
    launch_affinity_tiles<AF, false, false>(p, l, s);
}

// A[g][k] += sum_s partial[s][g][k] for g < G (row g = blockIdx.y), and s_down[k] +=
// sum_s partial[s][G][k] when s_down is given, in fp64 and in a fixed order: eight split
// groups (splits r, r + 8, r + 16, ...) summed in parallel, then the groups in order.
constexpr int kReduceGroups = 8;
__global__ void __launch_bounds__(256)
reduce_splits_kernel(const float* __restrict__ partial, int splits, int G, int I, int I_pad,
                     float* __restrict__ A, float* __restrict__ s_down) {
  __shared__ double part[kReduceGroups][32];
  const int kk = threadIdx.x & 31, r = threadIdx.x >> 5;
  const int g = blockIdx.y;
  const int k = blockIdx.x * 32 + kk;
  double s = 0.0;
  if (k < I)
    for (int sp = r; sp < splits; sp += kReduceGroups)
      s += (double)partial[((int64_t)sp * (G + 1) + g) * I_pad + k];
  part[r][kk] = s;
  __syncthreads();
  if (r == 0 && k < I) {
    float* out = g < G ? A + (int64_t)g * I + k : s_down + k;
    double t = (double)*out;
    for (int q = 0; q < kReduceGroups; ++q) t += part[q][kk];
    *out = (float)t;
  }
}

inline unsigned grid_for(int64_t n, int threads) {
  const int64_t b = (n + threads - 1) / threads;
  return (unsigned)std::min<int64_t>(b, 1 << 20);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace
}  // namespace dtp

using namespace dtp;

struct dtp_layer_s {
  dtp_layer_desc desc;
  int device = 0;
  int n_tiles = 0, I_pad = 0, Kt = 0;
  int dP = 0, dhP = 0;     // bf16 path: d and dh rounded up to whole stages
  bool has_weights = false;
  void* w = nullptr;       // folded rows [2 I_pad][Kt]; bf16 fragment-major, fp32 row-major
  void* woT = nullptr;     // bf16: W_o^T, fragment-major [H*dh rounded up to 256][dP], operand of the fold
  float* nd = nullptr;       // [I_pad]
  float* rinv = nullptr;     // [kSliceTokens]
  float* rinv_next = nullptr;  // [kSliceTokens], 1/r' for the down statistic
  float* partial = nullptr;  // [kMaxSplits][G][I_pad]
  uint16_t* xt = nullptr;    // bf16 path: one slice of token rows, fragment-major
  int64_t tile_slice = 0;    // tokens per bf16 slice
  bool profiling = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
};

namespace {

void layer_free(dtp_layer L) {
  void* bufs[] = {L->w, L->woT, L->nd, L->rinv, L->rinv_next, L->partial, L->xt};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  for (auto& e : L->events) {
    (void)hipEventDestroy(e.first);
    (void)hipEventDestroy(e.second);
  }
  delete L;
}

// n_d into L->nd, with the layer's split partials as the scratch of the row chunks (the
// affinity launches that use them are ordered after this on the stream).
template <typename T>
dtp_status down_norms(const T* w_down, dtp_layer L, hipStream_t s) {
  const dtp_layer_desc& d = L->desc;
  const int64_t cap = (int64_t)kMaxSplits * (d.n_kv_groups + 1) * L->I_pad;  // floats
  int chunk_rows = 32;
  while ((int64_t)((d.d_model + chunk_rows - 1) / chunk_rows) * d.n_neurons > cap) chunk_rows *= 2;
  const int chunks = (d.d_model + chunk_rows - 1) / chunk_rows;
  const dim3 grid((d.n_neurons + 8 * 256 - 1) / (8 * 256), chunks);
  if (d.n_neurons % 8 == 0 && aligned16(w_down))
    down_norm_part_kernel<T, true><<<grid, 256, 0, s>>>(w_down, d.d_model, d.n_neurons, chunk_rows,
                                                        L->partial);
  else
    down_norm_part_kernel<T, false><<<grid, 256, 0, s>>>(w_down, d.d_model, d.n_neurons, chunk_rows,
                                                         L->partial);
  DTP_HIP(hipGetLastError());
  down_norm_sum_kernel<<<(L->I_pad + 63) / 64, 64, 0, s>>>(L->partial, chunks, d.n_neurons, L->I_pad,
                                                           L->nd);
  DTP_HIP(hipGetLastError());
  return DTP_OK;
}

dtp_status check_device(dtp_layer L) {
  int dev = -1;
  DTP_HIP(hipGetDevice(&dev));
  DTP_CHECK(dev == L->device, DTP_ERR_INVALID_ARG,
            "layer was created on device %d but device %d is current", L->device, dev);
  return DTP_OK;
}

}  // namespace

namespace dtp {
namespace {

// Tokens of a call's bf16 slices but the last, which takes the rest: even shares, cut to where
// the slice's tiles fill whole rounds of the CUs if what that leaves to the last still fits.
int64_t choose_slice(const dtp_layer_s* L, int64_t n_tokens) {
  if (n_tokens <= L->tile_slice) return n_tokens;
  const int64_t even_most = L->tile_slice - kSliceSpare * kTokenPad;
  const int64_t n = (n_tokens + even_most - 1) / even_most;
  const int64_t share = pad_tokens((n_tokens + n - 1) / n) / kTokenPad;  // tiles
  const int64_t groups = L->I_pad / kBlockNeurons, cus = device_cus();
  const int64_t whole = share * groups / cus * cus / groups;
  const int64_t rest = n_tokens - (n - 1) * whole * kTokenPad;
  return (whole > 0 && rest <= L->tile_slice ? whole : share) * kTokenPad;
}

// Shared body of the two accumulate entry points; x_next / s_down are NULL for the up
// affinity alone.
dtp_status accumulate(dtp_layer L, const void* x, const void* attn, const void* x_next,
                      float eps_next, int64_t n_tokens, float* A, float* s_down, bool add,
                      void* stream) {
  DTP_CHECK(L != nullptr, DTP_ERR_INVALID_ARG, "layer is NULL");
  DTP_CHECK(n_tokens >= 0, DTP_ERR_INVALID_ARG, "n_tokens=%lld is negative", (long long)n_tokens);
  if (n_tokens == 0) return DTP_OK;
  DTP_CHECK(x && attn && A, DTP_ERR_INVALID_ARG, "x, attn or A is NULL");
  DTP_CHECK(aligned16(x) && aligned16(attn), DTP_ERR_INVALID_ARG,
            "x and attn must be 16-byte aligned");
  DTP_CHECK((x_next == nullptr) == (s_down == nullptr), DTP_ERR_INVALID_ARG,
            "x_next and s_down must be given together");
  DTP_CHECK(x_next == nullptr || aligned16(x_next), DTP_ERR_INVALID_ARG,
            "x_next must be 16-byte aligned");
  DTP_CHECK(std::isfinite(eps_next) && eps_next >= 0.0f, DTP_ERR_INVALID_ARG,
            "rms_eps_next=%g must be finite and >= 0", (double)eps_next);
  DTP_CHECK(L->has_weights, DTP_ERR_INVALID_ARG, "dtp_layer_set_weights was not called");
  dtp_status st = check_device(L);
  if (st != DTP_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  const dtp_layer_desc& d = L->desc;
  const int H = d.n_q_heads, dh = d.head_dim, HD = H * dh, G = d.n_kv_groups;
  const int I = d.n_neurons, dm = d.d_model;
  const size_t esz = d.dtype == DTP_BF16 ? 2 : 4;
  const size_t nt = (size_t)n_tokens;
  if ((st = check_dev_buffer(x, esz * nt * dm, "x")) != DTP_OK ||
      (st = check_dev_buffer(attn, esz * nt * HD, "attn")) != DTP_OK ||
      (st = check_dev_buffer(A, sizeof(float) * (size_t)G * I, "A")) != DTP_OK ||
      (st = check_dev_buffer(x_next, esz * nt * dm, "x_next", true)) != DTP_OK ||
      (st = check_dev_buffer(s_down, sizeof(float) * (size_t)I, "s_down", true)) != DTP_OK)
    return st;
  // Tokens per slice: the 1/r buffer size, and element offsets of a slice below 2^30.  On the
  // bf16 path the slices of a call are of even length, so that none is a short rest.
  const int64_t width = std::max(dm, HD);
  int64_t slice = std::max<int64_t>(256, std::min<int64_t>(kSliceTokens, ((int64_t)1 << 30) / width) / 256 * 256);
  if (d.dtype == DTP_BF16) slice = choose_slice(L, n_tokens);
  for (int64_t t0 = 0, T_next; t0 < n_tokens; t0 += T_next) {
    const int T = (int)(d.dtype == DTP_BF16 && n_tokens - t0 <= L->tile_slice ? n_tokens - t0
                                                                              : std::min(slice, n_tokens - t0));
    T_next = T;
    const char* xs = (const char*)x + esz * (size_t)t0 * dm;
    const char* as = (const char*)attn + esz * (size_t)t0 * HD;
    const char* xns = x_next ? (const char*)x_next + esz * (size_t)t0 * dm : nullptr;
    const float* rinv_next = xns ? L->rinv_next : nullptr;
    AffinityArgs p{};
    LaunchShape shape;
    if (d.dtype == DTP_BF16) {
      p.xt = L->xt;
      p.wcat = (const uint16_t*)L->w;
      p.rinv = L->rinv;
      p.rinv_next = rinv_next;
      p.nd = L->nd;
      p.partial = L->partial;
      p.ks = L->Kt / kStage;
      p.nq1 = L->dP / kStage;
      p.nqh = L->dhP / kStage;
      p.G = G;
      p.hpg = H / G;
      p.I_pad = L->I_pad;
      shape = choose_launch(p, add, T, L->tile_slice);
      TokenArgs t{(const uint16_t*)xs, (const uint16_t*)as, (const uint16_t*)xns, d.rms_eps, eps_next, T,
                  shape.mtiles * shape.tile, dm, H, dh, L->dP, L->dhP, L->xt, L->rinv, L->rinv_next};
      (shape.tile == 64 ? launch_tile_tokens<4> : shape.tile == 128 ? launch_tile_tokens<8> : launch_tile_tokens<12>)(t, s);
    } else if (xns) {  // the fp32 kernel takes 1/r from the rows that it stages
      rms_kernel<<<(unsigned)((T + 3) / 4), 256, 0, s>>>((const float*)xns, T, dm, eps_next, L->rinv_next);
    }
    DTP_HIP(hipGetLastError());

    int splits;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (L->profiling) {
      DTP_HIP(hipEventCreate(&e0));
      DTP_HIP(hipEventCreate(&e1));
      DTP_HIP(hipEventRecord(e0, s));
    }
    if (d.dtype == DTP_BF16) {
      (shape.tile == 64 ? launch_affinity<2> : shape.tile == 128 ? launch_affinity<4> : launch_affinity<6>)(
          p, shape, add, s);
      splits = shape.splits;
    } else {
      AffinityF32Args f;
      f.x = (const float*)xs;
      f.attn = (const float*)as;
      f.wcat = (const float*)L->w;
      f.rinv_next = rinv_next;
      f.nd = L->nd;
      f.partial = L->partial;
      f.eps = d.rms_eps;
      f.T = T;
      f.d = dm;
      f.H = H;
      f.G = G;
      f.dh = dh;
      f.Kt = L->Kt;
      f.I_pad = L->I_pad;
      f.splits = 0;
      f.add = add ? 1 : 0;
      splits = launch_affinity_f32(f, device_cus(), s);
    }
    DTP_HIP(hipGetLastError());
    if (L->profiling) {
      DTP_HIP(hipEventRecord(e1, s));
      L->events.emplace_back(e0, e1);
    }
    reduce_splits_kernel<<<dim3((I + 31) / 32, s_down ? G + 1 : G), 256, 0, s>>>(
        L->partial, splits, G, I, L->I_pad, A, s_down);
    DTP_HIP(hipGetLastError());
  }
  return DTP_OK;
}

}  // namespace
}  // namespace dtp

extern "C" {

dtp_status dtp_layer_create(const dtp_layer_desc* desc, dtp_layer* out) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(desc != nullptr && out != nullptr, DTP_ERR_INVALID_ARG, "desc or out is NULL");
    const dtp_layer_desc& d = *desc;
    DTP_CHECK(d.d_model > 0 && d.n_neurons > 0 && d.n_q_heads > 0 && d.n_kv_groups > 0 &&
                  d.head_dim > 0,
              DTP_ERR_INVALID_ARG, "every size must be positive (d=%d I=%d H=%d G=%d dh=%d)",
              d.d_model, d.n_neurons, d.n_q_heads, d.n_kv_groups, d.head_dim);
    DTP_CHECK(d.n_q_heads % d.n_kv_groups == 0, DTP_ERR_INVALID_ARG,
              "H=%d is not a multiple of G=%d", d.n_q_heads, d.n_kv_groups);
    DTP_CHECK(d.n_kv_groups <= kMaxAffinityGroups, DTP_ERR_UNSUPPORTED, "G=%d exceeds %d",
              d.n_kv_groups, kMaxAffinityGroups);
    DTP_CHECK(d.head_dim % 16 == 0, DTP_ERR_INVALID_ARG, "head_dim=%d is not a multiple of 16",
              d.head_dim);
    DTP_CHECK(d.d_model % 16 == 0, DTP_ERR_INVALID_ARG, "d_model=%d is not a multiple of 16",
              d.d_model);
    DTP_CHECK(d.d_model <= 65536 && d.n_neurons <= (1 << 20) &&
                  (int64_t)d.n_q_heads * d.head_dim <= 65536,
              DTP_ERR_UNSUPPORTED, "shape too large (d <= 65536, I <= 2^20, H*dh <= 65536)");
    DTP_CHECK(std::isfinite(d.rms_eps) && d.rms_eps >= 0.0f, DTP_ERR_INVALID_ARG,
              "rms_eps=%g must be finite and >= 0", (double)d.rms_eps);
    DTP_CHECK(d.dtype == DTP_BF16 || d.dtype == DTP_F32, DTP_ERR_UNSUPPORTED, "dtype %d",
              d.dtype);
    dtp_layer L = new (std::nothrow) dtp_layer_s();
    DTP_CHECK(L != nullptr, DTP_ERR_NO_MEMORY, "host allocation failed");
    L->desc = d;
    hipError_t e = hipGetDevice(&L->device);
    L->n_tiles = (d.n_neurons + kBlockNeurons - 1) / kBlockNeurons * (kBlockNeurons / kBN);
    L->I_pad = L->n_tiles * kBN;
    const int64_t HD = (int64_t)d.n_q_heads * d.head_dim;
    const size_t rows = 2 * (size_t)L->I_pad;
    if (d.dtype == DTP_BF16) {
      auto up = [](int v) { return (v + kStage - 1) / kStage * kStage; };
      L->dP = (d.d_model + 4 * kStage - 1) / (4 * kStage) * (4 * kStage);
      // Heads of one to six stages have kernels of their own; longer ones take fours of stages.
      L->dhP = up(d.head_dim);
      if (L->dhP > 6 * kStage) L->dhP = (d.head_dim + 4 * kStage - 1) / (4 * kStage) * (4 * kStage);
      L->Kt = L->dP + d.n_q_heads * L->dhP;
      // Element offsets inside the tiled slice stay below 2^30.
      L->tile_slice = std::max<int64_t>((kSliceSpare + 1) * kTokenPad,
                                        std::min<int64_t>(pad_tokens(kTileTokens) + kSliceSpare * kTokenPad,
                                                          ((int64_t)1 << 30) / L->Kt / kTokenPad * kTokenPad));
      if (e == hipSuccess) e = hipMalloc(&L->w, 2 * rows * L->Kt);
      if (e == hipSuccess) e = hipMalloc(&L->woT, 2 * (size_t)((HD + 255) / 256 * 256) * L->dP);
      if (e == hipSuccess) e = hipMalloc(&L->xt, 2 * (size_t)L->tile_slice * L->Kt);
    } else {
      L->Kt = d.d_model + (int)HD;
      if (e == hipSuccess) e = hipMalloc(&L->w, 4 * rows * L->Kt);
    }
    if (e == hipSuccess) e = hipMalloc(&L->nd, 4 * (size_t)L->I_pad);
    if (e == hipSuccess) e = hipMalloc(&L->rinv, 4 * (size_t)kSliceTokens);
    if (e == hipSuccess)
      e = hipMalloc(&L->partial, 4 * (size_t)kMaxSplits * (d.n_kv_groups + 1) * L->I_pad);
    if (e == hipSuccess) e = hipMalloc(&L->rinv_next, 4 * (size_t)kSliceTokens);
    if (e != hipSuccess) {
      layer_free(L);
      return fail(e == hipErrorOutOfMemory ? DTP_ERR_NO_MEMORY : DTP_ERR_HIP,
                  "layer allocation failed: %s", hipGetErrorString(e));
    }
    *out = L;
    return DTP_OK;
  });
}

dtp_status dtp_layer_destroy(dtp_layer layer) {
  return guarded([&]() -> dtp_status {
    clear_error();
    if (layer) layer_free(layer);
    return DTP_OK;
  });
}

dtp_status dtp_layer_set_weights(dtp_layer L, const void* w_o, const void* gamma,
                                 const void* w_gate, const void* w_up, const void* w_down,
                                 void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(L != nullptr, DTP_ERR_INVALID_ARG, "layer is NULL");
    DTP_CHECK(w_o && gamma && w_gate && w_up && w_down, DTP_ERR_INVALID_ARG,
              "a weight pointer is NULL");
    dtp_status st = check_device(L);
    if (st != DTP_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const dtp_layer_desc& d = L->desc;
    const int H = d.n_q_heads, dh = d.head_dim, HD = H * dh, I = d.n_neurons, dm = d.d_model;
    {
      const size_t esz = d.dtype == DTP_BF16 ? 2 : 4;
      const void* ptrs[5] = {w_o, gamma, w_gate, w_up, w_down};
      const size_t elems[5] = {(size_t)dm * HD, (size_t)dm, (size_t)I * dm, (size_t)I * dm,
                               (size_t)dm * I};
      const char* names[5] = {"w_o", "gamma", "w_gate", "w_up", "w_down"};
      for (int i = 0; i < 5; ++i)
        if ((st = check_dev_buffer(ptrs[i], esz * elems[i], names[i])) != DTP_OK) return st;
    }
    if (d.dtype == DTP_BF16) {
      launch_prep_gate_up((const uint16_t*)w_gate, (const uint16_t*)w_up, (const uint16_t*)gamma, I, dm,
                          L->dP, L->I_pad, L->Kt / kStage, (uint16_t*)L->w, s);
      DTP_HIP(hipGetLastError());
      launch_fold((const uint16_t*)w_o, HD, dm, dh, L->dP, L->dhP, L->I_pad, L->Kt / kStage, (uint16_t*)L->woT,
                  (uint16_t*)L->w, s);
      DTP_HIP(hipGetLastError());
      st = down_norms((const uint16_t*)w_down, L, s);
      if (st != DTP_OK) return st;
    } else {
      prep_gate_up_kernel<<<grid_for((int64_t)L->n_tiles * kCols * dm, 256), 256, 0, s>>>(
          (const float*)w_gate, (const float*)w_up, (const float*)gamma, I, dm, L->n_tiles, L->Kt,
          (float*)L->w);
      DTP_HIP(hipGetLastError());
      launch_fold_f32((float*)L->w, (const float*)w_o, L->n_tiles * kCols, HD, dm, L->Kt, s);
      DTP_HIP(hipGetLastError());
      st = down_norms((const float*)w_down, L, s);
      if (st != DTP_OK) return st;
    }
    L->has_weights = true;
    return DTP_OK;
  });
}

dtp_status dtp_affinity_accumulate(dtp_layer L, const void* x, const void* attn, int64_t n_tokens,
                                   float* A, void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    return dtp::accumulate(L, x, attn, nullptr, 0.0f, n_tokens, A, nullptr, false, stream);
  });
}

dtp_status dtp_affinity_accumulate_add(dtp_layer L, const void* x, const void* attn,
                                       int64_t n_tokens, float* A, void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    return dtp::accumulate(L, x, attn, nullptr, 0.0f, n_tokens, A, nullptr, true, stream);
  });
}

dtp_status dtp_affinity_accumulate_down(dtp_layer L, const void* x, const void* attn,
                                        const void* x_next, float rms_eps_next, int64_t n_tokens,
                                        float* A, float* s_down, void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(x_next && s_down, DTP_ERR_INVALID_ARG, "x_next or s_down is NULL");
    return dtp::accumulate(L, x, attn, x_next, rms_eps_next, n_tokens, A, s_down, false, stream);
  });
}

dtp_status dtp_layer_profile(dtp_layer L, int32_t enable) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(L != nullptr, DTP_ERR_INVALID_ARG, "layer is NULL");
    L->profiling = enable != 0;
    return DTP_OK;
  });
}

dtp_status dtp_layer_profile_read(dtp_layer L, double* total_ms, int64_t* launches) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(L != nullptr && total_ms && launches, DTP_ERR_INVALID_ARG, "NULL argument");
    double sum = 0.0;
    for (auto& e : L->events) {
      DTP_HIP(hipEventSynchronize(e.second));
      float ms = 0.0f;
      DTP_HIP(hipEventElapsedTime(&ms, e.first, e.second));
      sum += ms;
    }
    *total_ms = sum;
    *launches = (int64_t)L->events.size();
    for (auto& e : L->events) {
      (void)hipEventDestroy(e.first);
      (void)hipEventDestroy(e.second);
    }
    L->events.clear();
    return DTP_OK;
  });
}

}  // extern "C"
