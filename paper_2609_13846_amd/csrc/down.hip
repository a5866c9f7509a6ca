// Down-edge affinity on MI355X (gfx950): Section 3 of the paper, "Affinity scores", down
// edge.  Neuron k of layer i writes alpha_k w^d_k into the residual stream; through the
// attention pre-norm of layer i+1 (gain gamma', rms r') it reaches the q/k/v projections of
// KV group g as (alpha_k / r') b_gk with b_gk = W^{qkv}_g (gamma' * w^d_k), so
//   S_down[k, g] = sum_t alpha_k^2 / r'^2 * ||b_gk||^2      (raw token sum).
// The token statistic s[k] = sum_t alpha_k^2 / r'^2 comes out of the affinity kernel's
// operating point (dtp_affinity_accumulate_down).  This file holds the weight-only factor
// B[g, k] = ||b_gk||^2 and the product of the two.
//
// W^{qkv}_g stacks the q rows of the group's query heads (consecutive heads share a group),
// then its k rows and its v rows, from the q_proj / k_proj / v_proj weight layouts.
//
// Kernels:
//   transpose_fragments_kernel  gamma' * W_down transposed to bf16 fragments, once per call
//   qkv_fragments_kernel     the rows of every W^{qkv}_g as bf16 fragments, once per call
//   down_weight_frag_kernel  one block per (256 neurons, 256 or 128 rows of W^{qkv}_g, group):
//                            MFMA over d, then per-column sums of squares of each 128 rows
//   down_weight_bf16_kernel  the same straight from the caller's matrices, for the
//                            allocation-free call and where the copies' launches would
//                            be too large: 128 neurons x 128 rows per block
//   down_weight_f32_kernel   the same with plain FMAs, one thread per (group, neuron)
//   down_rows_reduce_kernel  B[g, k] = fixed-order fp64 sum over the row chunks
//   down_combine_kernel      S_down[k, g] = s[k] B[g, k]
#include <cmath>
#include <mutex>
#include <type_traits>

#include "dtp_internal.h"
#include "frag_gemm.h"
#include "tile_mfma.h"

namespace dtp {
namespace {

constexpr int kDKC = 32;              // contraction depth per LDS stage
constexpr int kDRow = kDKC + 8;       // bf16 per LDS row (16 bytes of padding)
constexpr int kDRows = 128;           // rows of W^{qkv}_g per block (4 waves x 32)
constexpr int kDCols = 128;           // neurons per block
constexpr int kDThreads = 256;

// Row rho of W^{qkv}_g inside the three projection matrices (each row d long).
template <typename T>
__device__ inline const T* qkv_row(const T* w_q, const T* w_k, const T* w_v, int g, int rho,
                                   int hpg, int dh, int d) {
  if (rho < hpg * dh) return w_q + ((int64_t)g * hpg * dh + rho) * d;
  rho -= hpg * dh;
  if (rho < dh) return w_k + ((int64_t)g * dh + rho) * d;
  return w_v + ((int64_t)g * dh + rho - dh) * d;
}

// The rows of every W^{qkv}_g in fragment-major layout, each group padded with zero rows to
// group_rows (and zero columns past d, a multiple of 8).  One wavefront per fragment: lane l
// reads piece l % 4 of row l / 4 (64 contiguous bytes per row) and the pieces change lanes
// into fragment order.  Fragments in memory order: F of a stage, then the next stage's.
template <int F>
__global__ void __launch_bounds__(256)
qkv_fragments_kernel(const uint16_t* __restrict__ w_q, const uint16_t* __restrict__ w_k,
                     const uint16_t* __restrict__ w_v, int d, int hpg, int dh, int group_rows, int ks,
                     int64_t n_frags, uint16_t* __restrict__ out) {
  const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (f >= n_frags) return;  // whole wavefronts
  const int lane = threadIdx.x & 63;
  const int64_t tile = f / (F * ks);
  const int at = (int)(f % (F * ks));
  const int j = at / F * 32 + 8 * (lane % 4);
  const int64_t row = (tile * F + at % F) * 16 + lane / 4;
  const int g = (int)(row / group_rows), rho = (int)(row % group_rows);
  u32x4 v = {0u, 0u, 0u, 0u};
  if (rho < (hpg + 2) * dh && j < d)
    v = *reinterpret_cast<const u32x4*>(qkv_row(w_q, w_k, w_v, g, rho, hpg, dh, d) + j);
  const int from = (lane % 16) * 4 + lane / 16;
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (uint32_t)__shfl((int)v[e], from, 64);
  *reinterpret_cast<u32x4*>(out + (f * 64 + lane) * 8) = o;
}

// Column l % 16's sum of squares over the 32 rows of two stacked 16 x 16 accumulators.
__device__ __forceinline__ float rows32_sum_sq(f32x4 lo, f32x4 hi) {
  float c = 0.0f;
#pragma unroll
  for (int e = 0; e < 4; ++e) c = fmaf(lo[e], lo[e], c);
#pragma unroll
  for (int e = 0; e < 4; ++e) c = fmaf(hi[e], hi[e], c);
  c += __shfl_xor(c, 16, 64);
  return c + __shfl_xor(c, 32, 64);
}

// partial[g][chunk][k] = sum over the chunk's 128 rows of (W^{qkv}_g[rho] . (gamma' * w^d_k))^2:
// a block takes 32 AF rows (one chunk or two) of one group x 256 neurons.  The products'
// order along the contraction and the order of the sums are those of
// down_weight_bf16_kernel, so both give the same bits.  Bound by the matrix cores and the clock
// that they leave: 721 GFLOP of the 8B-class shape in 522 us at best (1,380 TFLOP/s, as much as a
// large library product, at 1.90 GHz with the MFMAs busy 69% of the time and 1,344 blocks in
// 5.25 rounds of 256 CUs) and 533 to 608 over a row of calls, against 960 us for 128 x 128 tiles
// staged through registers.
template <int AF>
__global__ void __launch_bounds__(512, 2)
down_weight_frag_kernel(const uint16_t* __restrict__ qkv, const uint16_t* __restrict__ tw, int ks,
                        int n_row_tiles, int n_col_tiles, int I, float* __restrict__ partial) {
  using P = FragPipe<AF, 4>;
  __shared__ __attribute__((aligned(16))) uint16_t s0[P::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s1[P::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s2[P::kSlot];
  __shared__ __attribute__((aligned(16))) uint16_t s3[P::kSlot];
  __shared__ float red[P::kARows / 32][P::kBRows];  // sums over 32 rows
  int rt, ct;
  frag_work(blockIdx.x, n_row_tiles, n_col_tiles, 6, rt, ct);
  P p(qkv + (int64_t)rt * P::kARows * ks * 32, (uint32_t)P::kAFrags * ks * 1024u,
      tw + (int64_t)ct * P::kBRows * ks * 32, (uint32_t)P::kBFrags * ks * 1024u);
  p.contract(s0, s1, s2, s3, ks);
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < AF; i += 2) {
      const float c = rows32_sum_sq(p.acc[i][j], p.acc[i + 1][j]);
      if (p.lane < 16) red[(p.wm * AF + i) / 2][(p.wn * 4 + j) * 16 + p.lane] = c;
    }
  __syncthreads();
  for (int idx = threadIdx.x; idx < P::kARows / kDRows * P::kBRows; idx += 512) {
    const int chunk = idx / P::kBRows, c = idx % P::kBRows, k = ct * P::kBRows + c;
    if (k < I)
      partial[((int64_t)rt * (P::kARows / kDRows) + chunk) * I + k] =
          red[4 * chunk][c] + red[4 * chunk + 1][c] + red[4 * chunk + 2][c] + red[4 * chunk + 3][c];
  }
}

// partial[g][chunk][k] = sum over the chunk's rows rho of (W^{qkv}_g[rho] . (gamma' * w^d_k))^2.
// The allocation-free form: each stage scales and transposes its slice of W_down itself, for
// want of room for a copy.  Bound by that transposition's LDS writes: as words of two rows
// 265 us, as halves 431, for 128 groups of 24 rows at d = 1,024, I = 3,072.
__global__ void __launch_bounds__(kDThreads)
down_weight_bf16_kernel(const uint16_t* __restrict__ w_q, const uint16_t* __restrict__ w_k,
                        const uint16_t* __restrict__ w_v, const uint16_t* __restrict__ gamma,
                        const uint16_t* __restrict__ w_down, int d, int I, int hpg, int dh,
                        float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) uint16_t As[2][kDRows * kDRow];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kDCols * kDRow];
  __shared__ float red[4][kDCols];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int k0 = blockIdx.x * kDCols, chunk = blockIdx.y, g = blockIdx.z;
  const int n_chunks = gridDim.y;
  const int R = (hpg + 2) * dh;
  f32x4 acc[2][8] = {};
  // A stage's operands in registers: A, 128 rows x 32 columns of W^{qkv}_g, and B, 128
  // neurons x 32 columns of gamma' * W_down, 16 bytes per thread and pass (2 passes each).
  // Stage kc+32 is fetched into registers during stage kc's MFMAs and stored into the
  // other LDS buffer after them.
  u32x4 av[2], bv[2];
  float bg[2];
  auto fetch = [&](int kc) __attribute__((always_inline)) {
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const int row = threadIdx.x / 4 + 64 * pass, seg = threadIdx.x % 4;
      const int rho = chunk * kDRows + row, j = kc + 8 * seg;
      av[pass] = u32x4{0u, 0u, 0u, 0u};
      if (rho < R && j < d)
        av[pass] = *reinterpret_cast<const u32x4*>(qkv_row(w_q, w_k, w_v, g, rho, hpg, dh, d) + j);
    }
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      bv[pass] = u32x4{0u, 0u, 0u, 0u};
      const int j = kc + 2 * (threadIdx.x / 16) + pass, k = k0 + 8 * (threadIdx.x % 16);
      // I % 8 == 0: the 8 neurons are all valid or all past I
      if (j < d && k < I) bv[pass] = *reinterpret_cast<const u32x4*>(w_down + (int64_t)j * I + k);
      bg[pass] = j < d ? bf16_to_f32(gamma[j]) : 0.0f;
    }
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const int row = threadIdx.x / 4 + 64 * pass, seg = threadIdx.x % 4;
      *reinterpret_cast<u32x4*>(As[buf] + row * kDRow + 8 * seg) = av[pass];
    }
    // scaled by gamma'[j] and stored transposed, [k][j], the two rows of a thread as one word
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      uint16_t w[2];
#pragma unroll
      for (int pass = 0; pass < 2; ++pass)
        w[pass] = f32_to_bf16(bf16_to_f32((uint16_t)(bv[pass][e / 2] >> (16 * (e % 2)))) * bg[pass]);
      *reinterpret_cast<uint32_t*>(Bs[buf] + (8 * (threadIdx.x % 16) + e) * kDRow + 2 * (threadIdx.x / 16)) =
          (uint32_t)w[0] | ((uint32_t)w[1] << 16);
    }
  };
  fetch(0);
  store(0);
  __syncthreads();
  for (int kc = 0, buf = 0; kc < d; kc += kDKC, buf ^= 1) {
    const bool more = kc + kDKC < d;
    if (more) fetch(kc + kDKC);
    const int at = (lane & 15) * kDRow + 8 * (lane >> 4);
    bf16x8 a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a[i] = *reinterpret_cast<const bf16x8*>(As[buf] + (32 * wave + 16 * i) * kDRow + at);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bf16x8 bb = *reinterpret_cast<const bf16x8*>(Bs[buf] + 16 * b * kDRow + at);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], bb, acc[i][b], 0, 0, 0);
    }
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  // Sum of squares over the wave's 32 rows, per column; rows past R are zero.
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const float c = rows32_sum_sq(acc[0][b], acc[1][b]);
    if (lane < 16) red[wave][b * 16 + lane] = c;
  }
  __syncthreads();
  for (int c = threadIdx.x; c < kDCols; c += kDThreads) {
    const int k = k0 + c;
    if (k < I)
      partial[((int64_t)g * n_chunks + chunk) * I + k] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
  }
}

// B[g][k] directly, fp32 FMAs: one thread per (group, neuron).
__global__ void __launch_bounds__(256)
down_weight_f32_kernel(const float* __restrict__ w_q, const float* __restrict__ w_k,
                       const float* __restrict__ w_v, const float* __restrict__ gamma,
                       const float* __restrict__ w_down, int d, int I, int G, int hpg, int dh,
                       float* __restrict__ B) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)G * I) return;
  const int g = (int)(idx / I), k = (int)(idx % I);
  const int R = (hpg + 2) * dh;
  double acc = 0.0;
  for (int rho = 0; rho < R; ++rho) {
    const float* row = qkv_row(w_q, w_k, w_v, g, rho, hpg, dh, d);
    float b = 0.0f;
    for (int j = 0; j < d; ++j) b = fmaf(row[j], gamma[j] * w_down[(int64_t)j * I + k], b);
    acc += (double)b * b;
  }
  B[idx] = (float)acc;
}

__global__ void down_rows_reduce_kernel(const float* __restrict__ partial, int G, int n_chunks,
                                        int I, float* __restrict__ B) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)G * I) return;
  const int g = (int)(idx / I), k = (int)(idx % I);
  double s = 0.0;
  for (int c = 0; c < n_chunks; ++c) s += (double)partial[((int64_t)g * n_chunks + c) * I + k];
  B[idx] = (float)s;
}

__global__ void down_combine_kernel(const float* __restrict__ s, const float* __restrict__ B,
                                    int I, int G, float* __restrict__ A_down) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)I * G) return;
  const int k = (int)(idx / G), g = (int)(idx % G);
  A_down[idx] = s[k] * B[(int64_t)g * I + k];
}

unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

// Scratch of dtp_down_weights_noalloc: the per-chunk partial sums, in device memory the
// library never allocates.  Each device the library runs on holds its own copy until the
// process ends.  In host code `scratch` names a host-side stand-in, not a device address:
// the kernels only ever receive the address hipGetSymbolAddress returns for the current
// device (noalloc_scratch below).  Every slot a call reads is written earlier in the same
// call, so nothing needs clearing between calls.
constexpr size_t kNoAllocScratchFloats = size_t(1) << 20;  // 4 MiB
constexpr int kNoAllocMaxDevices = 64;
static __device__ __align__(256) float scratch[kNoAllocScratchFloats];

std::mutex g_scratch_mu;
float* g_scratch_dev[kNoAllocMaxDevices] = {};

// The current device's copy of `scratch`, looked up once per device on first use.
dtp_status noalloc_scratch(float** out) {
  int dev = -1;
  DTP_HIP(hipGetDevice(&dev));
  DTP_CHECK(dev >= 0 && dev < kNoAllocMaxDevices, DTP_ERR_UNSUPPORTED,
            "device %d: the allocation-free scratch is kept for devices 0..%d", dev,
            kNoAllocMaxDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[dev] == nullptr) {
    void* p = nullptr;
    DTP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    DTP_CHECK(p != nullptr, DTP_ERR_HIP, "no device address for the scratch on device %d", dev);
    g_scratch_dev[dev] = (float*)p;
  }
  *out = g_scratch_dev[dev];
  return DTP_OK;
}

// Whether the operands are copied fragment-major first: while the launches over the copies hold
// fewer than 2^32 threads each.  (Thousands of groups of a few rows, each padded to a chunk,
// do not: 4,096 at d = 65,536.)  The kernel of the allocation-free call, whose grid has the groups
// in a dimension of their own, takes those with the same bits; where both can run it is the
// slower one, 265 us against 104 for 128 groups of 24 rows at d = 1,024, I = 3,072.
bool copies_launch(int64_t rows, int64_t n_frags, int64_t col_tiles) {
  constexpr int64_t kThreads = (int64_t)1 << 32;
  return n_frags * 64 < kThreads && rows / kDRows * col_tiles * 512 < kThreads;
}

// Shared body of dtp_down_weights and dtp_down_weights_noalloc.  The scratch of the row-chunk
// sums comes from the stream-ordered allocator, or with `use_static` from the current
// device's copy of `scratch` (the call is refused when it would not fit).
dtp_status down_weights(int32_t d_model, int32_t n_neurons, int32_t n_q_heads, int32_t n_kv_groups,
                        int32_t head_dim, dtp_dtype dtype, const void* w_q, const void* w_k,
                        const void* w_v, const void* gamma_next, const void* w_down, float* B,
                        bool use_static, void* stream) {
  DTP_CHECK(d_model > 0 && n_neurons > 0 && n_q_heads > 0 && n_kv_groups > 0 && head_dim > 0,
            DTP_ERR_INVALID_ARG, "every size must be positive (d=%d I=%d H=%d G=%d dh=%d)",
            d_model, n_neurons, n_q_heads, n_kv_groups, head_dim);
  DTP_CHECK(n_q_heads % n_kv_groups == 0, DTP_ERR_INVALID_ARG, "H=%d is not a multiple of G=%d",
            n_q_heads, n_kv_groups);
  DTP_CHECK(d_model <= 65536 && n_neurons <= (1 << 20) && (int64_t)n_q_heads * head_dim <= 65536,
            DTP_ERR_UNSUPPORTED, "shape too large (d <= 65536, I <= 2^20, H*dh <= 65536)");
  DTP_CHECK(dtype == DTP_BF16 || dtype == DTP_F32, DTP_ERR_UNSUPPORTED, "dtype %d", dtype);
  const int hpg = n_q_heads / n_kv_groups;
  const int64_t GI = (int64_t)n_kv_groups * n_neurons;
  const int R = (hpg + 2) * head_dim;
  const int n_chunks = (R + kDRows - 1) / kDRows;
  if (use_static && dtype == DTP_BF16)
    DTP_CHECK((size_t)GI * n_chunks <= kNoAllocScratchFloats, DTP_ERR_UNSUPPORTED,
              "G * I * ceil((H/G + 2) * dh / 128) = %lld partial sums exceed the %zu floats of "
              "the allocation-free scratch (use dtp_down_weights)",
              (long long)(GI * n_chunks), kNoAllocScratchFloats);
  DTP_CHECK(w_q && w_k && w_v && gamma_next && w_down && B, DTP_ERR_INVALID_ARG,
            "a weight pointer or B is NULL");
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
  DTP_CHECK(al16(w_q) && al16(w_k) && al16(w_v) && al16(w_down), DTP_ERR_INVALID_ARG,
            "w_q, w_k, w_v and w_down must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  {
    const size_t esz = dtype == DTP_BF16 ? 2 : 4, dm = (size_t)d_model;
    const size_t gd = (size_t)n_kv_groups * head_dim;
    dtp_status st;
    if ((st = check_dev_buffer(w_q, esz * n_q_heads * head_dim * dm, "w_q")) != DTP_OK ||
        (st = check_dev_buffer(w_k, esz * gd * dm, "w_k")) != DTP_OK ||
        (st = check_dev_buffer(w_v, esz * gd * dm, "w_v")) != DTP_OK ||
        (st = check_dev_buffer(gamma_next, esz * dm, "gamma_next")) != DTP_OK ||
        (st = check_dev_buffer(w_down, esz * dm * n_neurons, "w_down")) != DTP_OK ||
        (st = check_dev_buffer(B, sizeof(float) * (size_t)GI, "B")) != DTP_OK)
      return st;
  }
  if (dtype == DTP_F32) {
    DTP_CHECK(d_model % 4 == 0, DTP_ERR_INVALID_ARG, "d_model=%d is not a multiple of 4", d_model);
    down_weight_f32_kernel<<<blocks_for(GI, 256), 256, 0, s>>>(
        (const float*)w_q, (const float*)w_k, (const float*)w_v, (const float*)gamma_next,
        (const float*)w_down, d_model, n_neurons, n_kv_groups, hpg, head_dim, B);
    DTP_HIP(hipGetLastError());
    return DTP_OK;
  }
  DTP_CHECK(d_model % 8 == 0, DTP_ERR_INVALID_ARG, "d_model=%d is not a multiple of 8", d_model);
  DTP_CHECK(n_neurons % 8 == 0, DTP_ERR_INVALID_ARG, "n_neurons=%d is not a multiple of 8",
            n_neurons);
  // Scratch of the copying form in one block: [partial sums | neuron fragments | row fragments].
  const int ks = (d_model + 31) / 32;
  const int col_tiles = (n_neurons + 255) / 256;
  const int64_t rows = (int64_t)n_kv_groups * n_chunks * kDRows;
  const int64_t n_frags = rows / 16 * ks;
  const size_t part_bytes = (sizeof(float) * (size_t)GI * n_chunks + 1023) / 1024 * 1024;
  const size_t tw_bytes = (size_t)col_tiles * 256 * ks * 64, qkv_bytes = (size_t)rows * ks * 64;
  float* partial = nullptr;
  char* base = nullptr;
  hipError_t e = hipSuccess;
  if (use_static) {
    dtp_status st = noalloc_scratch(&partial);
    if (st != DTP_OK) return st;
  } else {
    const bool copy = copies_launch(rows, n_frags, col_tiles);
    DTP_HIP(stream_alloc((void**)&partial, part_bytes + (copy ? tw_bytes + qkv_bytes : 0), s));
    if (copy) base = (char*)partial;
  }
  if (base == nullptr) {
    const dim3 grid((n_neurons + kDCols - 1) / kDCols, n_chunks, n_kv_groups);
    down_weight_bf16_kernel<<<grid, kDThreads, 0, s>>>(
        (const uint16_t*)w_q, (const uint16_t*)w_k, (const uint16_t*)w_v,
        (const uint16_t*)gamma_next, (const uint16_t*)w_down, d_model, n_neurons, hpg, head_dim,
        partial);
    e = hipGetLastError();
  } else {
    uint16_t* tw = (uint16_t*)(base + part_bytes);
    uint16_t* qkv = (uint16_t*)(base + part_bytes + tw_bytes);
    const dim3 tg(col_tiles * 4, (ks + 1) / 2);
    transpose_fragments_kernel<16, true, true><<<tg, 256, 0, s>>>((const uint16_t*)w_down, (const uint16_t*)gamma_next,
                                                   d_model, n_neurons, ks, tw);
    // Two chunks per block where a group has an even number of them: half the neuron
    // fragments read per product.
    auto launch = [&](auto af) {
      constexpr int AF = decltype(af)::value;
      const int row_tiles = (int)(rows / (32 * AF));
      qkv_fragments_kernel<2 * AF><<<blocks_for(n_frags, 4), 256, 0, s>>>(
          (const uint16_t*)w_q, (const uint16_t*)w_k, (const uint16_t*)w_v, d_model, hpg, head_dim,
          n_chunks * kDRows, ks, n_frags, qkv);
      down_weight_frag_kernel<AF><<<row_tiles * col_tiles, 512, 0, s>>>(qkv, tw, ks, row_tiles, col_tiles,
                                                                        n_neurons, partial);
    };
    if (n_chunks % 2 == 0)
      launch(std::integral_constant<int, 8>());
    else
      launch(std::integral_constant<int, 4>());
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    down_rows_reduce_kernel<<<blocks_for(GI, 256), 256, 0, s>>>(partial, n_kv_groups, n_chunks,
                                                                n_neurons, B);
    e = hipGetLastError();
  }
  const hipError_t ef = use_static ? hipSuccess : stream_free(partial, s);
  DTP_HIP(e);
  DTP_HIP(ef);
  return DTP_OK;
}

}  // namespace
}  // namespace dtp

using namespace dtp;

extern "C" {

dtp_status dtp_down_weights(int32_t d_model, int32_t n_neurons, int32_t n_q_heads,
                            int32_t n_kv_groups, int32_t head_dim, dtp_dtype dtype,
                            const void* w_q, const void* w_k, const void* w_v,
                            const void* gamma_next, const void* w_down, float* B, void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    return down_weights(d_model, n_neurons, n_q_heads, n_kv_groups, head_dim, dtype, w_q, w_k, w_v,
                        gamma_next, w_down, B, false, stream);
  });
}

dtp_status dtp_down_weights_noalloc(int32_t d_model, int32_t n_neurons, int32_t n_q_heads,
                                    int32_t n_kv_groups, int32_t head_dim, dtp_dtype dtype,
                                    const void* w_q, const void* w_k, const void* w_v,
                                    const void* gamma_next, const void* w_down, float* B,
                                    void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    return down_weights(d_model, n_neurons, n_q_heads, n_kv_groups, head_dim, dtype, w_q, w_k, w_v,
                        gamma_next, w_down, B, true, stream);
  });
}

dtp_status dtp_down_affinity(int32_t n_neurons, int32_t n_kv_groups, const float* s_down,
                             const float* B, float* A_down, void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(n_neurons > 0 && n_kv_groups > 0, DTP_ERR_INVALID_ARG, "I=%d and G=%d must be positive",
              n_neurons, n_kv_groups);
    DTP_CHECK(s_down && B && A_down, DTP_ERR_INVALID_ARG, "s_down, B or A_down is NULL");
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = (int64_t)n_neurons * n_kv_groups;
    dtp_status st;
    if ((st = check_dev_buffer(s_down, sizeof(float) * (size_t)n_neurons, "s_down")) != DTP_OK ||
        (st = check_dev_buffer(B, sizeof(float) * (size_t)n, "B")) != DTP_OK ||
        (st = check_dev_buffer(A_down, sizeof(float) * (size_t)n, "A_down")) != DTP_OK)
      return st;
    down_combine_kernel<<<blocks_for(n, 256), 256, 0, s>>>(s_down, B, n_neurons, n_kv_groups, A_down);
    DTP_HIP(hipGetLastError());
    return DTP_OK;
  });
}

}  // extern "C"
