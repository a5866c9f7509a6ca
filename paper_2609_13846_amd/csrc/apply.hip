// Applying a layout to a decoder layer's weights (Section 3, "The layout as a free
// variable").  Let group_order[p] be the original KV group placed at new position p and
// neuron_order[p] the original neuron at new position p, where each list runs through
// device 0's members in increasing original index, then device 1's, and so on.  With
// hpg = H/G query heads per group, the permuted weights are
//   w_q     row block p      (hpg*dh rows)  <- row block group_order[p]
//   w_k,w_v row block p      (dh rows)      <- row block group_order[p]
//   w_o     column block p   (hpg*dh cols)  <- column block group_order[p]
//   w_gate, w_up  row p      <- row neuron_order[p]
//   w_down  column p         <- column neuron_order[p]
// so device l's shard is one contiguous range of groups and of neurons.  Gains and
// per-head norm weights do not move.
//
// Kernels (pure data movement, bit-exact):
//   permute_units_kernel     matrices whose permuted pieces are whole 16-byte vectors: rows,
//                            and w_o's column blocks; all of them in one launch
//   permute_cols_lds_kernel  single columns, through rows held in LDS
//   permute_cols_kernel      out[:, c] = in[:, column of block order[c / block]], any size
#include <algorithm>
#include <vector>

#include "dtp_internal.h"

namespace dtp {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// A matrix as a sequence of units of `unit` 16-byte vectors: in every run of n_order units,
// unit u of `out` is unit order[u] of `in`.  A row permutation is one run of row blocks, a
// permutation of column blocks one run per row.
struct UnitMove {
  const u32x4* in;
  u32x4* out;
  const int32_t* order;
  int64_t n_vec, unit;
  int32_t n_order;
  uint32_t first_block;  // of the launch
};
constexpr int kMaxMoves = 6;
struct UnitMoves {
  UnitMove m[kMaxMoves];
  int n;
};
constexpr int kMoveVecs = 4;  // vectors per thread, a block's 256 threads side by side

// HBM-bound.  Four loads per thread are in flight before the first store; a block's place in
// its matrix is found once, in scalars.  All six matrices of the 8B-class shape (637 MB read
// and written): 127 us, 5.0 TB/s, where a large copy reaches 5.4; a launch per matrix, one vector
// per thread and 64-bit quotients took 148.
__global__ void __launch_bounds__(256)
permute_units_kernel(UnitMoves moves) {
  int k = 0;
  while (k + 1 < moves.n && blockIdx.x >= moves.m[k + 1].first_block) ++k;
  const UnitMove& m = moves.m[k];
  const int64_t i0 = (int64_t)(blockIdx.x - m.first_block) * (256 * kMoveVecs);
  const int64_t u0 = i0 / m.unit;
  const int64_t off0 = i0 - u0 * m.unit + threadIdx.x;
  const int64_t run0 = u0 / m.n_order;
  const uint32_t c0 = (uint32_t)(u0 - run0 * m.n_order);
  u32x4 v[kMoveVecs];
#pragma unroll
  for (int j = 0; j < kMoveVecs; ++j) {
    // Units past the block's first: a 32-bit quotient, at most one for units that need 64 bits.
    const int64_t off = off0 + 256 * j;
    const uint32_t past = m.unit < (int64_t)1 << 30 ? (uint32_t)off / (uint32_t)m.unit : off >= m.unit;
    const uint32_t c = c0 + past;
    const int64_t run = run0 + c / m.n_order;
    if (i0 + threadIdx.x + 256 * j < m.n_vec)
      v[j] = m.in[(run * m.n_order + m.order[c % m.n_order]) * m.unit + (off - past * m.unit)];
  }
#pragma unroll
  for (int j = 0; j < kMoveVecs; ++j) {
    const int64_t i = i0 + threadIdx.x + 256 * j;
    if (i < m.n_vec) m.out[i] = v[j];
  }
}

constexpr size_t kColsLds = 64 * 1024;  // rows held per block
constexpr int kColsThreads = 1024;      // two such blocks fill a CU

// out[r][c] = in[r][order[c]], rows of a multiple of 16 bytes: `per` rows at a time go into LDS with
// 16-byte loads and come out in the new order, four bytes per thread so that neighbouring lanes
// write neighbouring words (and read LDS words a device count apart: a shard holds its neurons
// in increasing order).  HBM-bound: w_down of the 8B-class shape 51 us (81 with a quarter
// of the threads), against 172 us for one
// 2-byte gather from memory per element.
template <typename T>
__global__ void __launch_bounds__(kColsThreads)
permute_cols_lds_kernel(const T* __restrict__ in, T* __restrict__ out, int64_t rows, int cols, int per,
                        const int32_t* __restrict__ order) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int kWord = 4 / sizeof(T);  // elements per 4-byte word
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int n = (int)min((int64_t)per, rows - r0);
  const int vecs = n * cols / (int)(16 / sizeof(T));
  const u32x4* src = reinterpret_cast<const u32x4*>(in + r0 * cols);
  u32x4* tile = reinterpret_cast<u32x4*>(lds);
#pragma unroll 4
  for (int i = threadIdx.x; i < vecs; i += kColsThreads) tile[i] = src[i];
  __syncthreads();
  const T* row = reinterpret_cast<const T*>(lds);
  uint32_t* dst = reinterpret_cast<uint32_t*>(out + r0 * cols);
  const int words = cols / kWord;
#pragma unroll 4
  for (int w = threadIdx.x; w < words; w += kColsThreads) {
    int32_t from[kWord];
#pragma unroll
    for (int e = 0; e < kWord; ++e) from[e] = order[w * kWord + e];
    for (int r = 0; r < n; ++r) {
      uint32_t v;
      if constexpr (kWord == 2)
        v = (uint32_t)row[r * cols + from[0]] | ((uint32_t)row[r * cols + from[1]] << 16);
      else
        v = __float_as_uint(row[r * cols + from[0]]);
      dst[(int64_t)r * words + w] = v;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
permute_cols_kernel(const T* __restrict__ in, T* __restrict__ out, int64_t rows, int64_t cols,
                    int block, const int32_t* __restrict__ order) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * cols) return;
  const int64_t r = i / cols, c = i % cols;
  out[i] = in[r * cols + (int64_t)order[c / block] * block + c % block];
}

unsigned grid1(int64_t n) { return (unsigned)((n + 255) / 256); }

// order[p]: original index at new position p of a balanced assignment of n items.  One pass with
// a cursor per device (a pass per device, with a branch on each item, cost the host as much
// as the copies of an 8B-class layer cost the GPU).
void order_of(int n, int L, const int32_t* a, int32_t* order) {
  std::vector<int32_t> at(L);
  for (int l = 0; l < L; ++l) at[l] = l * (n / L);
  for (int i = 0; i < n; ++i) order[at[a[i]]++] = i;
}

// group_order / neuron_order: new position -> original index.
void orders(int G, int I, int L, const int32_t* h, const int32_t* nu, int32_t* go, int32_t* no) {
  order_of(G, L, h, go);
  order_of(I, L, nu, no);
}

dtp_status check_assignment(const int32_t* a, int n, int L, const char* what) {
  std::vector<int> cnt(L, 0);
  for (int i = 0; i < n; ++i) {
    DTP_CHECK(a[i] >= 0 && a[i] < L, DTP_ERR_INVALID_ARG, "%s[%d] = %d is not a device in [0, %d)",
              what, i, a[i], L);
    ++cnt[a[i]];
  }
  for (int l = 0; l < L; ++l)
    DTP_CHECK(cnt[l] == n / L, DTP_ERR_INVALID_ARG, "%s is not balanced (device %d holds %d)",
              what, l, cnt[l]);
  return DTP_OK;
}

}  // namespace
}  // namespace dtp

using namespace dtp;

extern "C" {

dtp_status dtp_layout_orders(int32_t G, int32_t I, int32_t L, const int32_t* h, const int32_t* nu,
                             int32_t* group_order, int32_t* neuron_order) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(G > 0 && I > 0 && L > 0 && G % L == 0 && I % L == 0, DTP_ERR_INVALID_ARG,
              "G=%d and I=%d must be positive multiples of L=%d", G, I, L);
    DTP_CHECK(h && nu && group_order && neuron_order, DTP_ERR_INVALID_ARG, "a pointer is NULL");
    dtp_status st = check_assignment(h, G, L, "h");
    if (st != DTP_OK) return st;
    if ((st = check_assignment(nu, I, L, "nu")) != DTP_OK) return st;
    orders(G, I, L, h, nu, group_order, neuron_order);
    return DTP_OK;
  });
}

dtp_status dtp_apply_layout(const dtp_layer_desc* desc, int32_t L, const int32_t* h,
                            const int32_t* nu, const void* const* src, void* const* dst,
                            void* stream) {
  return guarded([&]() -> dtp_status {
    clear_error();
    DTP_CHECK(desc && h && nu && src && dst, DTP_ERR_INVALID_ARG, "a pointer is NULL");
    const dtp_layer_desc& d = *desc;
    const int G = d.n_kv_groups, H = d.n_q_heads, dh = d.head_dim, I = d.n_neurons, dm = d.d_model;
    DTP_CHECK(dm > 0 && I > 0 && H > 0 && G > 0 && dh > 0 && H % G == 0, DTP_ERR_INVALID_ARG,
              "invalid layer shape (d=%d I=%d H=%d G=%d dh=%d)", dm, I, H, G, dh);
    DTP_CHECK(L > 0 && G % L == 0 && I % L == 0, DTP_ERR_INVALID_ARG,
              "G=%d and I=%d must be multiples of L=%d", G, I, L);
    DTP_CHECK(d.dtype == DTP_BF16 || d.dtype == DTP_F32, DTP_ERR_UNSUPPORTED, "dtype %d", d.dtype);
    const int esz = d.dtype == DTP_BF16 ? 2 : 4;
    DTP_CHECK(((int64_t)dm * esz) % 16 == 0, DTP_ERR_INVALID_ARG,
              "rows of d=%d elements must be a multiple of 16 bytes", dm);
    for (int i = 0; i < 7; ++i) {
      DTP_CHECK(src[i] && dst[i], DTP_ERR_INVALID_ARG, "weight %d is NULL", i);
      DTP_CHECK(((uintptr_t)src[i] & 15u) == 0 && ((uintptr_t)dst[i] & 15u) == 0,
                DTP_ERR_INVALID_ARG, "weight %d is not 16-byte aligned", i);
      DTP_CHECK(src[i] != dst[i], DTP_ERR_INVALID_ARG, "weight %d: in-place permutation", i);
    }
    dtp_status st = check_assignment(h, G, L, "h");
    if (st != DTP_OK) return st;
    if ((st = check_assignment(nu, I, L, "nu")) != DTP_OK) return st;
    {
      const size_t hd = (size_t)H * dh, gd = (size_t)G * dh;
      const size_t elems[7] = {hd * dm, gd * dm, gd * dm, (size_t)dm * hd, (size_t)I * dm,
                               (size_t)I * dm, (size_t)dm * I};
      const char* src_names[7] = {"src w_q", "src w_k", "src w_v", "src w_o", "src w_gate",
                                  "src w_up", "src w_down"};
      const char* dst_names[7] = {"dst w_q", "dst w_k", "dst w_v", "dst w_o", "dst w_gate",
                                  "dst w_up", "dst w_down"};
      for (int i = 0; i < 7; ++i) {
        if ((st = check_dev_buffer(src[i], esz * elems[i], src_names[i])) != DTP_OK) return st;
        if ((st = check_dev_buffer(dst[i], esz * elems[i], dst_names[i])) != DTP_OK) return st;
      }
    }
    std::vector<int32_t> ord(G + I);
    orders(G, I, L, h, nu, ord.data(), ord.data() + G);
    hipStream_t s = (hipStream_t)stream;
    int32_t* dord = nullptr;
    DTP_HIP(stream_alloc((void**)&dord, sizeof(int32_t) * (G + I), s));
    hipError_t e = hipMemcpyAsync(dord, ord.data(), sizeof(int32_t) * (G + I), hipMemcpyHostToDevice, s);
    const int32_t* go = dord;
    const int32_t* no = dord + G;
    const int hpg = H / G;
    const int64_t vr = (int64_t)dm * esz / 16;  // 16-byte vectors per row of d elements
    UnitMoves moves{};
    uint32_t blocks = 0;
    auto move = [&](int i, int64_t n_vec, int64_t unit, int n_order, const int32_t* ord_dev) {
      moves.m[moves.n++] = {(const u32x4*)src[i], (u32x4*)dst[i], ord_dev, n_vec, unit, n_order, blocks};
      blocks += (uint32_t)((n_vec + 256 * kMoveVecs - 1) / (256 * kMoveVecs));
    };
    auto rows = [&](int i, int64_t n_rows, int block, const int32_t* ord_dev) {
      move(i, n_rows * vr, block * vr, (int)(n_rows / block), ord_dev);
    };
    auto cols = [&](int i, int64_t n_cols, int block, const int32_t* ord_dev) {
      if (e != hipSuccess) return;
      if (esz == 2)
        permute_cols_kernel<uint16_t><<<grid1((int64_t)dm * n_cols), 256, 0, s>>>(
            (const uint16_t*)src[i], (uint16_t*)dst[i], dm, n_cols, block, ord_dev);
      else
        permute_cols_kernel<float><<<grid1((int64_t)dm * n_cols), 256, 0, s>>>(
            (const float*)src[i], (float*)dst[i], dm, n_cols, block, ord_dev);
      e = hipGetLastError();
    };
    rows(0, (int64_t)H * dh, hpg * dh, go);  // w_q: a group's query heads are one block
    rows(1, (int64_t)G * dh, dh, go);        // w_k
    rows(2, (int64_t)G * dh, dh, go);        // w_v
    rows(4, I, 1, no);                       // w_gate
    rows(5, I, 1, no);                       // w_up
    // w_o columns, like the q rows; in vectors where a group's columns are whole ones
    const int64_t group_bytes = (int64_t)hpg * dh * esz;
    if (group_bytes % 16 == 0)
      move(3, (int64_t)dm * G * (group_bytes / 16), group_bytes / 16, G, go);
    else
      cols(3, (int64_t)H * dh, hpg * dh, go);
    if (e == hipSuccess) {
      permute_units_kernel<<<blocks, 256, 0, s>>>(moves);
      e = hipGetLastError();
    }
    // w_down columns, through LDS where rows are whole vectors and one fits
    const size_t row_bytes = (size_t)I * esz;
    if (e == hipSuccess && row_bytes % 16 == 0 && row_bytes <= kColsLds) {
      const int per = (int)std::min<size_t>(4, kColsLds / row_bytes);
      const unsigned grid = (unsigned)((dm + per - 1) / per);
      if (esz == 2)
        permute_cols_lds_kernel<uint16_t><<<grid, kColsThreads, per * row_bytes, s>>>(
            (const uint16_t*)src[6], (uint16_t*)dst[6], dm, I, per, no);
      else
        permute_cols_lds_kernel<float><<<grid, kColsThreads, per * row_bytes, s>>>((const float*)src[6], (float*)dst[6],
                                                                          dm, I, per, no);
      e = hipGetLastError();
    } else {
      cols(6, I, 1, no);
    }
    const hipError_t ef = stream_free(dord, s);
    DTP_HIP(e);
    DTP_HIP(ef);
    // The order upload reads `ord`, which dies on return.
    DTP_HIP(hipStreamSynchronize(s));
    return DTP_OK;
  });
}

}  // extern "C"
