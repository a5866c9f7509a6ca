// fp32 path of the affinity accumulation (dtype DTP_F32): the decomposition of the bf16
// path (one contraction over [x | a_0 | ... | a_{H-1}] against the folded rows
// [W' | F_0 | ... | F_{H-1}], with epilogues at the operating point and after each head)
// on the fp32 matrix instructions, every product and sum in fp32.
//
// Kernels:
//   fold_f32_kernel      F = W' W_o into the columns d .. d+H*dh of the folded rows
//   affinity_f32_kernel  1/r, operating point, per-head damage and token sums of one tile
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dtp_internal.h"

namespace dtp {
namespace {

constexpr int kFK = 16;          // contraction depth of a stage: d and dh are multiples of it
constexpr int kFRow = kFK + 4;   // floats per LDS row: 16 rows' 16-byte reads cover the 64 banks once
constexpr int kFThreads = 256;
constexpr int kMaxSplitsF32 = 128;  // token splits per launch (size of the partials)
constexpr int kFTile = 64;       // neurons per tile of the folded rows (64 gate rows, then 64 up)

typedef __attribute__((ext_vector_type(4))) float f32x4v;
typedef __attribute__((ext_vector_type(16))) float f32x16v;

// The fp32 matrix instruction of an S x S tile.  Lane l feeds row (column) l % S; its 64 / S
// lane groups hold one contraction element each, so a lane's 16-byte read is four
// instructions' operands: group g takes columns 4 (64 / S) s + 4 g .. + 3 of read s.
template <int S>
struct MfmaF32;

template <>
struct MfmaF32<32> {
  typedef f32x16v Acc;
  static constexpr int kElems = 16;
  __device__ static __forceinline__ Acc run(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int i, int lane) {
    return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
  }
};

template <>
struct MfmaF32<16> {
  typedef f32x4v Acc;
  static constexpr int kElems = 4;
  __device__ static __forceinline__ Acc run(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static __forceinline__ int row(int i, int lane) { return 4 * (lane >> 4) + i; }
};

// wcat[m][d + n] = sum_j wcat[m][j] W_o[j][n] for m < M (a multiple of 64), n < N = H*dh (a
// multiple of 16): a block of 64 x 64 outputs, one 32 x 32 tile per wavefront, the next
// stage fetched during the current one's products.  W_o may have any alignment, so its rows
// come as dwords (64 consecutive ones per wavefront) and stay [k][n] in LDS.  388 -> 29 us
// at d = 512, I = 1536, 8 heads of 64, against one thread per output element.
__global__ void __launch_bounds__(kFThreads)
fold_f32_kernel(float* __restrict__ wcat, const float* __restrict__ w_o, int N, int d, int64_t ld) {
  constexpr int kBRow = 64 + 8;  // the two lane groups read rows 4 apart: 288 floats, other banks
  __shared__ __attribute__((aligned(16))) float As[2][64 * kFRow];
  __shared__ __attribute__((aligned(16))) float Bs[2][kFK * kBRow];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t m0 = (int64_t)blockIdx.x * 64;
  const int n0 = blockIdx.y * 64;
  const int arow = threadIdx.x / 4, acol = 4 * (threadIdx.x % 4);
  const float* ap = wcat + (m0 + arow) * ld + acol;
  const int bn = n0 + lane;
  f32x4v av;
  float bv[4];
  auto fetch = [&](int k0) __attribute__((always_inline)) {
    av = *reinterpret_cast<const f32x4v*>(ap + k0);
#pragma unroll
    for (int j = 0; j < 4; ++j) bv[j] = bn < N ? w_o[(int64_t)(k0 + wave + 4 * j) * N + bn] : 0.0f;
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
    *reinterpret_cast<f32x4v*>(As[buf] + arow * kFRow + acol) = av;
#pragma unroll
    for (int j = 0; j < 4; ++j) Bs[buf][(wave + 4 * j) * kBRow + lane] = bv[j];
  };
  const int wm = wave & 1, wn = wave >> 1, r = lane & 31, grp = lane >> 5;
  f32x16v acc = {};
  fetch(0);
  store(0);
  __syncthreads();
  for (int k0 = 0, buf = 0; k0 < d; k0 += kFK, buf ^= 1) {
    const bool more = k0 + kFK < d;
    if (more) fetch(k0 + kFK);
#pragma unroll
    for (int s = 0; s < kFK / 8; ++s) {
      const f32x4v a = *reinterpret_cast<const f32x4v*>(As[buf] + (32 * wm + r) * kFRow + 8 * s + 4 * grp);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc = MfmaF32<32>::run(a[e], Bs[buf][(8 * s + 4 * grp + e) * kBRow + 32 * wn + r], acc);
    }
    if (more) store(buf ^ 1);
    __syncthreads();
  }
  const int n = n0 + 32 * wn + r;
  if (n < N) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      wcat[(m0 + 32 * wm + MfmaF32<32>::row(i, lane)) * ld + d + n] = acc[i];
  }
}

// One block: 2S tokens x 2S neurons (their gate and up rows), 2 x 2 wavefronts of S x S
// neurons each with a gate and an up accumulator, so both damage terms of a (token,
// neuron) pair sit in one lane.  Stages of 16 contraction columns go through registers into
// a padded LDS double buffer, the next one fetched during the current one's products.
// 1/r needs no pass of its own: the four threads that stage a token row sum its squares, in 64
// bits, since a quarter of a row is a long chain (in 32 the error of A grew by 3 to 5% and that
// of the down statistic by 4 to 8% from d = 2,048 on, against 64 threads per row).
// Bound by the fp32 matrix rate (64 FLOP per clock and SIMD): a stage's operands are 3
// 16-byte LDS reads per 8 instructions.  S = 32 reads each operand half as often from L2;
// S = 16 gives four times the blocks and a quarter of the serial work per tile, for launches
// that would leave CUs without a block.  Measured against one thread per (neuron, token
// lane), whose lanes each walked a weight row of their own: 15,318 -> 140 us at d = 512,
// I = 1536, 8 heads of 64, 2,048 tokens (93 TFLOP/s, matrix cores busy 62% at 2.25 GHz; a large
// fp32 product reaches 154), and with S = 16 52 -> 12 us at d = 64, I = 128, 8 heads of 16, 512
// tokens.  Of that, 180 -> 154 us are three wavefronts per SIMD, so that the 768 blocks run at
// once, and the rest the loops over stages in which nothing but the products touches the
// accumulators (epilogues inside a stage made the compiler copy all 32 in each).
template <int S>
__global__ void __launch_bounds__(kFThreads, 3)
affinity_f32_kernel(AffinityF32Args p) {
  using M = MfmaF32<S>;
  constexpr int kRows = 2 * S;
  constexpr int kBPer = 4 * S * (kFK / 4) / kFThreads;  // weight pieces of 16 bytes per thread
  constexpr int kReads = kFK / (4 * (64 / S));
  __shared__ __attribute__((aligned(16))) float As[2][kRows * kFRow];
  __shared__ __attribute__((aligned(16))) float Bs[2][4 * S * kFRow];
  __shared__ float rv[kRows];   // 1/r of the tile's rows, 0 past T
  __shared__ float rv2[kRows];  // 1/r' (down statistic)
  extern __shared__ float red[];  // [4 wavefronts][G + 1][S]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave & 1, wn = wave >> 1, r = lane % S, grp = lane / S;
  const int G1 = p.G + 1, hpg = p.H / p.G, HD = p.H * p.dh;
  const int group = blockIdx.x / p.splits, split = blockIdx.x % p.splits;
  for (int i = threadIdx.x; i < 4 * G1 * S; i += kFThreads) red[i] = 0.0f;

  // Staging: thread t moves 16-byte piece t % 4 of token row t / 4 and of weight rows t / 4,
  // t / 4 + 64; row R of the stage is the gate row of neuron R for R < 2S, else an up row.
  const int srow = threadIdx.x / 4, scol = 4 * (threadIdx.x % 4);
  const bool stages_tokens = srow < kRows;
  const float* wp[kBPer];
#pragma unroll
  for (int j = 0; j < kBPer; ++j) {
    const int R = srow + 64 * j;
    const int n = group * kRows + R % kRows;
    wp[j] = p.wcat + ((int64_t)(n / kFTile) * 2 * kFTile + (R / kRows) * kFTile + n % kFTile) * p.Kt + scol;
  }
  const int mtiles = (p.T + kRows - 1) / kRows;
  const int per = (mtiles + p.splits - 1) / p.splits;
  const int mt_begin = split * per, mt_end = min(mtiles, mt_begin + per);
  const int nq1 = p.d / kFK, nqh = p.dh / kFK, nq = nq1 + p.H * nqh;

  for (int mt = mt_begin; mt < mt_end; ++mt) {
    const int64_t t = (int64_t)mt * kRows + srow;
    const bool valid = stages_tokens && t < p.T;
    const float* xp = p.x + t * p.d + scol;
    const float* ap = p.attn + t * HD + scol;
    f32x4v av, bv[kBPer];
    double ss = 0.0;
    auto fetch = [&](int q) __attribute__((always_inline)) {
      av = f32x4v{0.0f, 0.0f, 0.0f, 0.0f};
      if (valid) av = *reinterpret_cast<const f32x4v*>(q < nq1 ? xp + q * kFK : ap + (q - nq1) * kFK);
#pragma unroll
      for (int j = 0; j < kBPer; ++j) bv[j] = *reinterpret_cast<const f32x4v*>(wp[j] + q * kFK);
    };
    auto store = [&](int q, bool op) __attribute__((always_inline)) {
      const int buf = q & 1;
      if (stages_tokens) *reinterpret_cast<f32x4v*>(As[buf] + srow * kFRow + scol) = av;
#pragma unroll
      for (int j = 0; j < kBPer; ++j)
        *reinterpret_cast<f32x4v*>(Bs[buf] + (srow + 64 * j) * kFRow + scol) = bv[j];
      if (op) {
        ss += (double)(fmaf(av[0], av[0], av[1] * av[1]) + fmaf(av[2], av[2], av[3] * av[3]));
      }
    };
    typename M::Acc acc[2] = {};
    float c1[M::kElems], c2[M::kElems];
    float colsum = 0.0f;
    fetch(0);
    store(0, true);
    if (p.rinv_next && threadIdx.x < kRows) {
      const int64_t tn = (int64_t)mt * kRows + threadIdx.x;
      rv2[threadIdx.x] = tn < p.T ? p.rinv_next[tn] : 0.0f;
    }
    __syncthreads();
    // Products of stage q while q + 1 is on its way into the other buffer; nothing else in a
    // stage touches the accumulators.
    auto stage = [&](int q, bool op, bool last) __attribute__((always_inline)) {
      const int buf = q & 1;
      if (!last || q + 1 < nq) fetch(q + 1);
      __builtin_amdgcn_sched_barrier(0);  // the loads first: they have the stage to land
#pragma unroll
      for (int s = 0; s < kReads; ++s) {
        const int col = 4 * ((64 / S) * s + grp);
        const f32x4v a = *reinterpret_cast<const f32x4v*>(As[buf] + (S * wm + r) * kFRow + col);
        const f32x4v bg = *reinterpret_cast<const f32x4v*>(Bs[buf] + (S * wn + r) * kFRow + col);
        const f32x4v bu = *reinterpret_cast<const f32x4v*>(Bs[buf] + (kRows + S * wn + r) * kFRow + col);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[0] = M::run(a[e], bg[e], acc[0]);
          acc[1] = M::run(a[e], bu[e], acc[1]);
        }
      }
      if (!last || q + 1 < nq) store(q + 1, op);
      __syncthreads();
    };
    int q = 0;
    for (; q < nq1 - 1; ++q) stage(q, true, false);
    // The row's last columns are in: its four threads are neighbours.
    ss += __shfl_xor(ss, 1, 64);
    ss += __shfl_xor(ss, 2, 64);
    if (stages_tokens && scol == 0) rv[srow] = valid ? (float)(1.0 / sqrt(ss / (double)p.d + (double)p.eps)) : 0.0f;
    stage(q++, false, false);
    // Operating point: c1 = silu'(g) u / r, c2 = silu(g) / r (both 1/r for the ADD score).
    float ds = 0.0f;
#pragma unroll
    for (int i = 0; i < M::kElems; ++i) {
      const int row = S * wm + M::row(i, lane);
      const float ri = rv[row];
      const float g = acc[0][i] * ri, u = acc[1][i] * ri;
      const float sg = 1.0f / (1.0f + expf(-g));
      if (p.rinv_next) {
        const float a = g * sg * u * rv2[row];
        ds = fmaf(a, a, ds);
      }
      c2[i] = p.add ? ri : g * sg * ri;
      c1[i] = p.add ? ri : sg * (1.0f + g * (1.0f - sg)) * u * ri;
    }
    if (p.rinv_next) {
#pragma unroll
      for (int off = S; off < 64; off *= 2) ds += __shfl_xor(ds, off, 64);
      if (lane < S) red[(wave * G1 + p.G) * S + lane] += ds;
    }
    for (int h = 0; h < p.H;) {
      acc[0] = typename M::Acc{};
      acc[1] = typename M::Acc{};
      for (int e = 0; e < nqh; ++e, ++q) stage(q, false, true);
#pragma unroll
      for (int i = 0; i < M::kElems; ++i) {
        const float dg = c1[i] * acc[0][i], du = c2[i] * acc[1][i];
        if (p.add) {
          colsum = fmaf(dg, dg, fmaf(du, du, colsum));
        } else {
          const float dl = dg + du;
          colsum = fmaf(dl, dl, colsum);
        }
      }
      if (++h % hpg == 0) {  // last query head of its KV group
#pragma unroll
        for (int off = S; off < 64; off *= 2) colsum += __shfl_xor(colsum, off, 64);
        if (lane < S) red[(wave * G1 + h / hpg - 1) * S + lane] += colsum;
        colsum = 0.0f;
      }
    }
  }
  __syncthreads();  // a split past the last tile ran none of the loop's barriers
  for (int i = threadIdx.x; i < G1 * kRows; i += kFThreads) {
    const int g = i / kRows, nl = i % kRows;
    const int w = 2 * (nl / S), k = nl % S;
    const float sum = red[(w * G1 + g) * S + k] + red[((w + 1) * G1 + g) * S + k];
    const int n = group * kRows + nl;
    p.partial[((int64_t)split * G1 + g) * p.I_pad + n] = g < p.G && !p.add ? sum * p.nd[n] : sum;
  }
}

// Token splits of a launch of `groups` neuron groups x `mtiles` token tiles.  Blocks of equal
// length run in rounds of one per CU (several share a CU, and its matrix cores), a block
// taking up to ceil(mtiles / S) tiles: the launch lasts about ceil(groups * S / CUs) *
// ceil(mtiles / S) tile times.  From the smallest count that gives each CU three blocks, up
// to four times it, the first that minimises that product.
int choose_splits(int groups, int mtiles, int64_t cus) {
  const int cap = std::min(mtiles, kMaxSplitsF32);
  const int lo = std::max(1, std::min((int)((3 * cus + groups - 1) / groups), cap));
  int best = lo;
  int64_t best_cost = -1;
  for (int s = lo; s <= std::min(4 * lo, cap); ++s) {
    const int64_t rounds = ((int64_t)groups * s + cus - 1) / cus;
    const int64_t cost = rounds * ((mtiles + s - 1) / s);
    if (best_cost < 0 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

template <int S>
int launch_affinity_f32_tiles(AffinityF32Args p, int cus, hipStream_t s) {
  const int groups = p.I_pad / (2 * S);
  p.splits = choose_splits(groups, (p.T + 2 * S - 1) / (2 * S), cus);
  const size_t shm = sizeof(float) * 4 * (p.G + 1) * S;
  affinity_f32_kernel<S><<<groups * p.splits, kFThreads, shm, s>>>(p);
  return p.splits;
}

}  // namespace

void launch_fold_f32(float* wcat, const float* w_o, int rows, int N, int d, int64_t ld, hipStream_t s) {
  fold_f32_kernel<<<dim3(rows / 64, (N + 63) / 64), kFThreads, 0, s>>>(wcat, w_o, N, d, ld);
}

int launch_affinity_f32(const AffinityF32Args& p, int cus, hipStream_t s) {
  const int64_t tiles = (int64_t)(p.I_pad / 64) * ((p.T + 63) / 64);
  return tiles < cus ? launch_affinity_f32_tiles<16>(p, cus, s) : launch_affinity_f32_tiles<32>(p, cus, s);
}

}  // namespace dtp
