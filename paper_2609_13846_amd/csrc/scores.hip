// Head step on the GPU (Section 3, "Optimiser"): score every labelled balanced partition
// of a layer's KV groups given the neighbouring neuron assignments.
//
// The objective is linear in h_i once nu_{i-1} and nu_i are fixed, so
//   score(h) = sum_g C[g, h(g)],
//   C[g, l]  = sum_{k: nu_i(k)=l} Q_up_i[g, k] + sum_{k: nu_{i-1}(k)=l} Q_down_{i-1}[k, g].
// All quantities are int64 fixed-point codes, so sums are exact in any order.
//
// Kernels (all over N layers at once):
//   head_gain_kernel      one block per (layer, group): C[g, :] in per-device LDS bins
//   partition_score_kernel one wavefront per (layer, partition): lane g adds C[g, h(g)]
//   best_partition_kernel one block per layer: best score, lowest rank on ties; in the
//                         coordinate ascent also the layer's new h and its part of J
//   layout_value_kernel   each layer's part of J where no layer's heads move
//   neuron_gain_kernel    the gain matrices of the neuron step
//   two_device_kernel     the neuron step for two devices, one block per layer
#include "dtp_internal.h"

namespace dtp {

namespace {

constexpr int kGainThreads = 256;

__device__ inline int64_t wave_sum_i64(int64_t v) {
  for (int off = 32; off > 0; off >>= 1) {
    const int lo = __shfl_xor((int)(uint32_t)(uint64_t)v, off, 64);
    const int hi = __shfl_xor((int)(uint32_t)((uint64_t)v >> 32), off, 64);
    v += (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
  }
  return v;
}

// At most kMaxGainDevices devices: a balanced layout over L devices has at least L!
// labelled partitions (G is a multiple of L), and 11! is beyond what the scoring accepts.
constexpr int kMaxGainDevices = 10;
static_assert(39916800 > kMaxPartitions, "11 devices would need more than 10 device sums");

// C[g, :] of one (layer, group) in one pass over the neurons: each lane keeps one register
// sum per device (DEV >= L of them, selects rather than a branch on the device index, so
// a thread's loads of successive neurons are in flight together), then each sum is added
// across the wavefront and one lane per wavefront adds it to the block's LDS bin.
// Integer sums: exact in any order.  A device index outside [0, L) adds to no sum.
template <int DEV>
__global__ void __launch_bounds__(kGainThreads)
head_gain_kernel(const int64_t* __restrict__ Q_up, const int32_t* __restrict__ nu,
                 const int64_t* __restrict__ Q_down, const int32_t* __restrict__ nu_down,
                 int G, int I, int L, int64_t* __restrict__ C) {
  __shared__ unsigned long long bins[DEV];
  const int layer = blockIdx.x / G;
  const int g = blockIdx.x % G;
  if (threadIdx.x < DEV) bins[threadIdx.x] = 0ull;
  __syncthreads();
  const int64_t* qu = Q_up + ((size_t)layer * G + g) * I;
  const int32_t* nl = nu + (size_t)layer * I;
  const bool down = Q_down != nullptr && layer > 0;
  const int64_t* qd = down ? Q_down + (size_t)(layer - 1) * I * G : nullptr;
  const int32_t* nd = down ? nu_down + (size_t)(layer - 1) * I : nullptr;
  int64_t sum[DEV] = {};
  auto add = [&](int l, int64_t v) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < DEV; ++j) sum[j] += l == j ? v : 0;
  };
#pragma unroll 4
  for (int k = threadIdx.x; k < I; k += kGainThreads) add(nl[k], qu[k]);
  if (down) {
#pragma unroll 4
    for (int k = threadIdx.x; k < I; k += kGainThreads) add(nd[k], qd[(size_t)k * G + g]);
  }
#pragma unroll
  for (int j = 0; j < DEV; ++j) {
    const int64_t t = wave_sum_i64(sum[j]);
    if ((threadIdx.x & 63) == 0) atomicAdd(&bins[j], (unsigned long long)t);
  }
  __syncthreads();
  for (int l = threadIdx.x; l < L; l += kGainThreads)
    C[((size_t)layer * G + g) * L + l] = (int64_t)bins[l];
}

// One wavefront per (layer, partition); lanes index KV groups (G <= 64).
__global__ void __launch_bounds__(256)
partition_score_kernel(const uint8_t* __restrict__ table, const int64_t* __restrict__ C,
                       int N, int G, int L, int64_t P, int64_t* __restrict__ scores) {
  const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wid >= (int64_t)N * P) return;  // whole wavefronts exit together
  const int layer = (int)(wid / P);
  const int64_t p = wid % P;
  int64_t v = 0;
  if (lane < G) {
    const int dev = table[p * G + lane];
    v = C[((size_t)layer * G + lane) * L + dev];
  }
  v = wave_sum_i64(v);
  if (lane == 0) scores[(size_t)layer * P + p] = v;
}

__device__ inline bool better(int64_t s, int64_t r, int64_t bs, int64_t br, int minimise) {
  if (s != bs) return minimise ? (s < bs) : (s > bs);
  return r < br;
}

__global__ void __launch_bounds__(256)
best_partition_kernel(const int64_t* __restrict__ scores, int64_t P, int minimise,
                      int64_t* __restrict__ best, const uint8_t* __restrict__ table, int G,
                      const uint8_t* __restrict__ moves, int32_t* __restrict__ h,
                      int64_t* __restrict__ value) {
  __shared__ int64_t ss[256];
  __shared__ int64_t sr[256];
  const int layer = blockIdx.x;
  const int64_t* sc = scores + (size_t)layer * P;
  int64_t bs = 0, br = -1;
  for (int64_t p = threadIdx.x; p < P; p += blockDim.x) {
    if (br < 0 || better(sc[p], p, bs, br, minimise)) {
      bs = sc[p];
      br = p;
    }
  }
  ss[threadIdx.x] = bs;
  sr[threadIdx.x] = br;
  __syncthreads();
  for (int step = 128; step > 0; step >>= 1) {
    if (threadIdx.x < step) {
      const int o = threadIdx.x + step;
      if (sr[o] >= 0 && (sr[threadIdx.x] < 0 ||
                         better(ss[o], sr[o], ss[threadIdx.x], sr[threadIdx.x], minimise))) {
        ss[threadIdx.x] = ss[o];
        sr[threadIdx.x] = sr[o];
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) best[layer] = sr[0];
  if (h == nullptr) return;
  const bool move = moves[layer] != 0;
  if (threadIdx.x == 0) value[layer] = move ? ss[0] : sc[0];
  if (move && threadIdx.x < G) h[(size_t)layer * G + threadIdx.x] = table[sr[0] * G + threadIdx.x];
}

// Where no layer's heads move, a sweep needs of its head step only each layer's part of J: one
// wavefront per layer, lane g adds C[g, h(g)].  An ascent of 28 layers of 12 groups over 4 devices (369,600 partitions each) takes
// 4.6 ms, and 9.2 where every sweep scores them; 4 layers of 20 groups over 2, 2.1 and 2.9 ms.
__global__ void __launch_bounds__(256)
layout_value_kernel(const int64_t* __restrict__ C, const int32_t* __restrict__ h, int N, int G, int L,
                    int64_t* __restrict__ value) {
  const int layer = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
  if (layer >= N) return;  // whole wavefronts
  int64_t v = 0;
  if (lane < G) v = C[((size_t)layer * G + lane) * L + h[(size_t)layer * G + lane]];
  v = wave_sum_i64(v);
  if (lane == 0) value[layer] = v;
}

// One thread per (layer, neuron): the up codes of a group are contiguous over the neurons, the
// down codes of a neuron over the groups; h is the same for the block.  The matrix is L / (2 G)
// of the codes that it sums, which is what goes to the host's neuron step.
template <int DEV>
__global__ void __launch_bounds__(256)
neuron_gain_kernel(const int64_t* __restrict__ Q_up, const int64_t* __restrict__ Q_down,
                   const int32_t* __restrict__ h, int N, int G, int I, int L, int minimise,
                   int64_t* __restrict__ M) {
  const int layer = blockIdx.y, k = blockIdx.x * 256 + threadIdx.x;
  if (k >= I) return;
  int64_t sum[DEV] = {};
  auto add = [&](int l, int64_t v) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < DEV; ++j) sum[j] += l == j ? v : 0;
  };
  const int64_t* up = Q_up + (size_t)layer * G * I + k;
#pragma unroll 4
  for (int g = 0; g < G; ++g) add(h[(size_t)layer * G + g], up[(size_t)g * I]);
  if (Q_down != nullptr && layer + 1 < N) {
    const int64_t* down = Q_down + ((size_t)layer * I + k) * G;
#pragma unroll 4
    for (int g = 0; g < G; ++g) add(h[(size_t)(layer + 1) * G + g], down[g]);
  }
  int64_t* out = M + ((size_t)layer * I + k) * L;
#pragma unroll
  for (int j = 0; j < DEV; ++j)
    if (j < L) out[j] = minimise ? -sum[j] : sum[j];
}

// The neuron step for two devices, as the host's: with d_k = M[k][0] - M[k][1], device 0 holds the
// neurons above the I/2-th largest value t and, of those at t, the first as many as fit.  One
// block per layer: the keys d + 2^50 (|d| is below 2^50: two matrices' codes sum to 2^48 each)
// in LDS or, for more than kTwoLds of them, in scratch; a radix selection of seven bytes;
// then the ties in index order.  Bound by its chain of barriers: 17 us at G = 8, I = 3072.
// With it the ascent of such a layer takes 135 us instead of 197, most of the difference being
// the copies and the round trip to the host between two sweeps.
constexpr int kTwoThreads = 1024;
constexpr int kTwoLds = 7168;  // keys held in LDS (56 KB)

template <bool LDS>
__global__ void __launch_bounds__(kTwoThreads)
two_device_kernel(const int64_t* __restrict__ Q_up, const int64_t* __restrict__ Q_down,
                  const int32_t* __restrict__ h, const uint8_t* __restrict__ moves, int N, int G, int I,
                  int minimise, uint64_t* __restrict__ scratch, int32_t* __restrict__ nu) {
  extern __shared__ uint64_t lds_keys[];
  __shared__ int hist[256];
  __shared__ int waves[kTwoThreads / 64];
  __shared__ int sel_bin, sel_rank;
  const int layer = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (moves[layer] == 0) return;
  uint64_t* keys = LDS ? lds_keys : scratch + (size_t)layer * I;  // a thread reads its own only
  const int64_t* up = Q_up + (size_t)layer * G * I;
  const bool down = Q_down != nullptr && layer + 1 < N;
  for (int k = tid; k < I; k += kTwoThreads) {
    int64_t d = 0;
#pragma unroll 8
    for (int g = 0; g < G; ++g) {
      const int64_t v = up[(size_t)g * I + k];
      d += h[(size_t)layer * G + g] == 0 ? v : -v;
    }
    if (down) {
      const int64_t* q = Q_down + ((size_t)layer * I + k) * G;
#pragma unroll 8
      for (int g = 0; g < G; ++g) d += h[(size_t)(layer + 1) * G + g] == 0 ? q[g] : -q[g];
    }
    keys[k] = (uint64_t)((minimise ? -d : d) + ((int64_t)1 << 50));
  }
  uint64_t prefix = 0, mask = 0;
  int rank = I / 2;  // of the wanted key among those that match the prefix, from the largest
  for (int shift = 48; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int k0 = 0; k0 < I; k0 += kTwoThreads) {  // whole wavefronts, for the ballots
      const int k = k0 + tid;
      const uint64_t key = k < I ? keys[k] : 0;
      const bool in = k < I && (key & mask) == prefix;
      const int bin = (int)(key >> shift) & 255;
      // The first bytes put most keys into one bin: a wavefront of one bin adds once.
      const uint64_t live = __ballot(in);
      if (live == 0) continue;
      const int first = __shfl(bin, __ffsll((unsigned long long)live) - 1, 64);
      const uint64_t same = __ballot(in && bin == first);
      if (same == live) {
        if (lane == 0) atomicAdd(&hist[first], __popcll(live));
      } else if (in) {
        atomicAdd(&hist[bin], 1);
      }
    }
    __syncthreads();
    if (wave == 0) {  // lane l: bins 255 - 4 l down to 252 - 4 l
      int c[4], sum = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) sum += c[j] = hist[255 - 4 * lane - j];
      int above = sum;
      for (int off = 1; off < 64; off *= 2) {
        const int v = __shfl_up(above, off, 64);
        if (lane >= off) above += v;
      }
      above -= sum;  // keys in the bins of the lanes before
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (above < rank && rank <= above + c[j]) {
          sel_bin = 255 - 4 * lane - j;
          sel_rank = rank - above;
        }
        above += c[j];
      }
    }
    __syncthreads();
    prefix |= (uint64_t)sel_bin << shift;
    mask |= (uint64_t)255 << shift;
    rank = sel_rank;
  }
  // `prefix` is t, and `rank` of the keys at t go to device 0.
  for (int k0 = 0; k0 < I; k0 += kTwoThreads) {
    const int k = k0 + tid;
    const uint64_t key = k < I ? keys[k] : 0;
    const bool tie = k < I && key == prefix;
    const uint64_t ties = __ballot(tie);
    if (lane == 0) waves[wave] = __popcll(ties);
    __syncthreads();
    int before = __popcll(ties & (((uint64_t)1 << lane) - 1)), total = 0;
    for (int w = 0; w < kTwoThreads / 64; ++w) {
      if (w < wave) before += waves[w];
      total += waves[w];
    }
    if (k < I) nu[(size_t)layer * I + k] = key > prefix || (tie && before < rank) ? 0 : 1;
    rank -= total;
    __syncthreads();
  }
}

dtp_status launch_two_device_neurons(const ScoreWorkspace& ws, const int64_t* Q_up, const int64_t* Q_down,
                                     int minimise, const uint8_t* moves, uint64_t* scratch, int32_t* nu,
                                     hipStream_t stream) {
  if (ws.I <= kTwoLds)
    two_device_kernel<true><<<ws.N, kTwoThreads, sizeof(uint64_t) * ws.I, stream>>>(
        Q_up, Q_down, ws.h, moves, ws.N, ws.G, ws.I, minimise, scratch, nu);
  else
    two_device_kernel<false><<<ws.N, kTwoThreads, 0, stream>>>(Q_up, Q_down, ws.h, moves, ws.N, ws.G, ws.I,
                                                               minimise, scratch, nu);
  DTP_HIP(hipGetLastError());
  return DTP_OK;
}

dtp_status launch_neuron_gains(const ScoreWorkspace& ws, const int64_t* Q_up, const int64_t* Q_down,
                               int minimise, int64_t* M, hipStream_t stream) {
  const dim3 grid((ws.I + 255) / 256, ws.N);
  if (ws.L <= 2)
    neuron_gain_kernel<2><<<grid, 256, 0, stream>>>(Q_up, Q_down, ws.h, ws.N, ws.G, ws.I, ws.L, minimise, M);
  else if (ws.L <= 4)
    neuron_gain_kernel<4><<<grid, 256, 0, stream>>>(Q_up, Q_down, ws.h, ws.N, ws.G, ws.I, ws.L, minimise, M);
  else
    neuron_gain_kernel<kMaxAssignDevices><<<grid, 256, 0, stream>>>(Q_up, Q_down, ws.h, ws.N, ws.G, ws.I, ws.L,
                                                                    minimise, M);
  DTP_HIP(hipGetLastError());
  return DTP_OK;
}

}  // namespace

dtp_status score_workspace_create(ScoreWorkspace* ws, int N, int G, int I, int L, hipStream_t s) {
  ws->stream = s;
  ws->N = N;
  ws->G = G;
  ws->I = I;
  ws->L = L;
  ws->P = count_partitions(G, L);
  ws->neuron_gains = launch_neuron_gains;
  ws->two_device_neurons = launch_two_device_neurons;
  DTP_CHECK(ws->P > 0 && ws->P <= kMaxPartitions, DTP_ERR_UNSUPPORTED,
            "%lld partitions of %d groups over %d devices exceed the limit of %lld",
            (long long)ws->P, G, L, (long long)kMaxPartitions);
  ws->host_table = enumerate_partitions(G, L);
  const std::vector<uint8_t>& table = ws->host_table;
  // One allocation: [C | scores | best | table], each part 256-byte aligned.
  auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t c_bytes = up(sizeof(int64_t) * (size_t)N * G * L);
  const size_t s_bytes = up(sizeof(int64_t) * (size_t)N * ws->P);
  const size_t b_bytes = up(sizeof(int64_t) * (size_t)N);
  char* base = nullptr;
  DTP_HIP(stream_alloc((void**)&base, c_bytes + s_bytes + b_bytes + table.size(), s));
  ws->C = (int64_t*)base;
  ws->scores = (int64_t*)(base + c_bytes);
  ws->best = (int64_t*)(base + c_bytes + s_bytes);
  ws->table = (uint8_t*)(base + c_bytes + s_bytes + b_bytes);
  DTP_HIP(hipMemcpyAsync(ws->table, table.data(), table.size(), hipMemcpyHostToDevice, s));
  return DTP_OK;
}

// The host table must outlive its upload: callers synchronise the stream before this.
void score_workspace_destroy(ScoreWorkspace* ws) {
  if (ws->C) (void)stream_free(ws->C, ws->stream);
  *ws = ScoreWorkspace();
}

dtp_status launch_partition_scores(const ScoreWorkspace& ws, const int64_t* Q_up,
                                   const int32_t* nu, const int64_t* Q_down,
                                   const int32_t* nu_down, int minimise, hipStream_t stream) {
  DTP_CHECK(ws.L <= kMaxGainDevices && ws.G <= kMaxGroups, DTP_ERR_UNSUPPORTED,
            "partition scoring supports G <= %d and L <= %d", kMaxGroups, kMaxGainDevices);
  const unsigned gain_blocks = (unsigned)(ws.N * ws.G);
  if (ws.L <= 2)
    head_gain_kernel<2><<<gain_blocks, kGainThreads, 0, stream>>>(Q_up, nu, Q_down, nu_down, ws.G,
                                                                  ws.I, ws.L, ws.C);
  else if (ws.L <= 4)
    head_gain_kernel<4><<<gain_blocks, kGainThreads, 0, stream>>>(Q_up, nu, Q_down, nu_down, ws.G,
                                                                  ws.I, ws.L, ws.C);
  else
    head_gain_kernel<kMaxGainDevices><<<gain_blocks, kGainThreads, 0, stream>>>(
        Q_up, nu, Q_down, nu_down, ws.G, ws.I, ws.L, ws.C);
  DTP_HIP(hipGetLastError());
  if (ws.frozen) {
    layout_value_kernel<<<(unsigned)((ws.N + 3) / 4), 256, 0, stream>>>(ws.C, ws.h, ws.N, ws.G, ws.L, ws.value);
    DTP_HIP(hipGetLastError());
    return DTP_OK;
  }
  const int64_t waves = (int64_t)ws.N * ws.P;
  const int64_t blocks = (waves + 3) / 4;
  partition_score_kernel<<<(unsigned)blocks, 256, 0, stream>>>(ws.table, ws.C, ws.N, ws.G,
                                                               ws.L, ws.P, ws.scores);
  DTP_HIP(hipGetLastError());
  best_partition_kernel<<<ws.N, 256, 0, stream>>>(ws.scores, ws.P, minimise, ws.best, ws.table, ws.G,
                                                  ws.moves, ws.h, ws.value);
  DTP_HIP(hipGetLastError());
  return DTP_OK;
}

}  // namespace dtp
