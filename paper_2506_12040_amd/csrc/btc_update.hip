// btc_update: M-step of the binary codebook clustering (section "Flash and Accurate Binary
// Codebook", step "M-step Centroid Update"; the loop over clusters in the algorithm of appendix
// "Binary Codebook Optimization"):  c_k = sign(mean of the vectors assigned to k), a zero mean
// giving +1; a cluster without members keeps its centroid.  Integer work, exact.
//
// Element t of the new centroid is +1 iff  2 * (members with element t = +1) >= members.  So the
// call counts, per cluster, its members and the +1s of every element: v + 1 counters per cluster
// in the caller's workspace.  Pass 1: a workgroup adds up its share of the vectors in an LDS copy
// of the counters and then adds its non-zero counters to the workspace.
//   * Short vectors (v <= 12, pattern_kernel): there are 2^v different vectors, and an E-step sends equal vectors to the
//     same cluster, so a workgroup counts patterns: one word per pattern holds the cluster of the first vector with that
//     pattern and the number of its vectors there -- one LDS read and one LDS atomic per vector instead of an atomic
//     per set bit.  A vector whose cluster is another one (any assignment is allowed) is counted element by element.
//     At the end the patterns are added to the counters.
//   * Otherwise (count_kernel): one LDS atomic per set bit and one per vector.
// When the counters of all clusters do not fit LDS (more than 16128) the clusters are cut into ranges that do, and
// every range gets its own workgroups, which read all the vectors and count only those of their range: re-reading 8
// bytes per vector is far cheaper than atomics that go to memory.  Pass 2: one thread per cluster forms the centroid
// and clears its counters, so the workspace is left zero-filled for the next call.  Integer sums: the result does not
// depend on the order of the atomics.
// 7.1 M vectors of v = 10, K = 256: pass 1 25.9 us element by element, see the kernel for patterns.
#include <algorithm>

#include "btc_internal.h"

namespace btc {
namespace update {

constexpr int kThreads = 1024;
constexpr int kMaxLdsCounters = 16128;   // 63 KB

__global__ __launch_bounds__(kThreads) void count_kernel(const uint32_t* __restrict__ vectors, const int32_t* __restrict__ z,
                                                        long long N, int v, int K, uint32_t* __restrict__ counts,
                                                        int KR, uint32_t* __restrict__ bad) {
  extern __shared__ uint32_t local[];                          // [KR][v + 1]: clusters k0 .. k0 + KR - 1
  const int W = v + 1;
  const int tid = threadIdx.x;
  const int k0 = blockIdx.y * KR;
  const int kn = min(KR, K - k0);
  for (int t = tid; t < kn * W; t += kThreads) local[t] = 0u;
  __syncthreads();
  const long long step = (long long)gridDim.x * kThreads;
  for (long long i = (long long)blockIdx.x * kThreads + tid; i < N; i += step) {
    const int k = z[i];
    if (k < 0 || k >= K) {                                     // reported by the host after the call; nothing is counted
      *bad = 1u;
      continue;
    }
    if (k < k0 || k >= k0 + kn) continue;                      // another range's cluster
    uint32_t b = vectors[i] & (v >= 32 ? 0xFFFFFFFFu : ((1u << v) - 1u));
    uint32_t* row = local + (size_t)(k - k0) * W;
    atomicAdd(row + v, 1u);
    while (b) {
      const int t = __builtin_ctz(b);
      b &= b - 1u;
      atomicAdd(row + t, 1u);
    }
  }
  __syncthreads();
  for (int t = tid; t < kn * W; t += kThreads) {
    const uint32_t c = local[t];
    if (c) atomicAdd(counts + (size_t)k0 * W + t, c);
  }
}

constexpr int kMaxPatternBits = 12;

// (a vector read and its cluster: 57 MB for 7.1 M vectors, 12 us at the rate of a copy)
__global__ __launch_bounds__(kThreads) void pattern_kernel(const uint32_t* __restrict__ vectors, const int32_t* __restrict__ z,
                                                          long long N, int v, int K, uint32_t* __restrict__ counts,
                                                          int KR, uint32_t* __restrict__ bad) {
  extern __shared__ uint32_t local[];                          // [KR][v + 1] counters, then a word per pattern
  const int W = v + 1;
  const int tid = threadIdx.x;
  const int k0 = blockIdx.y * KR;
  const int kn = min(KR, K - k0);
  const uint32_t mask = (1u << v) - 1u;
  uint32_t* const pat = local + KR * W;                        // cluster + 1 in the high half, vectors in the low half
  const long long step = (long long)gridDim.x * kThreads * 4;
  long long i = ((long long)blockIdx.x * kThreads + tid) * 4;
  int4 k4 = make_int4(0, 0, 0, 0);
  uint4 b4 = make_uint4(0u, 0u, 0u, 0u);
  if (i + 3 < N) {
    k4 = *(const int4*)(z + i);
    b4 = *(const uint4*)(vectors + i);
  }
  for (int t = tid; t < kn * W; t += kThreads) local[t] = 0u;
  for (int p = tid; p <= (int)mask; p += kThreads) pat[p] = 0u;
  __syncthreads();
  auto add = [&](int k, uint32_t b) {
    if (k < 0 || k >= K) {                                     // reported by the host after the call; nothing is counted
      *bad = 1u;
      return;
    }
    if (k < k0 || k >= k0 + kn) return;                        // another range's cluster
    b &= mask;
    uint32_t owner = pat[b] >> 16;
    const uint32_t own = (uint32_t)(k - k0) + 1u;              // (KR <= 8064)
    if (owner == 0u) {                                         // the first vector with this pattern, unless another thread is faster
      owner = atomicCAS(&pat[b], 0u, own << 16) >> 16;
      if (owner == 0u) owner = own;
    }
    if (owner == own) {
      atomicAdd(&pat[b], 1u);                                  // (a workgroup sees fewer than 65536 vectors)
      return;
    }
    uint32_t* row = local + (size_t)(k - k0) * W;
    atomicAdd(row + v, 1u);
    while (b) {
      const int t = __builtin_ctz(b);
      b &= b - 1u;
      atomicAdd(row + t, 1u);
    }
  };
  for (; i < N; i += step) {
    if (i + 3 < N) {
      const int4 k = k4;
      const uint4 b = b4;
      if (i + step + 3 < N) {                                  // the next ones are under way
        k4 = *(const int4*)(z + i + step);
        b4 = *(const uint4*)(vectors + i + step);
      }
      add(k.x, b.x);
      add(k.y, b.y);
      add(k.z, b.z);
      add(k.w, b.w);
    } else {
      for (long long j = i; j < N; ++j) add(z[j], vectors[j]);
    }
  }
  __syncthreads();
  for (int p = tid; p <= (int)mask; p += kThreads) {
    const uint32_t n = pat[p] & 0xFFFFu;
    if (n == 0u) continue;
    uint32_t* row = local + (size_t)((pat[p] >> 16) - 1u) * W;
    atomicAdd(row + v, n);
    for (uint32_t b = (uint32_t)p; b; b &= b - 1u) atomicAdd(row + __builtin_ctz(b), n);
  }
  __syncthreads();
  for (int t = tid; t < kn * W; t += kThreads) {
    const uint32_t c = local[t];
    if (c) atomicAdd(counts + (size_t)k0 * W + t, c);
  }
}

// A wave per 64 / 32 = two clusters: lane t of a half holds the counter of element t, so that the counters are read in one
// trip (as a loop of one thread per cluster: 5.7 us at v = 10, K = 256).
__global__ __launch_bounds__(256) void vote_kernel(uint32_t* __restrict__ counts, int v, int K,
                                                  uint32_t* __restrict__ codebook, uint32_t* __restrict__ bad,
                                                  uint32_t* __restrict__ host_flag) {
  const int k = blockIdx.x * 8 + (threadIdx.x >> 5), t = threadIdx.x & 31, half = threadIdx.x & 32;
  const uint32_t flag = *bad;
  if (k == 0 && t == 0) *host_flag = flag;                     // (pinned host memory)
  const bool have = k < K;
  uint32_t* row = counts + (size_t)(have ? k : 0) * (v + 1);
  const uint32_t members = have ? row[v] : 0u;
  const bool mine = have && t < v;
  const uint32_t ones = mine ? row[t] : 0u;
  const unsigned long long ballot = __ballot(mine && 2u * ones >= members);      // sum of +-1 >= 0
  if (mine) row[t] = 0u;
  if (have && t == 0) {
    row[v] = 0u;
    if (members != 0u && flag == 0u) codebook[k] = (uint32_t)(ballot >> half);
  }
}

__global__ void clear_word_kernel(uint32_t* word) { *word = 0u; }

}  // namespace update
}  // namespace btc

extern "C" {

size_t btc_update_workspace_bytes(int32_t v, int32_t K) {
  if (v < 1 || v > 32 || K < 1 || K > 65536) return 0;
  return ((size_t)K * (size_t)(v + 1) * 4 + 16 + 15) & ~(size_t)15;   // the counters and an error flag
}

btc_status btc_update(void* stream, const uint32_t* vectors, const int32_t* z, int64_t N, int32_t v,
                      uint32_t* codebook, int32_t K, void* workspace, size_t workspace_bytes) {
  using namespace btc;
  using namespace btc::update;
  if (!vectors || !z || !codebook) return BTC_ERR_NULL;
  if (N <= 0) return BTC_ERR_SHAPE;
  if (v < 1 || v > 32 || K < 1 || K > 65536) return BTC_ERR_UNSUPPORTED;
  if (N >= (1LL << 31)) return BTC_ERR_UNSUPPORTED;            // 32-bit counters
  if (!workspace || workspace_bytes < btc_update_workspace_bytes(v, K)) return BTC_ERR_WORKSPACE;
  if (!aligned16(vectors) || !aligned16(z) || !aligned16(codebook) || !aligned16(workspace)) return BTC_ERR_ALIGN;
  hipStream_t q = (hipStream_t)stream;
  uint32_t* counts = (uint32_t*)workspace;
  const size_t n_counters = (size_t)K * (size_t)(v + 1);
  uint32_t* bad = counts + ((n_counters + 3) & ~(size_t)3);
  uint32_t* host_flag = host_word();
  if (!host_flag) return BTC_ERR_HIP;
  // patterns pay once there are several vectors for each of them in a workgroup
  const bool patterns = v <= kMaxPatternBits && N >= (256LL << v);
  const int KR = std::min(K, (kMaxLdsCounters - (patterns ? 1 << v : 0)) / (v + 1));   // clusters per range
  const int ranges = (K + KR - 1) / KR;
  long long want = (N + kThreads - 1) / kThreads;
  // about two workgroups per compute unit in all; one for patterns (a workgroup ends with an atomic addition to memory
  // per counter: at 512 workgroups those take longer than the vectors)
  long long gx = (patterns ? 256 : 512) / ranges;
  if (patterns) gx = std::max<long long>(gx, N / 49152 + 1);              // (16-bit counts)
  if (gx < 1) gx = 1;
  if (gx > want) gx = want;
  const size_t lds = (size_t)KR * (v + 1) * 4;
  if (patterns)
    pattern_kernel<<<dim3((unsigned)gx, (unsigned)ranges), kThreads, lds + ((size_t)4 << v), q>>>(vectors, z, (long long)N, v,
                                                                                                 K, counts, KR, bad);
  else
    count_kernel<<<dim3((unsigned)gx, (unsigned)ranges), kThreads, lds, q>>>(vectors, z, (long long)N, v, K, counts, KR, bad);
  if (launch_status() != BTC_OK) return BTC_ERR_HIP;
  vote_kernel<<<(K + 7) / 8, 256, 0, q>>>(counts, v, K, codebook, bad, host_flag);
  if (launch_status() != BTC_OK) return BTC_ERR_HIP;
  // one of the two calls that wait: an assignment outside [0, K) is an error of the caller's data
  if (hipStreamSynchronize(q) != hipSuccess) return BTC_ERR_HIP;
  const uint32_t flag = *(volatile uint32_t*)host_flag;
  if (flag) {
    clear_word_kernel<<<1, 1, 0, q>>>(bad);                     // the workspace is handed back zero-filled
    return BTC_ERR_INDEX_RANGE;
  }
  return BTC_OK;
}

}  // extern "C"
