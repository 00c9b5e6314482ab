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
//   * Otherwise (count_kernel): the counters of four elements are one 64-bit LDS word, so a vector costs an atomic per four
//     elements and one for the member.
// LDS counters have 16 bits (a workgroup sees fewer than 65536 vectors), so that 4096 clusters of v = 16 fit it; when the
// counters of all clusters do not, the clusters are cut into ranges that do, and every range gets its own workgroups,
// which read all the vectors and count only those of their range.  A workgroup ends with an atomic addition to memory per
// non-zero counter, 2.5e11 of them a second on the whole chip: the number of workgroups balances that against the
// vectors (workgroups()).  Pass 2 forms the centroids and clears the counters, so the workspace is left zero-filled for
// the next call.  Integer sums: the result does not depend on the order of the atomics.
// 7.1 M vectors of v = 10, K = 256: pass 1 25.9 us element by element, see the kernel for patterns.  10.2 M vectors of v = 16,
// K = 4096: 84 us (137 us with an atomic per set bit and 32-bit counters in five ranges); what bounds it there are the LDS atomics,
// five per vector (0.64 ns), and the additions at the end.
#include <cmath>
#include <algorithm>

#include "btc_internal.h"

namespace btc {
namespace update {

constexpr int kThreads = 1024;
constexpr int kMaxLdsCounters = 16128;   // 63 KB (pattern_kernel)
constexpr int kMaxLdsBytes = 159 << 10;  // count_kernel

// bits 0 and 1 -> the lowest bits of the two halves of a word
__device__ __forceinline__ uint32_t spread2(uint32_t b) { return __umul24(b, 0x8001u) & 0x10001u; }

// NW = ceil(v / 4) words of four counters per cluster
template <int NW>
__global__ __launch_bounds__(kThreads) void count_kernel(const uint32_t* __restrict__ vectors, const int32_t* __restrict__ z,
                                                        long long N, int v, int K, uint32_t* __restrict__ counts,
                                                        int KR, uint32_t* __restrict__ bad) {
  // [KR][NW] words of four counters, then KR 16-bit counters of the members: clusters k0 .. k0 + KR - 1.  Word w of cluster k
  // stands at place w ^ (k % NW) where NW is a power of two: else one word of all clusters meets few banks.
  extern __shared__ __align__(16) unsigned long long fours[];
  constexpr uint32_t kTurn = (NW & (NW - 1)) == 0 ? NW - 1 : 0;
  uint32_t* const members = (uint32_t*)(fours + (size_t)KR * NW);
  const int W = v + 1;
  const int tid = threadIdx.x;
  const int k0 = blockIdx.y * KR;
  const int kn = min(KR, K - k0);
  const uint32_t mask = v >= 32 ? 0xFFFFFFFFu : ((1u << v) - 1u);
  const long long step = (long long)gridDim.x * kThreads * 4;
  long long i = ((long long)blockIdx.x * kThreads + tid) * 4;
  int4 k4 = make_int4(0, 0, 0, 0);
  uint4 b4 = make_uint4(0u, 0u, 0u, 0u);
  if (i + 3 < N) {
    k4 = *(const int4*)(z + i);
    b4 = *(const uint4*)(vectors + i);
  }
  for (int t = tid; t < KR * NW; t += kThreads) fours[t] = 0ull;
  for (int t = tid; t < (KR + 1) / 2; t += kThreads) members[t] = 0u;
  __syncthreads();
  auto add = [&](int k, uint32_t b) {
    if (k < 0 || k >= K) {                                     // reported by the host after the call; nothing is counted
      *bad = 1u;
      return;
    }
    k -= k0;
    if (k < 0 || k >= kn) return;                              // another range's cluster
    b &= mask;
    const uint32_t row = (uint32_t)(k * NW) | ((uint32_t)k & kTurn);
#pragma unroll
    for (uint32_t w = 0; w < NW; ++w)
      atomicAdd(fours + (kTurn ? row ^ w : row + w),
                (unsigned long long)spread2((b >> (4 * w)) & 15u) | ((unsigned long long)spread2((b >> (4 * w + 2)) & 3u) << 32));
    atomicAdd(members + (k >> 1), 1u << (16 * (k & 1)));
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
  const uint16_t* c16 = (const uint16_t*)fours;
  const uint16_t* m16 = (const uint16_t*)members;
  uint32_t* const mine = counts + (size_t)k0 * W;
  const int total = kn * W;
  const int dk = kThreads / W, de = kThreads - dk * W;         // a thread's next counter is dk clusters and de elements on
  const int first = (int)((long long)total * blockIdx.x / gridDim.x);      // not all workgroups at the same addresses
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    const int end = part == 0 ? total : first;
    int g = (part == 0 ? first : 0) + tid;
    int k = g / W, e = g - k * W;
    while (g < end) {
      uint32_t c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {                            // four LDS reads in flight
        c[u] = g + u * kThreads >= end ? 0u
               : e == v                ? m16[k]
                                       : c16[(((k * NW) | (k & kTurn)) ^ (kTurn ? e >> 2 : 0)) * 4 + (kTurn ? e & 3 : e)];
        k += dk;
        e += de;
        if (e >= W) {
          e -= W;
          ++k;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c[u]) atomicAdd(mine + g + u * kThreads, c[u]);
      g += 4 * kThreads;
    }
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

// Half a wave per cluster: lane t holds the counter of element t, so that the counters are read in one trip (as a loop of
// one thread per cluster: 5.7 us at v = 10, K = 256).  The block that comes last tells the waiting host (waiting for the
// stream instead takes 6 us longer): every block writes its results back before it counts itself in `arrivals`.
__global__ __launch_bounds__(kThreads) void vote_kernel(uint32_t* __restrict__ counts, int v, int K,
                                                       uint32_t* __restrict__ codebook, uint32_t* __restrict__ bad,
                                                       uint32_t* __restrict__ arrivals, uint32_t* __restrict__ host_word) {
  const int t = threadIdx.x & 31, half = threadIdx.x & 32;
  const uint32_t flag = *bad;
  for (int base = blockIdx.x * (kThreads / 32); base < K; base += gridDim.x * (kThreads / 32)) {      // (whole waves)
    const int k = base + (threadIdx.x >> 5);
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
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence_system();
    if (atomicAdd(arrivals, 1u) == gridDim.x - 1) {
      *arrivals = 0u;
      *bad = 0u;
      __threadfence_system();
      __hip_atomic_store(host_word, 1u | (flag << 1), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

template <int NW>
static btc_status launch_count(hipStream_t q, dim3 grid, size_t lds, const uint32_t* vectors, const int32_t* z, long long N,
                               int v, int K, uint32_t* counts, int KR, uint32_t* bad) {
  static bool attr_set = false;  // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)count_kernel<NW>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  count_kernel<NW><<<grid, kThreads, lds, q>>>(vectors, z, N, v, K, counts, KR, bad);
  return launch_status();
}

// Workgroups per range: streaming takes N * per_vector / g nanoseconds, the additions at the end g * K * (v + 1) * 4e-3.
static long long workgroups(long long N, int v, int K, double per_vector) {
  return (long long)std::sqrt((double)N * per_vector / ((double)K * (v + 1) * 4e-3)) + 1;
}

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
  uint32_t* arrivals = bad + 1;
  uint32_t* word = host_word();
  if (!word) return BTC_ERR_HIP;
  // patterns pay once there are several vectors for each of them in a workgroup
  const bool patterns = v <= kMaxPatternBits && N >= (256LL << v);
  const long long want = (N + 4 * kThreads - 1) / (4 * kThreads);
  if (patterns) {
    const int KR = std::min(K, (kMaxLdsCounters - (1 << v)) / (v + 1));   // clusters per range
    const int ranges = (K + KR - 1) / KR;
    long long gx = std::min<long long>(workgroups(N, v, K, 0.5), std::max(256 / ranges, 1));
    gx = std::min<long long>(std::max<long long>(gx, N / 49152 + 1), want);                     // (16-bit counts)
    pattern_kernel<<<dim3((unsigned)gx, (unsigned)ranges), kThreads, (size_t)KR * (v + 1) * 4 + ((size_t)4 << v), q>>>(
        vectors, z, (long long)N, v, K, counts, KR, bad);
  } else {
    const int per_cluster = 8 * ((v + 3) / 4) + 2;
    const int KR = std::min(K, (kMaxLdsBytes - 4) / per_cluster);
    const int ranges = (K + KR - 1) / KR;
    const size_t lds = (size_t)KR * per_cluster + 4;
    long long gx = workgroups(N, v, K, 0.64);
    gx = std::max(gx, std::min<long long>(32, want));
    gx = std::min<long long>(gx, std::max(256 / ranges, 1));
    gx = std::min<long long>(std::max<long long>(gx, N / 61440 + 1), want);                     // (16-bit counts)
    const dim3 grid((unsigned)gx, (unsigned)ranges);
    constexpr decltype(&launch_count<1>) launch[] = {launch_count<1>, launch_count<2>, launch_count<3>, launch_count<4>,
                                                     launch_count<5>, launch_count<6>, launch_count<7>, launch_count<8>};
    if (launch[(v - 1) / 4](q, grid, lds, vectors, z, (long long)N, v, K, counts, KR, bad) != BTC_OK) return BTC_ERR_HIP;
  }
  if (launch_status() != BTC_OK) return BTC_ERR_HIP;
  vote_kernel<<<std::min((K + kThreads / 32 - 1) / (kThreads / 32), 32), kThreads, 0, q>>>(counts, v, K, codebook, bad, arrivals, word);
  if (launch_status() != BTC_OK) return BTC_ERR_HIP;
  // one of the two calls that wait: an assignment outside [0, K) is an error of the caller's data
  return wait_host_word(q, word);
}

}  // extern "C"
