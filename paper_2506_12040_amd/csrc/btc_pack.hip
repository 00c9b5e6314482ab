// btc_pack / btc_unpack: index matrix <-> per-row LSB-first bit stream.
// Integer work only; bit-exact by construction.  (Section "Compression
// Analysis": each length-v vector costs ceil(log2 c) index bits; appendix
// "Binary Codebook LUT-GEMM": index matrix I of shape m x n/v.)
#include <algorithm>
#include <mutex>

#include "btc_internal.h"

namespace btc {

// A wave per 64 output words of a row.  The codes whose fields overlap them are fetched coalesced, every one of them
// range-checked by the wave that fetches it, and parked in LDS; lane w then gathers the fields of word w.  Bound by
// memory: 28 MB of codes and 7 MB of words on 13824 x 5120 at 8 bits.  (One thread per word straight from memory, with
// its fields 16 bytes apart from the neighbour's, took 14.5 us there.)
constexpr int kPackWaves = 4;
constexpr int kPackFields = 2048 + 2;            // fields that can overlap 64 words (1-bit indices)

// Where a call's kernel notes an index out of range, on each device (zero between calls): a word per calling thread.
constexpr int kSlots = 1024;
static __device__ uint32_t bad_index[kSlots];

// The thread's word; threads beyond kSlots - 1 share the last one, under a mutex.
class Slot {
 public:
  Slot() {
    static thread_local Own own;
    if (own.n < 0) shared_ = std::unique_lock<std::mutex>(all().in_use);
    n_ = own.n < 0 ? kSlots - 1 : own.n;
  }
  int n() const { return n_; }

 private:
  struct All {
    std::mutex m, in_use;
    bool taken[kSlots - 1] = {};
  };
  static All& all() {
    static All* a = new All;               // (outlives the threads that give their words back)
    return *a;
  }
  struct Own {
    int n = -1;
    Own() {
      std::lock_guard<std::mutex> lock(all().m);
      bool* end = all().taken + kSlots - 1;
      bool* p = std::find(all().taken, end, false);
      if (p != end) {
        *p = true;
        n = (int)(p - all().taken);
      }
    }
    ~Own() {
      if (n < 0) return;
      std::lock_guard<std::mutex> lock(all().m);
      all().taken[n] = false;
    }
  };
  std::unique_lock<std::mutex> shared_;
  int n_;
};

template <int FIELDS>
__global__ __launch_bounds__(kPackWaves * 64) void pack_kernel(Dims d, const int32_t* __restrict__ idx,
                                                               uint32_t* __restrict__ packed, int slot) {
  __shared__ uint16_t codes[kPackWaves][FIELDS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float per_bit = 1.0f / (float)d.b;
  const int w0 = (int)blockIdx.y << 6;
  const long long bit0 = (long long)w0 * 32;
  const int j0 = (int)(bit0 / d.b);                                          // first field that overlaps the words
  const int j1 = (int)min((long long)d.nchunks, (bit0 + 2048 + d.b - 1) / d.b);     // one past the last
  for (int i = blockIdx.x * kPackWaves + wave; i < d.out; i += gridDim.x * kPackWaves) {
    const int32_t* row = idx + (long long)i * d.nchunks;
    bool bad = false;
    for (int base = j0 + lane; base < j1; base += 5 * 64) {                    // five loads in flight per lane
      int32_t code[5];
#pragma unroll
      for (int u = 0; u < 5; ++u) code[u] = base + 64 * u < j1 ? row[base + 64 * u] : 0;
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        bad |= code[u] < 0 || code[u] >= d.K;
        if (base + 64 * u < j1) codes[wave][base - j0 + 64 * u] = (uint16_t)((uint32_t)code[u] & ((1u << d.b) - 1u));
      }
    }
    if (bad) bad_index[slot] = 1u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();                                         // (LDS operations of a wave complete in order)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int w = w0 + lane;
    if (w < d.wpr) {
      const int lo_bit = 32 * lane + (int)(bit0 - (long long)j0 * d.b);      // of word w, counted from field j0
      uint32_t word = 0u;
      // (lo_bit < 2064: the quotient is exact)
      for (int f = (int)(((float)lo_bit + 0.5f) * per_bit); f < j1 - j0 && f * d.b < lo_bit + 32; ++f) {
        const int start = f * d.b - lo_bit;                                  // may be negative: the field began in word w - 1
        const uint32_t c = codes[wave][f];
        word |= start >= 0 ? (c << start) : (c >> (-start));
      }
      packed[(long long)i * d.wpr + w] = word;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Behind pack_kernel, whose results are in memory when this one starts: tells the waiting host (waiting for the stream
// instead takes 3 us longer).
__global__ void report_kernel(int slot, uint32_t* host_word) {
  const uint32_t bad = bad_index[slot];
  if (bad) bad_index[slot] = 0u;
  __hip_atomic_store(host_word, 1u | (bad << 1), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One thread per index.
__global__ __launch_bounds__(256) void unpack_kernel(Dims d, const uint32_t* __restrict__ packed,
                                                     int32_t* __restrict__ idx) {
  const long long total = (long long)d.out * d.nchunks;
  for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < total;
       g += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(g / d.nchunks);
    const int j = (int)(g - (long long)i * d.nchunks);
    idx[g] = (int32_t)field_at(packed + (long long)i * d.wpr, d.wpr, j * d.b, d.b);
  }
}

static int grid_for(long long total) {
  long long blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  return (int)blocks;
}

}  // namespace btc

extern "C" {

btc_status btc_pack(void* stream, const btc_shape* s, const int32_t* idx, uint32_t* packed,
                    void* workspace, size_t workspace_bytes) {
  btc_status st = btc::check_shape(s);
  if (st != BTC_OK) return st;
  if (!idx || !packed) return BTC_ERR_NULL;
  if (!workspace || workspace_bytes < 16) return BTC_ERR_WORKSPACE;
  if (!btc::aligned16(idx) || !btc::aligned16(packed) || !btc::aligned16(workspace)) return BTC_ERR_ALIGN;
  hipStream_t q = (hipStream_t)stream;
  uint32_t* word = btc::host_word();
  if (!word) return BTC_ERR_HIP;
  const btc::Slot slot;
  const btc::Dims d = btc::dims_of(*s);
  const int segments = (d.wpr + 63) / 64;
  if (segments > 65535) return BTC_ERR_UNSUPPORTED;      // (rows of 130 million index bits)
  const dim3 grid((unsigned)std::min((d.out + btc::kPackWaves - 1) / btc::kPackWaves, 65536), (unsigned)segments);
  if (d.b >= 7)      // at most 295 fields overlap 64 words
    btc::pack_kernel<320><<<grid, btc::kPackWaves * 64, 0, q>>>(d, idx, packed, slot.n());
  else
    btc::pack_kernel<btc::kPackFields><<<grid, btc::kPackWaves * 64, 0, q>>>(d, idx, packed, slot.n());
  if (btc::launch_status() != BTC_OK) return BTC_ERR_HIP;
  btc::report_kernel<<<1, 1, 0, q>>>(slot.n(), word);
  if (btc::launch_status() != BTC_OK) return BTC_ERR_HIP;
  return btc::wait_host_word(q, word);
}

btc_status btc_unpack(void* stream, const btc_shape* s, const uint32_t* packed, int32_t* idx) {
  btc_status st = btc::check_shape(s);
  if (st != BTC_OK) return st;
  if (!idx || !packed) return BTC_ERR_NULL;
  if (!btc::aligned16(idx) || !btc::aligned16(packed)) return BTC_ERR_ALIGN;
  const btc::Dims d = btc::dims_of(*s);
  btc::unpack_kernel<<<btc::grid_for((long long)d.out * d.nchunks), 256, 0, (hipStream_t)stream>>>(d, packed, idx);
  return btc::launch_status();
}

}  // extern "C"
