// btc_pack / btc_unpack: index matrix <-> per-row LSB-first bit stream.
// Integer work only; bit-exact by construction.  (Section "Compression
// Analysis": each length-v vector costs ceil(log2 c) index bits; appendix
// "Binary Codebook LUT-GEMM": index matrix I of shape m x n/v.)
#include <algorithm>

#include "btc_internal.h"

namespace btc {

// A wave per 64 output words of a row.  The codes whose fields overlap them are fetched coalesced, every one of them
// range-checked by the wave that fetches it, and parked in LDS; lane w then gathers the fields of word w.  Bound by
// memory: 28 MB of codes and 7 MB of words on 13824 x 5120 at 8 bits.  (One thread per word straight from memory, with
// its fields 16 bytes apart from the neighbour's, took 14.5 us there.)
constexpr int kPackWaves = 4;
constexpr int kPackFields = 2048 + 2;            // fields that can overlap 64 words (1-bit indices)

template <int FIELDS>
__global__ __launch_bounds__(kPackWaves * 64) void pack_kernel(Dims d, const int32_t* __restrict__ idx,
                                                               uint32_t* __restrict__ packed, uint32_t* __restrict__ host_flag) {
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
    if (bad) *host_flag = 1u;                                                // (pinned host memory)
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
  uint32_t* flag = btc::host_word();
  if (!flag) return BTC_ERR_HIP;
  const btc::Dims d = btc::dims_of(*s);
  const int segments = (d.wpr + 63) / 64;
  if (segments > 65535) return BTC_ERR_UNSUPPORTED;      // (rows of 130 million index bits)
  const dim3 grid((unsigned)std::min((d.out + btc::kPackWaves - 1) / btc::kPackWaves, 65536), (unsigned)segments);
  if (d.b >= 7)      // at most 295 fields overlap 64 words
    btc::pack_kernel<320><<<grid, btc::kPackWaves * 64, 0, q>>>(d, idx, packed, flag);
  else
    btc::pack_kernel<btc::kPackFields><<<grid, btc::kPackWaves * 64, 0, q>>>(d, idx, packed, flag);
  if (btc::launch_status() != BTC_OK) return BTC_ERR_HIP;
  if (hipStreamSynchronize(q) != hipSuccess) return BTC_ERR_HIP;
  return *(volatile uint32_t*)flag ? BTC_ERR_INDEX_RANGE : BTC_OK;
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
