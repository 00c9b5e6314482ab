// btc_assign: E-step of the binary codebook clustering (section "Flash and Accurate Binary
// Codebook", step "E-step Assignment"): every +-1 vector of length v goes to its nearest centroid,
//     z_i = argmin_k || b_i - c_k ||^2 = argmin_k 4 d_H(b_i, c_k),   d_H = POPCNT(b_i xor c_k),
// a vector identical to a centroid going to that centroid (distance 0).  Among equally near
// centroids the lowest index wins (the paper leaves ties open; duplicates in the codebook make
// them common).  Integer work, exact.
//
// Few different vectors: a table of all 2^v patterns per workgroup (one kernel up to v = 15, one for v = 16).  Otherwise all
// pairs on the integer matrix cores.
#include <algorithm>

#include "btc_internal.h"

namespace btc {
namespace assign {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;

// ---- all pairs.  For +-1 vectors ||b - c||^2 = 2 v - 2 <b, c>, and the inner products of 32 codewords with 32 vectors
// are one MFMA i32 32x32x32 (v <= 32; positions past v are zero).  The codewords enter as +-kA, the vectors as -+kB,
// and the accumulators start at the codeword's number within its block of 32, so a result is the key
//     -kS <b, c> + row,   kS = kA kB > row,
// which orders by distance first and codeword second: no instruction per pair but half a three-way minimum.
// A wave holds kCols blocks of 32 vectors as operands and walks the codebook; a lane turns 16 bits of its codeword into
// an operand (spread over bytes by a 24-bit multiply and a byte permute), shared by the kCols products.  Codewords
// past K repeat the last one: a larger key.  kSeg codewords at a time have keys below kS + .. apart; between segments
// the key goes over into  distance, index.  Measured on 1.0 M vectors of v = 16 against 4096 codewords: see below.
constexpr int kThreads = 256;
constexpr int kCols = 4;                 // blocks of 32 vectors per wave
constexpr int kA = 64, kB = 127, kS = kA * kB;
constexpr int kSeg = 8096;               // codewords per segment: a multiple of 32 below kS

// 16 sign bits -> 16 bytes, bit set => byte 1 of `pair`, else byte 0
__device__ __forceinline__ i32x4 spread16(uint32_t bits, uint32_t pair) {
  i32x4 r;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    r[q] = (int)__builtin_amdgcn_perm(0u, pair, __umul24((bits >> (4 * q)) & 0xFu, 0x204081u) & 0x01010101u);
  return r;
}

__global__ __launch_bounds__(kThreads) void assign_mfma_kernel(const uint32_t* __restrict__ vectors, long long N, int v,
                                                              const uint32_t* __restrict__ codebook, int K,
                                                              int32_t* __restrict__ z, int32_t* __restrict__ dist2) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = threadIdx.x >> 6;
  const long long first = ((long long)blockIdx.x * (kThreads / 64) + wave) * (32 * kCols);
  if (first >= N) return;
  // this lane half's 16 positions: bytes past v are zero in both operands (cleared in the vectors)
  const int keep = min(max(v - 16 * h, 0), 16);
  const uint32_t bytes[4] = {keep >= 4 ? 0xFFFFFFFFu : (1u << (8 * max(keep, 0))) - 1u,
                             keep >= 8 ? 0xFFFFFFFFu : keep > 4 ? (1u << (8 * (keep - 4))) - 1u : 0u,
                             keep >= 12 ? 0xFFFFFFFFu : keep > 8 ? (1u << (8 * (keep - 8))) - 1u : 0u,
                             keep >= 16 ? 0xFFFFFFFFu : keep > 12 ? (1u << (8 * (keep - 12))) - 1u : 0u};
  i32x4 b[kCols];
  int best[kCols], bk[kCols];            // over the finished segments: -<b, c> and the codeword
#pragma unroll
  for (int c = 0; c < kCols; ++c) {
    const long long i = first + 32 * c + l32;
    const uint32_t w = vectors[i < N ? i : N - 1];
    b[c] = spread16(w >> (16 * h), (uint32_t)(uint8_t)kB | ((uint32_t)(uint8_t)(-kB) << 8));   // +1 => -kB
#pragma unroll
    for (int q = 0; q < 4; ++q) b[c][q] &= (int)bytes[q];
    best[c] = 0x7FFFFFFF;
    bk[c] = 0;
  }
  i32x16 rows;                           // the codeword of every accumulator, within a block
#pragma unroll
  for (int e = 0; e < 16; ++e) rows[e] = 8 * (e >> 2) + 4 * h + (e & 3);
  for (int s0 = 0; s0 < K; s0 += kSeg) {
    const int s1 = min(K, s0 + kSeg);
    int m[kCols];
#pragma unroll
    for (int c = 0; c < kCols; ++c) m[c] = 0x7FFFFFFF;
    uint32_t next = codebook[min(s0 + l32, K - 1)];
    for (int k0 = s0; k0 < s1; k0 += 32) {
      const uint32_t w = next;
      next = codebook[min(k0 + 32 + l32, K - 1)];
      const i32x4 a = spread16(w >> (16 * h), (uint32_t)(uint8_t)(-kA) | ((uint32_t)kA << 8));
#pragma unroll
      for (int c = 0; c < kCols; ++c) {
        const i32x16 d = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[c], rows, 0, 0, 0);
        int t = min(min(d[0], d[1]), d[2]);
#pragma unroll
        for (int e = 3; e < 15; e += 2) t = min(min(t, d[e]), d[e + 1]);
        t = min(t, d[15]);
        m[c] = min(m[c], t + (k0 - s0));
      }
    }
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
      const int o = __shfl_xor(m[c], 32, 64);            // the other half of the codewords
      const int key = min(m[c], o);
      const int shifted = key + 32 * kS;                 // >= 0
      const int q = shifted / kS;                        // 32 - <b, c>
      const int k = s0 + (shifted - q * kS);
      if (q < best[c]) {                                 // (an earlier segment wins a tie)
        best[c] = q;
        bk[c] = k;
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kCols; ++c) {
    const long long i = first + 32 * c + l32;
    if (i < N && h == (c & 1)) {
      z[i] = bk[c];
      if (dist2) dist2[i] = 2 * (best[c] - 32 + v);      // 4 d_H = 2 v - 2 <b, c>
    }
  }
}

// ---- short vectors (v <= 15): there are only 2^v different ones, so every workgroup first makes a table
// of all of them -- key  distance << 16 | codeword, the least over the codebook -- and then looks its share of the
// vectors up.  The table is a distance transform over the v-cube: the entries of the codewords start at distance 0, all
// others at infinity, and for every bit the two entries that differ in it exchange  key + (1 << 16):  v steps of 2^(v-1)
// pairs instead of 2^v K pairs (1.0 instead of 6 us at v = 10, K = 256).  After it the call is bound by reading the
// vectors and writing the results.
constexpr int kLutThreads = 1024;

__global__ __launch_bounds__(kLutThreads) void assign_lut_kernel(const uint32_t* __restrict__ vectors, long long N, int v,
                                                                const uint32_t* __restrict__ codebook, int K,
                                                                int32_t* __restrict__ z, int32_t* __restrict__ dist2) {
  extern __shared__ uint32_t table[];                          // [2^v] keys
  const uint32_t mask = (1u << v) - 1u;
  const int tid = threadIdx.x;
  const int P = 1 << v;
  const long long step = (long long)gridDim.x * kLutThreads * 4;
  long long i = ((long long)blockIdx.x * kLutThreads + tid) * 4;
  uint4 w = make_uint4(0u, 0u, 0u, 0u);
  if (i + 3 < N) w = *(const uint4*)(vectors + i);             // (under way while the table is built)
  for (int p = tid; p < P; p += kLutThreads) table[p] = 0x7FFF0000u;
  __syncthreads();
  for (int k = tid; k < K; k += kLutThreads) atomicMin(&table[codebook[k] & mask], (uint32_t)k);
  __syncthreads();
  for (int t = 0; t < v; ++t) {
    const int low = (1 << t) - 1;
    for (int q = tid; q < P / 2; q += kLutThreads) {
      const int p0 = ((q & ~low) << 1) | (q & low), p1 = p0 | (1 << t);
      const uint32_t a = table[p0], b = table[p1];
      table[p0] = min(a, b + (1u << 16));
      table[p1] = min(b, a + (1u << 16));
    }
    __syncthreads();
  }
  for (; i < N; i += step) {
    if (i + 3 < N) {
      const uint4 b = w;
      if (i + step + 3 < N) w = *(const uint4*)(vectors + i + step);
      const uint32_t k0 = table[b.x & mask], k1 = table[b.y & mask], k2 = table[b.z & mask], k3 = table[b.w & mask];
      *(int4*)(z + i) = make_int4((int)(k0 & 0xFFFFu), (int)(k1 & 0xFFFFu), (int)(k2 & 0xFFFFu), (int)(k3 & 0xFFFFu));
      if (dist2)
        *(int4*)(dist2 + i) = make_int4((int)(k0 >> 16) * 4, (int)(k1 >> 16) * 4, (int)(k2 >> 16) * 4, (int)(k3 >> 16) * 4);
    } else {
      for (long long j = i; j < N; ++j) {
        const uint32_t key = table[vectors[j] & mask];
        z[j] = (int32_t)(key & 0xFFFFu);
        if (dist2) dist2[j] = (int32_t)(key >> 16) * 4;
      }
    }
  }
}

// ---- the same for v = 16 and K <= 4096: 65536 keys  distance << ib | codeword  (ib <= 12 index bits) of 16 bits, 128 KB of
// LDS.  A thread takes 64 entries into registers, two to a register, so that five or six of the bits exchange inside a
// thread with saturating packed 16-bit arithmetic; three trips through LDS cover the 16 bits (bit by bit through LDS: 16
// trips).  All ones stands for "further than the key can say": no codebook of 4096 different codewords has such a
// pattern, but one with many duplicates can, and a vector with that pattern is compared with the codebook directly.
// About 9 us for the table on every compute unit; 10.2 M vectors against 4096 codewords: 33 us (1751 us as pairs on
// the matrix cores), 123 MB of it memory; 59 k vectors: 14 us (61 us).
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;

__device__ __forceinline__ uint32_t nearer(uint32_t a, uint32_t b, uint32_t step) {      // min(a, b + step), both halves
  const u16x2 far = __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, b), __builtin_bit_cast(u16x2, step));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), far));
}

// the exchange along bit BIT of the register number
template <int BIT>
__device__ __forceinline__ void exchange(uint32_t (&r)[32], uint32_t step) {
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    if (e & (1 << BIT)) continue;
    const uint32_t a = r[e], b = r[e | (1 << BIT)];
    r[e] = nearer(a, b, step);
    r[e | (1 << BIT)] = nearer(b, a, step);
  }
}

__device__ __forceinline__ void exchange5(uint32_t (&r)[32], uint32_t step) {
  exchange<0>(r, step);
  exchange<1>(r, step);
  exchange<2>(r, step);
  exchange<3>(r, step);
  exchange<4>(r, step);
}

__device__ __noinline__ uint32_t nearest(uint32_t b, const uint32_t* __restrict__ codebook, int K) {
  uint32_t best = 0xFFFFFFFFu;
  for (int k = 0; k < K; ++k) best = min(best, ((uint32_t)__popc((codebook[k] ^ b) & 0xFFFFu) << 16) | (uint32_t)k);
  return best;
}

__global__ __launch_bounds__(kLutThreads) void assign_lut16_kernel(const uint32_t* __restrict__ vectors, long long N,
                                                                  const uint32_t* __restrict__ codebook, int K, int ib,
                                                                  int32_t* __restrict__ z, int32_t* __restrict__ dist2) {
  extern __shared__ __align__(16) uint32_t pairs[];            // [2^15]: patterns 2w (low half) and 2w + 1
  const int tid = threadIdx.x;
  const long long step = (long long)gridDim.x * kLutThreads * 4;
  long long i = ((long long)blockIdx.x * kLutThreads + tid) * 4;
  uint4 w0 = make_uint4(0u, 0u, 0u, 0u), w1 = w0;              // two trips ahead
  if (i + 3 < N) w0 = *(const uint4*)(vectors + i);
  if (i + step + 3 < N) w1 = *(const uint4*)(vectors + i + step);
  uint4* quads = (uint4*)pairs;
#pragma unroll
  for (int j = 0; j < 8; ++j) quads[tid + j * kLutThreads] = make_uint4(~0u, ~0u, ~0u, ~0u);
  __syncthreads();
  for (int k = tid; k < K; k += kLutThreads) {                 // the lowest codeword of a pattern
    const uint32_t p = codebook[k] & 0xFFFFu, sh = (p & 1u) * 16u;
    uint32_t old = pairs[p >> 1];
    while (((old >> sh) & 0xFFFFu) > (uint32_t)k) {
      const uint32_t seen = old;
      old = atomicCAS(&pairs[p >> 1], seen, (seen & ~(0xFFFFu << sh)) | ((uint32_t)k << sh));
      if (old == seen) break;
    }
  }
  __syncthreads();
  const uint32_t one = 0x10001u << ib;
  uint32_t r[32];
  // bits 0..5: a thread's 64 neighbouring entries; quad j ^ (tid % 8) in place j (bank conflicts), which only reflects bits
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint4 t = quads[tid * 8 + (j ^ (tid & 7))];
    r[4 * j] = t.x; r[4 * j + 1] = t.y; r[4 * j + 2] = t.z; r[4 * j + 3] = t.w;
  }
#pragma unroll
  for (int e = 0; e < 32; ++e) r[e] = nearer(r[e], __builtin_amdgcn_alignbit(r[e], r[e], 16), one);
  exchange5(r, one);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    quads[tid * 8 + (j ^ (tid & 7))] = make_uint4(r[4 * j], r[4 * j + 1], r[4 * j + 2], r[4 * j + 3]);
  __syncthreads();
  // bits 6..10, then 11..15
#pragma unroll
  for (int at = 5; at <= 10; at += 5) {
    const int base = (tid & ((1 << at) - 1)) | ((tid >> at) << (at + 5));
#pragma unroll
    for (int e = 0; e < 32; ++e) r[e] = pairs[base + (e << at)];
    exchange5(r, one);
#pragma unroll
    for (int e = 0; e < 32; ++e) pairs[base + (e << at)] = r[e];
    __syncthreads();
  }
  const uint16_t* table = (const uint16_t*)pairs;
  const uint32_t index = (1u << ib) - 1u;
  auto look = [&](uint32_t b, int& k, int& d2) {
    const uint32_t key = table[b & 0xFFFFu];
    k = (int)(key & index);
    d2 = (int)(key >> ib) * 4;
    if (key == 0xFFFFu) {
      const uint32_t best = nearest(b, codebook, K);
      k = (int)(best & 0xFFFFu);
      d2 = (int)(best >> 16) * 4;
    }
  };
  for (; i < N; i += step) {
    if (i + 3 < N) {
      const uint4 b = w0;
      w0 = w1;
      if (i + 2 * step + 3 < N) w1 = *(const uint4*)(vectors + i + 2 * step);
      int4 k, d2;
      look(b.x, k.x, d2.x);
      look(b.y, k.y, d2.y);
      look(b.z, k.z, d2.z);
      look(b.w, k.w, d2.w);
      *(int4*)(z + i) = k;
      if (dist2) *(int4*)(dist2 + i) = d2;
    } else {
      for (long long j = i; j < N; ++j) {
        int k, d2;
        look(vectors[j], k, d2);
        z[j] = k;
        if (dist2) dist2[j] = d2;
      }
    }
  }
}

}  // namespace assign
}  // namespace btc

extern "C" {

btc_status btc_assign(void* stream, const uint32_t* vectors, int64_t N, int32_t v, const uint32_t* codebook,
                      int32_t K, int32_t* z, int32_t* dist2) {
  using namespace btc;
  using namespace btc::assign;
  if (!vectors || !codebook || !z) return BTC_ERR_NULL;
  if (N <= 0) return BTC_ERR_SHAPE;
  if (v < 1 || v > 32 || K < 1 || K > 65536) return BTC_ERR_UNSUPPORTED;
  if (!aligned16(vectors) || !aligned16(codebook) || !aligned16(z) || (dist2 && !aligned16(dist2))) return BTC_ERR_ALIGN;
  // Tables pay when the pairs they replace take longer than making them on every compute unit (microseconds; the matrix
  // cores take 2.4e7 pairs in one, and a wave 60 for its walk through 4096 codewords however few vectors there are).
  const double pairs_us = std::max((double)N * K / 2.4e7, K * (60.0 / 4096));
  const double table_us = v == 16 ? 9.0 : v <= 15 ? 0.7 + 2.4e-5 * v * (1 << v) : 1e30;
  const long long want = (N + 4 * kLutThreads - 1) / (4 * kLutThreads);
  const bool many = pairs_us > table_us;
  if (v <= 15 && many) {
    const unsigned most = v <= 14 ? 512 : 256;     // two tables per compute unit where they fit: 32 waves for the streaming part
    const unsigned grid = (unsigned)(want < most ? want : most);
    static bool attr_set = false;  // one-time kernel attribute, not call state
    if (v > 13 && !attr_set) {
      if (hipFuncSetAttribute((const void*)assign_lut_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 4 << 15) != hipSuccess)
        return BTC_ERR_HIP;
      attr_set = true;
    }
    assign_lut_kernel<<<grid, kLutThreads, (size_t)4 << v, (hipStream_t)stream>>>(vectors, (long long)N, v, codebook, K, z, dist2);
    return launch_status();
  }
  if (v == 16 && K <= 4096 && many) {
    static bool attr_set = false;
    if (!attr_set) {
      if (hipFuncSetAttribute((const void*)assign_lut16_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 2 << 16) != hipSuccess)
        return BTC_ERR_HIP;
      attr_set = true;
    }
    int ib = 1;
    while ((1 << ib) < K) ++ib;
    assign_lut16_kernel<<<(unsigned)(want < 256 ? want : 256), kLutThreads, 2 << 16, (hipStream_t)stream>>>(
        vectors, (long long)N, codebook, K, ib, z, dist2);
    return launch_status();
  }
  const long long per_block = (long long)(kThreads / 64) * 32 * kCols;
  const long long blocks = (N + per_block - 1) / per_block;
  if (blocks > 0x7FFFFFFFLL) return BTC_ERR_SHAPE;
  assign_mfma_kernel<<<(unsigned)blocks, kThreads, 0, (hipStream_t)stream>>>(vectors, (long long)N, v, codebook, K, z, dist2);
  return launch_status();
}

}  // extern "C"
