// btc_assign: E-step of the binary codebook clustering (section "Flash and Accurate Binary
// Codebook", step "E-step Assignment"): every +-1 vector of length v goes to its nearest centroid,
//     z_i = argmin_k || b_i - c_k ||^2 = argmin_k 4 d_H(b_i, c_k),   d_H = POPCNT(b_i xor c_k),
// a vector identical to a centroid going to that centroid (distance 0).  Among equally near
// centroids the lowest index wins (the paper leaves ties open; duplicates in the codebook make
// them common).  Integer work, exact.
//
// Two kernels: few different vectors (a table of all 2^v patterns per workgroup), and all pairs on the integer matrix
// cores.
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

// ---- many vectors (N >= 64 * 2^v, v <= 14): there are only 2^v different ones, so every workgroup first makes a table
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
  if (v <= 14 && N >= (64LL << v)) {
    const long long want = (N + 4 * kLutThreads - 1) / (4 * kLutThreads);
    const unsigned grid = (unsigned)(want < 512 ? want : 512);   // two tables per compute unit: 32 waves for the streaming part
    assign_lut_kernel<<<grid, kLutThreads, (size_t)4 << v, (hipStream_t)stream>>>(vectors, (long long)N, v, codebook, K, z, dist2);
    return launch_status();
  }
  const long long per_block = (long long)(kThreads / 64) * 32 * kCols;
  const long long blocks = (N + per_block - 1) / per_block;
  if (blocks > 0x7FFFFFFFLL) return BTC_ERR_SHAPE;
  assign_mfma_kernel<<<(unsigned)blocks, kThreads, 0, (hipStream_t)stream>>>(vectors, (long long)N, v, codebook, K, z, dist2);
  return launch_status();
}

}  // extern "C"
