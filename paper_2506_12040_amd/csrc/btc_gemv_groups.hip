// Decode-time product for the storage variant with several (alpha, mu) pairs per weight row (Table "Study
// of Number of Split Points"; appendix hyper-parameters: 2 split points by default, 3 for higher accuracy):
//   W_hat[i][k] = alpha[i][g] * B_hat[i][k] + mu[i][g],   g = group[i][k] in [0, G),  G <= 4
//   y[i] = sum_g ( alpha[i][g] * sum_{k in g} B_hat[i][k] x[k]  +  mu[i][g] * sum_{k in g} x[k] )
// The partition is an explicit map of 2 bits per weight (bits [2k, 2k+2) of row i's map, LSB-first like the
// index stream, ceil(2 in / 32) words per row): three times the bytes of a 0.8-bit index stream.
//
// Chunk lengths 9 and 10 with up to 10 index bits (gemv_groups_pairs_kernel): the 64 combinations of signs and groups
// that two neighbouring weights can have give 64 pairs of weight values per row, so a wave writes its row's table into
// LDS -- each value as two fp16 parts of a number scaled by a power of two (22 bits) -- and a pair of weights costs one
// 8-byte table read and two packed dot products (fp32), whatever the number of groups.  Lane l takes the chunks l, l +
// 64, ..; the activations of a chunk are read once for the R rows of a wave; a lane's index and map fields sit at bit
// positions that do not depend on the slot, inside an 8-byte window each, requested one slot ahead.  Per chunk and row
// about 40 vector instructions and 41 LDS clocks bound it: 13.3 us on 13824 x 5120 with three groups, 51 with the kernel
// below, 20 with a table of memberships and two dot products per group; the bytes (25 MB) need 5.4 us.
// Every other setting (gemv_groups_kernel): a wave per row, per weight a sign select and two fused multiply-adds per
// group with a 0 / 1 factor (branch-free); fp32 sums, fixed order.
#include <hip/hip_fp16.h>

#include <algorithm>

#include "btc_internal.h"

namespace btc {
namespace groups {

constexpr int kWaves = 16;
constexpr int kMaxIn = 32768;           // activation row in LDS: 64 KB
constexpr int kCodebookLds = 8192;      // codebook entries held in LDS (32 KB)

__device__ __forceinline__ float wave_sum(float a) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
  return a;
}

template <int G, bool CB_LDS>
__global__ __launch_bounds__(kWaves * 64) void gemv_groups_kernel(Dims d, const uint32_t* __restrict__ packed,
                                                                  const uint32_t* __restrict__ codebook,
                                                                  const float* __restrict__ alpha,
                                                                  const float* __restrict__ mu,
                                                                  const uint32_t* __restrict__ gmap,
                                                                  const uint16_t* __restrict__ x, void* __restrict__ y,
                                                                  int y_is_f32) {
  extern __shared__ __align__(16) unsigned char smem[];
  __half* xs = (__half*)smem;                            // [in]
  uint32_t* cb = (uint32_t*)(smem + (((size_t)d.in * 2 + 15) & ~(size_t)15));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int k = tid; k < d.in; k += kWaves * 64) xs[k] = __builtin_bit_cast(__half, x[k]);
  if (CB_LDS)
    for (int k = tid; k < (1 << d.b); k += kWaves * 64) cb[k] = codebook[k];
  __syncthreads();
  const uint32_t mask = (1u << d.b) - 1u;
  const int gwpr = (2 * d.in + 31) >> 5;
  for (int i = blockIdx.x * kWaves + wave; i < d.out; i += gridDim.x * kWaves) {
    const uint32_t* row = packed + (size_t)i * d.wpr;
    const uint32_t* grow = gmap + (size_t)i * gwpr;
    float acc[G], sx[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = sx[g] = 0.f;
    for (int j = lane; j < d.nchunks; j += 64) {
      const uint32_t p = (uint32_t)j * (uint32_t)d.b;
      const uint32_t w = p >> 5, sh = p & 31u;
      const uint32_t lo = row[w];
      const uint32_t hi = (sh + d.b > 32u) ? row[w + 1] : 0u;   // inside the row whenever the field crosses
      const uint32_t code = __builtin_amdgcn_alignbit(hi, lo, sh) & mask;
      const uint32_t pat = CB_LDS ? cb[code] : codebook[code];
      const int k0 = j * d.v;
      const int len = min(d.v, d.in - k0);
      // the 2 * len <= 64 map bits of the chunk: three words cover them whatever the alignment
      const int gw = (2 * k0) >> 5;
      const uint32_t gs = (uint32_t)(2 * k0) & 31u;
      const uint32_t g0 = grow[gw];
      const uint32_t g1 = gw + 1 < gwpr ? grow[gw + 1] : 0u;
      const uint32_t g2 = gw + 2 < gwpr ? grow[gw + 2] : 0u;
      const uint32_t mlo = __builtin_amdgcn_alignbit(g1, g0, gs), mhi = __builtin_amdgcn_alignbit(g2, g1, gs);
      for (int t = 0; t < len; ++t) {
        const float xv = __half2float(xs[k0 + t]);
        const float sv = ((pat >> t) & 1u) ? xv : -xv;
        const uint32_t gi = ((t < 16 ? mlo : mhi) >> (2 * (t & 15))) & 3u;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float on = gi == (uint32_t)g ? 1.0f : 0.0f;
          acc[g] = fmaf(on, sv, acc[g]);
          sx[g] = fmaf(on, xv, sx[g]);
        }
      }
    }
    float r = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float a = wave_sum(acc[g]), sxx = wave_sum(sx[g]);
      r += alpha[(size_t)i * G + g] * a + mu[(size_t)i * G + g] * sxx;
    }
    if (lane == 0) {
      if (y_is_f32) ((float*)y)[i] = r;
      else ((__half*)y)[i] = __float2half_rn(r);
    }
  }
}

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
constexpr int kPairWaves = 4;
constexpr int kRsrcFlags = 0x00020000;

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b), c, false);
}
__device__ __forceinline__ uint32_t half_bits(float v) { return (uint32_t)__builtin_bit_cast(uint16_t, __float2half_rn(v)); }

// bytes of LDS: row tables (512 per row of a wave), sign fields (4 per codeword), activations (16 + 4 per chunk slot)
static size_t pairs_lds_bytes(const Dims& d, int R) {
  return (size_t)kPairWaves * R * 512 + ((size_t)4 << d.b) + (size_t)((d.nchunks + 63) & ~63) * 20;
}

template <int G, int R>
__global__ __launch_bounds__(kPairWaves * 64, 7) void gemv_groups_pairs_kernel(
    Dims d, const uint32_t* __restrict__ packed, const uint32_t* __restrict__ codebook, const float* __restrict__ alpha,
    const float* __restrict__ mu, const uint32_t* __restrict__ gmap, const uint16_t* __restrict__ x, void* __restrict__ y,
    int y_is_f32) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kRows = kPairWaves * R * 512;
  const int slots = (d.nchunks + 63) >> 6, nc = slots << 6;
  uint32_t* const sf = (uint32_t*)(smem + kRows);        // sign fields of a codeword: pair t in bits 6 t, 6 t + 1
  u32x4* const xa = (u32x4*)(sf + ((size_t)1 << d.b));   // pairs 0..3 of a chunk of activations
  uint32_t* const xb = (uint32_t*)(xa + nc);             // pair 4
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mw = (2 * d.in + 31) >> 5;                   // words of a row's map
  const __amdgpu_buffer_rsrc_t rP =
      __builtin_amdgcn_make_buffer_rsrc((void*)packed, 0, (int)((uint32_t)d.out * (uint32_t)d.wpr * 4u), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rM =
      __builtin_amdgcn_make_buffer_rsrc((void*)gmap, 0, (int)((uint32_t)d.out * (uint32_t)mw * 4u), kRsrcFlags);
  // this lane's fields of slot s: 64 chunks further on are 2 b and 4 v whole words further on
  const uint32_t pbit = (uint32_t)(lane * d.b), mbit = (uint32_t)(lane * 2 * d.v);
  const uint32_t psh = pbit & 31u, msh = mbit & 31u;
  const int units = (d.out + R - 1) / R;
  int q = blockIdx.x * kPairWaves + wave;
  u32x2 pw[R], mp[R];
  uint32_t poff[R], moff[R];
  float al[R][G], mn[R][G];                              // of the rows of this wave (every lane)
  auto begin = [&]() {                                   // (rows past the end: zeros from past the end of the buffers)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      poff[r] = (uint32_t)(q * R + r) * (uint32_t)d.wpr * 4u + (pbit >> 5) * 4u;
      moff[r] = (uint32_t)(q * R + r) * (uint32_t)mw * 4u + (mbit >> 5) * 4u;
      const int i = min(q * R + r, d.out - 1);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        al[r][g] = alpha[(size_t)i * G + g];
        mn[r][g] = mu[(size_t)i * G + g];
      }
    }
  };
  auto fetch = [&]() {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      pw[r] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rP, poff[r], 0, 0));
      mp[r] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rM, moff[r], 0, 0));
      poff[r] += (uint32_t)(8 * d.b);
      moff[r] += (uint32_t)(16 * d.v);
    }
  };
  begin();
  fetch();
  // ---- sign fields and activations
  for (int c = tid; c < nc; c += kPairWaves * 64) {
    uint32_t w[5] = {0u, 0u, 0u, 0u, 0u};
    const int k0 = c * d.v;
    if (d.v == 10 && (d.in & 1) == 0 && k0 + 10 <= d.in) {               // 20 bytes at 4-byte alignment
#pragma unroll
      for (int t = 0; t < 5; ++t) w[t] = ((const uint32_t*)x)[5 * c + t];
    } else {
#pragma unroll
      for (int t = 0; t < 10; ++t)                       // zero past the row, in the surplus slot of v = 9, in phantom chunks
        if (t < d.v && k0 + t < d.in) w[t >> 1] |= (uint32_t)x[k0 + t] << (16 * (t & 1));
    }
    xa[c] = u32x4{w[0], w[1], w[2], w[3]};
    xb[c] = w[4];
  }
  for (int k = tid; k < (1 << d.b); k += kPairWaves * 64) {
    const uint32_t n = codebook[k];
    uint32_t w = 0u;
#pragma unroll
    for (int t = 0; t < 5; ++t) w |= ((n >> (2 * t)) & 3u) << (6 * t);
    sf[k] = w;
  }
  __syncthreads();
  const uint32_t imask = (1u << d.b) - 1u;
  // LDS addresses as numbers (LDS starts at this array, at address 0): the compiler adds the array's base to every
  // access otherwise
  const uint32_t rows = (uint32_t)(uintptr_t)(lds_u8*)smem + (uint32_t)(wave * R * 512);
  const uint32_t signs = (uint32_t)(uintptr_t)(lds_u8*)smem + kRows;
  while (q < units) {
    // ---- the table of each row: entry s0 + 2 s1 + 4 g0 + 16 g1 = the values of two weights with signs s0, s1 in groups g0, g1
    float scale[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float top = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g) top = fmaxf(top, fabsf(al[r][g]) + fabsf(mn[r][g]));
      // a power of two that brings the largest value into [1, 2) (exponents at the ends of the range: clamped)
      const int e = min(max((int)(__float_as_uint(top) >> 23), 2), 252);
      const float up = __uint_as_float((uint32_t)(254 - e) << 23);
      scale[r] = __uint_as_float((uint32_t)e << 23);
      float v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int g = (lane >> (2 + 2 * h)) & 3;
        float a = al[r][0], m = mn[r][0];
#pragma unroll
        for (int k = 1; k < G; ++k)
          if (g == k) { a = al[r][k]; m = mn[r][k]; }
        v[h] = (((lane >> h) & 1) ? m + a : m - a) * up;
      }
      const uint32_t h0 = half_bits(v[0]), h1 = half_bits(v[1]);
      const float l0 = (v[0] - __half2float(__ushort_as_half((uint16_t)h0))) * 2048.f;
      const float l1 = (v[1] - __half2float(__ushort_as_half((uint16_t)h1))) * 2048.f;
      *(lds_u32x2*)(uintptr_t)(rows + r * 512 + lane * 8) = u32x2{h0 | (h1 << 16), half_bits(l0) | (half_bits(l1) << 16)};
    }
    __builtin_amdgcn_wave_barrier();                     // (this wave's own table; its LDS operations complete in order)
    float hi[R], lo[R];
#pragma unroll
    for (int r = 0; r < R; ++r) hi[r] = lo[r] = 0.f;
    for (int s = 0; s < slots; ++s) {
      uint32_t f[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t code = __builtin_amdgcn_alignbit(pw[r].y, pw[r].x, psh) & imask;
        const uint32_t m = __builtin_amdgcn_alignbit(mp[r].y, mp[r].x, msh);
        f[r] = *(const lds_u32*)(uintptr_t)(signs + code * 4);
#pragma unroll
        for (int t = 0; t < 5; ++t) f[r] |= (m & (0xFu << (4 * t))) << (2 * t + 2);   // group fields between the sign fields
      }
      const u32x4 x4 = xa[s * 64 + lane];
      const uint32_t x1 = xb[s * 64 + lane];
      fetch();                                           // the next slot (behind the last one: unused)
      const uint32_t xw[5] = {x4.x, x4.y, x4.z, x4.w, x1};
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < 5; ++t) {
          // address = field * 8 + table: one shift and one "and, or" (the tables are aligned to their size)
          uint32_t at;
          asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(at) : "v"(t ? f[r] >> (6 * t - 3) : f[r] << 3), "s"(0x1F8u), "v"(rows));
          const u32x2 w = *(const lds_u32x2*)(uintptr_t)(at + r * 512);
          hi[r] = dot2(xw[t], w.x, hi[r]);
          lo[r] = dot2(xw[t], w.y, lo[r]);
        }
    }
    const int row0 = q * R;
    q += gridDim.x * kPairWaves;
    begin();
    fetch();                                             // the next rows (past the end: zeros)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float v = wave_sum(hi[r] + lo[r] * (1.f / 2048.f)) * scale[r];
      if (lane == 0 && row0 + r < d.out) {
        if (y_is_f32) ((float*)y)[row0 + r] = v;
        else ((__half*)y)[row0 + r] = __float2half_rn(v);
      }
    }
  }
}

// 32-bit buffer offsets; the next slot's and the next rows' windows stay below 2^32
static bool pairs_cover(const Dims& d) {
  return (d.v == 9 || d.v == 10) && d.b <= 10 && (long long)d.out * d.wpr * 4 < (1LL << 30) &&
         (long long)d.out * ((2 * d.in + 31) / 32) * 4 < (1LL << 30) && pairs_lds_bytes(d, 2) <= 160 * 1024;
}

template <int G, int R>
static btc_status launch_pairs(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                               const float* alpha, const float* mu, const uint32_t* gmap, const void* x, void* y,
                               int y_is_f32) {
  static bool attr_set = false;  // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)gemv_groups_pairs_kernel<G, R>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  const int lds = (int)pairs_lds_bytes(d, R);
  const int groups = ((d.out + R - 1) / R + kPairWaves - 1) / kPairWaves;
  // resident workgroups per compute unit: as many as balance the units of rows best (every workgroup fills its tables
  // once, so fewer of them on a tie)
  int per_cu = 1;
  long long best = 1LL << 60;
  for (int w = 1; w <= std::min(7, 160 * 1024 / lds); ++w) {
    const long long steps = (long long)((groups + 256 * w - 1) / (256 * w)) * w;   // units of work per compute unit
    const long long cost = steps * 8 + w + (w < 4 ? (4 - w) * steps * 2 : 0);      // (fewer than 4 waves per SIMD hide less)
    if (cost < best) {
      best = cost;
      per_cu = w;
    }
  }
  const int grid = std::min(groups, 256 * per_cu);
  gemv_groups_pairs_kernel<G, R><<<grid, kPairWaves * 64, lds, q>>>(d, packed, codebook, alpha, mu, gmap,
                                                                  (const uint16_t*)x, y, y_is_f32);
  return launch_status();
}

template <int G>
static btc_status launch(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                         const float* alpha, const float* mu, const uint32_t* gmap, const void* x, void* y, int y_is_f32) {
  // two rows per wave share the reads of the activations; one where that would leave waves without rows
  if (pairs_cover(d))
    return d.out > 4096 ? launch_pairs<G, 2>(q, d, packed, codebook, alpha, mu, gmap, x, y, y_is_f32)
                        : launch_pairs<G, 1>(q, d, packed, codebook, alpha, mu, gmap, x, y, y_is_f32);
  const bool cb_lds = (1 << d.b) <= kCodebookLds;
  const size_t lds = (((size_t)d.in * 2 + 15) & ~(size_t)15) + (cb_lds ? (size_t)4 << d.b : 0);
  const int grid = std::min(512, (d.out + kWaves - 1) / kWaves);
  static bool attr_set = false;  // one-time kernel attributes, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)gemv_groups_kernel<G, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024) != hipSuccess ||
        hipFuncSetAttribute((const void*)gemv_groups_kernel<G, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  if (cb_lds)
    gemv_groups_kernel<G, true><<<grid, kWaves * 64, lds, q>>>(d, packed, codebook, alpha, mu, gmap, (const uint16_t*)x, y, y_is_f32);
  else
    gemv_groups_kernel<G, false><<<grid, kWaves * 64, lds, q>>>(d, packed, codebook, alpha, mu, gmap, (const uint16_t*)x, y, y_is_f32);
  return launch_status();
}

}  // namespace groups
}  // namespace btc

extern "C" btc_status btc_gemv_groups(void* stream, const btc_shape* s, const uint32_t* packed, const uint32_t* codebook,
                                      const float* alpha, const float* mu, const uint32_t* group_map, int32_t ngroups,
                                      const void* x, void* y, btc_dtype y_dtype) {
  using namespace btc;
  btc_status st = check_shape(s);
  if (st != BTC_OK) return st;
  if (!packed || !codebook || !alpha || !mu || !group_map || !x || !y) return BTC_ERR_NULL;
  if (ngroups < 1 || ngroups > 4 || s->in > groups::kMaxIn) return BTC_ERR_UNSUPPORTED;
  if (y_dtype != BTC_F16 && y_dtype != BTC_F32) return BTC_ERR_UNSUPPORTED;
  if (!aligned16(packed) || !aligned16(codebook) || !aligned16(alpha) || !aligned16(mu) || !aligned16(group_map) ||
      !aligned16(x) || !aligned16(y))
    return BTC_ERR_ALIGN;
  const Dims d = dims_of(*s);
  hipStream_t q = (hipStream_t)stream;
  const int f32 = y_dtype == BTC_F32;
  switch (ngroups) {
    case 1: return groups::launch<1>(q, d, packed, codebook, alpha, mu, group_map, x, y, f32);
    case 2: return groups::launch<2>(q, d, packed, codebook, alpha, mu, group_map, x, y, f32);
    case 3: return groups::launch<3>(q, d, packed, codebook, alpha, mu, group_map, x, y, f32);
    default: return groups::launch<4>(q, d, packed, codebook, alpha, mu, group_map, x, y, f32);
  }
}
