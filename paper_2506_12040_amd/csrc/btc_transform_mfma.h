// btc_transform for several rows: the matrix-core kernel (one translation unit per alignment of the rows of the view).
#pragma once
#include <algorithm>
#include <type_traits>

#include "btc_internal.h"

namespace btc {
namespace transform {

// n2 a multiple of 16; even; odd.  BTC_ERR_UNSUPPORTED: the operands of the factors do not fit LDS.
btc_status mfma_16(hipStream_t q, const void* X, int is_bf16, int M, int n1, int n2, const uint32_t* sign_bits, const float* P1,
                   const float* P2, void* Y, int y_dtype);
btc_status mfma_2(hipStream_t q, const void* X, int is_bf16, int M, int n1, int n2, const uint32_t* sign_bits, const float* P1,
                  const float* P2, void* Y, int y_dtype);
btc_status mfma_1(hipStream_t q, const void* X, int is_bf16, int M, int n1, int n2, const uint32_t* sign_bits, const float* P1,
                  const float* P2, void* Y, int y_dtype);

// ---- device side, for the translation units that define one of the above
#ifdef BTC_TRANSFORM_ALIGN
// The two stages are small dense contractions and run on the matrix cores (MFMA 32x32x16 bf16,
// fp32 accumulate).  A wave owns one row of X and one block of 32 columns j2:
//   stage 1:  D1[i1][j2] = sum_i2 (sigma x)[i1][i2] P2[i2][j2]    A = the row itself, read from
//             global memory in operand layout (16 bytes per lane, signs applied in registers);
//             B = P2 from LDS
//   stage 2:  Z[j1][j2]  = sum_i1 P1[i1][j1] D1[i1][j2]           A = P1^T from LDS; B = D1 as it
//             sits in the accumulators: a lane of D1 holds column j2 = lane % 32 and the 16 rows
//             8 (e / 4) + 4 (lane / 32) + e % 4, which is a valid B operand once the contraction
//             index of a 16-row step is permuted the same way in A -- P1^T is staged in that order.
// The fp32 factors and the fp32 D1 enter as sums of NP bf16 numbers: three (24 bits; products whose weight is below 2^-24
// are dropped) for the accuracy of the fp32 kernel above, two (16 bits) where 64 or more rows of bf16
// activations, n2 a multiple of 16, end in a 16-bit output.  bf16 activations enter exactly as they are, fp16 ones exactly as the sum of two bf16 numbers.
//
// ALIGN: the largest of 16, 2 and 1 that divides n2.  Below 16 the last step reaches past the end of a row of the n1 x n2 view:
// the elements there are cleared.  With odd n2 rows start inside words: the loads start at the word below and are shifted
// into place.
//
// What bounds it: instructions, not bytes.  So the operands of the factors, which take longer to make than a few rows to
// transform, are made once per compute unit for all columns that fit LDS (a workgroup per column block made them 768
// times), the signs of eight elements come from a table of masks in LDS (four exclusive ors), and a pair of lanes trades
// halves so that outputs leave as words.  2048 x 5120 (64 x 80, bf16 to bf16): 22.8 -> 16.8 us; 2048 x 13824 (108 x 128):
// 71 -> 59 us.  Odd n2 and fp16 ran on the vector ALU: 2048 x 4672 (64 x 73) 207 -> 23 us, 2048 x 5120 in fp16 136 -> 24 us.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// two floats -> two bf16 bit patterns, round to nearest even (the hardware conversion of gfx950)
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// (a, b) = the sum of the NP pairs p[0] + .. up to 2^-8 NP relative
template <int NP>
__device__ __forceinline__ void split_pair(float a, float b, uint32_t (&p)[NP]) {
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    p[k] = bf16_pair(a, b);
    a -= bf16_lo(p[k]);
    b -= bf16_hi(p[k]);
  }
}

__device__ __forceinline__ f32x16 mfma32(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// f(integral_constant<int, I>) for I = Begin .. End - 1, fully unrolled
template <int Begin, int End, class F>
__device__ __forceinline__ void static_for_it(F&& f) {
  if constexpr (Begin < End) {
    f(std::integral_constant<int, Begin>{});
    static_for_it<Begin + 1, End>(f);
  }
}

constexpr int kSignTable = 256 * 16;
constexpr int kMfmaLds = 160 * 1024 - 256;

// waves per workgroup at most: with three or four blocks of rows a wave needs more than 128 registers
template <int IT>
constexpr int mfma_waves() { return IT <= 2 ? 16 : 12; }

// IT = ceil(n1 / 32): blocks of 32 rows i1 (and of 32 rows j1).  ncb column blocks of 32 per workgroup, from blockIdx.x * ncb.
template <int IT, int NP, bool F16, int ALIGN>
__global__ __launch_bounds__(64 * mfma_waves<IT>()) void transform_mfma_kernel(const uint16_t* __restrict__ X, int M, int n1, int n2,
                                                                 const uint32_t* __restrict__ sign_bits,
                                                                 const float* __restrict__ P1,
                                                                 const float* __restrict__ P2, void* __restrict__ Y,
                                                                 int y_dtype, int ncb) {
  constexpr int KS1 = 2 * IT;                // 16-row steps of stage 2
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  constexpr int waves = mfma_waves<IT>(), NT = 64 * waves;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int n = n1 * n2, KS2 = (n2 + 15) >> 4;
  const int cb0 = blockIdx.x * ncb, my_ncb = min(ncb, (n2 + 31) / 32 - cb0);
  u32x4* const signs = (u32x4*)smem;                             // [byte]: the masks of its eight elements, a clear bit flips
  u32x4* const P1op = (u32x4*)(smem + kSignTable);               // [block j1][step][part][lane]: A operands of stage 2
  u32x4* const P2op = P1op + IT * KS1 * NP * 64;                 // [column block][step][part][lane]: B operands of stage 1

  // ---- operands of the factors: a wave makes the NP parts of a step's operand, U steps' loads under way
  constexpr int U = 4;
  const int n_p1 = IT * KS1, n_ops = n_p1 + my_ncb * KS2;
#pragma unroll 1
  for (int base = wave; base < n_ops; base += U * waves) {
    float v[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int op = base + u * waves;
      if (op < n_p1) {
        const int ks = op % KS1, j1 = op / KS1 * 32 + l32;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int i1 = 16 * ks + 8 * (e >> 2) + 4 * h + (e & 3);   // the row of D1 that element e of a lane's step holds
          v[u][e] = (i1 < n1 && j1 < n1) ? P1[i1 * n1 + j1] : 0.f;
        }
      } else {
        const int s = op - n_p1, cb = s / KS2, ks = s - cb * KS2, c = (cb0 + cb) * 32 + l32;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int i2 = 16 * ks + 8 * h + e;
          v[u][e] = (i2 < n2 && c < n2 && op < n_ops) ? P2[i2 * n2 + c] : 0.f;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int op = base + u * waves;
      uint32_t q[4][NP];
#pragma unroll
      for (int e = 0; e < 4; ++e) split_pair<NP>(v[u][2 * e], v[u][2 * e + 1], q[e]);
      if (op < n_ops) {
#pragma unroll
        for (int p = 0; p < NP; ++p) P1op[(op * NP + p) * 64 + lane] = u32x4{q[0][p], q[1][p], q[2][p], q[3][p]};
      }
    }
  }
  for (int t = tid; t < 256; t += NT) {
    const uint32_t minus = ~(uint32_t)t;
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (((minus >> (2 * e)) & 1u) << 15) | (((minus >> (2 * e + 1)) & 1u) << 31);
    signs[t] = w;
  }

  // ---- One block of 32 rows i1 at a time: its stage 1 (all steps over i2), the split of its 32 x 32 result, and its
  // share of stage 2 for every block j1 -- so only one block of the intermediate is alive, next to the IT
  // accumulators of the output.  A operands of stage 1 come straight from global memory, PD steps ahead: slot u of
  // the ring holds step ks0 + u of the current chunk of PD steps; once used it is refilled with step ks0 + PD + u
  // of the same block or, in a block's last chunk, with step u of the next block (of the wave's next item after
  // the last block), so the loads always fly during the arithmetic of the block before.
  constexpr int PD = 4;
  const __amdgpu_buffer_rsrc_t rX =
      __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)(((uint32_t)M * (uint32_t)n * 2u + 3u) & ~3u), 0x00020000);
  const uint32_t sign_bytes = (uint32_t)((n + 31) >> 5) * 4u;
  const __amdgpu_buffer_rsrc_t rS = __builtin_amdgcn_make_buffer_rsrc((void*)sign_bits, 0, (int)sign_bytes, 0x00020000);
  u32x4 ring[PD];
  uint32_t after[ALIGN == 1 ? PD : 1], rsg[PD];                  // the word behind them; their signs
  auto load_a = [&](int mm, int it, int ks, int u) __attribute__((always_inline)) {
    const int i1 = min(it * 32 + l32, n1 - 1);                   // rows past the end: a valid row, which meets zeros of P1
    const uint32_t k = (uint32_t)(i1 * n2 + 16 * ks + 8 * h), at = 2u * (uint32_t)(mm * n);
    if constexpr (ALIGN == 1) {
      const uint32_t off = (at + 2u * k) & ~3u;
      ring[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rX, off, 0, 0));
      after[u] = __builtin_amdgcn_raw_buffer_load_b32(rX, off + 16u, 0, 0);
    } else {
      ring[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rX, 2u * k, (int)at, 0));
    }
    if constexpr (ALIGN == 16) {
      rsg[u] = __builtin_amdgcn_raw_buffer_load_b8(rS, k >> 3, 0, 0);
    } else {                                                     // (the eight bits may straddle two bytes)
      const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b8(rS, k >> 3, 0, 0);
      const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b8(rS, (k >> 3) + 1u, 0, 0);
      rsg[u] = (lo | (hi << 8)) >> (k & 7u);
    }
  };
  // item t of the workgroup: column block t % my_ncb of its row t / my_ncb
  const int rows = (M - (int)blockIdx.y + (int)gridDim.y - 1) / (int)gridDim.y, items = rows * my_ncb;
  auto row_of = [&](int t) { return (int)blockIdx.y + (t / my_ncb) * (int)gridDim.y; };
  if (wave < items) {
#pragma unroll
    for (int u = 0; u < PD; ++u)
      if (u < KS2) load_a(row_of(wave), 0, u, u);
  }
  __syncthreads();

  u32x4 keep;                                                    // elements of the last step inside a row of the view
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i2 = 16 * (KS2 - 1) + 8 * h + 2 * e;
    keep[e] = (i2 < n2 ? 0xFFFFu : 0u) | (i2 + 1 < n2 ? 0xFFFF0000u : 0u);
  }
  const uint32_t swap = (lane & 1) ? 0x03020706u : 0x05040100u;  // halves of (neighbour's pair, own pair): see the stores
#pragma unroll 1
  for (int t = wave; t < items; t += waves) {
    const int m = row_of(t), cb = t % my_ncb;
    const int m_next = t + waves < items ? row_of(t + waves) : -1;
    const u32x4* const p2 = P2op + cb * KS2 * NP * 64 + lane;
    f32x16 z[IT];
#pragma unroll
    for (int jt = 0; jt < IT; ++jt)
#pragma unroll
      for (int e = 0; e < 16; ++e) z[jt][e] = 0.f;
    static_for_it<0, IT>([&](auto it_c) {
      constexpr int it = decltype(it_c)::value;
      asm volatile("" ::: "memory");                             // (else the operands of P1 are kept in registers from item to item, spilt)
      f32x16 d1;
#pragma unroll
      for (int e = 0; e < 16; ++e) d1[e] = 0.f;
#pragma unroll 1
      for (int ks0 = 0; ks0 < KS2; ks0 += PD) {
        const bool last_chunk = ks0 + PD >= KS2;
#pragma unroll
        for (int u = 0; u < PD; ++u) {
          const int ks = ks0 + u;
          if (ks < KS2) {
            u32x4 a = ring[u];
            if constexpr (ALIGN == 1) {
              const uint32_t by = (uint32_t)((m * n + min(it * 32 + l32, n1 - 1) * n2) & 1) * 16u;
#pragma unroll
              for (int e = 0; e < 4; ++e) a[e] = __builtin_amdgcn_alignbit(e < 3 ? ring[u][e + 1] : after[u], ring[u][e], by);
            }
            a ^= signs[rsg[u] & 0xFFu];
            if (ALIGN < 16 && ks == KS2 - 1) a &= keep;
            u32x4 b[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) b[p] = p2[(ks * NP + p) * 64];
            if constexpr (F16) {                                 // a = a0 + a1, both bf16, exactly
              u32x4 a0, a1;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const f16x2 w = __builtin_bit_cast(f16x2, (uint32_t)a[e]);
                uint32_t p[2];
                split_pair<2>((float)w[0], (float)w[1], p);
                a0[e] = p[0];
                a1[e] = p[1];
              }
#pragma unroll
              for (int p = NP - 2; p >= 0; --p) d1 = mfma32(a1, b[p], d1);
              a = a0;
            }
#pragma unroll
            for (int p = NP - 1; p >= 0; --p) d1 = mfma32(a, b[p], d1);
          }
          if (ks + PD < KS2) {
            load_a(m, it, ks + PD, u);
          } else if (last_chunk && u < KS2) {
            if (it + 1 < IT) load_a(m, it + 1, u, u);
            else if (m_next >= 0) load_a(m_next, 0, u, u);
          }
        }
      }
      // the block as NP bf16 parts, in B-operand form: step s2 takes elements 8 s2 .. 8 s2 + 7
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        u32x4 y[NP];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t p[NP];
          split_pair<NP>(d1[8 * s2 + 2 * e], d1[8 * s2 + 2 * e + 1], p);
#pragma unroll
          for (int k = 0; k < NP; ++k) y[k][e] = p[k];
        }
#pragma unroll
        for (int jt = 0; jt < IT; ++jt) {
          const u32x4* ap = P1op + ((jt * KS1 + 2 * it + s2) * NP) * 64 + lane;
          const u32x4 a0 = ap[0], a1 = ap[64];
          if constexpr (NP == 3) {                               // small terms first
            z[jt] = mfma32(ap[128], y[0], z[jt]);
            z[jt] = mfma32(a1, y[1], z[jt]);
            z[jt] = mfma32(a0, y[2], z[jt]);
          }
          z[jt] = mfma32(a1, y[0], z[jt]);
          z[jt] = mfma32(a0, y[1], z[jt]);
          z[jt] = mfma32(a0, y[0], z[jt]);
        }
      }
    });
    // ---- outputs, through a buffer of the row (what lies past its end is not stored).  16-bit ones leave as words where
    // pairs of columns are aligned: of the rows e and e + 1 of its column an even lane takes row e, an odd one row e + 1,
    // of both columns.
    const int j2 = (cb0 + cb) * 32 + l32;
    const uint32_t size = y_dtype == BTC_F32 ? 4u : 2u;
    const __amdgpu_buffer_rsrc_t rY = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((char*)Y + (size_t)m * (uint32_t)n * size), 0, (int)((uint32_t)n * size), 0x00020000);
    constexpr bool kPairs = ALIGN != 1;
    if (kPairs && y_dtype != BTC_F32) {
      const uint32_t row0 = (uint32_t)(4 * h + (lane & 1));
      const uint32_t off = j2 < n2 ? 2u * (row0 * (uint32_t)n2 + (uint32_t)(j2 & ~1)) : 0x80000000u;
      auto store_all = [&](auto to16) __attribute__((always_inline)) {
#pragma unroll
        for (int jt = 0; jt < IT; ++jt)
#pragma unroll
          for (int e = 0; e < 16; e += 2) {
            const uint32_t own = to16(z[jt][e], z[jt][e + 1]);
            const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, true);   // lane ^ 1
            const uint32_t w = __builtin_amdgcn_perm(other, own, swap);
            __builtin_amdgcn_raw_buffer_store_b32(w, rY, off, (jt * 32 + 8 * (e >> 2) + (e & 3)) * n2 * 2, 0);
          }
      };
      if (y_dtype == BTC_BF16) store_all([](float a, float b) { return bf16_pair(a, b); });
      else store_all([](float a, float b) {
        return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a) | ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)b) << 16);
      });
    } else {
      const uint32_t off = j2 < n2 ? size * ((uint32_t)(4 * h) * (uint32_t)n2 + (uint32_t)j2) : 0x80000000u;
#pragma unroll
      for (int jt = 0; jt < IT; ++jt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int at = (jt * 32 + 8 * (e >> 2) + (e & 3)) * n2 * (int)size;
          if (y_dtype == BTC_F32)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)z[jt][e]), rY, off, at, 0);
          else if (y_dtype == BTC_BF16)
            __builtin_amdgcn_raw_buffer_store_b16((short)bf16_pair(z[jt][e], 0.f), rY, off, at, 0);
          else
            __builtin_amdgcn_raw_buffer_store_b16((short)__builtin_bit_cast(uint16_t, (_Float16)z[jt][e]), rY, off, at, 0);
        }
    }
  }
}

template <int IT, int NP, bool F16, int ALIGN>
static btc_status launch_mfma(hipStream_t q, const uint16_t* X, int M, int n1, int n2, const uint32_t* sign_bits,
                              const float* P1, const float* P2, void* Y, int y_dtype) {
  static bool attr_set = false;              // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)transform_mfma_kernel<IT, NP, F16, ALIGN>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kMfmaLds) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  const int blocks = (n2 + 31) / 32, p1_bytes = IT * 2 * IT * NP * 1024, p2_bytes = ((n2 + 15) >> 4) * NP * 1024;
  // Column blocks per workgroup: all that fit beside P1 and the signs, evenly; one where there are not rows enough for every
  // compute unit.  One workgroup per compute unit: the operands of the factors are made as seldom as can be.
  const int fit = (kMfmaLds - kSignTable - p1_bytes) / p2_bytes;
  if (fit < 1) return BTC_ERR_UNSUPPORTED;
  int groups = (blocks + fit - 1) / fit;
  if (M < 128) groups = blocks;
  const int ncb = (blocks + groups - 1) / groups;
  groups = (blocks + ncb - 1) / ncb;
  const int lds = kSignTable + p1_bytes + ncb * p2_bytes;
  const int gy = std::max(1, std::min(M, 256 / groups));
  transform_mfma_kernel<IT, NP, F16, ALIGN><<<dim3(groups, gy), 64 * mfma_waves<IT>(), lds, q>>>(X, M, n1, n2, sign_bits, P1, P2, Y, y_dtype, ncb);
  return launch_status();
}

template <int IT, int ALIGN>
static btc_status launch_mfma_it(hipStream_t q, const uint16_t* X, int is_bf16, int M, int n1, int n2, const uint32_t* sign_bits,
                                 const float* P1, const float* P2, void* Y, int y_dtype) {
  if (!is_bf16) return launch_mfma<IT, 3, true, ALIGN>(q, X, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
  if constexpr (ALIGN == 16) {
    if (y_dtype != BTC_F32 && M >= 64) return launch_mfma<IT, 2, false, ALIGN>(q, X, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
  }
  return launch_mfma<IT, 3, false, ALIGN>(q, X, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
}

template <int ALIGN>
static btc_status run_mfma(hipStream_t q, const void* X, int is_bf16, int M, int n1, int n2, const uint32_t* sign_bits,
                           const float* P1, const float* P2, void* Y, int y_dtype) {
  const uint16_t* x = (const uint16_t*)X;
  switch ((n1 + 31) / 32) {
    case 1: return launch_mfma_it<1, ALIGN>(q, x, is_bf16, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
    case 2: return launch_mfma_it<2, ALIGN>(q, x, is_bf16, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
    case 3: return launch_mfma_it<3, ALIGN>(q, x, is_bf16, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
    case 4: return launch_mfma_it<4, ALIGN>(q, x, is_bf16, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
    default: return BTC_ERR_UNSUPPORTED;
  }
}

#endif

}  // namespace transform
}  // namespace btc
