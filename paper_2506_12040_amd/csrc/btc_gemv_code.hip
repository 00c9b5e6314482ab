// Decode-time product for the long-vector settings of the paper's vector-length study (Table
// "Ablation study on vector length / centroids": v = 12 .. 20 and beyond, codebooks of up to 65536
// centroids), one activation row.
//
// With 11 to 16 index bits neither the expanded-codeword tables of the tuned engines nor a table of
// chunk sums fits LDS: the codebook itself (128 KB as 16-bit patterns for v <= 16, or as 32-bit
// patterns up to 32768 centroids) is what LDS can hold, and the blockwise dot product <x_j, C[I_rj]>
// (appendix "Binary Codebook LUT-GEMM") is evaluated from the pattern's bits.  Layout of the work:
//   * a workgroup of 16 waves fills LDS with the codebook once;
//   * lane l takes chunks l, l + 64, .. of an output row: it reads its index from the row's bit stream (consecutive lanes,
//     consecutive fields: coalesced), gathers the pattern from LDS and adds the chunk's activations with the pattern's
//     signs, two at a time: the two sign bits are moved onto the sign positions of a packed (1, 1) and the pair is summed in
//     fp32 by a packed dot product;
//   * the index loads of a wave's next row are issued before the current row is summed up.
// Vector lengths 12, 14, .. 20 (gemv_code_kernel): a lane's activations, the same for every row, stay in registers.  That is four
// chunks at most, so longer rows are shared by 2, 4, 8 or 16 waves; the shares meet in LDS at the end.  Three vector instructions per
// two weights, no LDS reads but the patterns: 8192 x 8192 at v = 16, K = 65536 18.6 -> 15.4 us, 4 of them for the 128 KB of
// codebook; 13829 x 12214 at v = 20 54 -> 29.  Other even lengths (gemv_code_any_kernel): activations from LDS, a wave per row.
// Patterns of 18 and 20 bits with 16 index bits fill LDS to the last byte (16 + 4 bits: 160 KB), so sums stay in registers until
// the codebook has been read.  A codebook that does not fit (v > 20 with 16 index bits) is gathered from memory instead --
// it stays in the L2 of every XCD, but every pattern costs a cache line -- and so is any where a compute unit has fewer than
// 64 gathers of a wave to do (110 where LDS would have to be split): filling LDS takes longer (1024 x 8192 at v = 16, K = 65536: 9.5
// against 8.2 us).
// Epilogue: y = alpha * acc + mu * sum(x)  (Algorithm "Binary Transformation and Compression").
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>

#include "btc_internal.h"

namespace btc {
namespace code {

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
constexpr int kWaves = 16;
constexpr int kMaxIn = 16384;           // activation row in LDS: 32 KB
constexpr int kMaxSteps = 16;           // chunks per lane and row held in flight

// Sum over the 64 lanes by data-parallel moves (no LDS traffic), valid in lane 63.
__device__ __forceinline__ float wave_sum_to_lane63(float v) {
  auto dpp = [](float x, auto ctrl, auto row_mask, auto bound_ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                 decltype(row_mask)::value, 0xF, decltype(bound_ctrl)::value));
  };
  using std::integral_constant;
  v += dpp(v, integral_constant<int, 0xB1>{}, integral_constant<int, 0xF>{}, integral_constant<bool, true>{});    // quad: lane ^ 1
  v += dpp(v, integral_constant<int, 0x4E>{}, integral_constant<int, 0xF>{}, integral_constant<bool, true>{});    // quad: lane ^ 2
  v += dpp(v, integral_constant<int, 0x141>{}, integral_constant<int, 0xF>{}, integral_constant<bool, true>{});   // row_half_mirror
  v += dpp(v, integral_constant<int, 0x140>{}, integral_constant<int, 0xF>{}, integral_constant<bool, true>{});   // row_mirror
  v += dpp(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{}, integral_constant<bool, false>{});  // row_bcast:15
  v += dpp(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{}, integral_constant<bool, false>{});  // row_bcast:31
  return v;
}

constexpr int kSteps = 4;                // chunks per lane and row at most
constexpr int kHigh = 2 << 16;           // ESZ = 3: the upper four bits of 65536 patterns of up to 20, behind the lower sixteen

// inverted codebook -> LDS, four entries per load, eight loads in flight per thread
template <int ESZ>
__device__ __forceinline__ void fill_codebook(unsigned char* cb, const uint32_t* __restrict__ codebook, int b) {
  const int tid = threadIdx.x, quads = (1 << b) >> 2;
  if (ESZ == 4 && b < 2 && tid < (1 << b)) ((uint32_t*)cb)[tid] = ~codebook[tid];   // a codebook of two
  for (int k0 = tid; k0 < quads; k0 += 8 * kWaves * 64) {
    uint4 c[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = k0 + r * kWaves * 64;
      c[r] = k < quads ? ((const uint4*)codebook)[k] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = k0 + r * kWaves * 64;
      if (k < quads) {
        if (ESZ == 4) ((uint4*)cb)[k] = make_uint4(~c[r].x, ~c[r].y, ~c[r].z, ~c[r].w);
        if (ESZ == 3) ((uint16_t*)(cb + kHigh))[k] = (uint16_t)(((~c[r].x >> 16) & 15u) | (((~c[r].y >> 16) & 15u) << 4) |
                                                                 (((~c[r].z >> 16) & 15u) << 8) | (((~c[r].w >> 16) & 15u) << 12));
        if (ESZ != 4) ((uint2*)cb)[k] = make_uint2((~c[r].x & 0xFFFFu) | (~c[r].y << 16), (~c[r].z & 0xFFFFu) | (~c[r].w << 16));
      }
    }
  }
}

// PAIRS = v / 2.  ESZ: bytes of a codebook entry in LDS, 2 or 4; 3 = patterns of up to 20 bits in 2.5 bytes (160 KB: all of LDS);
// 0 = codebook read from memory.  The rows of a workgroup: rows_per_wg from blockIdx.x * rows_per_wg; share s of `shares` of a
// row: the chunks 64 (shares t + s) + lane.
template <int ESZ, int PAIRS>
__global__ __launch_bounds__(kWaves * 64) void gemv_code_kernel(Dims d, const uint32_t* __restrict__ packed,
                                                                const uint32_t* __restrict__ codebook,
                                                                const float* __restrict__ alpha, const float* __restrict__ mu,
                                                                const uint16_t* __restrict__ x, void* __restrict__ y,
                                                                int y_is_f32, int rows_per_wg, int shares) {
  constexpr int S = kSteps;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* const cb = smem;
  float* const res = (float*)smem;                       // at the end: [row][share], then [share]: sums of the activations
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int groups = kWaves / shares, share = wave % shares, group = wave / shares;
  const int row0 = blockIdx.x * rows_per_wg, rows = min(rows_per_wg, d.out - row0);
  const int blocks = (d.nchunks + 63) >> 6;              // of 64 chunks
  const int steps = (blocks - share + shares - 1) / shares;
  const __amdgpu_buffer_rsrc_t rP =
      __builtin_amdgcn_make_buffer_rsrc((void*)packed, 0, (int)((uint32_t)d.out * (uint32_t)d.wpr * 4u), 0x00020000);
  const __amdgpu_buffer_rsrc_t rX = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (d.in * 2 + 3) & ~3, 0x00020000);
  // index words of a row, the two that hold a field; two rows ahead
  u32x2 field[2][S];
  auto fetch = [&](auto set, int row) {                  // (uniform; a row past the last: zeros or another workgroup's)
    const uint32_t at = (uint32_t)(row0 + row) * (uint32_t)d.wpr * 4u;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      if (t < steps) {
        const uint32_t j = (uint32_t)(64 * (shares * t + share) + lane);
        // (past the row's last chunk: fields of the next row, or zeros; their activations are zeros)
        field[decltype(set)::value][t] =
            __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rP, ((j * (uint32_t)d.b) >> 5) * 4u + at, 0, 0));
      }
    }
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  fetch(even, group);
  fetch(odd, group + groups);
  // ---- this lane's activations, zeros past the end of the row
  uint32_t xw[S][PAIRS];
#pragma unroll
  for (int t = 0; t < S; ++t) {
    if (t < steps) {
      const uint32_t k = (uint32_t)(64 * (shares * t + share) + lane) * (4u * PAIRS);
#pragma unroll
      for (int u = 0; u + 4 <= PAIRS; u += 4) {
        typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
        const u32x4 w = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rX, k + 4u * u, 0, 0));
        xw[t][u] = w.x; xw[t][u + 1] = w.y; xw[t][u + 2] = w.z; xw[t][u + 3] = w.w;
      }
#pragma unroll
      for (int u = PAIRS & ~3; u < PAIRS; ++u) xw[t][u] = __builtin_amdgcn_raw_buffer_load_b32(rX, k + 4u * u, 0, 0);
    } else {
#pragma unroll
      for (int u = 0; u < PAIRS; ++u) xw[t][u] = 0u;
    }
  }
  if (ESZ != 0) fill_codebook<ESZ>(cb, codebook, d.b);
  const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
  float sx = 0.f;
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int k = (64 * (shares * t + share) + lane) * (2 * PAIRS);
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
      if (k + 2 * u + 1 >= d.in) xw[t][u] = k + 2 * u >= d.in ? 0u : xw[t][u] & 0xFFFFu;
      sx = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, xw[t][u]), one, sx, false);
    }
  }
  sx = wave_sum_to_lane63(sx);
  __syncthreads();

  const uint32_t mask = (1u << d.b) - 1u;
  uint32_t ones = 0x3C003C00u;
  asm volatile("" : "+v"(ones));                         // (an instruction takes one constant that is not in a register)
  int kept = 0, n_kept = 0;                              // lane l: the sum of this wave's row l (LDS may be full)
  auto one_row = [&](auto set, int row) {
    uint32_t np[S];                                      // inverted patterns (bit set: -1)
#pragma unroll
    for (int t = 0; t < S; ++t) {
      if (t < steps) {
        const uint32_t j = (uint32_t)(64 * (shares * t + share) + lane);
        const u32x2 f = field[decltype(set)::value][t];
        const uint32_t idx = __builtin_amdgcn_alignbit(f.y, f.x, (j * (uint32_t)d.b) & 31u) & mask;
        if (ESZ == 4) np[t] = ((const uint32_t*)cb)[idx];
        else if (ESZ == 0) np[t] = ~codebook[idx];
        else np[t] = ((const uint16_t*)cb)[idx];
        if (ESZ == 3) np[t] |= ((cb[kHigh + (idx >> 1)] >> (4u * (idx & 1u))) & 15u) << 16;
      }
    }
    fetch(set, row + 2 * groups);
    float acc[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < S; ++t) {
      if (t < steps) {
#pragma unroll
        for (int h = 0; h < (PAIRS + 7) / 8; ++h) {      // sixteen bits at a time
          const uint32_t n = ESZ == 2 ? np[t] : h ? np[t] >> 16 : np[t] & 0xFFFFu;
          const uint32_t w = (n << 15) | n;              // bit 2 u of the pattern at 2 u, bit 2 u + 1 at 16 + 2 u
#pragma unroll
          for (int u = 0; u < 8 && 8 * h + u < PAIRS; ++u) {
            const uint32_t sign = ((w << (15 - 2 * u)) & 0x80008000u) | ones;
            acc[u & 1] = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, xw[t][8 * h + u]), __builtin_bit_cast(f16x2, sign), acc[u & 1], false);
          }
        }
      }
    }
    const int a = __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_sum_to_lane63(acc[0] + acc[1])), 63);
    kept = lane == n_kept ? a : kept;
    ++n_kept;
  };
  for (int row = group; row < rows; row += 2 * groups) {
    one_row(even, row);
    if (row + groups < rows) one_row(odd, row + groups);
  }
  __syncthreads();                                       // the codebook has been read
  if (group + lane * groups < rows) res[(group + lane * groups) * shares + share] = __builtin_bit_cast(float, kept);
  if (group == 0 && lane == 63) res[rows_per_wg * shares + share] = sx;
  __syncthreads();
  float sum_x = 0.f;
  for (int s = 0; s < shares; ++s) sum_x += res[rows_per_wg * shares + s];
  for (int row = tid; row < rows; row += kWaves * 64) {
    float a = 0.f;
    for (int s = 0; s < shares; ++s) a += res[row * shares + s];
    const int i = row0 + row;
    const float r = alpha[i] * a + mu[i] * sum_x;
    if (y_is_f32) ((float*)y)[i] = r;
    else ((__half*)y)[i] = __float2half_rn(r);
  }
}

// ESZ: bytes of a codebook entry in LDS (2 or 4), 0 = codebook read from memory.
template <int ESZ>
__global__ __launch_bounds__(kWaves * 64) void gemv_code_any_kernel(Dims d, const uint32_t* __restrict__ packed,
                                                                const uint32_t* __restrict__ codebook,
                                                                const float* __restrict__ alpha,
                                                                const float* __restrict__ mu,
                                                                const uint16_t* __restrict__ x, void* __restrict__ y,
                                                                int y_is_f32) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* xs = (uint16_t*)smem;                        // [in rounded up to the chunk grid] fp16, zeros past `in`
  const int xpad = d.nchunks * d.v;
  float* sxp = (float*)(smem + ((xpad * 2 + 15) & ~15));     // [kWaves] partial sums of x
  unsigned char* cb = (unsigned char*)(sxp + kWaves);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_id = blockIdx.x * kWaves + wave, n_waves = gridDim.x * kWaves;
  const uint32_t mask = (1u << d.b) - 1u;
  const int steps = (d.nchunks + 63) >> 6;               // chunks per lane and row

  // index of chunk j of row i; past the row's last chunk: 0 (its activations in LDS are zero)
  auto index_of = [&](int i, int j) -> uint32_t {
    if (j >= d.nchunks) return 0u;
    const uint32_t* row = packed + (size_t)i * d.wpr;
    const uint32_t p = (uint32_t)j * (uint32_t)d.b;
    const uint32_t w = p >> 5, sh = p & 31u;
    const uint32_t lo = row[w];
    const uint32_t hi = (sh + d.b > 32u) ? row[w + 1] : 0u;   // inside the row whenever the field crosses
    return __builtin_amdgcn_alignbit(hi, lo, sh) & mask;
  };
  // the first row's indices fly while LDS is filled
  uint32_t idx[kMaxSteps];
  int i = wave_id;
  if (i < d.out) {
#pragma unroll
    for (int s = 0; s < kMaxSteps; ++s)
      if (s < steps) idx[s] = index_of(i, lane + 64 * s);
  }
  float sx_part = 0.f;                                   // this thread's share of sum(x), the factor of mu
  for (int k = tid; k < xpad / 2; k += kWaves * 64) {    // v is even: whole pairs
    const uint32_t lo = 2 * k < d.in ? x[2 * k] : 0u, hi = 2 * k + 1 < d.in ? x[2 * k + 1] : 0u;
    const uint32_t w = lo | (hi << 16);
    ((uint32_t*)xs)[k] = w;
    const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
    sx_part = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w), one, sx_part, false);
  }
  sx_part = wave_sum_to_lane63(sx_part);
  if (lane == 63) sxp[wave] = sx_part;
  if (ESZ != 0) fill_codebook<ESZ>(cb, codebook, d.b);   // (inverted: bit set = -1)
  __syncthreads();
  float sx = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) sx += sxp[w];

  const int pairs = d.v >> 1;
  while (i < d.out) {
    // inverted patterns (bit set: -1) of this row's chunks
    uint32_t np[kMaxSteps];
#pragma unroll
    for (int s = 0; s < kMaxSteps; ++s) {
      if (s < steps) {
        if (ESZ == 4) np[s] = ((const uint32_t*)cb)[idx[s]];
        else if (ESZ == 2) np[s] = ((const uint16_t*)cb)[idx[s]];
        else np[s] = ~codebook[idx[s]];
      }
    }
    const int i_next = i + n_waves;
    uint32_t idx_next[kMaxSteps];
    if (i_next < d.out) {
#pragma unroll
      for (int s = 0; s < kMaxSteps; ++s)
        if (s < steps) idx_next[s] = index_of(i_next, lane + 64 * s);
    }
    float acc = 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSteps; ++s) {
      if (s < steps) {
        const int j = min(lane + 64 * s, d.nchunks - 1);  // (lanes past the last chunk: index 0 times real
        const bool live = lane + 64 * s < d.nchunks;     //  activations -- masked out below)
        const uint32_t* xc = (const uint32_t*)xs + (size_t)j * pairs;
        float a = 0.f;
        auto pair_step = [&](int u, uint32_t xw) {
          const uint32_t n = (np[s] >> (2 * u)) & 3u;
          const uint32_t sg = ((n << 15) | (n << 30)) & 0x80008000u;   // bit 0 -> sign of the low half, bit 1 -> of the high half
          const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
          a = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, xw ^ sg), one, a, false);
        };
        for (int u = 0; u < pairs; ++u) pair_step(u, xc[u]);
        acc += live ? a : 0.f;
      }
    }
    acc = wave_sum_to_lane63(acc);
    if (lane == 63) {
      const float r = alpha[i] * acc + mu[i] * sx;
      if (y_is_f32) ((float*)y)[i] = r;
      else ((__half*)y)[i] = __float2half_rn(r);
    }
    i = i_next;
#pragma unroll
    for (int s = 0; s < kMaxSteps; ++s) idx[s] = idx_next[s];
  }
}

static int entry_bytes(const Dims& d) {
  if ((4LL << d.b) <= 128 * 1024) return 4;
  if (d.v <= 16 && (2LL << d.b) <= 128 * 1024) return 2;
  return 0;
}
static size_t any_lds_bytes(const Dims& d) {
  return (((size_t)d.nchunks * d.v * 2 + 15) & ~(size_t)15) + kWaves * sizeof(float) + ((size_t)entry_bytes(d) << d.b);
}

// The kernel with the activations in registers, for v / 2 = 6 .. 10.
struct Plan {
  int shares, rows_per_wg, grid, esz;
  size_t lds;
};
static bool make_plan(const Dims& d, Plan* p) {
  if (d.v < 12 || d.v > 20 || (d.v & 1)) return false;
  const int blocks = (d.nchunks + 63) / 64;
  // The number of shares with the shortest wave: its rows times the steps of a share (and what a row costs besides).  A
  // workgroup per compute unit, each with as many rows, a share of a row for every wave at least.
  p->shares = 0;
  double best = 1e30;
  for (int s = 1; s <= kWaves; s *= 2) {
    const int steps = (blocks + s - 1) / s, rows = std::max((d.out + 255) / 256, kWaves / s), per_wave = (rows * s + kWaves - 1) / kWaves;
    if (steps > kSteps || per_wave > 64) continue;       // (a wave keeps its sums in a register)
    const double cost = per_wave * (steps + 0.35);
    if (cost < best) {
      best = cost;
      p->shares = s;
      p->rows_per_wg = rows;
    }
  }
  if (p->shares == 0) return false;
  p->grid = (d.out + p->rows_per_wg - 1) / p->rows_per_wg;
  p->esz = entry_bytes(d);
  if (p->esz == 0 && d.b == 16) p->esz = 3;
  if ((long long)p->rows_per_wg * blocks < (p->esz == 3 ? 110 : 65)) p->esz = 0;
  const size_t cb = p->esz == 3 ? (size_t)kHigh + (1 << 15) : (size_t)p->esz << d.b;
  p->lds = std::max((size_t)(p->rows_per_wg + 1) * p->shares * 4, cb);
  return p->lds <= 160 * 1024;
}

template <int ESZ, int PAIRS>
static btc_status launch(hipStream_t q, const Dims& d, const Plan& p, const uint32_t* packed, const uint32_t* codebook,
                         const float* alpha, const float* mu, const void* x, void* y, int y_is_f32) {
  static bool attr_set = false;  // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)gemv_code_kernel<ESZ, PAIRS>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  gemv_code_kernel<ESZ, PAIRS><<<p.grid, kWaves * 64, p.lds, q>>>(d, packed, codebook, alpha, mu, (const uint16_t*)x, y, y_is_f32,
                                                                  p.rows_per_wg, p.shares);
  return launch_status();
}

template <int ESZ>
static btc_status launch_any(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook, const float* alpha,
                             const float* mu, const void* x, void* y, int y_is_f32) {
  static bool attr_set = false;  // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)gemv_code_any_kernel<ESZ>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  gemv_code_any_kernel<ESZ><<<std::min(256, (d.out + kWaves - 1) / kWaves), kWaves * 64, any_lds_bytes(d), q>>>(
      d, packed, codebook, alpha, mu, (const uint16_t*)x, y, y_is_f32);
  return launch_status();
}

template <int ESZ>
static btc_status launch_esz(hipStream_t q, const Dims& d, const Plan& p, const uint32_t* packed, const uint32_t* codebook,
                             const float* alpha, const float* mu, const void* x, void* y, int y_is_f32) {
  switch (d.v / 2) {
    case 6: return launch<ESZ, 6>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    case 7: return launch<ESZ, 7>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    case 8: return launch<ESZ, 8>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    case 9: return launch<ESZ, 9>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    case 10: return launch<ESZ, 10>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    default: return BTC_ERR_UNSUPPORTED;
  }
}

}  // namespace code

bool gemv_code_covers(const Dims& d) {
  if (d.v < 2 || (d.v & 1) || d.v > 32 || d.b > 16) return false;
  if ((long long)d.out * d.wpr * 4 >= (1LL << 31)) return false;
  code::Plan p;
  if (d.in <= code::kMaxIn && code::make_plan(d, &p)) return true;
  return d.in <= code::kMaxIn && d.nchunks <= 64 * code::kMaxSteps && code::any_lds_bytes(d) <= 160 * 1024;
}

btc_status gemv_code(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                     const float* alpha, const float* mu, const void* x, void* y, int y_is_f32) {
  using namespace code;
  Plan p;
  if (make_plan(d, &p)) {
    if (p.esz == 4) return launch_esz<4>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    if (p.esz == 3) return d.v == 18 ? launch<3, 9>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32)
                                     : launch<3, 10>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    if (p.esz == 2) return launch_esz<2>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
    return launch_esz<0>(q, d, p, packed, codebook, alpha, mu, x, y, y_is_f32);
  }
  switch (entry_bytes(d)) {
    case 4: return launch_any<4>(q, d, packed, codebook, alpha, mu, x, y, y_is_f32);
    case 2: return launch_any<2>(q, d, packed, codebook, alpha, mu, x, y, y_is_f32);
    default: return launch_any<0>(q, d, packed, codebook, alpha, mu, x, y, y_is_f32);
  }
}

}  // namespace btc
