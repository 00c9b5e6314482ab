// Decode product on the matrix cores for 2..16 activation rows in one kernel; chunk lengths 9 and 10, 7..10 index bits, rows of
// any length.  The operand scheme (table entries in LDS that ARE the A operands, chunk-aligned permutation of the
// contraction index, super-groups of 64 chunks) is that of btc_gemv_mfma.hip.
//
// There the columns are cut into tiles whose partial sums a second kernel adds: that launch and its trip through memory are
// 3.5 us of the 10 that a call on 4096 x 4096 takes.  Here the sixteen waves of a workgroup are RB blocks of 16 weight rows
// times KS shares of the columns (RB KS = 16), the workgroup walks ALL columns, and the KS sums meet in LDS.  The activation
// rows are staged in operand order NJ = 2, 4, 8 or 16 to a chunk, S super-groups at a time (S <= 64 / NJ: a thread takes four
// chunks of a row, five 16-byte loads whose words map to operand places at compile time), the next S on their way while
// these are contracted.
//
// A row of activations may start on any even address (rows of odd length), a row of codes on any: the loads start at the
// word below and the words are shifted into place.
#pragma once
#include <algorithm>

#include "btc_mfma_decode.h"

namespace btc {
namespace few {

using namespace skinny;   // operand types, table geometry

constexpr int kLds = 160 * 1024 - 256;

// What the activations are: fp16, bf16, or 8-bit codes of rows  lo + step * code  (exact as fp16 operands).
enum { kF16 = 0, kBf16 = 1, kCodes = 2 };

struct CodeArgs {
  const float *wsum, *lo, *step;                                 // sum of each weight row; offset and step of each row of codes
};

template <int NJ>
constexpr int sg_bytes() { return kSG * NJ * 20; }

constexpr int max_sg(int nj) { return 64 / nj; }                 // super-groups staged at a time: one task per thread

// Place of (chunk c, row 0) in X8, in bytes: 16 / NJ chunks share 256 bytes (every bank once), turned so that the quads of
// chunks that a wave writes together meet different banks.
template <int NJ>
__host__ __device__ constexpr uint32_t x8_place(int c) {
  constexpr int G = 16 / NJ;
  const int quad = c >> 2;
  const int turn = NJ == 8 ? quad & 1 : NJ == 4 ? quad & 3 : NJ == 2 ? (quad >> 1) & 3 : 0;
  return (uint32_t)((c / G) * 256 + ((c % G) ^ turn) * (NJ * 16));
}

template <int V, int B, int NJ, int T>
__global__ __launch_bounds__(kWaves * 64) void gemv_few_kernel(
    Dims d, const uint32_t* __restrict__ packed, const uint32_t* __restrict__ codebook, const float* __restrict__ alpha,
    const float* __restrict__ mu, const void* __restrict__ x, CodeArgs ca, int batch, int ks_log2, int S,
    void* __restrict__ y, int y_dtype) {
  constexpr bool BF16 = T == kBf16;
  constexpr int kSize = T == kCodes ? 1 : 2;                     // bytes of an activation
  static_assert(V == 9 || V == 10, "chunk lengths 9 (one tail value) and 10 (two)");
  using C = Cfg<B>;
  constexpr int NW = C::kNW;
  static_assert(Cfg<B>::kE8Bytes + max_sg(NJ) * sg_bytes<NJ>() <= kLds, "LDS budget");
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* E8 = smem;                                      // [code][copy] x 16 B: values 0..7 as +-1 (+ 2 flag bits)
  unsigned char* X8 = smem + C::kE8Bytes;                        // x8_place(chunk) + row x 16 B
  uint32_t* X2 = (uint32_t*)(X8 + S * kSG * NJ * 16);            // [chunk / 4][NJ rows][chunk % 4] x 4 B
  float* red = (float*)X8;                                       // at the end: [wave][NJ rows][16 weight rows], and
  float* xs_w = red + kWaves * NJ * 16;                             // [wave][NJ]: sums of the activations

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, q = lane >> 4;
  const int KS = 1 << ks_log2, RB = kWaves >> ks_log2;
  const int rb = wave >> ks_log2, ks = wave & (KS - 1);
  const int n0 = blockIdx.x * (16 * RB);                         // first weight row of the workgroup
  const int sgs = (d.nchunks + kSG - 1) / kSG;

  // ---- every load of the prologue first
  constexpr int NC = (C::kK2 + kWaves * 64 - 1) / (kWaves * 64);
  uint32_t cw[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int code = tid + k * kWaves * 64;
    cw[k] = code < C::kK2 ? codebook[code] : 0u;
  }
  const int my_row = tid & (NJ - 1), my_quad = tid / NJ;         // staging: four chunks of one activation row
  const bool stager = my_row < batch && my_quad < S * (kSG / 4);
  const uint32_t row_byte = (uint32_t)my_row * (uint32_t)d.in * kSize;
  const uint32_t off_by = row_byte & 3u;                         // a row may start inside a word (its quads of chunks keep that)
  const __amdgpu_buffer_rsrc_t rX =
      __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)(((long long)batch * d.in * kSize + 3) & ~3LL), kRsrcFlags);
  constexpr int kLoads = T == kCodes ? 3 : 5;
  uint4 xv[kLoads];
  uint32_t xn = 0u;                                              // the word behind them
  auto load_x = [&](int first) {                                 // first: super-group
    const int k = (first * kSG + 4 * my_quad) * V;
    const uint32_t off = row_byte - off_by + (uint32_t)k * kSize;
#pragma unroll
    for (int m = 0; m < kLoads; ++m)
      xv[m] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(rX, stager && k + 16 / kSize * m < d.in + (T == kCodes ? 3 : 0) ? off + 16u * m : kOob, 0, 0));
    if constexpr (T != kCodes)
      xn = __builtin_amdgcn_raw_buffer_load_b32(rX, off_by && stager && k + 39 < d.in ? off + 80u : kOob, 0, 0);
  };
  load_x(0);
  const __amdgpu_buffer_rsrc_t rP =
      __builtin_amdgcn_make_buffer_rsrc((void*)packed, 0, (int)((uint32_t)d.out * (uint32_t)d.wpr * 4u), kRsrcFlags);
  const int n_row = n0 + rb * 16 + i;
  auto load_words = [&](int sg, uint32_t (&W)[NW]) {
    const int cs = sg * kSG;
    const int w0 = ((cs + 16 * q) * B) >> 5;
    const bool row_ok = sg < sgs && n_row < d.out;
    // does every lane's window lie inside its row?  (uniform; false only in the last super-group of a row)
    if ((((cs + kSG) * B + 31) >> 5) <= d.wpr) {
      const uint32_t off = row_ok ? ((uint32_t)n_row * (uint32_t)d.wpr + (uint32_t)w0) * 4u : kOob;
      const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rP, off, 0, 0));
      W[0] = v.x; W[1] = v.y; W[2] = v.z; W[3] = v.w;
      if constexpr (NW == 5) W[4] = __builtin_amdgcn_raw_buffer_load_b32(rP, off + 16u, 0, 0);
    } else {
#pragma unroll
      for (int k = 0; k < NW; ++k)
        W[k] = __builtin_amdgcn_raw_buffer_load_b32(
            rP, (row_ok && w0 + k < d.wpr) ? ((uint32_t)n_row * (uint32_t)d.wpr + (uint32_t)(w0 + k)) * 4u : kOob, 0, 0);
    }
  };
  uint32_t Wc[NW], Wx[NW];
  load_words(ks, Wc);
  const int n_out = n0 + (tid & (16 * RB - 1));                  // this thread's weight row in the epilogue
  const float my_alpha = n_out < d.out ? alpha[n_out] : 0.f, my_mu = n_out < d.out ? mu[n_out] : 0.f;
  float my_wsum = 0.f, my_lo = 0.f, my_step = 0.f;
  if constexpr (T == kCodes) {
    if (n_out < d.out) my_wsum = ca.wsum[n_out];
    if (tid < batch) my_lo = ca.lo[tid], my_step = ca.step[tid];
  }

  // ---- table: a thread writes all copies of its entries
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int code = tid + k * kWaves * 64;
    if (code < C::kK2) {
      const uint32_t npat = ~cw[k];
      uint32_t p[4];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        p[m] = (BF16 ? 0x3F803F80u : 0x3C003C00u) | ((npat << (15 - 2 * m)) & 0x8000u) | ((npat << (30 - 2 * m)) & 0x80000000u);
      // the signs of values 8 and 9 ride in the lowest mantissa bit of values 0 and 1
      p[0] |= ((npat >> 8) & 1u) | (V == 10 ? ((npat >> 9) & 1u) << 16 : 0u);
#pragma unroll
      for (int c = 0; c < C::kRep; ++c)   // copies in an order rotated by the code: neighbouring threads write different bank groups
        *(uint4*)(E8 + (code * C::kRep + ((c + code) & (C::kRep - 1))) * 16) = make_uint4(p[0], p[1], p[2], p[3]);
    }
  }

  // ---- activations into operand order, zeros past the end of a row (which makes the rest of the last chunk and the chunks
  // past the end contribute nothing)
  float xsum = 0.f;
  auto put_x = [&](int first) {
    if (!stager) return;
    uint32_t w[21];
    if constexpr (T == kCodes) {                                 // four codes a word -> two pairs of fp16
      uint32_t c[13];
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        c[4 * m] = xv[m].x; c[4 * m + 1] = xv[m].y; c[4 * m + 2] = xv[m].z; c[4 * m + 3] = xv[m].w;
      }
      c[12] = 0u;
      const f16x2 bias = {(_Float16)1024.0f, (_Float16)1024.0f};
#pragma unroll
      for (int u = 0; u < 10; ++u) {
        const uint32_t p = __builtin_amdgcn_alignbit(c[u + 1], c[u], off_by * 8u);
#pragma unroll
        for (int h = 0; h < 2; ++h)                              // 0x6400 | code is 1024 + code
          w[2 * u + h] = __builtin_bit_cast(
              uint32_t, (f16x2)(__builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x64646464u, p, h ? 0x04030402u : 0x04010400u)) - bias));
      }
      w[20] = 0u;
    } else {
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        w[4 * m] = xv[m].x; w[4 * m + 1] = xv[m].y; w[4 * m + 2] = xv[m].z; w[4 * m + 3] = xv[m].w;
      }
      w[20] = xn;
#pragma unroll
      for (int u = 0; u < 20; ++u) w[u] = __builtin_amdgcn_alignbit(w[u + 1], w[u], off_by * 8u);
    }
    constexpr int kWords = 2 * V;                                // words of four chunks
    if ((first + S) * (kSG * V) > d.in) {                        // uniform: this pass reaches past the rows' end
      const int k = (first * kSG + 4 * my_quad) * V;
#pragma unroll
      for (int u = 0; u < kWords; ++u)
        if (k + 2 * u + 1 >= d.in) w[u] = k + 2 * u >= d.in ? 0u : w[u] & 0xFFFFu;
    }
#pragma unroll
    for (int u = 0; u < kWords; ++u) xsum = pair_sum<BF16>(w[u], xsum);
    uint32_t tail[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t o[4];
      if constexpr (V == 10) {
#pragma unroll
        for (int m = 0; m < 4; ++m) o[m] = w[5 * e + m];
        tail[e] = w[5 * e + 4];
      } else {                                                   // chunk e starts at value 9 e; its second tail slot is zero
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int at = 9 * e + 2 * m;
          o[m] = (at & 1) ? __builtin_amdgcn_alignbit(w[at / 2 + 1], w[at / 2], 16u) : w[at / 2];
        }
        tail[e] = ((9 * e + 8) & 1) ? w[(9 * e + 8) / 2] >> 16 : w[(9 * e + 8) / 2] & 0xFFFFu;
      }
      *(uint4*)(X8 + x8_place<NJ>(4 * my_quad + e) + my_row * 16) = make_uint4(o[0], o[1], o[2], o[3]);
    }
    *(uint4*)((unsigned char*)X2 + (my_quad * NJ + my_row) * 16) = make_uint4(tail[0], tail[1], tail[2], tail[3]);
  };

  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  const uint32_t shift = (uint32_t)(16 * q * B) & 31u;           // where the lane's first index starts in its window
  typedef __attribute__((address_space(3))) const u32x4* lds_u4;
  const uint32_t e8_lane32 = (uint32_t)(uintptr_t)(lds_u4)(const u32x4*)(E8 + (i & (C::kRep - 1)) * 16);
  const int col = i < batch ? i : 0;                             // (columns past the batch: any row will do)
  const uint32_t x8_lane = x8_place<NJ>(16 * q) + (uint32_t)col * 16u, x2_lane = (uint32_t)(q * 4 * NJ + col) * 16u;
  uint32_t one2;                                                 // 1.0 | 1.0 (chunk length 9: the second tail slot is 0.0)
  if constexpr (V == 10) asm volatile("s_mov_b32 %0, %1" : "=s"(one2) : "i"(BF16 ? 0x3f803f80 : 0x3c003c00));
  else asm volatile("s_mov_b32 %0, %1" : "=s"(one2) : "i"(BF16 ? 0x00003f80 : 0x00003c00));

  for (int first = 0; first < sgs; first += S) {
    put_x(first);
    load_x(first + S);                                           // (two passes ahead: slower, the registers are full)
    __syncthreads();
    for (int g = ks; g < S; g += KS) {
      // the next super-group of this wave: in this pass or at the front of the next
      load_words(g + KS < S ? first + g + KS : first + S + ks, Wx);
      if (first + g < sgs) {
        uint32_t Wn[NW];                                         // the lane's 16 indices, aligned to bit 0
#pragma unroll
        for (int k = 0; k + 1 < NW; ++k) Wn[k] = __builtin_amdgcn_alignbit(Wc[k + 1], Wc[k], shift);
        Wn[NW - 1] = Wc[NW - 1] >> shift;
        const unsigned char* x8 = X8 + g * (kSG * NJ * 16);
        const unsigned char* x2 = (const unsigned char*)X2 + g * (kSG * NJ * 4) + x2_lane;
        static_for<0, 4>([&](auto t_c) {
          constexpr int t = decltype(t_c)::value;
          uint4 a8[4], b8[4];
          uint32_t a2w[4];
          static_for<0, 4>([&](auto w_c) {
            constexpr int w = decltype(w_c)::value;
            constexpr int u = 4 * t + w;
            // (only NJ = 2 has a turn that depends on q: its bits are disjoint from the others)
            b8[w] = *(const uint4*)(x8 + (NJ == 2 ? x8_lane ^ x8_place<NJ>(u) : x8_lane + x8_place<NJ>(u)));
            constexpr int pos = u * B;
            constexpr int wi = pos >> 5, sh = pos & 31;
            uint32_t src = Wn[wi];
            if constexpr (sh + B > 32) src = __builtin_amdgcn_alignbit(Wn[wi + 1 < NW ? wi + 1 : wi], Wn[wi], (uint32_t)sh);
            uint32_t code, addr;
            asm("v_bfe_u32 %0, %1, %2, %3" : "=v"(code) : "v"(src), "n"(sh + B > 32 ? 0 : sh), "n"(B));
            asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(addr) : "v"(code), "n"(B <= 8 ? 8 : B == 9 ? 7 : 6), "v"(e8_lane32));
            a8[w] = __builtin_bit_cast(uint4, *(lds_u4)(uintptr_t)addr);
          });
          const uint4 b2 = *(const uint4*)(x2 + t * (NJ * 16));
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            uint32_t flags;
            asm("v_and_b32 %0, 0x10001, %1" : "=v"(flags) : "v"(a8[w].x));
            a2w[w] = (flags << 15) | one2;                       // (not in assembly: an MFMA may follow at once)
            a8[w].x &= 0xFFFEFFFEu;
          }
          acc[0] = mfma16<BF16>(a8[0], b8[0], acc[0]);
          acc[1] = mfma16<BF16>(a8[1], b8[1], acc[1]);
          acc[0] = mfma16<BF16>(a8[2], b8[2], acc[0]);
          acc[1] = mfma16<BF16>(a8[3], b8[3], acc[1]);
          acc[0] = mfma16<BF16>(make_uint4(a2w[0], a2w[1], a2w[2], a2w[3]), b2, acc[0]);
        });
      }
#pragma unroll
      for (int k = 0; k < NW; ++k) Wc[k] = Wx[k];
    }
    __syncthreads();                                             // everybody is done with the pass
  }

  // ---- the column shares meet in LDS: lane (j, q) holds weight rows 4 q .. 4 q + 3 for activation row j
#pragma unroll
  for (int o = 32; o >= NJ; o >>= 1) xsum += __shfl_xor(xsum, o, 64);      // (lane l: row l % NJ)
  if (i < NJ) {
    const f32x4 v = acc[0] + acc[1];
    *(float4*)(red + (wave * NJ + i) * 16 + 4 * q) = make_float4(v[0], v[1], v[2], v[3]);
    if (q == 0) xs_w[wave * NJ + i] = xsum;
  }
  float* const lo_step = xs_w + kWaves * NJ;                     // [2][NJ]
  if (T == kCodes && tid < batch) {
    lo_step[tid] = my_lo;
    lo_step[NJ + tid] = my_step;
  }
  __syncthreads();
  const int rows_log2 = 8 - ks_log2, row = tid & ((1 << rows_log2) - 1);      // 16 RB weight rows
  if (n_out < d.out) {
    for (int j = tid >> rows_log2; j < batch; j += 1024 >> rows_log2) {
      float sum = 0.f, sx = 0.f;
      const float* p = red + ((((row >> 4) << ks_log2) * NJ + j) * 16 + (row & 15));
      for (int s = 0; s < KS; ++s) sum += p[s * (NJ * 16)];
#pragma unroll
      for (int s = 0; s < kWaves; ++s) sx += xs_w[s * NJ + j];
      float v = my_alpha * sum + my_mu * sx;
      if constexpr (T == kCodes) v = lo_step[NJ + j] * v + lo_step[j] * my_wsum;
      const size_t at = (size_t)j * d.out + n_out;
      if (y_dtype == BTC_F32) ((float*)y)[at] = v;
      else if (y_dtype == BTC_BF16) ((__hip_bfloat16*)y)[at] = __float2bfloat16(v);
      else ((__half*)y)[at] = __float2half_rn(v);
    }
  }
}

struct Plan {
  int ks_log2, S, grid;
  double us;
};

// The number of column shares that makes the call shortest.  Microseconds, fitted to measurements on 500 x 1000 .. 28672 x
// 8192: rounds of workgroups (one per compute unit), each with its table and tail, its passes and its super-groups; the
// index stream.
static Plan make_plan(const Dims& d, int batch) {
  const int nj = batch <= 2 ? 2 : batch <= 4 ? 4 : batch <= 8 ? 8 : 16;
  const int sgs = (d.nchunks + kSG - 1) / kSG;
  const double unit = nj == 2 || nj == 16 ? 1.3 : 1.62;          // a super-group on each of the sixteen waves
  Plan best{0, 0, 0, 1e30};
  for (int l = 4; l >= 0; --l) {
    const int KS = 1 << l, rows = 16 * (kWaves >> l);
    const int per_wave = (sgs + KS - 1) / KS;
    int S = std::min(max_sg(nj) / KS, per_wave) * KS;
    if (S == 0) continue;
    const int passes = (sgs + S - 1) / S;
    S = (per_wave + passes - 1) / passes * KS;                   // passes of equal length
    const int grid = (d.out + rows - 1) / rows;
    const int rounds = (grid + 255) / 256;
    const double us = 1.0 + rounds * (3.2 + passes * (0.4 + 0.03 * std::min(S, sgs) * nj) + unit * per_wave) +
                      0.09e-6 * d.out * d.wpr * 4;
    if (us < best.us) best = Plan{l, S, grid, us};
  }
  return best;
}

template <int V, int B, int NJ, int T>
static btc_status launch(hipStream_t q, const Dims& d, const Plan& p, const uint32_t* packed, const uint32_t* codebook,
                         const float* alpha, const float* mu, const void* x, const CodeArgs& ca, int batch, void* y, int y_dtype) {
  static bool attr_set = false;  // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)gemv_few_kernel<V, B, NJ, T>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  const int x_bytes = std::max(p.S * sg_bytes<NJ>(), kWaves * NJ * 68 + 8 * NJ);
  gemv_few_kernel<V, B, NJ, T><<<p.grid, kWaves * 64, Cfg<B>::kE8Bytes + x_bytes, q>>>(d, packed, codebook, alpha, mu, x, ca,
                                                                                     batch, p.ks_log2, p.S, y, y_dtype);
  return launch_status();
}

template <int V, int B, int T>
static btc_status launch_vb(hipStream_t q, const Dims& d, const Plan& p, const uint32_t* packed, const uint32_t* codebook,
                            const float* alpha, const float* mu, const void* x, const CodeArgs& ca, int batch, void* y, int y_dtype) {
  if (batch <= 2) return launch<V, B, 2, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
  if (batch <= 4) return launch<V, B, 4, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
  if (batch <= 8) return launch<V, B, 8, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
  return launch<V, B, 16, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
}

template <int T>
static btc_status run(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook, const float* alpha,
                      const float* mu, const void* x, const CodeArgs& ca, int batch, void* y, int y_dtype) {
  const Plan p = make_plan(d, batch);
  switch (d.v * 16 + d.b) {
    case 10 * 16 + 7: return launch_vb<10, 7, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 10 * 16 + 8: return launch_vb<10, 8, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 10 * 16 + 9: return launch_vb<10, 9, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 10 * 16 + 10: return launch_vb<10, 10, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 9 * 16 + 7: return launch_vb<9, 7, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 9 * 16 + 8: return launch_vb<9, 8, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 9 * 16 + 9: return launch_vb<9, 9, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    case 9 * 16 + 10: return launch_vb<9, 10, T>(q, d, p, packed, codebook, alpha, mu, x, ca, batch, y, y_dtype);
    default: return BTC_ERR_UNSUPPORTED;
  }
}

}  // namespace few
}  // namespace btc
