// Prefill product that decodes the weights inside the contraction:  Y[M][out] = X[M][in] . W_hat^T, for chunk
// lengths 9 and 10 and up to 10 index bits; 16-bit activations, or 8-bit activation codes (btc_gemm_aq).
//
// The weights reach a compute unit as what they are stored as -- b index bits for v weights -- and become matrix-core
// operands in LDS; nothing of the sign matrix B_hat (Algorithm "Binary Transformation and Compression":
// W_hat = alpha * B_hat + mu) is ever written to memory.  alpha and mu are applied in fp32 afterwards.
//
// A workgroup owns BM = 128 MA activation rows x BN = 32 NF weight rows and walks k-tiles of KT columns (80 for 16-bit
// operands, 128 for codes: 160 / 128 bytes per activation row):
//   * 4 contraction waves, stacked along M, 32 MA rows each: MA x NF accumulators of MFMA 32x32 (bf16, fp16 or int8).
//     Both operands come from LDS, read one k-slice ahead of the MFMAs that use them.  A weight is one byte in LDS:
//     the int8 number itself, or the HIGH byte of +-1.0, which four byte permutes turn into eight 16-bit elements in
//     the shadow of the MFMAs.
//   * 1 loader wave issues the load-to-LDS instructions of the activation tile (memory -> LDS, no registers).
//   * 3 decoder waves: a lane owns one weight row of the tile (half a row where BN <= 64).  The row's chunk indices are
//     fetched three tiles ahead as 8-byte windows of three fields (3 b <= 30 bits), the inverted codewords looked up
//     in a 2-byte table in LDS, strung together to the tile's KT sign bits by shifts that are the same for all rows,
//     and every 8 bits spread over 8 bytes by a second table of 2 KB (by a 24-bit multiply and a byte permute per 4
//     bits where LDS has no room for it).
// Three tile buffers, one barrier per tile: tile t + 2 is staged while tile t is contracted.
// LDS layout: as the load-to-LDS instruction wants it (lane l of a wave writes 16 bytes at base + 16 l), so bank
// conflicts are avoided by choosing WHICH 16 bytes a lane fetches: 160-byte activation rows keep piece p at
// p ^ ((row / 8) % 2), 128-byte rows at p ^ ((row / 2) % 8); 80-byte weight rows are conflict-free as they stand (5
// pieces of 16, read 16 bytes = two k-slices at a time), 128-byte ones are swizzled like the codes.
//
// k split: where the output tiles leave compute units idle, the k-tiles of an output tile are dealt to several
// workgroups, whose raw sums a second kernel adds in split order.
//
// What bounds it: at 256 busy compute units the clock and the traffic into LDS as much as the matrix pipe (5120 x 5120 at
// M = 2048: 88 us = 1215 TFLOP/s; without the decoders 70 us, with half the activation loads 73 us -- timing-only
// builds), on few activation rows prologue, epilogue and the second pass.  Against the kernels it took over from:
// 13824 x 5120 at M = 2048 237 us (251 with the signs expanded to memory first), at M = 512 69 us (85 with a table of
// expanded codewords and activations through registers); the seven products of a 7B-shaped layer at v = 9, M = 203
// 212 us (generic kernel: 2510); of a 13B-shaped layer on codes at M = 1024 541 us (825 as 16-bit copies of the codes).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>

#include "btc_internal.h"

namespace btc {
namespace dec {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) void lds_void;

enum Op { kF16 = 0, kBF16 = 1, kI8 = 2 };

constexpr int kMW = 4;                  // contraction waves
constexpr int kThreads = 512;           // + 1 loader wave + 3 decoder waves
constexpr uint32_t kOob = 0x80000000u;  // buffer offset that is always out of range
constexpr int kRsrcFlags = 0x00020000;
constexpr int kLut = 2048;              // bytes of the table that spreads 8 sign bits over 8 bytes

template <int OP>
struct Geo {
  static constexpr int KT = OP == kI8 ? 128 : 80;          // columns per k-tile
  static constexpr int XR = OP == kI8 ? 128 : 160;         // bytes of a staged activation row
  static constexpr int WR = OP == kI8 ? 128 : 80;          // bytes of a decoded weight row
  static constexpr int NS = OP == kI8 ? 4 : 5;             // k-slices of a tile
  static constexpr int XS = OP == kI8 ? 1 : 2;             // bytes of an activation
  static constexpr int LPR = XR / 16;                      // load instructions per 64 rows
};

__device__ __forceinline__ uint32_t bf16_bits(float v) { return (uint32_t)__builtin_bit_cast(uint16_t, __float2bfloat16(v)); }
__device__ __forceinline__ uint32_t f16_bits(float v) { return (uint32_t)__builtin_bit_cast(uint16_t, __float2half_rn(v)); }

// LDS traffic inside one wave (writes by some lanes, reads by others): LDS operations of a
// wave complete in order, so waiting for them is enough; the fences pin the compiler.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }

// 8 weight bytes (the high bytes of +-1.0) -> 8 16-bit operand elements; `low` holds the
// low byte of 1.0 in the operand's format (0x80 for bf16, 0x00 for fp16) in its byte 0.
__device__ __forceinline__ u32x4 widen_weights(uint32_t lo, uint32_t hi, uint32_t low) {
  u32x4 r;
  r.x = __builtin_amdgcn_perm(lo, low, 0x05000400u);
  r.y = __builtin_amdgcn_perm(lo, low, 0x07000600u);
  r.z = __builtin_amdgcn_perm(hi, low, 0x05000400u);
  r.w = __builtin_amdgcn_perm(hi, low, 0x07000600u);
  return r;
}

// 64 lanes x 16 bytes from memory straight into LDS: lane l's bytes land at dst + 16 l (dst is
// wave-uniform); an out-of-range offset stores zeros.  The host pass of the compiler does not
// know the 16-byte form of the builtin, so it only sees an empty body.
__device__ __forceinline__ void load_to_lds_16(const __amdgpu_buffer_rsrc_t& rsrc, unsigned char* dst, uint32_t voffset,
                                               int soffset) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)dst, 16, voffset, soffset, 0, 0);
#else
  (void)rsrc; (void)dst; (void)voffset; (void)soffset;
#endif
}

template <int OP>
struct AccOf { using type = f32x16; };
template <>
struct AccOf<kI8> { using type = i32x16; };

template <int OP>
__device__ __forceinline__ typename AccOf<OP>::type mfma(const u32x4& a, const u32x4& b, const typename AccOf<OP>::type& c) {
  if constexpr (OP == kBF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else if constexpr (OP == kF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(i32x4, a), __builtin_bit_cast(i32x4, b), c, 0, 0, 0);
}

// sum of the elements of one activation word, added to a running sum (fp32, or an integer for codes)
template <int OP, class T>
__device__ __forceinline__ T word_sum(uint32_t w, T acc) {
  if constexpr (OP == kBF16) {
    const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), one, acc, false);
  } else if constexpr (OP == kF16) {
    const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w), one, acc, false);
  } else {
    return __builtin_amdgcn_udot4(w, 0x01010101u, acc, false);
  }
}

// What the epilogue of the products on codes needs besides alpha and mu (see btc_gemm_aq).
struct CodeArgs {
  const float* wsum;
  const float* lo;
  const float* step;
};

// LDS: spreading table (LUT), codeword table (2 bytes per entry), activation tiles [3][BM][XR], weight tiles [3][BN][WR].
// The largest 16-bit tile leaves 2560 bytes for the tables: both for up to 8 index bits, else the codewords alone.
constexpr int kLdsMax = 160 * 1024;
template <int OP, int MA, int NF>
constexpr int tile_bytes() { return 3 * 128 * MA * Geo<OP>::XR + 3 * 32 * NF * Geo<OP>::WR; }
template <int OP, int MA, int NF>
constexpr bool tight() { return tile_bytes<OP, MA, NF>() + kLut + 2048 > kLdsMax; }
template <int OP, int MA, int NF, bool LUT>
constexpr int table_bytes() { return (LUT ? kLut : 0) + (LUT && tight<OP, MA, NF>() ? 512 : 2048); }
template <int OP, int MA, int NF, bool LUT>
constexpr int lds_bytes() { return tile_bytes<OP, MA, NF>() + table_bytes<OP, MA, NF, LUT>(); }

// waves per SIMD that the registers are cut for: two workgroups per compute unit where two of them fit LDS
template <int OP, int MA, int NF>
constexpr int waves_per_simd() { return 2 * lds_bytes<OP, MA, NF, true>() <= kLdsMax ? 4 : 2; }

template <int OP, int MA, int NF, bool LUT>
__global__ __launch_bounds__(kThreads, (waves_per_simd<OP, MA, NF>())) void gemm_decode_kernel(
    Dims d, const uint32_t* __restrict__ packed, const uint32_t* __restrict__ codebook, const float* __restrict__ alpha,
    const float* __restrict__ mu, const void* __restrict__ X, CodeArgs ca, int M, void* __restrict__ Y, int y_dtype,
    int m_blocks, int n_blocks, int gm, int per_split, int tiles_per_split, const float* __restrict__ rs_all,
    float* __restrict__ part) {
  using G = Geo<OP>;
  using Acc = typename AccOf<OP>::type;
  constexpr int BM = 128 * MA, BN = 32 * NF;
  constexpr int KT = G::KT, XB = BM * G::XR, WB = BN * G::WR;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kTab = LUT ? kLut : 0;                   // offsets in LDS
  constexpr int kX0 = table_bytes<OP, MA, NF, LUT>(), kW0 = kX0 + 3 * XB;
  uint16_t* const tab = (uint16_t*)(smem + kTab);

  int mb, nb, sp;                                        // activation-row block, weight-row block, k split
  {
    // Workgroup L of a split runs on XCD L % 8 (every split has a multiple of eight workgroups).  The XCDs form a grid
    // of gm x gn (gm gn = 8): XCD (xm, xn) takes the m blocks = xm (mod gm) and the n blocks = xn (mod gn), so that the
    // chip reads the index stream gm times and the activations gn times through its eight separate L2 caches.
    sp = blockIdx.x / per_split;
    const int L = blockIdx.x - sp * per_split;
    const int x = L & 7, sq = L >> 3;
    const int gn = 8 / gm;
    const int xm = x % gm, xn = x / gm;
    const int pm = (m_blocks + gm - 1) / gm;
    mb = xm + gm * (sq % pm);
    nb = xn + gn * (sq / pm);
    if (mb >= m_blocks || nb >= n_blocks) return;
  }
  const int m0 = mb * BM, n0 = nb * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntiles = (d.in + KT - 1) / KT;
  const int t_begin = sp * tiles_per_split;              // (the host makes every split non-empty)
  const int nt = min(ntiles, t_begin + tiles_per_split) - t_begin;

  if (wave == kMW) {
    // =============================== loader wave ===============================
    constexpr int LPR = G::LPR, XJ = 2 * MA * LPR;       // loads of a tile
    static_assert(XJ <= 63, "the number of loads of a tile must fit the wait counter");
    const __amdgpu_buffer_rsrc_t rX =
        __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)((long long)M * d.in * G::XS), kRsrcFlags);
    // Load i of a group of 64 rows fills positions 64 i + lane of the group (LPR per row).  Rows m >= M need no
    // test of their own: X is row-major, so they lie past the end of the buffer and the hardware range check
    // makes the load store zeros.
    uint32_t xv[LPR];                                    // byte offset of this lane's piece in tile 0, first group
    int xk[LPR];                                         // its first column inside a tile (for the ragged last tile)
#pragma unroll
    for (int i = 0; i < LPR; ++i) {
      const int g = 64 * i + lane;
      const int row = g / LPR, pos = g - LPR * row;
      const int p = OP == kI8 ? pos ^ ((row >> 1) & 7) : pos ^ ((row >> 3) & 1);
      xk[i] = p * (16 / G::XS);
      xv[i] = (uint32_t)((long long)(m0 + row) * d.in * G::XS + 16 * p);
    }
    const uint32_t group = (uint32_t)(64 * d.in * G::XS);
    auto issue = [&](int t, int buf) {
      if (t >= nt) return;                               // (uniform)
      unsigned char* const xb = smem + kX0 + buf * XB;
      const int k0 = (t_begin + t) * KT;
      if (k0 + KT <= d.in) {                             // the whole tile lies inside the rows: scalar column offset
#pragma unroll
        for (int g = 0; g < 2 * MA; ++g)
#pragma unroll
          for (int i = 0; i < LPR; ++i)
            load_to_lds_16(rX, xb + (g * LPR + i) * 1024, xv[i] + (uint32_t)g * group, k0 * G::XS);
      } else {
        // `in` is a multiple of 16 for this kernel, so a piece lies wholly inside or outside the row
#pragma unroll
        for (int g = 0; g < 2 * MA; ++g)
#pragma unroll
          for (int i = 0; i < LPR; ++i) {
            const uint32_t off = k0 + xk[i] >= d.in ? kOob : xv[i] + (uint32_t)g * group + (uint32_t)(k0 * G::XS);
            load_to_lds_16(rX, xb + (g * LPR + i) * 1024, off, 0);
          }
      }
    };
    // Tile t lives in buffer t % 3.  Its loads are issued right after the barrier that ends tile
    // t - 3 (whose buffer it takes over) and must have landed at the barrier that ends tile t - 1.
    issue(0, 0);
    issue(1, 1);
    __builtin_amdgcn_s_barrier();                        // the tables are complete
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();                        // tiles 0 and 1 are in LDS
    int buf = 2;
    for (int t = 0; t < nt; ++t) {
      issue(t + 2, buf);
      buf = buf == 2 ? 0 : buf + 1;
      // everything but the loads just issued has landed (a wave's loads complete in order)
      if (t + 2 >= nt) wait_vmcnt<0>();
      else wait_vmcnt<XJ>();
      __builtin_amdgcn_s_barrier();                      // tile t consumed, tile t + 1 in LDS
    }
    return;
  }

  const uint32_t pair = OP == kI8 ? 0x0000FF01u : OP == kBF16 ? 0x0000BF3Fu : 0x0000BC3Cu;   // bytes of +1 and -1
  auto spread = [&](uint32_t n4) {                       // 4 sign bits -> 4 bytes
    return __builtin_amdgcn_perm(0u, pair, __umul24(n4, 0x204081u) & 0x01010101u);
  };
  auto build_tables = [&](int first) {                   // by all waves but the loader
    for (int k = first; k < (1 << d.b); k += kThreads - 64)
      tab[k] = (uint16_t)(~codebook[k] & ((1u << d.v) - 1u));          // inverted codewords: bit set => -1
    if (LUT && first < 256) *(u32x2*)(smem + 8 * first) = u32x2{spread(first & 15), spread(first >> 4)};
  };

  if (wave > kMW) {
    // =============================== decoder waves ===============================
    constexpr int HS = NF <= 2 ? 2 : 1;                  // items per weight row and tile
    constexpr int KI = KT / HS;                          // columns of an item
    constexpr int NW = KI == 40 ? 2 : KI == 64 ? 3 : KI == 80 ? 4 : 6;   // windows of three chunks that cover KI + 8 columns
    constexpr int NB = (KI + 31) / 32;                   // words of sign bits
    const int dw = wave - kMW - 1;
    const int half = HS == 2 ? dw : 0;                   // (HS = 2: BN <= 64 rows per wave, waves 0 and 1 take a half each)
    const int r = min(HS == 2 ? lane : dw * 64 + lane, BN - 1);   // (lanes without a row repeat the last one)
    const bool any = HS == 2 ? dw < 2 : dw * 64 < BN;    // (uniform) whether this wave has rows at all
    const __amdgpu_buffer_rsrc_t rP =
        __builtin_amdgcn_make_buffer_rsrc((void*)packed, 0, (int)((uint32_t)d.out * (uint32_t)d.wpr * 4u), kRsrcFlags);
    // rows past the end of the matrix start past the end of the buffer: zeros, i.e. index 0
    const uint32_t row_off = (uint32_t)(n0 + r) * (uint32_t)d.wpr * 4u;
    const int b = d.b, v = d.v;
    // first chunk of the item and the columns of it that belong to the item before; both advance with the tile (the
    // same for all rows: scalar registers)
    int cj, ct;
    {
      const int k = t_begin * KT + half * KI;
      cj = k / v;
      ct = k - cj * v;
    }
    const int sj = KT / v, st = KT - sj * v;
    u32x2 win[3][NW];                                    // index windows of three tiles
    int wbit[3], wt[3];                                  // their first bit, their first column inside the first chunk
    auto fetch = [&](auto slot) {
      constexpr int S = decltype(slot)::value;
      wbit[S] = cj * b;
      wt[S] = ct;
#pragma unroll
      for (int g = 0; g < NW; ++g) {
        const uint32_t off = row_off + (uint32_t)(((wbit[S] + 3 * b * g) >> 5) << 2);   // (past the stream: zeros)
        win[S][g] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rP, off, 0, 0));
      }
      cj += sj;
      ct += st;
      if (ct >= v) {
        ct -= v;
        ++cj;
      }
    };
    const uint32_t mask2 = ((1u << b) - 1u) << 1;
    uint32_t neg = 0u;                                   // weights -1 of the item so far (codes: see the epilogue)
    auto decode = [&](auto slot) {                       // into tile buffer `slot`
      constexpr int S = decltype(slot)::value;
      uint32_t W[NW];                                    // sign bits of three chunks
#pragma unroll
      for (int g = 0; g < NW; ++g) {
        const uint32_t x = __builtin_amdgcn_alignbit(win[S][g].y, win[S][g].x, (uint32_t)(wbit[S] + 3 * b * g) & 31u);
        const uint32_t p0 = *(const uint16_t*)(smem + kTab + ((x << 1) & mask2));
        const uint32_t p1 = *(const uint16_t*)(smem + kTab + ((x >> (b - 1)) & mask2));
        const uint32_t p2 = *(const uint16_t*)(smem + kTab + ((x >> (2 * b - 1)) & mask2));
        W[g] = p0 | (p1 << v) | (p2 << (2 * v));
      }
      // Window g starts at bit 3 v g of the item's string: 27 g or 30 g, which lie in the same word for both.
      uint32_t Bs[NB + 1];
      Bs[0] = W[0] | (W[1] << (3 * v));
      Bs[1] = W[1] >> (32 - 3 * v);
      if constexpr (NW > 2) Bs[1] |= W[2] << (6 * v - 32);
      if constexpr (NB > 1) {
        Bs[2] = 0u;
        if constexpr (NW > 2) Bs[2] = W[2] >> (64 - 6 * v);
        if constexpr (NW > 3) Bs[2] |= W[3] << (9 * v - 64);
      }
      if constexpr (NB > 2) {
        Bs[3] = 0u;
        if constexpr (NW > 3) Bs[3] = W[3] >> (96 - 9 * v);
        if constexpr (NW > 4) Bs[3] |= W[4] << (12 * v - 96);
      }
      if constexpr (NB > 3) {
        Bs[4] = W[4] >> (128 - 12 * v);
        Bs[4] |= W[5] << (15 * v - 128);
      }
      const uint32_t dst = (uint32_t)(kW0 + S * WB + r * G::WR);
      u32x2 o[KI / 8];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const uint32_t x = __builtin_amdgcn_alignbit(Bs[i + 1], Bs[i], (uint32_t)wt[S]);
        if constexpr (OP == kI8) neg += (uint32_t)__builtin_popcount(x);
#pragma unroll
        for (int q = 4 * i; q < 4 * i + 4 && q < KI / 8; ++q) {          // 8 bytes at a time
          const uint32_t x8 = x >> (8 * (q & 3));
          if constexpr (LUT) o[q] = *(const u32x2*)(smem + (((q & 3) ? x >> (8 * (q & 3) - 3) : x << 3) & 0x7F8u));
          else o[q] = u32x2{spread(x8 & 0xFu), spread((x8 >> 4) & 0xFu)};
        }
      }
#pragma unroll
      for (int q = 0; q < KI / 8; q += (KI % 16 == 0 ? 2 : 1)) {
        const int at = 8 * q + half * KI;
        if constexpr (OP == kI8) *(u32x4*)(smem + dst + (((at >> 4) ^ ((r >> 1) & 7)) << 4)) = u32x4{o[q].x, o[q].y, o[q + 1].x, o[q + 1].y};
        else if constexpr (KI % 16 == 0) *(u32x4*)(smem + dst + at) = u32x4{o[q].x, o[q].y, o[q + 1].x, o[q + 1].y};
        else *(u32x2*)(smem + dst + at) = o[q];
      }
    };
    if (!any) {                                          // keep the barriers only
      build_tables(tid - 64);
      __syncthreads();
      __syncthreads();
      for (int t = 0; t < nt; ++t) __syncthreads();
      return;
    }
    fetch(std::integral_constant<int, 0>{});
    fetch(std::integral_constant<int, 1>{});
    fetch(std::integral_constant<int, 2>{});
    build_tables(tid - 64);
    __syncthreads();                                     // the tables are complete
    auto step = [&](auto slot) {
      decode(slot);
      fetch(slot);                                       // three tiles on
    };
    step(std::integral_constant<int, 0>{});
    if (nt > 1) step(std::integral_constant<int, 1>{});
    __syncthreads();                                     // tiles 0 and 1 are in LDS
    auto finish = [&]() {                                // the last tile is decoded everywhere: the tables are free
      if constexpr (OP == kI8) ((uint32_t*)smem)[half * BN + r] = neg;
      __syncthreads();
    };
    int left = nt - 2;                                   // tiles that are not decoded yet
    for (;;) {
      if (left <= 0) break;
      step(std::integral_constant<int, 2>{});
      __syncthreads();                                   // a tile consumed, the next one in LDS
      if (--left <= 0) break;
      step(std::integral_constant<int, 0>{});
      __syncthreads();
      if (--left <= 0) break;
      step(std::integral_constant<int, 1>{});
      __syncthreads();
      --left;
    }
    if (nt > 1) __syncthreads();
    finish();
    return;
  }

  // ================================= contraction waves =================================
  build_tables(tid);
  __syncthreads();                                       // the tables are complete
  if (m0 + wave * 32 * MA >= M) {                        // no activation rows for this wave: keep the barriers only
    __syncthreads();
    for (int t = 0; t < nt; ++t) __syncthreads();
    return;
  }
  __builtin_amdgcn_s_setprio(2);                         // the matrix pipe is the bottleneck: issue these first
  const int h = lane >> 5, l32 = lane & 31;
  Acc acc[MA][NF];
#pragma unroll
  for (int a = 0; a < MA; ++a)
#pragma unroll
    for (int c = 0; c < NF; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][c][e] = 0;
  u32x4 afr[2][MA];                                      // [register set][fragment]

  if constexpr (OP == kI8) {
    // Lane (l32, h) holds bytes 16 h .. 16 h + 15 of a k-slice of 32, of activation row l32 of a fragment (A)
    // and of weight row l32 of a block (B): piece 2 s + h of the row, stored at that number ^ swz,
    // swz = (row / 2) % 8 -- the same for every row this lane reads (rows differ by multiples of 32).
    const int swz = (l32 >> 1) & 7;
    const uint32_t a_row = (uint32_t)(kX0 + (wave * 32 * MA + l32) * G::XR);
    const uint32_t b_row = (uint32_t)(kW0 + l32 * G::WR);
    uint32_t p_off[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) p_off[s] = (uint32_t)(((2 * s + h) ^ swz) * 16);
    u32x4 bfr[2][NF];
    auto read_slice = [&](int set, int xoff, int woff, int s) {
#pragma unroll
      for (int a = 0; a < MA; ++a) afr[set][a] = *(const u32x4*)(smem + (uint32_t)xoff + a_row + p_off[s] + a * 32 * G::XR);
#pragma unroll
      for (int c = 0; c < NF; ++c) bfr[set][c] = *(const u32x4*)(smem + (uint32_t)woff + b_row + p_off[s] + c * 32 * G::WR);
    };
    __syncthreads();                                     // tiles 0 and 1 are in LDS
    read_slice(0, 0, 0, 0);
    // the operands of slice s + 1 are read while slice s is contracted, those of the next tile's first slice right
    // after the barrier that the last slice starts with
    for (int t = 0, b0 = 0; t < nt; ++t) {
      const int b1 = b0 == 2 ? 0 : b0 + 1;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int set = s & 1;
        __builtin_amdgcn_sched_barrier(0);
        if (s < 3) {
          read_slice(set ^ 1, b0 * XB, b0 * WB, s + 1);
        } else {
          __syncthreads();                               // this tile is in registers; the next one is in LDS
          read_slice(set ^ 1, b1 * XB, b1 * WB, 0);     // (behind the last tile: bytes that nobody uses)
        }
        __builtin_amdgcn_sched_barrier(0);
        // the matrix cores take SIGNED bytes: code - 128 (top bit flipped) goes in, and the epilogue adds
        // 128 * (sum of the signs) back
#pragma unroll
        for (int a = 0; a < MA; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) afr[set][a][e] ^= 0x80808080u;
#pragma unroll
        for (int c = 0; c < NF; ++c)
#pragma unroll
          for (int a = 0; a < MA; ++a) acc[a][c] = mfma<OP>(afr[set][a], bfr[set][c], acc[a][c]);
      }
      b0 = b1;
    }
  } else {
    // Slices of a tile: 0, 1 = the two of columns 0..31; 2, 3 = of columns 32..63; 4 = columns 64..79.  A 16-byte
    // weight read covers two slices, so inside a block of 32 columns lane half h owns columns 16 h .. 16 h + 15 (first
    // eight: first slice, last eight: second slice), for both operands; the last 16 columns form a plain slice.
    // Activation piece (8 columns) of lane half h in slice s: 4 (s / 2) + 2 h + (s % 2) for s < 4, 8 + h for s = 4;
    // stored at that number ^ swz, swz = (row / 8) % 2.
    const int swz = (l32 >> 3) & 1;
    // two per-lane addresses serve all slices (the rest are instruction offsets): even slices (odd
    // slices: the neighbouring piece, bit 4 flipped) and slice 4
    const uint32_t a_base = (uint32_t)(kX0 + (wave * 32 * MA + l32) * G::XR);
    const uint32_t a_even = a_base + (uint32_t)((2 * h + swz) * 16);
    const uint32_t a_last = a_base + (uint32_t)((8 + (h ^ swz)) * 16);
    const uint32_t b_pair = (uint32_t)(kW0 + l32 * G::WR + 16 * h);   // + c * 32 * 80 + 16 s  (s = 0, 2)
    const uint32_t b_last = (uint32_t)(kW0 + l32 * G::WR + 64 + 8 * h);
    const uint32_t low = OP == kBF16 ? 0x80u : 0x00u;
    u32x4 bq[2][NF];                                     // [register set][weight block]: 16 bytes = two slices
    u32x4 bw[2];                                         // widened weights, two sets in turn
    auto read_a = [&](int set, int xoff, int s) {
      const uint32_t at = (uint32_t)xoff + (s == 4 ? a_last : (s & 1) ? (a_even ^ 16u) : a_even);
#pragma unroll
      for (int a = 0; a < MA; ++a)
        afr[set][a] = *(const u32x4*)(smem + at + a * 32 * G::XR + (s < 4 ? 64 * (s >> 1) : 0));
    };
    auto read_b = [&](int set, int woff, int s) {        // s = 0, 2: 16 bytes; s = 4: 8 bytes
#pragma unroll
      for (int c = 0; c < NF; ++c) {
        if (s < 4) {
          bq[set][c] = *(const u32x4*)(smem + ((uint32_t)woff + b_pair) + c * 32 * G::WR + 16 * s);
        } else {
          const u32x2 w = *(const u32x2*)(smem + ((uint32_t)woff + b_last) + c * 32 * G::WR);
          bq[set][c].x = w.x;
          bq[set][c].y = w.y;
        }
      }
    };
    auto widen = [&](int set, int c, int s) {
      return (s & 1) ? widen_weights(bq[set][c].z, bq[set][c].w, low) : widen_weights(bq[set][c].x, bq[set][c].y, low);
    };
    __syncthreads();                                     // tiles 0 and 1 are in LDS
    read_a(0, 0, 0);
    read_b(0, 0, 0);
    // Register sets: activations alternate per slice, weights per 16-byte read (slices 0, 2, 4); a tile
    // has an odd number of either, so both follow the tile's parity P.  Weight set of slices 0, 1 and
    // 4: P; of slices 2, 3: P ^ 1; the next tile's first read goes to P ^ 1.
    auto tile = [&](int xoff, int woff, int xnext, int wnext, auto parity) {
      constexpr int P = decltype(parity)::value;
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int aset = (P + s) & 1;
        const int bset = (s == 2 || s == 3) ? (P ^ 1) : P;
        __builtin_amdgcn_sched_barrier(0);
        if (s < 4) {
          read_a(aset ^ 1, xoff, s + 1);
          if (s == 1) read_b(P ^ 1, woff, 2);
          if (s == 3) read_b(P, woff, 4);
        } else {
          __syncthreads();                               // this tile is in registers; the next one is in LDS
          // (behind the last tile: bytes that nobody uses; reading them without a test of its own keeps the registers
          // of both sets in place -- with the test the compiler spilled 750 values)
          read_a(aset ^ 1, xnext, 0);
          read_b(P ^ 1, wnext, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s == 0) bw[0] = widen(bset, 0, s);
#pragma unroll
        for (int c = 0; c < NF; ++c) {
          // order pinned: the permutes for the next block are issued in the shadow of this block's MFMAs and write
          // registers no MFMA in flight reads
          const int g = s * NF + c;
          __builtin_amdgcn_sched_barrier(0);
          acc[0][c] = mfma<OP>(afr[aset][0], bw[g & 1], acc[0][c]);
          __builtin_amdgcn_sched_barrier(0);
          if (c + 1 < NF) bw[(g + 1) & 1] = widen(bset, c + 1, s);
          else if (s + 1 < 5) bw[(g + 1) & 1] = widen((s + 1 == 2 || s + 1 == 3) ? (P ^ 1) : P, 0, s + 1);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (MA == 2) acc[1][c] = mfma<OP>(afr[aset][1], bw[g & 1], acc[1][c]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    int b0 = 0;                                          // buffer of the current tile
    for (int t = 0; t < nt; t += 2) {
      const int b1 = b0 == 2 ? 0 : b0 + 1, b2 = b1 == 2 ? 0 : b1 + 1;
      tile(b0 * XB, b0 * WB, b1 * XB, b1 * WB, std::integral_constant<int, 0>{});
      if (t + 1 < nt) tile(b1 * XB, b1 * WB, b2 * XB, b2 * WB, std::integral_constant<int, 1>{});
      b0 = b2;
    }
  }

  // ---- epilogue.  After the last barrier the tile buffers are free; each wave uses a part of
  // them to turn its accumulators (lane = weight row n, 16 activation rows per register set)
  // into rows of Y, so that a lane stores 4 consecutive outputs at once.
  constexpr int TS = BN + 4;                                   // floats per staged row
  float* Tw = (float*)(smem + kX0) + wave * (32 * TS);         // 32 rows x BN of this wave
  float* rowp = (float*)(smem + kX0) + kMW * (32 * TS) + wave * 96 * MA;   // per activation row: sum (, step, offset)
  // With a k split the workgroup leaves its raw sums in the workspace; a second kernel finishes.
  const bool split = part != nullptr;
  if (split) {
    Y = part + (size_t)sp * M * d.out;
    y_dtype = BTC_F32;
  }
  float al[NF], mn[NF], ws[NF];
  int kc[NF];                                            // codes: 128 * (sum of the signs that met code - 128)
#pragma unroll
  for (int c = 0; c < NF; ++c) {
    const int n = n0 + c * 32 + l32;
    al[c] = split ? 1.f : n < d.out ? alpha[n] : 0.f;
    mn[c] = split ? 0.f : n < d.out ? mu[n] : 0.f;
    if constexpr (OP == kI8) {
      // The columns of the last tile past the end of the rows count too: whatever signs were decoded for them met the
      // code 0, i.e. -128.  The decoders left the number of weights -1 of every row where the tables were.
      constexpr int HS = NF <= 2 ? 2 : 1;
      const uint32_t* cnt = (const uint32_t*)smem + c * 32 + l32;
      kc[c] = 128 * (nt * KT - 2 * (int)(cnt[0] + (HS == 2 ? cnt[BN] : 0u)));
      ws[c] = !split && n < d.out ? ca.wsum[n] : 0.f;
    }
  }
  if (lane < 32 * MA) {                                  // every lane then picks up the rows it needs
    const int m = m0 + wave * 32 * MA + lane;
    const bool have = m < M && !split;
    rowp[lane] = have ? rs_all[m] : 0.f;
    if constexpr (OP == kI8) {
      rowp[32 * MA + lane] = have ? ca.step[m] : 1.f;
      rowp[64 * MA + lane] = have ? ca.lo[m] : 0.f;
    }
  }
  wave_lds_sync();
  const bool vec = (d.out & 3) == 0;                           // 4 outputs of a row are aligned and inside
#pragma unroll
  for (int a = 0; a < MA; ++a) {
    const int mrow0 = m0 + wave * 32 * MA + a * 32;
    f32x4 rs[4], sv[4], lv[4];                                 // of the 16 activation rows this lane's registers hold
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      rs[g] = *(const f32x4*)(rowp + a * 32 + 8 * g + 4 * h);
      if constexpr (OP == kI8) {
        sv[g] = *(const f32x4*)(rowp + 32 * MA + a * 32 + 8 * g + 4 * h);
        lv[g] = *(const f32x4*)(rowp + 64 * MA + a * 32 + 8 * g + 4 * h);
      }
    }
#pragma unroll
    for (int c = 0; c < NF; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        float r;
        if constexpr (OP == kI8) {
          r = al[c] * (float)(acc[a][c][e] + kc[c]) + mn[c] * rs[e >> 2][e & 3];   // exact integers inside
          r = sv[e >> 2][e & 3] * r + lv[e >> 2][e & 3] * ws[c];
        } else {
          r = al[c] * acc[a][c][e] + mn[c] * rs[e >> 2][e & 3];
        }
        Tw[(8 * (e >> 2) + 4 * h + (e & 3)) * TS + c * 32 + l32] = r;
      }
    wave_lds_sync();
    if (vec) {
      // The staged rows leave in batches: all LDS reads of a batch are issued, then its stores, and the output
      // type is tested outside the loops.
      constexpr int NI = BN / 8, NBT = 5;
      auto rows_out = [&](auto kind) {
        constexpr int KIND = decltype(kind)::value;
#pragma unroll
        for (int b0 = 0; b0 < NI; b0 += NBT) {
          f32x4 vv[NBT];   // (a vector type: an array of structs would live in scratch memory)
#pragma unroll
          for (int u = 0; u < NBT; ++u) {
            const int idx = (b0 + u) * 64 + lane;
            const int rr = idx / (BN / 4), c4 = idx - rr * (BN / 4);
            if (b0 + u < NI) vv[u] = *(const f32x4*)(Tw + rr * TS + 4 * c4);
          }
#pragma unroll
          for (int u = 0; u < NBT; ++u) {
            const int idx = (b0 + u) * 64 + lane;
            const int rr = idx / (BN / 4), c4 = idx - rr * (BN / 4);
            const int m = mrow0 + rr, n = n0 + 4 * c4;
            if (b0 + u < NI && m < M && n < d.out) {
              const long long o = (long long)m * d.out + n;
              if constexpr (KIND == BTC_F32) {
                *(f32x4*)((float*)Y + o) = vv[u];
              } else if constexpr (KIND == BTC_BF16) {
                *(uint2*)((uint16_t*)Y + o) = make_uint2(bf16_bits(vv[u].x) | (bf16_bits(vv[u].y) << 16),
                                                         bf16_bits(vv[u].z) | (bf16_bits(vv[u].w) << 16));
              } else {
                *(uint2*)((uint16_t*)Y + o) = make_uint2(f16_bits(vv[u].x) | (f16_bits(vv[u].y) << 16),
                                                         f16_bits(vv[u].z) | (f16_bits(vv[u].w) << 16));
              }
            }
          }
        }
      };
      if (y_dtype == BTC_F32) rows_out(std::integral_constant<int, BTC_F32>{});
      else if (y_dtype == BTC_BF16) rows_out(std::integral_constant<int, BTC_BF16>{});
      else rows_out(std::integral_constant<int, BTC_F16>{});
    } else {
      for (int idx = lane; idx < 32 * BN; idx += 64) {
        const int rr = idx / BN, cc = idx - rr * BN;
        const int m = mrow0 + rr, n = n0 + cc;
        if (m < M && n < d.out) {
          const float r = Tw[rr * TS + cc];
          const long long o = (long long)m * d.out + n;
          if (y_dtype == BTC_F32) ((float*)Y)[o] = r;
          else if (y_dtype == BTC_BF16) ((__hip_bfloat16*)Y)[o] = __float2bfloat16(r);
          else ((__half*)Y)[o] = __float2half_rn(r);
        }
      }
    }
    wave_lds_sync();                                           // before the second half overwrites the rows
  }
}

// Sum of activation row m over all its columns (in fp32, or of the codes: an exact integer), the factor of mu, by a
// workgroup of 256 threads; every thread returns it.
template <int OP>
__device__ __forceinline__ float row_sum(const void* X, int m, int in, float* red) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int n = in * Geo<OP>::XS / 16;                   // 16-byte pieces (`in` is a multiple of 16)
  const u32x4* row = (const u32x4*)((const char*)X + (size_t)m * in * Geo<OP>::XS);
  using Sum = std::conditional_t<OP == kI8, uint32_t, float>;
  Sum s = 0;
  for (int i0 = 0; i0 < n; i0 += 4 * 256) {              // four loads in flight per lane
    u32x4 w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 256 * u + tid;
      w[u] = i < n ? row[i] : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = word_sum<OP>(w[u][e], s);
  }
  float f = (float)s;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) f += __shfl_xor(f, o, 64);
  if (lane == 0) red[tid >> 6] = f;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// In front of a call without a k split: rs[m] = sum of activation row m.  (Inside the contraction's loop the packed dot
// products cost 10 of 75 us at 5120 x 5120, M = 512: its waves have no issue slots to spare.)
template <int OP>
__global__ __launch_bounds__(256) void row_sums_kernel(const void* __restrict__ X, int in, float* __restrict__ rs) {
  __shared__ float red[4];
  const float s = row_sum<OP>(X, blockIdx.x, in, red);
  if (threadIdx.x == 0) rs[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void clear_kernel(float* __restrict__ p, int n) {
  for (int i = threadIdx.x; i < n; i += 256) p[i] = 0.f;
}

// Second pass of a k-split call: the splits' raw sums in split order, then what the epilogue above does.  A workgroup
// finishes the outputs [n_part blockIdx.x, + n_part) of one activation row and adds that row up on the way.  It is the
// only reader of its partial sums, so with `clear` it can hand the workspace back zero-filled (the decode entry point
// promises that to its callers).
template <int OP>
__global__ __launch_bounds__(256) void decode_reduce_kernel(float* __restrict__ part, const float* __restrict__ alpha,
                                                            const float* __restrict__ mu, const void* __restrict__ X,
                                                            CodeArgs ca, int M, int in, int out, int n_part, int splits,
                                                            void* __restrict__ Y, int y_dtype, int clear) {
  __shared__ float red[4];
  const int m = blockIdx.y, tid = threadIdx.x;
  const size_t total = (size_t)M * out;
  const size_t row = (size_t)m * out;
  const int n_begin = blockIdx.x * n_part, n_end = min(out, n_begin + n_part);
  // Everything the first outputs need is requested before the row is added up: the call is a chain of latencies.
  const bool vec = (out & 3) == 0;
  const int n_first = n_begin + 4 * tid;
  f32x4 first = {0.f, 0.f, 0.f, 0.f}, al = first, mn = first, ws = first;
  if (vec && n_first < n_end) {
    al = *(const f32x4*)(alpha + n_first);
    mn = *(const f32x4*)(mu + n_first);
    if (OP == kI8) ws = *(const f32x4*)(ca.wsum + n_first);
#pragma unroll 4
    for (int sp = 0; sp < splits; ++sp) first += *(const f32x4*)(part + (size_t)sp * total + row + n_first);
  }
  const float rs = row_sum<OP>(X, m, in, red);
  const float sv = OP == kI8 ? ca.step[m] : 1.f, lv = OP == kI8 ? ca.lo[m] : 0.f;
  auto finish = [&](float s, float a, float u, float w) {
    const float r = a * s + u * rs;
    return OP == kI8 ? sv * r + lv * w : r;
  };
  if (vec) {
    for (int n = n_first; n < n_end; n += 4 * 256) {
      f32x4 v = first;
      if (n != n_first) {
        v = f32x4{0.f, 0.f, 0.f, 0.f};
        al = *(const f32x4*)(alpha + n);
        mn = *(const f32x4*)(mu + n);
        if (OP == kI8) ws = *(const f32x4*)(ca.wsum + n);
#pragma unroll 4
        for (int sp = 0; sp < splits; ++sp) v += *(const f32x4*)(part + (size_t)sp * total + row + n);
      }
      if (clear)
        for (int sp = 0; sp < splits; ++sp) *(f32x4*)(part + (size_t)sp * total + row + n) = f32x4{0.f, 0.f, 0.f, 0.f};
      float r[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = finish(v[e], al[e], mn[e], ws[e]);
      if (y_dtype == BTC_F32) {
        *(f32x4*)((float*)Y + row + n) = f32x4{r[0], r[1], r[2], r[3]};
      } else if (y_dtype == BTC_BF16) {
        *(uint2*)((uint16_t*)Y + row + n) =
            make_uint2(bf16_bits(r[0]) | (bf16_bits(r[1]) << 16), bf16_bits(r[2]) | (bf16_bits(r[3]) << 16));
      } else {
        *(uint2*)((uint16_t*)Y + row + n) =
            make_uint2(f16_bits(r[0]) | (f16_bits(r[1]) << 16), f16_bits(r[2]) | (f16_bits(r[3]) << 16));
      }
    }
  } else {
    for (int n = n_begin + tid; n < n_end; n += 256) {
      float v = 0.f;
      for (int sp = 0; sp < splits; ++sp) {
        float* p = part + (size_t)sp * total + row + n;
        v += *p;
        if (clear) *p = 0.f;
      }
      const float r = finish(v, alpha[n], mu[n], OP == kI8 ? ca.wsum[n] : 0.f);
      if (y_dtype == BTC_F32) ((float*)Y)[row + n] = r;
      else if (y_dtype == BTC_BF16) ((__hip_bfloat16*)Y)[row + n] = __float2bfloat16(r);
      else ((__half*)Y)[row + n] = __float2half_rn(r);
    }
  }
}

struct Plan {
  int ma;               // activation rows per workgroup / 128
  int nf;               // weight rows per workgroup / 32
  int splits;           // workgroups that share one output tile along k
  int tiles_per_split;
  double est_us;        // modelled duration of the call
};

constexpr int kMaxSplits = 16;

// Tile shape and k split: the least modelled time, the model fitted to 400 measured calls (33 .. 2048 activation rows on
// the 7B and 13B shapes; 5 % rms).  A round of workgroups lasts (k-tiles) x (time per k-tile) + a start and an end that
// grow with the tile.  A k-tile costs the more the fuller the chip is (clock, L2 bandwidth); two workgroups of the
// smallest tile share a compute unit at the price of one and a half.  The second pass of a split costs its launch and
// the partial sums at about 2.6 TB/s, written and read.
static Plan make_plan(const Dims& d, int M, int op) {
  struct Fit { double t0, t_ma, t_nf, full, c0, c_area, split, per_mb; };
  const Fit f = op == kI8 ? Fit{0.013, 0.152, 0.130, 0.167, 1.62, 0.626, 1.55, 0.300}
                          : Fit{0.050, 0.144, 0.106, 0.289, 1.45, 0.193, 1.53, 0.381};
  const int kt = op == kI8 ? 128 : 80;
  const int ntiles = (d.in + kt - 1) / kt;
  Plan best{1, 5, 1, ntiles, 1e300};
  for (int ma = 1; ma <= 2; ++ma)
    for (int nf = 2; nf <= 5; ++nf) {
      const int m_blocks = (M + 128 * ma - 1) / (128 * ma);
      const long long tiles_out = (long long)m_blocks * ((d.out + 32 * nf - 1) / (32 * nf));
      const int resident = ma == 1 && nf == 2 ? 512 : 256;       // workgroups at once
      for (int sp = 1; sp <= kMaxSplits; ++sp) {
        const int tps = (ntiles + sp - 1) / sp;
        if (sp > 1 && (tps < 3 || (sp - 1) * tps >= ntiles || M > 65535)) continue;   // short or empty splits; grid limit of the second pass
        const long long wgs = tiles_out * sp, rounds = (wgs + resident - 1) / resident;
        const double per_round = (double)wgs / (double)rounds;
        double t = f.t0 + f.t_ma * ma + f.t_nf * nf;
        t *= 1.0 + f.full * std::min(1.0, per_round / 256.0) * ma * nf / 10.0;
        if (per_round > 256.0) t *= 1.3 + 0.2 * (per_round / 256.0 - 1.0);
        double cost = (double)rounds * (tps * t + f.c0 + f.c_area * ma * nf) + 5.0;
        if (sp > 1) cost += f.split + f.per_mb * sp * M * (double)d.out * 4e-6;
        if (cost < best.est_us) best = Plan{ma, nf, sp, tps, cost};
      }
    }
  return best;
}

// the splits' raw sums, or the sums of the activation rows
static size_t workspace_bytes_of(const Dims& d, int M, const Plan& p) {
  return p.splits == 1 ? (size_t)M * sizeof(float) : (size_t)p.splits * M * d.out * sizeof(float);
}

template <int OP, int MA, int NF, bool LUT>
static btc_status launch(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                         const float* alpha, const float* mu, const void* X, const CodeArgs& ca, int M, void* Y,
                         int y_dtype, const Plan& plan, void* workspace, int clear_workspace) {
  constexpr int kLds = lds_bytes<OP, MA, NF, LUT>();
  static bool attr_set = false;  // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)gemm_decode_kernel<OP, MA, NF, LUT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kLds) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  const int m_blocks = (M + 128 * MA - 1) / (128 * MA), n_blocks = (d.out + 32 * NF - 1) / (32 * NF);
  // split of the eight XCDs over m blocks (gm) and n blocks (8 / gm): least bytes read by the chip,
  // gm x (index bytes) + (8 / gm) x (activation bytes); no more XCD rows than m blocks
  int gm = 1;
  {
    const double wbytes = (double)d.out * d.wpr * 4, abytes = (double)M * d.in * Geo<OP>::XS;
    double best = 1e300;
    for (int g = 1; g <= 8; g *= 2) {
      if (g > m_blocks && g > 1) break;
      if (8 / g > n_blocks && g < 8) continue;
      const double t = g * wbytes + (8 / g) * abytes;
      if (t < best) {
        best = t;
        gm = g;
      }
    }
  }
  const int per_split = 8 * ((m_blocks + gm - 1) / gm) * ((n_blocks + 8 / gm - 1) / (8 / gm));
  float* const ws = (float*)workspace;
  if (plan.splits == 1) {
    row_sums_kernel<OP><<<M, 256, 0, q>>>(X, d.in, ws);
    if (launch_status() != BTC_OK) return BTC_ERR_HIP;
  }
  gemm_decode_kernel<OP, MA, NF, LUT><<<per_split * plan.splits, kThreads, kLds, q>>>(
      d, packed, codebook, alpha, mu, X, ca, M, Y, y_dtype, m_blocks, n_blocks, gm, per_split, plan.tiles_per_split, ws,
      plan.splits > 1 ? ws : nullptr);
  btc_status st = launch_status();
  if (st != BTC_OK) return st;
  if (plan.splits == 1) {
    if (clear_workspace) {
      clear_kernel<<<1, 256, 0, q>>>(ws, M);
      st = launch_status();
    }
    return st;
  }
  // 2048 workgroups or so, each with at least 1024 outputs
  const int parts = std::max(1, std::min((d.out + 1023) / 1024, 2048 / M));
  const int n_part = ((d.out + parts - 1) / parts + 3) / 4 * 4;
  decode_reduce_kernel<OP><<<dim3((d.out + n_part - 1) / n_part, M), 256, 0, q>>>(
      ws, alpha, mu, X, ca, M, d.in, d.out, n_part, plan.splits, Y, y_dtype, clear_workspace);
  return launch_status();
}

template <int OP, int MA, int NF>
static btc_status pick(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                       const float* alpha, const float* mu, const void* X, const CodeArgs& ca, int M, void* Y,
                       int y_dtype, const Plan& plan, void* workspace, int clear_workspace) {
  if constexpr (tight<OP, MA, NF>()) {                   // no room for both tables beyond 8 index bits
    if (d.b > 8) return launch<OP, MA, NF, false>(q, d, packed, codebook, alpha, mu, X, ca, M, Y, y_dtype, plan, workspace, clear_workspace);
  }
  return launch<OP, MA, NF, true>(q, d, packed, codebook, alpha, mu, X, ca, M, Y, y_dtype, plan, workspace, clear_workspace);
}

template <int OP>
static btc_status run(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook, const float* alpha,
                      const float* mu, const void* X, const CodeArgs& ca, int M, void* Y, int y_dtype, void* workspace,
                      size_t workspace_bytes, int clear_workspace) {
  const Plan plan = make_plan(d, M, OP);
  if (!workspace || workspace_bytes < workspace_bytes_of(d, M, plan)) return BTC_ERR_WORKSPACE;
#define BTC_DEC_CASE(MAV, NFV) \
  if (plan.ma == MAV && plan.nf == NFV) \
    return pick<OP, MAV, NFV>(q, d, packed, codebook, alpha, mu, X, ca, M, Y, y_dtype, plan, workspace, clear_workspace)
  BTC_DEC_CASE(1, 2);
  BTC_DEC_CASE(1, 3);
  BTC_DEC_CASE(1, 4);
  BTC_DEC_CASE(1, 5);
  BTC_DEC_CASE(2, 2);
  BTC_DEC_CASE(2, 3);
  BTC_DEC_CASE(2, 4);
  BTC_DEC_CASE(2, 5);
#undef BTC_DEC_CASE
  return BTC_ERR_UNSUPPORTED;
}

static bool covers(const Dims& d, int M, int xs) {
  if ((d.v != 9 && d.v != 10) || d.b > 10) return false;
  if (d.in % 16 != 0 || d.in >= (1 << 20) || M < 1) return false;   // 16-byte aligned activation rows, whole pieces
  // 32-bit buffer offsets, 0x80000000 being the out-of-range one; rows of a tile past the end stay below 2^32
  return (long long)M * d.in * xs < (1LL << 31) && (long long)d.out * d.wpr * 4 < (1LL << 31);
}

}  // namespace dec

bool gemm_decode_covers(const Dims& d, int M) { return dec::covers(d, M, 2); }
bool gemm_decode_i8_covers(const Dims& d, int M) { return dec::covers(d, M, 1); }
double gemm_decode_estimate_us(const Dims& d, int M) { return dec::make_plan(d, M, dec::kBF16).est_us; }
size_t gemm_decode_workspace_bytes(const Dims& d, int M) {
  return dec::workspace_bytes_of(d, M, dec::make_plan(d, M, dec::kBF16));
}
size_t gemm_decode_i8_workspace_bytes(const Dims& d, int M) {
  return dec::workspace_bytes_of(d, M, dec::make_plan(d, M, dec::kI8));
}

btc_status gemm_decode(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                       const float* alpha, const float* mu, const void* X, int is_bf16, int M, void* Y, int y_dtype,
                       void* workspace, size_t workspace_bytes, int clear_workspace) {
  const dec::CodeArgs none{nullptr, nullptr, nullptr};
  return is_bf16 ? dec::run<dec::kBF16>(q, d, packed, codebook, alpha, mu, X, none, M, Y, y_dtype, workspace,
                                        workspace_bytes, clear_workspace)
                 : dec::run<dec::kF16>(q, d, packed, codebook, alpha, mu, X, none, M, Y, y_dtype, workspace,
                                       workspace_bytes, clear_workspace);
}

btc_status gemm_decode_i8(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook,
                          const float* alpha, const float* mu, const float* wsum, const uint8_t* Q, const float* lo,
                          const float* step, int M, void* Y, int y_dtype, void* workspace, size_t workspace_bytes) {
  return dec::run<dec::kI8>(q, d, packed, codebook, alpha, mu, Q, dec::CodeArgs{wsum, lo, step}, M, Y, y_dtype, workspace,
                            workspace_bytes, 0);
}

}  // namespace btc
