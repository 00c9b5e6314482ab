// btc_transform: the online activation transform that precedes the layer at inference,
//     X <- X T,   T = D P,   D = diag(sigma), sigma_k = +-1,   P = P1 (x) P2
// (section "Learnable Transformation": transformation pair, Kronecker-factored P;
// "Integration into Transformer Architecture": Y = X W^T = (X T)(T^-1 W^T), the weights
// are compressed after T^-1 was folded in, the activations are transformed on the fly).
//
// A Kronecker-factored P never has to be formed: with a row of X reshaped to n1 x n2
// (channel i = i1 n2 + i2),  row . (P1 (x) P2)  reshaped the same way is  P1^T (X_m) P2.
// That is 2 n (n1 + n2) flop per row against 2 n^2 for the full matrix (144 against 5120
// multiply-adds per channel at n = 5120 = 64 x 80).
//
// Work split.  Output column j = j1 n2 + j2 depends on column j2 of P2 only, so a block of
// kCB columns j2 of ALL rows j1 is computed by one workgroup without help from any other:
//   stage 1:  Y1[i1][jj] = sum_i2 sigma x[i1 n2 + i2] P2[i2][j0 + jj]      (n1 x kCB values)
//   stage 2:  Z[j1][jj]  = sum_i1 P1[i1][j1] Y1[i1][jj]
// The workgroup keeps P1 and its slice of P2 in LDS and walks over the rows of X dealt to it; a
// row is staged with its signs applied (a flip of the sign bit: exact).  fp32 accumulation in a
// fixed order: deterministic.  Two shapes of this kernel: below a few hundred workgroups
// a workgroup has 1024 threads and every dot product of both stages is
// cut into KS = 4 pieces held by neighbouring lanes, whose sums meet by two cross-lane additions;
// for more rows than the matrix-core kernel can address 256 threads, whole dot products,
// four columns per thread, and the rows are dealt to about five workgroups per compute unit.
// Every global load of a phase is issued before the first one is used.  One row or a few (decode)
// take row_kernel below instead, more of them (prefill) the matrix-core kernel of
// btc_transform_mfma.h.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "btc_transform_mfma.h"

namespace btc {
namespace transform {

constexpr int kThreads = 256;
constexpr int kCB = 8;         // columns of P2 per workgroup
constexpr int kMaxN1 = 128;
constexpr int kMaxN2 = 256;

struct Layout {                // byte offsets into dynamic LDS
  int rs;                      // staged row stride in 16-bit elements (even; rs / 2 odd: rows start in different banks)
  int p1, p2, y1, total;
};

static Layout layout_of(int n1, int n2, int KS) {
  Layout L;
  L.rs = 2 * (((n2 + 1) / 2) | 1);
  auto up16 = [](int b) { return (b + 15) & ~15; };
  L.p1 = up16(n1 * L.rs * 2);
  L.p2 = L.p1 + up16((n1 * n1 + KS * 32) * 4);                // up to 31 words of padding per piece, here and in Y1
  L.y1 = L.p2 + up16((n2 + KS) * kCB * 4);
  L.total = L.y1 + up16((n1 * kCB + KS * 32) * 4);
  return L;
}

template <bool BF16>
__device__ __forceinline__ float widen(uint32_t h) {
  if constexpr (BF16) return __uint_as_float(h << 16);
  else return __half2float(__ushort_as_half((uint16_t)h));
}

__device__ __forceinline__ void store_out(void* Y, size_t at, float v, int y_dtype) {
  if (y_dtype == BTC_F32) {
    ((float*)Y)[at] = v;
  } else if (y_dtype == BTC_F16) {
    ((__half*)Y)[at] = __float2half_rn(v);
  } else {                                   // bf16, round to nearest even
    ((__bf16*)Y)[at] = (__bf16)v;
  }
}

// KS: pieces per dot product (threads = 256 KS); CPI: columns per work item.
template <bool BF16, int KS, int CPI>
__global__ __launch_bounds__(kThreads * KS) void transform_kernel(const uint16_t* __restrict__ X, int M, int n1, int n2,
                                                                 const uint32_t* __restrict__ sign_bits,
                                                                 const float* __restrict__ P1,
                                                                 const float* __restrict__ P2, void* __restrict__ Y,
                                                                 int y_dtype, Layout L) {
  constexpr int T = kThreads * KS;
  constexpr int IPR = kCB / CPI;             // work items per row index
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* xs = (uint16_t*)smem;
  float* p1s = (float*)(smem + L.p1);
  float* p2s = (float*)(smem + L.p2);        // row i2 at i2 * kCB + (i2 / len2) * kCB: a pad per piece, against bank conflicts
  float* y1 = (float*)(smem + L.y1);         // [n1][kCB], row i1 at i1 * kCB + (i1 / len1) * pady
  const int tid = threadIdx.x;
  const int n = n1 * n2;
  const int j0 = blockIdx.x * kCB;
  const int ncol = min(kCB, n2 - j0);
  const int len2 = (((n2 + KS - 1) / KS) + 1) & ~1;   // piece of a stage-1 dot product (even)
  const int len1 = (n1 + KS - 1) / KS;                // piece of a stage-2 dot product
  const float rcp_n2 = 1.0f / (float)n2, rcp_n1 = 1.0f / (float)n1, rcp_len1 = 1.0f / (float)len1;
  // The KS lanes that hold the pieces of one dot product are neighbours (a quad): their sums meet by two
  // cross-lane additions, ((p0 + p1) + (p2 + p3)), and the lane of piece 0 keeps the result.  The rows of P1 and
  // of Y1 that belong to piece ks are shifted by a few words, so that the four lanes of a quad, which read the same
  // column of different pieces, hit different banks: the start of piece ks is 8 ks words (mod 32) after that of
  // piece 0, whatever the sizes.
  const int pad1 = (8 - len1 * n1) & 31, pady = (8 - len1 * kCB) & 31;
  auto quad_sum = [](float a) __attribute__((always_inline)) {
    if constexpr (KS == 4) {
      a += __shfl_xor(a, 1, 64);
      a += __shfl_xor(a, 2, 64);
    }
    return a;
  };
  auto piece_of = [&](int i1) __attribute__((always_inline)) {
    return KS > 1 ? (int)(((float)i1 + 0.5f) * rcp_len1) : 0;  // i1 / len1, exact for these sizes
  };
  const bool x_vec = (n2 & 7) == 0;          // a group of 8 channels stays inside one row of the n1 x n2 view, and
                                             // rows of X start 16-byte aligned

  // A row of X with its signs applied -> LDS (row i1 of the n1 x n2 view at xs + i1 * rs).
  auto stage_x = [&](int m) __attribute__((always_inline)) {
    const uint16_t* xrow = X + (size_t)m * n;
    if (x_vec) {
      constexpr int U = 4;
      const int groups = n >> 3;
      for (int base = tid; base < groups; base += T * U) {
        uint4 v[U];
        uint32_t sw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int g = min(base + u * T, groups - 1);            // past the end: a valid group, not stored
          v[u] = *(const uint4*)(xrow + 8 * g);
          sw[u] = sign_bits[g >> 2];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int g = base + u * T;
          if (g < groups) {
            const int k = 8 * g;
            const int i1 = (int)(((float)k + 0.5f) * rcp_n2);     // exact for k < 2^20
            const int i2 = k - i1 * n2;
            const uint32_t minus = ~(sw[u] >> (k & 31)) & 0xFFu;    // bit e set: channel k + e is flipped
            uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              w[e] ^= (((minus >> (2 * e)) & 1u) << 15) | (((minus >> (2 * e + 1)) & 1u) << 31);
            uint32_t* dst = (uint32_t*)(xs + i1 * L.rs + i2);       // 4-byte aligned (rs and i2 are even)
            dst[0] = w[0]; dst[1] = w[1]; dst[2] = w[2]; dst[3] = w[3];
          }
        }
      }
    } else {
      for (int k = tid; k < n; k += T) {
        const int i1 = (int)(((float)k + 0.5f) * rcp_n2);
        const int i2 = k - i1 * n2;
        const uint32_t plus = (sign_bits[k >> 5] >> (k & 31)) & 1u;
        xs[i1 * L.rs + i2] = (uint16_t)(xrow[k] ^ (plus ? 0u : 0x8000u));
      }
    }
  };

  // ---- the first row's activations are requested first, then the factors (once per workgroup)
  stage_x(blockIdx.y);
  if ((n2 & 3) == 0) {                       // columns j0 .. j0 + kCB - 1 of a row of P2 are aligned 16-byte pieces
    constexpr int PR = kCB / 4;
    for (int t = tid; t < PR * n2; t += T) {
      const int i2 = t / PR, h = t % PR;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (j0 + 4 * h < n2) v = *(const float4*)(P2 + (size_t)i2 * n2 + j0 + 4 * h);
      *(float4*)(p2s + i2 * kCB + (i2 / len2) * kCB + 4 * h) = v;
    }
  } else {
    for (int t = tid; t < n2 * kCB; t += T) {
      const int i2 = t / kCB, jj = t - i2 * kCB;
      p2s[i2 * kCB + (i2 / len2) * kCB + jj] = jj < ncol ? P2[(size_t)i2 * n2 + j0 + jj] : 0.f;
    }
  }
  if ((n1 & 3) == 0) {                       // four consecutive elements stay inside one row of P1
    constexpr int U = 4;
    const int quads = (n1 * n1) >> 2;
    for (int base = tid; base < quads; base += T * U) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = *(const float4*)(P1 + 4 * (size_t)min(base + u * T, quads - 1));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int qd = base + u * T;
        if (qd < quads) {
          const int i1 = (int)(((float)(4 * qd) + 0.5f) * rcp_n1);
          *(float4*)(p1s + 4 * qd + piece_of(i1) * pad1) = v[u];   // pad1 is a multiple of 4 here
        }
      }
    }
  } else {
    for (int t = tid; t < n1 * n1; t += T) {
      const int i1 = (int)(((float)t + 0.5f) * rcp_n1);
      p1s[t + piece_of(i1) * pad1] = P1[t];
    }
  }

  const int items = n1 * IPR * KS;           // item = (row index, group of CPI columns, piece)
  for (int m = blockIdx.y; m < M; m += gridDim.y) {
    if (m != (int)blockIdx.y) {
      __syncthreads();                       // the previous row's readers are done
      stage_x(m);
    }
    __syncthreads();
    // ---- stage 1: piece ks of  Y1[i1][c0 .. c0 + CPI - 1]
    for (int it = tid; it < items; it += T) {
      const int ks = it % KS, rest = it / KS;
      const int c0 = (rest % IPR) * CPI, i1 = rest / IPR;
      const uint16_t* xr = xs + i1 * L.rs;
      const float* pc = p2s + ks * kCB + c0;
      const int lo = ks * len2, hi = min(n2, lo + len2);
      float a[CPI];
#pragma unroll
      for (int c = 0; c < CPI; ++c) a[c] = 0.f;
      int i2 = lo;
      for (; i2 + 1 < hi; i2 += 2) {
        const uint32_t pr = *(const uint32_t*)(xr + i2);
        const float x0 = widen<BF16>(pr & 0xFFFFu), x1 = widen<BF16>(pr >> 16);
        float p[CPI], q[CPI];
        if constexpr (CPI == 4) {
          const float4 pv = *(const float4*)(pc + i2 * kCB), qv = *(const float4*)(pc + (i2 + 1) * kCB);
          p[0] = pv.x; p[1] = pv.y; p[2] = pv.z; p[3] = pv.w;
          q[0] = qv.x; q[1] = qv.y; q[2] = qv.z; q[3] = qv.w;
        } else {
          const float2 pv = *(const float2*)(pc + i2 * kCB), qv = *(const float2*)(pc + (i2 + 1) * kCB);
          p[0] = pv.x; p[1] = pv.y; q[0] = qv.x; q[1] = qv.y;
        }
#pragma unroll
        for (int c = 0; c < CPI; ++c) a[c] = fmaf(x1, q[c], fmaf(x0, p[c], a[c]));
      }
      if (i2 < hi) {
        const float x0 = widen<BF16>(xr[i2]);
#pragma unroll
        for (int c = 0; c < CPI; ++c) a[c] = fmaf(x0, pc[i2 * kCB + c], a[c]);
      }
#pragma unroll
      for (int c = 0; c < CPI; ++c) a[c] = quad_sum(a[c]);
      if (ks == 0) {
        float* dst = y1 + i1 * kCB + piece_of(i1) * pady + c0;
#pragma unroll
        for (int c = 0; c < CPI; ++c) dst[c] = a[c];
      }
    }
    __syncthreads();
    // ---- stage 2: piece ks of  Z[j1][c0 .. c0 + CPI - 1]; a wave's lanes: 16 neighbouring j1 x KS pieces
    for (int it = tid; it < items; it += T) {
      const int ks = it % KS, rest = it / KS;
      const int j1 = rest % n1, c0 = (rest / n1) * CPI;
      const int lo = ks * len1, hi = min(n1, lo + len1);
      const float* pc = p1s + ks * pad1 + j1;
      const float* yc = y1 + ks * pady + c0;
      float a[CPI];
#pragma unroll
      for (int c = 0; c < CPI; ++c) a[c] = 0.f;
      for (int i1 = lo; i1 < hi; ++i1) {
        const float p = pc[i1 * n1];
#pragma unroll
        for (int c = 0; c < CPI; ++c) a[c] = fmaf(p, yc[i1 * kCB + c], a[c]);
      }
#pragma unroll
      for (int c = 0; c < CPI; ++c) a[c] = quad_sum(a[c]);
      if (ks == 0) {
        const size_t at = (size_t)m * n + (size_t)j1 * n2 + j0 + c0;
#pragma unroll
        for (int c = 0; c < CPI; ++c)
          if (c0 + c < ncol) store_out(Y, at + c, a[c], y_dtype);
      }
    }
  }
}

// ---- one or a few rows -------------------------------------------------------------------------------------------
// A decode call transforms one row: 2 n (n1 + n2) flops, a chain of latencies.  A workgroup computes four columns j2 of
// one row, and nothing is asked for late: every load of the call -- the row, its signs, P1, the four columns of P2 -- is
// issued by its first instructions, and only the columns of P2 pass through LDS before they are used.
//   stage 1: half-wave h holds rows 4 h .. 4 h + 3 of the n1 x n2 view, lane l their elements 8 l .. 8 l + 7, in
//            registers (a row is one contiguous piece of at most 512 bytes per half-wave); 16 sums per lane -- four rows,
//            four columns -- meet over the 32 lanes by exchanges that halve their number.
//   stage 2: the rows of Y1 that a half-wave has just made are the ones it contracts with its rows of P1 (lane l: columns
//            4 l .. 4 l + 3, in registers since the start), so the stages need no barrier in between; the half-waves'
//            partial sums of Z meet in LDS, eight threads per row j1.
// Alignment: rows start at any element; n2 odd: a row that starts inside a word is loaded from the word's start and
// shifted.  Elements past the end of a row are made zero (they belong to the next one).
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
constexpr uint32_t kOob = 0x80000000u;       // a byte offset past the end of every buffer
constexpr int kPart = 146;                   // float4 per half-wave of partial sums: 128 + 7 of skew, and 2 mod 16
constexpr int kRowFixed = 256 + 32 + 32 * 4; // float4: columns of P2 (one of padding per 8), Y1

static int row_half_waves(int n1) { return (((n1 + 3) / 4) + 1) & ~1; }

__device__ __forceinline__ float lane_xor1(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor2(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor4(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), (4 << 10) | 0x1F));
}
__device__ __forceinline__ float lane_xor8(float v) {      // rotation by 8 in a row of 16 lanes
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor16(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), (16 << 10) | 0x1F));
}

template <bool BF16, bool ODD>
__global__ __launch_bounds__(1024) void row_kernel(const uint16_t* __restrict__ X, int M, int n1, int n2,
                                                   const uint32_t* __restrict__ sign_bits, const float* __restrict__ P1,
                                                   const float* __restrict__ P2, void* __restrict__ Y, int y_dtype) {
  extern __shared__ __align__(16) float4 sm4[];
  float4* p2s = sm4;                         // row i2 at i2 + i2 / 8
  float4* y1s = sm4 + 256 + 32;              // [half-wave][row]
  float4* part = sm4 + kRowFixed;            // [half-wave][kPart]: row j1 at j1 + j1 / 16
  const int tid = threadIdx.x, l = tid & 31, hw = tid >> 5, n_hw = blockDim.x >> 5;
  const int j0 = blockIdx.x * 4, m = blockIdx.y;
  const uint32_t n = (uint32_t)n1 * (uint32_t)n2;
  const __amdgpu_buffer_rsrc_t rX =
      __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)(((uint32_t)M * n * 2u + 3u) & ~3u), 0x00020000);
  const __amdgpu_buffer_rsrc_t rS =
      __builtin_amdgcn_make_buffer_rsrc((void*)sign_bits, 0, (int)((n + 31u) / 32u * 4u), 0x00020000);
  const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc((void*)P1, 0, n1 * n1 * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc((void*)P2, 0, n2 * n2 * 4, 0x00020000);
  auto load4 = [](__amdgpu_buffer_rsrc_t r, uint32_t off) __attribute__((always_inline)) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return u32x4{v[0], v[1], v[2], v[3]};
  };
  auto p2_offset = [&](int t) { return t < 256 ? (uint32_t)(t * n2 + j0) * 4u : kOob; };   // rows past n2: zeros
  const u32x4 pv = load4(r2, p2_offset(tid));
  u32x4 xv[4], p1[4];
  uint32_t xt[4];
  u32x2 sg[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i1 = 4 * hw + r;
    const uint32_t k = (uint32_t)i1 * (uint32_t)n2 + 8u * l;
    const bool live = i1 < n1 && 8 * l < n2;
    const uint32_t off = live ? (((uint32_t)m * n + k) * 2u) & ~3u : kOob;
    xv[r] = load4(rX, off);
    if (ODD) xt[r] = __builtin_amdgcn_raw_buffer_load_b32(rX, off + 16u, 0, 0);
    const auto s2 = __builtin_amdgcn_raw_buffer_load_b64(rS, live ? (k >> 5) * 4u : kOob, 0, 0);
    sg[r] = u32x2{s2[0], s2[1]};
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) p1[r] = load4(r1, 4 * l < n1 ? (uint32_t)((4 * hw + r) * n1 + 4 * l) * 4u : kOob);
  if (tid < 256) p2s[tid + (tid >> 3)] = __builtin_bit_cast(float4, pv);
  for (int t = tid + (int)blockDim.x; t < 256; t += (int)blockDim.x)
    p2s[t + (t >> 3)] = __builtin_bit_cast(float4, load4(r2, p2_offset(t)));
  // the row's elements, signs applied, zeros past its end
  float x[4][8];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t k = (uint32_t)(4 * hw + r) * (uint32_t)n2 + 8u * l;
    uint32_t w[4] = {xv[r][0], xv[r][1], xv[r][2], xv[r][3]};
    if (ODD) {
      const uint32_t sh = (((uint32_t)m * n + k) & 1u) * 16u;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = __builtin_amdgcn_alignbit(e < 3 ? xv[r][e + 1] : xt[r], xv[r][e], sh);
    }
    const uint32_t minus = ~__builtin_amdgcn_alignbit(sg[r][1], sg[r][0], k & 31u);   // bit e set: element e is flipped
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int left = n2 - 8 * l - 2 * e;   // elements from this pair on
      w[e] = left >= 2 ? w[e] : left == 1 ? w[e] & 0xFFFFu : 0u;
      w[e] ^= (((minus >> (2 * e)) & 1u) << 15) | (((minus >> (2 * e + 1)) & 1u) << 31);
      x[r][2 * e] = widen<BF16>(w[e] & 0xFFFFu);
      x[r][2 * e + 1] = widen<BF16>(w[e] >> 16);
    }
  }
  __syncthreads();
  float a[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float4 p = p2s[9 * l + e];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a[4 * r + 0] = fmaf(x[r][e], p.x, a[4 * r + 0]);
      a[4 * r + 1] = fmaf(x[r][e], p.y, a[4 * r + 1]);
      a[4 * r + 2] = fmaf(x[r][e], p.z, a[4 * r + 2]);
      a[4 * r + 3] = fmaf(x[r][e], p.w, a[4 * r + 3]);
    }
  }
  // lane l: sum number l % 16 over the 32 lanes
  const bool b0 = l & 1, b1 = l & 2, b2 = l & 4, b3 = l & 8;
  float c8[8], c4[4], c2[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) c8[i] = (b0 ? a[2 * i + 1] : a[2 * i]) + lane_xor1(b0 ? a[2 * i] : a[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < 4; ++i) c4[i] = (b1 ? c8[2 * i + 1] : c8[2 * i]) + lane_xor2(b1 ? c8[2 * i] : c8[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < 2; ++i) c2[i] = (b2 ? c4[2 * i + 1] : c4[2 * i]) + lane_xor4(b2 ? c4[2 * i] : c4[2 * i + 1]);
  float y1 = (b3 ? c2[1] : c2[0]) + lane_xor8(b3 ? c2[0] : c2[1]);
  y1 += lane_xor16(y1);
  if (l < 16) ((float*)y1s)[hw * 16 + l] = y1;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // read by lanes of this wave only
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  float4 z[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) z[j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float4 v = y1s[hw * 4 + r];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float p = __uint_as_float(p1[r][j]);
      z[j].x = fmaf(p, v.x, z[j].x);
      z[j].y = fmaf(p, v.y, z[j].y);
      z[j].z = fmaf(p, v.z, z[j].z);
      z[j].w = fmaf(p, v.w, z[j].w);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) part[hw * kPart + 4 * l + j + (l >> 2)] = z[j];
  __syncthreads();
  const int j1 = tid >> 3, g = tid & 7;
  float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (8 * k + g < n_hw) {
      const float4 v = part[(8 * k + g) * kPart + j1 + (j1 >> 4)];
      t.x += v.x;
      t.y += v.y;
      t.z += v.z;
      t.w += v.w;
    }
  }
  const float t0 = (b0 ? t.y : t.x) + lane_xor1(b0 ? t.x : t.y), t1 = (b0 ? t.w : t.z) + lane_xor1(b0 ? t.z : t.w);
  float v = (b1 ? t1 : t0) + lane_xor2(b1 ? t0 : t1);      // lane: column lane % 4
  v += lane_xor4(v);
  const int c = tid & 3;
  if ((tid & 4) == 0 && j1 < n1 && j0 + c < n2) store_out(Y, (size_t)m * n + (size_t)j1 * n2 + j0 + c, v, y_dtype);
}

template <bool BF16, bool ODD>
static btc_status launch_row(hipStream_t q, const void* X, int M, int n1, int n2, const uint32_t* sign_bits, const float* P1,
                             const float* P2, void* Y, int y_dtype) {
  static bool attr_set = false;              // one-time kernel attribute, not call state
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)row_kernel<BF16, ODD>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (kRowFixed + 32 * kPart) * 16) != hipSuccess)
      return BTC_ERR_HIP;
    attr_set = true;
  }
  const int n_hw = row_half_waves(n1);
  row_kernel<BF16, ODD><<<dim3((n2 + 3) / 4, M), 32 * n_hw, (kRowFixed + n_hw * kPart) * 16, q>>>(
      (const uint16_t*)X, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
  return launch_status();
}

}  // namespace transform
}  // namespace btc

extern "C" {

btc_status btc_transform(void* stream, const void* X, btc_dtype x_dtype, int32_t M, int32_t n1, int32_t n2,
                         const uint32_t* sign_bits, const float* P1, const float* P2, void* Y, btc_dtype y_dtype) {
  using namespace btc;
  using namespace btc::transform;
  if (!X || !sign_bits || !P1 || !P2 || !Y) return BTC_ERR_NULL;
  if (M <= 0 || n1 <= 0 || n2 <= 0) return BTC_ERR_SHAPE;
  if (n1 > kMaxN1 || n2 > kMaxN2) return BTC_ERR_UNSUPPORTED;
  if (x_dtype != BTC_F16 && x_dtype != BTC_BF16) return BTC_ERR_UNSUPPORTED;
  if (y_dtype != BTC_F16 && y_dtype != BTC_BF16 && y_dtype != BTC_F32) return BTC_ERR_UNSUPPORTED;
  if ((long long)M * n1 * n2 >= (1LL << 40)) return BTC_ERR_SHAPE;
  if (!aligned16(X) || !aligned16(sign_bits) || !aligned16(P1) || !aligned16(P2) || !aligned16(Y)) return BTC_ERR_ALIGN;
  if (X == Y) return BTC_ERR_UNSUPPORTED;    // workgroups read whole rows that others write slices of
  hipStream_t q = (hipStream_t)stream;
  // One or a few rows: while the workgroups of row_kernel run in one go, 256 of them, or 512 where two fit a compute unit
  // (n1 <= 96) or where the other kernels' preparation of large factors costs more than a second round (n2 > 144).  Alone,
  // warm: one row of 110 x 160 8.0 -> 6.1 us, of 128 x 198 10.3 -> 6.2; 108 x 128, 8 rows 7.8 -> 6.6, 12 rows 10.3 against
  // 11.0 here; 72 x 104, 16 rows 8.0 -> 7.1; 64 x 64, 16 rows 5.6 -> 4.9, 24 rows 5.6 against 5.9.
  const long long row_wgs = (long long)M * ((n2 + 3) / 4);
  if (row_wgs <= (n2 > 144 || (n1 <= 96 && n2 > 96) ? 512 : 256) && (long long)M * n1 * n2 < (1LL << 30)) {   // (32-bit byte offsets)
    const bool odd = n2 & 1;
    if (x_dtype == BTC_BF16)
      return odd ? launch_row<true, true>(q, X, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype)
                 : launch_row<true, false>(q, X, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype);
    return odd ? launch_row<false, true>(q, X, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype)
               : launch_row<false, false>(q, X, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype);
  }
  // The matrix cores from where the kernel above needs a second round of workgroups on (it has one per row and eight columns,
  // and large factors leave room for one per compute unit): 108 x 128, 12 rows 10.2 against 11.3 us, 17 rows 18.6 against
  // 11.3; 64 x 80, 24 rows 6.0 against 7.2 (fp16: 8.6), 48 rows 8.4 against 7.3 (8.7).
  const long long vector_wgs = (long long)M * ((n2 + 7) / 8);
  const bool many = vector_wgs > (n1 > 64 ? 256 : x_dtype == BTC_BF16 && (n2 & 1) == 0 ? 360 : 400);
  if (many && (long long)M * n1 * n2 < (1LL << 30)) {   // (32-bit byte offsets)
    const btc_status st = (n2 & 15) == 0  ? mfma_16(q, X, x_dtype == BTC_BF16, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype)
                          : (n2 & 1) == 0 ? mfma_2(q, X, x_dtype == BTC_BF16, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype)
                                          : mfma_1(q, X, x_dtype == BTC_BF16, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype);
    if (st != BTC_ERR_UNSUPPORTED) return st;
  }
  int n_cb = (n2 + kCB - 1) / kCB;
  // Not many rows: one workgroup of 1024 threads per (column block, row), dot products cut in four.
  // Many rows: 256 threads, and the rows are dealt to about five workgroups per compute unit.
  // Large factors leave room for one workgroup per compute unit only: then the 1024-thread shape serves
  // many rows too (16 waves per compute unit instead of 4).
  const bool few = (long long)M * n_cb <= 512;
  const bool big = layout_of(n1, n2, 1).total > 48 * 1024;
  int KS = (few || big) ? 4 : 1;
  if (KS == 4 && layout_of(n1, n2, 4).total > 160 * 1024 - 256) KS = 1;   // the largest factors: no room for the pads
  const Layout L = layout_of(n1, n2, KS);
  if (L.total > 160 * 1024 - 256) return BTC_ERR_UNSUPPORTED;
  int gy = few ? M : big ? 256 / n_cb : 1280 / n_cb;
  if (gy < 1) gy = 1;
  if (gy > M) gy = M;
  static bool attr_set = false;              // one-time kernel attributes, not call state
  if (!attr_set) {
    const void* fns[4] = {(const void*)transform_kernel<false, 4, 2>, (const void*)transform_kernel<true, 4, 2>,
                          (const void*)transform_kernel<false, 1, 4>, (const void*)transform_kernel<true, 1, 4>};
    for (const void* fn : fns)
      if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) != hipSuccess)
        return BTC_ERR_HIP;
    attr_set = true;
  }
  const bool bf = x_dtype == BTC_BF16;
  const dim3 grid(n_cb, gy);
  const uint16_t* Xp = (const uint16_t*)X;
  if (KS == 4) {
    if (bf) transform_kernel<true, 4, 2><<<grid, kThreads * 4, L.total, q>>>(Xp, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype, L);
    else transform_kernel<false, 4, 2><<<grid, kThreads * 4, L.total, q>>>(Xp, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype, L);
  } else {
    if (bf) transform_kernel<true, 1, 4><<<grid, kThreads, L.total, q>>>(Xp, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype, L);
    else transform_kernel<false, 1, 4><<<grid, kThreads, L.total, q>>>(Xp, M, n1, n2, sign_bits, P1, P2, Y, (int)y_dtype, L);
  }
  return launch_status();
}

}  // extern "C"
