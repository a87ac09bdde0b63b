// Row quantiser Q_a(h) (Eq.8-10 applied to the hidden activation of Eq.5), the weighted
// combine of Eq.2 + Eq.4, and the calibration copy kernel.
#include <stdlib.h>
#include "common.h"
#include "launch.h"
#include "quant_body.h"

namespace mote {

constexpr int kRowThreads = 256;

constexpr int kRowChunks = 6;

template <int THREADS>
__global__ __launch_bounds__(THREADS) void quant_rows_kernel(const uint16_t* __restrict__ h, int F,
                                                             int8_t* __restrict__ q, float* __restrict__ beta,
                                                             int32_t* __restrict__ rowsum) {
  __shared__ QuantRowScratch<THREADS> lds;
  quant_row<THREADS, kRowChunks>(lds, blockIdx.x, h, F, q, beta, rowsum);
}

hipError_t launch_quant_rows(const uint16_t* h, int rows, int F, int8_t* q, float* beta, int32_t* rowsum,
                             hipStream_t stream) {
  if (rows == 0) return hipSuccess;
  // short rows: half the threads per row still read a row in one sweep, and twice as many rows are resident
  const bool narrow = knob(kKnobQuantWide) != 1;
  if (narrow && (F >> 3) <= 128 * kRowChunks) quant_rows_kernel<128><<<rows, 128, 0, stream>>>(h, F, q, beta, rowsum);
  else quant_rows_kernel<kRowThreads><<<rows, kRowThreads, 0, stream>>>(h, F, q, beta, rowsum);
  return hipGetLastError();
}

// Most tokens of a decode step: up to here combine_few_kernel's workgroups (64 of them at d = 2048) are fewer than the CUs.
constexpr int kCombineFewTokens = 64;

// Combine (Eq.2 + Eq.4): one thread per (token, 8 channels).
//   y_e[c] = float(D[row, c]) * ((beta_h[row] / 127) * alpha_down[e])      (ternary linear, Section 3.1)
//   out[t, c] = y_s[t, c] + sum_j p[t, j] * y_{e_j}[c]
// D and y_s may arrive as partial planes of a K split; they are added in plane order.
template <int KMAX>
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a) {
  const int d = a.d, k = a.k;
  const int chunks = d >> 3;
  const int64_t gid = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (gid >= static_cast<int64_t>(a.T) * chunks) return;
  const int t = static_cast<int>(gid / chunks);
  const int c0 = static_cast<int>(gid - static_cast<int64_t>(t) * chunks) << 3;
  const int64_t yo = static_cast<int64_t>(t) * d + c0;
  // Partial planes are requested four at a time (the loads of a batch are in flight together: a
  // plane-by-plane loop pays one memory round trip per plane) and added in plane order.
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int p0 = 0; p0 < a.y_planes; p0 += 4) {
    float4 s0[4], s1[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u < a.y_planes) {
        s0[u] = *reinterpret_cast<const float4*>(a.y_s + (p0 + u) * a.y_stride + yo);
        s1[u] = *reinterpret_cast<const float4*>(a.y_s + (p0 + u) * a.y_stride + yo + 4);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u < a.y_planes) {
        o[0] += s0[u].x; o[1] += s0[u].y; o[2] += s0[u].z; o[3] += s0[u].w;
        o[4] += s1[u].x; o[5] += s1[u].y; o[6] += s1[u].z; o[7] += s1[u].w;
      }
    }
  }
  if (a.tap_y_s) {
    *reinterpret_cast<float4*>(a.tap_y_s + yo) = make_float4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<float4*>(a.tap_y_s + yo + 4) = make_float4(o[4], o[5], o[6], o[7]);
  }
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    if (j < k) {
      const int row = a.row_of[t * k + j];
      const int e = a.topk_idx[t * k + j];
      const float p = a.topk_p[t * k + j];
      const float sc = (a.beta_h[row] / 127.0f) * a.alpha[e * 3 + 2];
      const int64_t ro = static_cast<int64_t>(row) * d + c0;
      int dsum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      const int d_planes = a.row_planes ? 1 + ((a.row_planes[row] >> (2 * (c0 / a.d_tile_n))) & 3) : a.d_planes;
      for (int p0 = 0; p0 < d_planes; p0 += 4) {
        int4 d0[4], d1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (p0 + u < d_planes) {
            d0[u] = *reinterpret_cast<const int4*>(a.acc_down + (p0 + u) * a.d_stride + ro);
            d1[u] = *reinterpret_cast<const int4*>(a.acc_down + (p0 + u) * a.d_stride + ro + 4);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (p0 + u < d_planes) {
            dsum[0] += d0[u].x; dsum[1] += d0[u].y; dsum[2] += d0[u].z; dsum[3] += d0[u].w;
            dsum[4] += d1[u].x; dsum[5] += d1[u].y; dsum[6] += d1[u].z; dsum[7] += d1[u].w;
          }
        }
      }
      if (a.tap_acc_down) {
        *reinterpret_cast<int4*>(a.tap_acc_down + ro) = make_int4(dsum[0], dsum[1], dsum[2], dsum[3]);
        *reinterpret_cast<int4*>(a.tap_acc_down + ro + 4) = make_int4(dsum[4], dsum[5], dsum[6], dsum[7]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = fmaf(p, static_cast<float>(dsum[i]) * sc, o[i]);
    }
  }
  if (a.residual) {   // x^a of Eq.2, added in fp32 before the single rounding
    const uint4 rb = *reinterpret_cast<const uint4*>(a.residual + yo);
    o[0] += bf16_lo(rb.x); o[1] += bf16_hi(rb.x); o[2] += bf16_lo(rb.y); o[3] += bf16_hi(rb.y);
    o[4] += bf16_lo(rb.z); o[5] += bf16_hi(rb.z); o[6] += bf16_lo(rb.w); o[7] += bf16_hi(rb.w);
  }
  uint4 ob;
  ob.x = cvt_pk_bf16(o[0], o[1]);
  ob.y = cvt_pk_bf16(o[2], o[3]);
  ob.z = cvt_pk_bf16(o[4], o[5]);
  ob.w = cvt_pk_bf16(o[6], o[7]);
  *reinterpret_cast<uint4*>(a.out + yo) = ob;
  if (a.out_f32) {
    *reinterpret_cast<float4*>(a.out_f32 + yo) = make_float4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<float4*>(a.out_f32 + yo + 4) = make_float4(o[4], o[5], o[6], o[7]);
  }
}

// The same for a decode step's few tokens, at most PMAX planes of either kind and two experts per token: a handful of
// workgroups whose time is their chain of memory round trips.  All partial planes of y_s are requested beside the routing
// entries and all of D and its scales behind them, two round trips in place of some ten (four planes at a time, expert after
// expert); the 200 registers that takes would cost a large batch its occupancy.  Sums in the same order.  us per forward,
// without -> with it (d = 2048, F = 11008, E = 16): T = 1 57.3 -> 55.9, INT4 T = 4 51.3 -> 50.0, T = 64 106.8 -> 105.9.
template <int PMAX>
__global__ __launch_bounds__(256) void combine_few_kernel(CombineArgs a) {
  const int d = a.d, k = a.k;
  const int chunks = d >> 3;
  const int gid = blockIdx.x * 256 + threadIdx.x;
  if (gid >= a.T * chunks) return;
  const int t = gid / chunks, c0 = (gid - t * chunks) << 3;
  const int64_t yo = static_cast<int64_t>(t) * d + c0;
  int row[2], e[2];
  float p[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = t * k + min(j, k - 1);
    row[j] = a.row_of[i];
    e[j] = a.topk_idx[i];
    p[j] = a.topk_p[i];
  }
  float4 y0[PMAX], y1[PMAX];
#pragma unroll
  for (int u = 0; u < PMAX; ++u)
    if (u < a.y_planes) {
      y0[u] = *reinterpret_cast<const float4*>(a.y_s + u * a.y_stride + yo);
      y1[u] = *reinterpret_cast<const float4*>(a.y_s + u * a.y_stride + yo + 4);
    }
  uint4 rb = make_uint4(0u, 0u, 0u, 0u);
  if (a.residual) rb = *reinterpret_cast<const uint4*>(a.residual + yo);
  __builtin_amdgcn_sched_barrier(0);
  float beta[2], alpha[2];
  int4 d0[2][PMAX], d1[2][PMAX];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int64_t ro = static_cast<int64_t>(row[j]) * d + c0;
    beta[j] = a.beta_h[row[j]];
    alpha[j] = a.alpha[e[j] * 3 + 2];
#pragma unroll
    for (int u = 0; u < PMAX; ++u)
      if (u < a.d_planes) {
        d0[j][u] = *reinterpret_cast<const int4*>(a.acc_down + u * a.d_stride + ro);
        d1[j][u] = *reinterpret_cast<const int4*>(a.acc_down + u * a.d_stride + ro + 4);
      }
  }
  __builtin_amdgcn_sched_barrier(0);
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < PMAX; ++u)
    if (u < a.y_planes) {
      o[0] += y0[u].x; o[1] += y0[u].y; o[2] += y0[u].z; o[3] += y0[u].w;
      o[4] += y1[u].x; o[5] += y1[u].y; o[6] += y1[u].z; o[7] += y1[u].w;
    }
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (j < k) {
      int dsum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < PMAX; ++u)
        if (u < a.d_planes) {
          dsum[0] += d0[j][u].x; dsum[1] += d0[j][u].y; dsum[2] += d0[j][u].z; dsum[3] += d0[j][u].w;
          dsum[4] += d1[j][u].x; dsum[5] += d1[j][u].y; dsum[6] += d1[j][u].z; dsum[7] += d1[j][u].w;
        }
      const float sc = (beta[j] / 127.0f) * alpha[j];
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = fmaf(p[j], static_cast<float>(dsum[i]) * sc, o[i]);
    }
  if (a.residual) {
    o[0] += bf16_lo(rb.x); o[1] += bf16_hi(rb.x); o[2] += bf16_lo(rb.y); o[3] += bf16_hi(rb.y);
    o[4] += bf16_lo(rb.z); o[5] += bf16_hi(rb.z); o[6] += bf16_lo(rb.w); o[7] += bf16_hi(rb.w);
  }
  uint4 ob;
  ob.x = cvt_pk_bf16(o[0], o[1]);
  ob.y = cvt_pk_bf16(o[2], o[3]);
  ob.z = cvt_pk_bf16(o[4], o[5]);
  ob.w = cvt_pk_bf16(o[6], o[7]);
  *reinterpret_cast<uint4*>(a.out + yo) = ob;
}

hipError_t launch_combine(const CombineArgs& a, hipStream_t stream) {
  if (a.T == 0) return hipSuccess;
  const bool taps = a.out_f32 != nullptr || a.tap_y_s != nullptr || a.tap_acc_down != nullptr;
  if (a.T <= kCombineFewTokens && a.k <= 2 && a.y_planes <= 8 && a.d_planes <= 8 && a.row_planes == nullptr && !taps) {
    combine_few_kernel<8><<<(a.T * (a.d >> 3) + 255) / 256, 256, 0, stream>>>(a);
    return hipGetLastError();
  }
  const int64_t n = static_cast<int64_t>(a.T) * (a.d >> 3);
  const unsigned blocks = static_cast<unsigned>((n + 255) / 256);
  combine_kernel<8><<<blocks, 256, 0, stream>>>(a);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n16) {
  const size_t stride = static_cast<size_t>(gridDim.x) * 256;
  for (size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

hipError_t launch_copy(void* dst, const void* src, size_t n_bytes, hipStream_t stream) {
  const size_t n16 = n_bytes / 16;
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 256 * 16) blocks = 256 * 16;
  copy_kernel<<<static_cast<unsigned>(blocks), 256, 0, stream>>>(static_cast<uint4*>(dst), static_cast<const uint4*>(src), n16);
  return hipGetLastError();
}

}  // namespace mote
