// Straight-through estimator of Section 3.2 for the grouped ternary linear layer of Section 3.1,
// Y_e = Q_a(X_e) Q_w(W_e)^T: the quantisers are skipped on the way back, so with the rows of dY
// grouped by expert
//
//   dX[r, c]   = alpha_e * sum_n dY[r, n] * t_e[n, c]
//   dW_e[n, c] = sum_{r in e} bf16(dY[r, n] * beta_r / 127) * q[r, c]
//
// Both are dense bf16 contractions with fp32 accumulation (ternary values and int8 codes are
// exact in bf16) and run on the bf16 MFMA GEMM of the shared expert, which contracts two
// row-major operands along their rows: dX of all experts as one launch over groups of rows, each
// with its own weight matrix; dW of all experts as one launch whose K ranges are the experts.  The
// kernels here bring the operands into that form, each in one launch over all experts:
//
//   reblock_ternary_t_kernel: packed 2-bit codes of W_e [N, K] -> 2-bit blocks of t_e^T along the contraction;
//                             the GEMM unpacks them in registers
//   transpose_groups_kernel : dY [R, N] bf16, scaled by beta_r / 127 and rounded once -> [N, sum_pad],
//                             q [R, K] int8 -> bf16 [K, sum_pad]; expert e in the columns pad0[e] ..,
//                             its rows rounded up to 64 with zeros
//   fill_alpha_kernel       : alpha_e broadcast over the K output channels of dX (the GEMM
//                             epilogue multiplies per output channel)
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace mote {

constexpr int kSteThreads = 256;

// One wavefront re-blocks one packed tile (32 output rows x 128 input channels): the operand of dX contracts over
// the rows, so its blocks (described in shared_ffn.hip) are [channel block 4][this row tile] of 32 x 32 codes.
// Lane (s, b, Q) takes the channels 32s + 4b .. +3 and 16 further on, byte-parallel, and the rows 8Q .. 8Q+7 of their words.  Memory-bound: 90 MB in and out for 16 experts of 11008 x 2048, where the bf16
// matrices they replaced were 721 MB (136 us to write, and the GEMM read them back).
__device__ __forceinline__ void reblock_ternary_t_tile(const uint32_t* __restrict__ tile, uint32_t* __restrict__ out, int64_t block_stride,
                                                       uint32_t* s_in, uint32_t* s_out) {
  const int lane = threadIdx.x & 63;
  reinterpret_cast<u4*>(s_in)[lane] = reinterpret_cast<const u4*>(tile)[lane];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int Q = lane & 3, b = (lane >> 2) & 3, s = lane >> 4;
  // codes t + 1 = 0, 1, 2: the low bit is set for t = 0 only, the high bit for t = +1 only
  uint32_t x[4];   // byte j of x[m]: byte m of word 4b + j (bit J: pair J & 3 of channel 4b + j + 16 * (J >> 2))
#pragma unroll
  for (int odd = 0; odd < 2; ++odd) {
    uint32_t lo = 0u, hi = 0u;
#pragma unroll
    for (int J = 0; J < 8; ++J) {
      const int row = 8 * Q + 2 * (J & 3) + odd;
      const uint32_t w = s_in[(32 * (J >> 2) + row) * 4 + s] >> (2 * b);
      lo |= (w & 0x01010101u) << J;
      hi |= ((w >> 1) & 0x01010101u) << J;
    }
    x[2 * odd] = ~lo;                 // non-zero
    x[2 * odd + 1] = ~(lo | hi);      // negative
  }
  // 4 x 4 byte transpose: word j = bytes j of x[0..3]
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t w = ((x[0] >> (8 * j)) & 0xFFu) | (((x[1] >> (8 * j)) & 0xFFu) << 8) | (((x[2] >> (8 * j)) & 0xFFu) << 16) |
                       ((x[3] >> (8 * j)) << 24);
    s_out[s * 64 + 16 * Q + 4 * b + j] = w;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // block c of the four: 256 bytes, sixteen lanes of 16 bytes
  reinterpret_cast<u4*>(out + (lane >> 4) * block_stride)[lane & 15] = reinterpret_cast<const u4*>(s_out)[lane];
}

// Expert e0 + blockIdx.y of `packed` ([experts][N, K] packed) into matrix blockIdx.y of `out`; experts
// without rows (row0[e] == row0[e + 1]) are skipped, their matrices are never read.  A workgroup takes four
// consecutive row tiles of one channel tile (consecutive K steps: 1 KiB runs of the output).
struct SteGroups {
  int n;
  int row0[65];
  int col0[65];   // first column of the expert's block in the transposed operands (rows padded to 64 per expert)
};
__global__ __launch_bounds__(kSteThreads) void reblock_ternary_t_kernel(const uint32_t* __restrict__ packed, int N, int K,
                                                                        SteGroups grp, int e0, uint32_t* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint32_t s_in[4][256], s_out[4][256];
  const int e = e0 + blockIdx.y;
  if (grp.row0[e] == grp.row0[e + 1]) return;
  const int tiles_k = K >> 7, wave = threadIdx.x >> 6;
  const int kt = blockIdx.x % tiles_k, nt = (blockIdx.x / tiles_k) * 4 + wave;
  const int64_t words = static_cast<int64_t>(N) * K / 16, block_stride = static_cast<int64_t>(N >> 5) * 64;
  reblock_ternary_t_tile(packed + e * words + (static_cast<int64_t>(nt) * tiles_k + kt) * 256,
                         out + blockIdx.y * words + kt * 4 * block_stride + nt * 64, block_stride, s_in[wave], s_out[wave]);
}

// in [rows, C] (bf16 bit patterns scaled by beta[r] / 127, or int8 codes) -> out [C, ld] bf16, columns
// 0 .. rows_pad - 1 of it (the caller offsets `out` to the expert's first column), 64 x 64 tiles
// through LDS.  Rows from `rows` up to rows_pad are written as zeros.
template <bool INT8>
__device__ __forceinline__ void transpose_rows_body(const void* __restrict__ in, const float* __restrict__ beta, int rows,
                                                    int C, int64_t ld, uint16_t* __restrict__ out) {
  __shared__ uint16_t s_t[64][64 + 2];   // [c][r]
  const int c_tiles = C >> 6;
  const int ct = blockIdx.x % c_tiles, rt = blockIdx.x / c_tiles;
  const int tid = threadIdx.x;
  // load: thread t reads 16 consecutive channels of row rt * 64 + t / 4
  {
    const int r = rt * 64 + (tid >> 2), c0 = ct * 64 + (tid & 3) * 16;
    uint16_t v[16];
    if (r < rows) {
      if constexpr (INT8) {
        const u4 raw = *reinterpret_cast<const u4*>(static_cast<const int8_t*>(in) + static_cast<int64_t>(r) * C + c0);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int q = static_cast<int8_t>((w[i >> 2] >> (8 * (i & 3))) & 0xFF);
          v[i] = f32_to_bf16(static_cast<float>(q));   // |q| <= 128: exact
        }
      } else {
        const float s = beta[r] / 127.0f;   // the scale of Q_a, as the forward pass forms it
        const uint16_t* src = static_cast<const uint16_t*>(in) + static_cast<int64_t>(r) * C + c0;
        const u4 a = *reinterpret_cast<const u4*>(src), b = *reinterpret_cast<const u4*>(src + 8);
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          v[2 * i] = f32_to_bf16(bf16_lo(w[i]) * s);
          v[2 * i + 1] = f32_to_bf16(bf16_hi(w[i]) * s);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = 0;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s_t[(tid & 3) * 16 + i][tid >> 2] = v[i];
  }
  __syncthreads();
  // store: thread t writes 16 consecutive rows of channel ct * 64 + t / 4
  {
    const int c = tid >> 2, r0 = (tid & 3) * 16;
    const uint16_t* src = &s_t[c][r0];
    u4 a, b;
    a.x = src[0] | (static_cast<uint32_t>(src[1]) << 16);
    a.y = src[2] | (static_cast<uint32_t>(src[3]) << 16);
    a.z = src[4] | (static_cast<uint32_t>(src[5]) << 16);
    a.w = src[6] | (static_cast<uint32_t>(src[7]) << 16);
    b.x = src[8] | (static_cast<uint32_t>(src[9]) << 16);
    b.y = src[10] | (static_cast<uint32_t>(src[11]) << 16);
    b.z = src[12] | (static_cast<uint32_t>(src[13]) << 16);
    b.w = src[14] | (static_cast<uint32_t>(src[15]) << 16);
    uint16_t* dst = out + static_cast<int64_t>(ct * 64 + c) * ld + rt * 64 + r0;
    *reinterpret_cast<u4*>(dst) = a;
    *reinterpret_cast<u4*>(dst + 8) = b;
  }
}

// Every expert in one launch (blockIdx.y = expert): expert e owns the rows row0[e] .. row0[e+1]-1
// of `in` and the columns col0[e] .. col0[e+1]-1 of `out` ([C, ld]; the block is padded with zeros to a
// multiple of 64 columns).  The grid covers the longest block; workgroups past an expert's block leave.
template <bool INT8>
__global__ __launch_bounds__(kSteThreads) void transpose_groups_kernel(const void* __restrict__ in, const float* __restrict__ beta,
                                                                       SteGroups grp, int C, int64_t ld, uint16_t* __restrict__ out) {
  const int e = blockIdx.y, r0 = grp.row0[e], c0 = grp.col0[e];
  if (static_cast<int>(blockIdx.x / (C >> 6)) * 64 >= grp.col0[e + 1] - c0) return;
  const void* const in_e = INT8 ? static_cast<const void*>(static_cast<const int8_t*>(in) + static_cast<int64_t>(r0) * C)
                                : static_cast<const void*>(static_cast<const uint16_t*>(in) + static_cast<int64_t>(r0) * C);
  transpose_rows_body<INT8>(in_e, INT8 ? nullptr : beta + r0, grp.row0[e + 1] - r0, C, ld, out + c0);
}

__global__ __launch_bounds__(kSteThreads) void fill_alpha_kernel(const float* __restrict__ alpha, int alpha_stride, int E,
                                                                 int K, float* __restrict__ out) {
  const int i = blockIdx.x * kSteThreads + threadIdx.x;
  if (i < E * K) out[i] = alpha[(i / K) * alpha_stride];
}

__global__ __launch_bounds__(kSteThreads) void fill_zero_kernel(float* __restrict__ out, int64_t n4) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kSteThreads;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kSteThreads + threadIdx.x; i < n4; i += stride)
    reinterpret_cast<float4*>(out)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// out[i] = scale * (plane 0 + plane 1 + ...)[i], planes added in order; alpha == nullptr: scale 1
__global__ __launch_bounds__(kSteThreads) void sum_planes_kernel(const float* __restrict__ planes, int n_planes, int64_t n4,
                                                                 const float* __restrict__ alpha, float* __restrict__ out) {
  const float scale = alpha != nullptr ? alpha[0] : 1.0f;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kSteThreads;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kSteThreads + threadIdx.x; i < n4; i += stride) {
    float4 acc = reinterpret_cast<const float4*>(planes)[i];
    for (int p = 1; p < n_planes; ++p) {
      const float4 v = reinterpret_cast<const float4*>(planes)[p * n4 + i];
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    reinterpret_cast<float4*>(out)[i] = make_float4(acc.x * scale, acc.y * scale, acc.z * scale, acc.w * scale);
  }
}

static inline size_t ste_align(size_t v) { return (v + 255) / 256 * 256; }

// The GEMMs address each operand of a launch with 32-bit byte offsets: the experts of one launch have operands below this.
constexpr int64_t kSteOperandBytes = int64_t{1} << 32;

// K planes of the dX contraction at most; dX runs as one grouped GEMM over as many experts as have their
// weights, counted as bf16, below 4 GiB together (the blocks are an eighth of that; the limit is a tuning knob so that
// tests reach the loop over batches with small matrices) and their gradient rows below kSteOperandBytes.
constexpr int kSteMaxPlanes = 8;
static int ste_dx_batch(int N, int K, int E) {
  const int64_t per = static_cast<int64_t>(N) * K * 2;
  const int64_t lim_mib = std::min(std::max(knob(kKnobSteBatchMiB), 1), 4095);
  const int64_t g = ((lim_mib << 20) + ((int64_t{1} << 20) - 1)) / per;
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(g, E)));
}

// Workspace: the re-blocked transposed weights of one batch of experts [experts][K, N] (2 bits each), the transposed
// scaled gradient rows and codes of every expert (sum of rows_pad_e <= R + 63 E columns, a sixteenth
// more when near-equal blocks are padded to the longest), alpha
// broadcast [E, K], partial planes of dX.
static size_t ste_pad_rows(int R, int E) { return (static_cast<size_t>(R) + 64 * static_cast<size_t>(E)) * 17 / 16 + 64; }
size_t ste_backward_workspace_bytes(int R, int N, int K, int E) {
  const size_t rp = ste_pad_rows(R, E);
  const size_t plane_bytes = static_cast<size_t>(kSteMaxPlanes) * R * K * 4;
  return ste_align(static_cast<size_t>(ste_dx_batch(N, K, E)) * K * N / 4) + ste_align(rp * N * 2) + ste_align(rp * K * 2) +
         ste_align(static_cast<size_t>(E) * K * 4) + ste_align(plane_bytes);
}

hipError_t launch_ste_backward(const uint16_t* dy, const int32_t* offsets_host, const uint32_t* packed, const float* alpha,
                               int alpha_stride, const int8_t* q, const float* beta, int R, int N, int K, int E,
                               float* dx, float* dw, void* workspace, hipStream_t stream) {
  char* ws = static_cast<char*>(workspace);
  const size_t rp_total = ste_pad_rows(R, E);
  const int batch = ste_dx_batch(N, K, E);
  uint32_t* wt = reinterpret_cast<uint32_t*>(ws);
  ws += ste_align(static_cast<size_t>(batch) * K * N / 4);
  uint16_t* dyt = reinterpret_cast<uint16_t*>(ws);
  ws += ste_align(rp_total * N * 2);
  uint16_t* qt = reinterpret_cast<uint16_t*>(ws);
  ws += ste_align(rp_total * K * 2);
  float* alpha_vec = reinterpret_cast<float*>(ws);
  ws += ste_align(static_cast<size_t>(E) * K * 4);
  float* dx_planes = reinterpret_cast<float*>(ws);

  SteGroups grp;
  grp.n = E;
  int64_t tight = 0;
  int longest = 0;
  for (int e = 0; e < E; ++e) {
    const int rows_pad = (offsets_host[e + 1] - offsets_host[e] + 63) / 64 * 64;
    tight += rows_pad;
    longest = std::max(longest, rows_pad);
  }
  // near-equal groups: every block as long as the longest (at most 1/16 more contraction steps); tiles of
  // equal length keep the workgroups of the dW GEMM in step (3B width, 16 groups of about 1024 rows:
  // 966 -> 921 us for the GEMM)
  const bool uniform = static_cast<int64_t>(E) * longest * 16 <= tight * 17;
  int block[64];   // columns of an expert's block in the transposed operands
  for (int e = 0; e < E; ++e) block[e] = uniform ? longest : (offsets_host[e + 1] - offsets_host[e] + 63) / 64 * 64;
  for (int e = 0; e <= 64; ++e) grp.row0[e] = offsets_host[std::min(e, E)], grp.col0[e] = 0;

  fill_alpha_kernel<<<(E * K + kSteThreads - 1) / kSteThreads, kSteThreads, 0, stream>>>(alpha, alpha_stride, E, K, alpha_vec);
  // dX: the codes of a batch of experts re-blocked along the contraction, then one grouped GEMM over their rows, scaled by alpha
  for (int e0 = 0, nb; e0 < E; e0 += nb) {
    const int row0 = offsets_host[e0];
    for (nb = 1; nb < std::min(batch, E - e0) && static_cast<int64_t>(offsets_host[e0 + nb + 1] - row0) * N * 2 < kSteOperandBytes;) ++nb;
    const int rows = offsets_host[e0 + nb] - row0;
    if (rows == 0) continue;
    reblock_ternary_t_kernel<<<dim3((N / 128) * (K / 128), nb), kSteThreads, 0, stream>>>(packed, N, K, grp, e0, wt);
    const GemmSplit sp = grouped_gemm_split(offsets_host + e0, nb, K, N, kSteMaxPlanes);
    const uint16_t* dy_b = dy + static_cast<int64_t>(row0) * N;
    float* dx_b = dx + static_cast<int64_t>(row0) * K;
    const float* alpha_b = alpha_vec + static_cast<int64_t>(e0) * K;
    hipError_t err = launch_gemm_grouped_f32(dy_b, wt, offsets_host + e0, nb, K, N, dx_b, dx_planes, alpha_b, sp, stream);
    if (err != hipSuccess) return err;
    if (sp.planes > 1) {   // rows whose contraction over N was cut into planes, added in order here
      const int64_t n4 = static_cast<int64_t>(rows - sp.split_row) * K / 4;
      sum_planes_kernel<<<static_cast<unsigned>(std::min<int64_t>((n4 + kSteThreads - 1) / kSteThreads, 2048)), kSteThreads,
                          0, stream>>>(dx_planes, sp.planes, n4, nullptr, dx_b + static_cast<int64_t>(sp.split_row) * K);
    }
  }
  // dW: the scaled gradient rows and the codes of every expert transposed into [N, columns] and [K, columns]
  // (an expert's block padded with zeros to a multiple of 64 columns), then ONE GEMM whose K ranges are the experts:
  // plane e = dW_e, zeros for an expert without rows.  Experts whose blocks reach kSteOperandBytes together go in several
  // such rounds, which use the same scratch one after the other.
  for (int e0 = 0, nb; e0 < E; e0 += nb) {
    int32_t col0[65] = {0};   // first column of every block = K ranges of the contraction
    int rows_max = 0;
    for (nb = 0; e0 + nb < E; ++nb) {
      const int64_t cols = static_cast<int64_t>(col0[nb]) + block[e0 + nb];
      if (nb > 0 && cols * std::max(N, K) * 2 >= kSteOperandBytes) break;
      col0[nb + 1] = static_cast<int32_t>(cols);
      rows_max = std::max(rows_max, block[e0 + nb]);
    }
    float* const dw_b = dw + static_cast<int64_t>(e0) * N * K;
    const int64_t ld = col0[nb];
    if (ld == 0) {
      fill_zero_kernel<<<1024, kSteThreads, 0, stream>>>(dw_b, static_cast<int64_t>(nb) * N * K / 4);
      continue;
    }
    SteGroups part;
    part.n = nb;
    for (int i = 0; i <= 64; ++i) part.row0[i] = offsets_host[std::min(e0 + i, E)], part.col0[i] = col0[std::min(i, nb)];
    const unsigned tiles_r = static_cast<unsigned>(rows_max / 64);
    transpose_groups_kernel<false><<<dim3(tiles_r * (N / 64), nb), kSteThreads, 0, stream>>>(dy, beta, part, N, ld, dyt);
    transpose_groups_kernel<true><<<dim3(tiles_r * (K / 64), nb), kSteThreads, 0, stream>>>(q, nullptr, part, K, ld, qt);
    hipError_t err = launch_gemm_tn_f32_kgroups(dyt, qt, N, K, col0, nb, dw_b, stream);
    if (err != hipSuccess) return err;
  }
  return hipGetLastError();
}

}  // namespace mote
