// Q_w (absmean ternary quantiser, Eq.7, Eq.9, Eq.10 of Section 3.1) and the 2-bit pack.
//
// Three launches on the caller's stream:
//   1. abs_sum_kernel   : fixed grid, each block writes one fp64 partial of sum|W| into the
//                         (not yet used) packed buffer -- deterministic, no atomics
//   2. alpha_kernel     : one block folds the partials in a fixed order, writes
//                         alpha = max(fp32(sum / (N*K)), 1e-5)
//   3. pack_kernel      : one workgroup per packed tile (32 rows x 128 channels):
//                         W / alpha -> RNE -> clip -> code t+1 at bit 8*(i%4) + 2*(i/4)
//
// Bound: HBM, the matrix is read twice (alpha is known only after the first pass; a matrix below the
// 256 MB of the memory-side cache is served from there the second time).
#include "common.h"
#include "launch.h"

namespace mote {

constexpr int kPackThreads = 256;

// The values of 16 bytes of a matrix: 4 fp32 or 8 bf16.
template <typename T>
struct Chunk;
template <>
struct Chunk<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void values(const u4& p, float (&v)[4]) {
    v[0] = __uint_as_float(p.x); v[1] = __uint_as_float(p.y); v[2] = __uint_as_float(p.z); v[3] = __uint_as_float(p.w);
  }
};
template <>
struct Chunk<uint16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void values(const u4& p, float (&v)[8]) {
    v[0] = bf16_lo(p.x); v[1] = bf16_hi(p.x); v[2] = bf16_lo(p.y); v[3] = bf16_hi(p.y);
    v[4] = bf16_lo(p.z); v[5] = bf16_hi(p.z); v[6] = bf16_lo(p.w); v[7] = bf16_hi(p.w);
  }
};

// Every thread keeps four 16-byte loads in flight (one 4-byte load at a time before: 11008 x 2048 fp32
// 30.2 -> 16.5 us = 5.5 TB/s, the rate of a large copy and more); the sums stay fp64.
constexpr int kSumUnroll = 4;
constexpr int kSumBlocks = 1024;

template <typename T>
__global__ __launch_bounds__(kPackThreads) void abs_sum_kernel(const u4* __restrict__ w, int64_t n_chunks,
                                                               double* __restrict__ partial) {
  __shared__ double s_part[kPackThreads / kWave];
  double acc[kSumUnroll] = {0.0, 0.0, 0.0, 0.0};
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kPackThreads;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kPackThreads + threadIdx.x; i < n_chunks; i += kSumUnroll * stride) {
    u4 c[kSumUnroll];
#pragma unroll
    for (int u = 0; u < kSumUnroll; ++u) c[u] = i + u * stride < n_chunks ? w[i + u * stride] : u4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < kSumUnroll; ++u) {
      float v[Chunk<T>::N];
      Chunk<T>::values(c[u], v);
#pragma unroll
      for (int j = 0; j < Chunk<T>::N; ++j) acc[u] += static_cast<double>(fabsf(v[j]));
    }
  }
  double a = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < kPackThreads / kWave; ++i) t += s_part[i];
    partial[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(kPackThreads) void alpha_kernel(const double* __restrict__ partial, int n_partial,
                                                            double count, float* __restrict__ alpha) {
  __shared__ double s_part[kPackThreads / kWave];
  double v[kSumBlocks / kPackThreads];   // every partial is requested before the first one is added
#pragma unroll
  for (int j = 0; j < kSumBlocks / kPackThreads; ++j) {
    const int i = threadIdx.x + j * kPackThreads;
    v[j] = i < n_partial ? partial[i] : 0.0;
  }
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < kSumBlocks / kPackThreads; ++j) acc += v[j];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < kPackThreads / kWave; ++i) t += s_part[i];
    const float a = static_cast<float>(t / count);
    alpha[0] = fmaxf(a, kEps);
  }
}

// t + 1 of clip(round_half_even(w / alpha), -1, 1), w / alpha rounded to fp32, without the division:
// the rounded quotient is above 1/2 exactly when |w| > alpha * (1/2 + 2^-25) (the midpoint between 1/2 and
// the next fp32 value; at the midpoint itself the division rounds to the even 1/2, whose round-half-even
// is 0).  alpha * (1/2 + 2^-25) has at most 49 significant bits, so it is exact in fp64, and |w| exceeds it
// exactly when |w| exceeds the largest fp32 value c that does not.  A NaN weight gives t = -1.
__device__ __forceinline__ float ternary_threshold(float alpha) {
  const double thr = static_cast<double>(alpha) * (0.5 + 0x1p-25);
  const float c = static_cast<float>(thr);
  return static_cast<double>(c) > thr ? __uint_as_float(__float_as_uint(c) - 1u) : c;
}
// finite is false for an infinite scale (a matrix with infinite weights): w / alpha is then 0 or NaN
__device__ __forceinline__ uint32_t ternary_code(float w, float c, bool finite, bool binary) {
  if (binary) return w < 0.0f ? 0u : 2u;   // 1-bit quantiser of the routed-expert ablation: sign(w), sign(0) = +1
  if (!finite) return fabsf(w) < __builtin_inff() ? 1u : 0u;
  return w > c ? 2u : (w >= -c ? 1u : 0u);
}

// One workgroup per tile.  A row of the tile is read by consecutive lanes, 16 bytes each (whole cache lines;
// a thread that owned a whole word read 64 bytes at a stride of 128), the lanes that share a word combine
// their bits with two DPP moves and each stores the word of one pass.  11008 x 2048: fp32 16.8 -> 15.1 us
// (6.3 TB/s, the matrix comes from the memory-side cache), bf16 10.3 us.  With the correctly rounded
// division (about 12 instructions per weight instead of 3) the vector pipe took half of the kernel's time.
template <typename T>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(const T* __restrict__ w, int tiles_k, int64_t n_in,
                                                            const float* __restrict__ alpha_ptr, bool binary,
                                                            uint32_t* __restrict__ packed) {
  constexpr int N = Chunk<T>::N;              // channels per thread and pass
  constexpr int TPR = 128 / N;                // threads per row
  constexpr int ROWS = kPackThreads / TPR;    // rows per pass
  constexpr int PASSES = 32 / ROWS;           // = threads that share a word of 16 channels
  static_assert(PASSES == 16 / N, "each of the threads that share a word stores the word of one pass");
  const int tid = threadIdx.x, c = tid % TPR, r0 = tid / TPR;
  const int64_t nt = blockIdx.x / static_cast<unsigned>(tiles_k);
  const int kt = blockIdx.x % static_cast<unsigned>(tiles_k);
  const T* const src = w + (nt * 32 + r0) * n_in + kt * 128 + c * N;
  u4 raw[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) raw[p] = *reinterpret_cast<const u4*>(src + p * ROWS * n_in);
  const float alpha = load_uniform(alpha_ptr);
  const float thr = ternary_threshold(alpha);
  const bool finite = alpha < __builtin_inff();
  const int part = c % PASSES;                // which N channels of the word
  uint32_t mine = 0;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    float v[N];
    Chunk<T>::values(raw[p], v);
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) word |= ternary_code(v[i], thr, finite, binary) << (8 * (i & 3) + 2 * (i >> 2));
    int b = static_cast<int>(word << (2 * (N / 4) * part));
    b |= __builtin_amdgcn_mov_dpp(b, 0xB1, 0xF, 0xF, true);                              // lane ^ 1
    if constexpr (PASSES == 4) b |= __builtin_amdgcn_mov_dpp(b, 0x4E, 0xF, 0xF, true);   // lane ^ 2
    mine = part == p ? static_cast<uint32_t>(b) : mine;
  }
  const int r = part * ROWS + r0, run = c / PASSES;   // run of 16 channels: 2 s + g
  packed[static_cast<int64_t>(blockIdx.x) * 256 + 4 * (32 * (run & 1) + r) + (run >> 1)] = mine;
}

template <typename T>
static hipError_t pack_impl(const T* w, int64_t n_out, int64_t n_in, uint32_t* packed, float* alpha, bool binary,
                            hipStream_t stream) {
  const int64_t n = n_out * n_in;
  const int64_t n_chunks = n / Chunk<T>::N;
  // The packed buffer holds n/4 bytes >= 1024, i.e. room for >= 128 fp64 partials.
  const int64_t max_partials = (n / 4) / 8;
  const int64_t want = (n_chunks + kPackThreads * kSumUnroll - 1) / (kPackThreads * kSumUnroll);
  int n_partial = static_cast<int>(want < kSumBlocks ? want : kSumBlocks);
  if (n_partial > max_partials) n_partial = static_cast<int>(max_partials);
  double* partial = reinterpret_cast<double*>(packed);
  abs_sum_kernel<T><<<n_partial, kPackThreads, 0, stream>>>(reinterpret_cast<const u4*>(w), n_chunks, partial);
  alpha_kernel<<<1, kPackThreads, 0, stream>>>(partial, n_partial, static_cast<double>(n), alpha);
  pack_kernel<T><<<static_cast<unsigned>(n / 4096), kPackThreads, 0, stream>>>(w, static_cast<int>(n_in / 128), n_in, alpha,
                                                                               binary, packed);
  return hipGetLastError();
}

hipError_t launch_pack_ternary(const void* w, bool is_bf16, int64_t n_out, int64_t n_in, uint32_t* packed,
                               float* alpha, bool binary, hipStream_t stream) {
  if (is_bf16) return pack_impl<uint16_t>(static_cast<const uint16_t*>(w), n_out, n_in, packed, alpha, binary, stream);
  return pack_impl<float>(static_cast<const float*>(w), n_out, n_in, packed, alpha, binary, stream);
}

}  // namespace mote
