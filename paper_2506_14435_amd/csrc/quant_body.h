// Device code of the row quantiser Q_a(h), shared by quant_rows_kernel and by the decode kernel that runs it
// beside the shared expert's down projection.
#pragma once
#include "common.h"

namespace mote {

template <int THREADS>
__device__ __forceinline__ float block_max(float v, float* s_buf) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) s_buf[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = s_buf[0];
#pragma unroll
  for (int i = 1; i < THREADS / kWave; ++i) r = fmaxf(r, s_buf[i]);
  __syncthreads();
  return r;
}

template <int THREADS>
__device__ __forceinline__ int block_sum(int v, int* s_buf) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) s_buf[threadIdx.x >> 6] = v;
  __syncthreads();
  int r = 0;
#pragma unroll
  for (int i = 0; i < THREADS / kWave; ++i) r += s_buf[i];
  __syncthreads();
  return r;
}

// One workgroup per dispatch row.  Rows of up to THREADS * CHUNKS 8-element chunks are
// read once: every thread requests all its chunks before it looks at the first (the loads are in
// flight together), takes the absmax, and quantises out of registers.  Longer rows take a second
// sweep (L2 hits) for the part that did not fit.
__device__ __forceinline__ float chunk_absmax(const uint4& p) {
  return fmaxf(fmaxf(fmaxf(fabsf(bf16_lo(p.x)), fabsf(bf16_hi(p.x))), fmaxf(fabsf(bf16_lo(p.y)), fabsf(bf16_hi(p.y)))),
               fmaxf(fmaxf(fabsf(bf16_lo(p.z)), fabsf(bf16_hi(p.z))), fmaxf(fabsf(bf16_lo(p.w)), fabsf(bf16_hi(p.w)))));
}

__device__ __forceinline__ int chunk_quant(const uint4& p, float s, uint2* o) {
  const int q0 = quant_i8(bf16_lo(p.x), s), q1 = quant_i8(bf16_hi(p.x), s);
  const int q2 = quant_i8(bf16_lo(p.y), s), q3 = quant_i8(bf16_hi(p.y), s);
  const int q4 = quant_i8(bf16_lo(p.z), s), q5 = quant_i8(bf16_hi(p.z), s);
  const int q6 = quant_i8(bf16_lo(p.w), s), q7 = quant_i8(bf16_hi(p.w), s);
  o->x = (q0 & 0xFF) | ((q1 & 0xFF) << 8) | ((q2 & 0xFF) << 16) | (static_cast<uint32_t>(q3 & 0xFF) << 24);
  o->y = (q4 & 0xFF) | ((q5 & 0xFF) << 8) | ((q6 & 0xFF) << 16) | (static_cast<uint32_t>(q7 & 0xFF) << 24);
  return q0 + q1 + q2 + q3 + q4 + q5 + q6 + q7;
}

template <int THREADS>
struct QuantRowScratch {   // LDS of a workgroup
  float f[THREADS / kWave];
  int i[THREADS / kWave];
};

// One row by a workgroup of THREADS threads, CHUNKS 16-byte chunks per thread in registers.
template <int THREADS, int CHUNKS>
__device__ __forceinline__ void quant_row(QuantRowScratch<THREADS>& lds, int64_t row, const uint16_t* __restrict__ h, int F, int8_t* __restrict__ q,
                                          float* __restrict__ beta, int32_t* __restrict__ rowsum) {
  const uint16_t* hp = h + row * F;
  const int n_chunks = F >> 3;
  uint4 keep[CHUNKS];
#pragma unroll
  for (int i = 0; i < CHUNKS; ++i) {
    const int ch = threadIdx.x + i * THREADS;
    keep[i] = ch < n_chunks ? *reinterpret_cast<const uint4*>(hp + ch * 8) : make_uint4(0u, 0u, 0u, 0u);
  }
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < CHUNKS; ++i) amax = fmaxf(amax, chunk_absmax(keep[i]));
  for (int ch = threadIdx.x + CHUNKS * THREADS; ch < n_chunks; ch += THREADS)
    amax = fmaxf(amax, chunk_absmax(*reinterpret_cast<const uint4*>(hp + ch * 8)));
  const float b = fmaxf(block_max<THREADS>(amax, lds.f), kEps);
  const float s = 127.0f / b;
  int rs = 0;
#pragma unroll
  for (int i = 0; i < CHUNKS; ++i) {
    const int ch = threadIdx.x + i * THREADS;
    uint2 o;
    const int part = chunk_quant(keep[i], s, &o);
    if (ch < n_chunks) {
      rs += part;
      *reinterpret_cast<uint2*>(q + row * F + ch * 8) = o;
    }
  }
  for (int ch = threadIdx.x + CHUNKS * THREADS; ch < n_chunks; ch += THREADS) {
    uint2 o;
    rs += chunk_quant(*reinterpret_cast<const uint4*>(hp + ch * 8), s, &o);
    *reinterpret_cast<uint2*>(q + row * F + ch * 8) = o;
  }
  const int total = block_sum<THREADS>(rs, lds.i);
  if (threadIdx.x == 0) {
    beta[row] = b;
    rowsum[row] = total;
  }
}

}  // namespace mote
