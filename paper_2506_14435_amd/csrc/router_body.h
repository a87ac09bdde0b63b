// Device code of the vector router: logits, gate softmax, top-k and Q_a(x) of a group of TPW tokens,
// shared by router_quant_kernel and by the decode kernel that runs the router beside the shared expert.
#pragma once
#include "common.h"

namespace mote {

template <int OFF, int N>
__device__ __forceinline__ void reduce_scatter_step(double (&v)[N], int lane) {
  constexpr int kHalf = OFF;  // values kept after this step == OFF (64 -> 32 -> ... -> 1)
  const bool up = (lane & OFF) != 0;
#pragma unroll
  for (int i = 0; i < kHalf; ++i) {
    const double keep = up ? v[i + kHalf] : v[i];
    const double send = up ? v[i] : v[i + kHalf];
    v[i] = keep + __shfl_xor(send, OFF, kWave);
  }
  if constexpr (OFF > 1) reduce_scatter_step<OFF / 2, N>(v, lane);
}

template <int EMAX>
__device__ __forceinline__ void load_router_row(const uint16_t* __restrict__ row, int E, bool vec_ok,
                                                double (&w)[EMAX]) {
  if (vec_ok) {
#pragma unroll
    for (int v = 0; v < EMAX / 8; ++v) {
      if (v * 8 < E) {
        const uint4 p = *reinterpret_cast<const uint4*>(row + v * 8);
        w[v * 8 + 0] = bf16_lo(p.x); w[v * 8 + 1] = bf16_hi(p.x);
        w[v * 8 + 2] = bf16_lo(p.y); w[v * 8 + 3] = bf16_hi(p.y);
        w[v * 8 + 4] = bf16_lo(p.z); w[v * 8 + 5] = bf16_hi(p.z);
        w[v * 8 + 6] = bf16_lo(p.w); w[v * 8 + 7] = bf16_hi(p.w);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) w[v * 8 + j] = 0.0;
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < EMAX; ++e) w[e] = (e < E) ? static_cast<double>(bf16_to_f32(row[e])) : 0.0;
  }
}

// The same in two steps, so that all rows of a chunk can be on their way together: the bf16 patterns of a row, two
// per register, and their conversion.  vec: 8 for rows of whole 16-byte runs, 4 for 8-byte runs (of an aligned matrix).
template <int EMAX>
__device__ __forceinline__ void load_router_row_raw(const uint16_t* __restrict__ row, int E, int vec, uint32_t (&r)[EMAX / 2]) {
#pragma unroll
  for (int i = 0; i < EMAX / 2; ++i) r[i] = 0u;
  if (vec == 8) {
#pragma unroll
    for (int v = 0; v < EMAX / 8; ++v)
      if (v * 8 < E) {
        const uint4 p = *reinterpret_cast<const uint4*>(row + v * 8);
        r[v * 4] = p.x; r[v * 4 + 1] = p.y; r[v * 4 + 2] = p.z; r[v * 4 + 3] = p.w;
      }
  } else if (vec == 4) {
#pragma unroll
    for (int v = 0; v < EMAX / 4; ++v)
      if (v * 4 < E) {
        const uint2 p = *reinterpret_cast<const uint2*>(row + v * 4);
        r[v * 2] = p.x; r[v * 2 + 1] = p.y;
      }
  } else {
#pragma unroll
    for (int e = 0; e < EMAX; ++e)
      if (e < E) r[e / 2] |= static_cast<uint32_t>(row[e]) << (16 * (e & 1));
  }
}

// Gate softmax (Eq.3) and top-k of one token on the EMAX consecutive lanes that hold its logits
// (lane's expert e; logits beyond E are padding).  `store`: whether this lane group's token exists
// and is this group's to write (the lanes still take part in the shuffles otherwise).
template <int EMAX>
__device__ __forceinline__ void gate_topk(double l, int e, bool store, int tok, const float* __restrict__ bias, int E,
                                          int k, int32_t* __restrict__ topk_idx, float* __restrict__ topk_p,
                                          float* __restrict__ gate_p) {
  const bool valid = e < E;
  if (bias != nullptr && valid) l += static_cast<double>(bias[e]);
  // A non-finite hidden state must not be able to select a padding lane: NaN and -inf logits
  // are ranked as the lowest finite value, still above the padding (-1e300) and the taken
  // (-1.7e300) lanes, so the k winners are always experts below E.
  if (!(l > -1.0e299)) l = -1.0e299;
  if (!valid) l = -1.0e300;
  // gate softmax (Eq.3) over the EMAX lanes of a token: max and sum by xor shuffles
  double mx = l;
#pragma unroll
  for (int off = EMAX / 2; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, kWave));
  // fp64 like the logits; P is rounded to fp32 once
  const double ex = valid ? exp(l - mx) : 0.0;
  double sum = ex;
#pragma unroll
  for (int off = EMAX / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
  const float pr = static_cast<float>(ex / sum);
  if (gate_p != nullptr && valid && store)
    gate_p[static_cast<int64_t>(tok) * E + e] = pr;   // the whole gate distribution (Eq.12 needs it)
  // top-k: k rounds of an arg-max butterfly over the EMAX lanes of a token.  Every lane of the
  // group ends a round with the winner (largest logit, ties to the lower expert index); the
  // winner's own lane then leaves the contest.
  double cur = l;                      // invalid experts sit at -1e300, taken ones go below that
  for (int j = 0; j < k; ++j) {
    double bl = cur;
    int be = e;
    float bp = pr;
#pragma unroll
    for (int off = EMAX / 2; off > 0; off >>= 1) {
      const double ol = __shfl_xor(bl, off, kWave);
      const int oe = __shfl_xor(be, off, kWave);
      const float op = __shfl_xor(bp, off, kWave);
      const bool take = (ol > bl) || (ol == bl && oe < be);
      bl = take ? ol : bl;
      be = take ? oe : be;
      bp = take ? op : bp;
    }
    if (be == e) cur = -1.7e300;
    if (e == 0 && store) {
      topk_idx[static_cast<int64_t>(tok) * k + j] = be;
      topk_p[static_cast<int64_t>(tok) * k + j] = bp;
    }
  }
}

template <int TPW, int NW>
struct RouterScratch {   // LDS of a workgroup
  double logit[NW][64];
  float amax[NW][TPW];
  int rsum[NW][TPW];
};

// One token group = TPW tokens from t0 on; the NW wavefronts of the workgroup split its channels.
// ROWS: router rows of a chunk requested together (registers against latency); 8: all of them, as raw patterns, in front
// of the first multiplication - one memory round trip per chunk, for workgroups whose time is that chain.
template <int EMAX, int TPW, int NW, int ROWS>
__device__ __forceinline__ void router_quant_group(
    RouterScratch<TPW, NW>& lds, int t0, const uint16_t* __restrict__ x, const uint16_t* __restrict__ w_router, const float* __restrict__ bias, int T,
    int d, int E, int k, int32_t* __restrict__ topk_idx, float* __restrict__ topk_p, int8_t* __restrict__ q_x,
    float* __restrict__ beta_x, int32_t* __restrict__ rowsum_x, float* __restrict__ gate_p) {
  constexpr int NV = EMAX * TPW;           // logits of a token group; lane l ends up with logit l % NV
  static_assert(NV <= 64 && 64 % NV == 0, "at most one finished logit per lane");
  constexpr int kWaves = NW;               // wavefronts that split the channels of one token group
  constexpr int kThreads = 64 * NW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n_chunks = d >> 3;
  const bool vec_ok = (E & 7) == 0;
  const int vec = vec_ok ? 8 : (E & 3) == 0 && (reinterpret_cast<uintptr_t>(w_router) & 7) == 0 ? 4 : 0;

  const uint16_t* xrow[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) xrow[t] = x + static_cast<int64_t>(min(t0 + t, T - 1)) * d;

  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.0;
  float amax[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) amax[t] = 0.0f;

  // with at most one chunk per lane the token values stay in registers for the quantisation pass
  const bool single_pass = n_chunks <= kThreads;
  u4 xkeep[TPW];   // plain register vectors
#pragma unroll
  for (int t = 0; t < TPW; ++t) xkeep[t] = u4{0u, 0u, 0u, 0u};
  for (int ch = wave * kWave + lane; ch < n_chunks; ch += kThreads) {
    const int c0 = ch << 3;
    float xf[TPW][8];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const uint4 p = *reinterpret_cast<const uint4*>(xrow[t] + c0);
      xkeep[t] = u4{p.x, p.y, p.z, p.w};
      xf[t][0] = bf16_lo(p.x); xf[t][1] = bf16_hi(p.x); xf[t][2] = bf16_lo(p.y); xf[t][3] = bf16_hi(p.y);
      xf[t][4] = bf16_lo(p.z); xf[t][5] = bf16_hi(p.z); xf[t][6] = bf16_lo(p.w); xf[t][7] = bf16_hi(p.w);
#pragma unroll
      for (int i = 0; i < 8; ++i) amax[t] = fmaxf(amax[t], fabsf(xf[t][i]));
    }
    if constexpr (ROWS == 8) {
      uint32_t raw[8][EMAX / 2];
#pragma unroll
      for (int i = 0; i < 8; ++i) load_router_row_raw<EMAX>(w_router + static_cast<int64_t>(c0 + i) * E, E, vec, raw[i]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
          const double xv = static_cast<double>(xf[t][i]);
#pragma unroll
          for (int e = 0; e < EMAX; ++e) {
            const uint32_t p = raw[i][e / 2];
            acc[t * EMAX + e] = fma(xv, static_cast<double>(e & 1 ? bf16_hi(p) : bf16_lo(p)), acc[t * EMAX + e]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);   // a row at a time: all conversions at once would take 256 registers
      }
    } else
#pragma unroll ROWS
    for (int i = 0; i < 8; ++i) {
      double w[EMAX];
      load_router_row<EMAX>(w_router + static_cast<int64_t>(c0 + i) * E, E, vec_ok, w);
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const double xv = static_cast<double>(xf[t][i]);
#pragma unroll
        for (int e = 0; e < EMAX; ++e) acc[t * EMAX + e] = fma(xv, w[e], acc[t * EMAX + e]);
      }
    }
  }

  // lane l holds this wavefront's share of logit(token (l % NV) / EMAX, expert l % EMAX): reduce-scatter
  // over the low lane bits, then (fewer than 64 logits) a butterfly sum over the remaining ones
  if constexpr (NV > 1) reduce_scatter_step<NV / 2, NV>(acc, lane);
#pragma unroll
  for (int off = NV; off < 64; off <<= 1) acc[0] += __shfl_xor(acc[0], off, kWave);
  lds.logit[wave][lane] = acc[0];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    amax[t] = wave_max(amax[t]);
    if (lane == 0) lds.amax[wave][t] = amax[t];
  }
  __syncthreads();
  if (wave == 0) {   // fixed summation order over the channel slices
    double l = lds.logit[0][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) l += lds.logit[w][lane];
    const int e = lane % EMAX;
    const int tok = t0 + (lane % NV) / EMAX;
    gate_topk<EMAX>(l, e, lane < NV && tok < T, tok, bias, E, k, topk_idx, topk_p, gate_p);
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    float m = lds.amax[0][t];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, lds.amax[w][t]);
    amax[t] = m;
  }

  if (q_x == nullptr) return;
  // Q_a(x): beta = max(absmax, 1e-5); s = 127 / beta (IEEE divide); q = clip(rne(x * s)).
  float scale[TPW];
  int rs[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    amax[t] = fmaxf(amax[t], kEps);
    scale[t] = 127.0f / amax[t];
    rs[t] = 0;
  }
  for (int ch = wave * kWave + lane; ch < n_chunks; ch += kThreads) {
    const int c0 = ch << 3;
    // all token rows are in registers before the first store: a wait for a load would otherwise
    // also wait for the stores issued before it (one counter for both)
    u4 px[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) px[t] = single_pass ? xkeep[t] : *reinterpret_cast<const u4*>(xrow[t] + c0);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const u4 p = px[t];
      const int q0 = quant_i8(bf16_lo(p.x), scale[t]), q1 = quant_i8(bf16_hi(p.x), scale[t]);
      const int q2 = quant_i8(bf16_lo(p.y), scale[t]), q3 = quant_i8(bf16_hi(p.y), scale[t]);
      const int q4 = quant_i8(bf16_lo(p.z), scale[t]), q5 = quant_i8(bf16_hi(p.z), scale[t]);
      const int q6 = quant_i8(bf16_lo(p.w), scale[t]), q7 = quant_i8(bf16_hi(p.w), scale[t]);
      rs[t] += q0 + q1 + q2 + q3 + q4 + q5 + q6 + q7;
      uint2 o;
      o.x = (q0 & 0xFF) | ((q1 & 0xFF) << 8) | ((q2 & 0xFF) << 16) | (static_cast<uint32_t>(q3 & 0xFF) << 24);
      o.y = (q4 & 0xFF) | ((q5 & 0xFF) << 8) | ((q6 & 0xFF) << 16) | (static_cast<uint32_t>(q7 & 0xFF) << 24);
      if (t0 + t < T) *reinterpret_cast<uint2*>(q_x + static_cast<int64_t>(t0 + t) * d + c0) = o;
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int part = wave_sum(rs[t]);
    if (lane == 0) lds.rsum[wave][t] = part;
  }
  __syncthreads();
  if (threadIdx.x < TPW && t0 + threadIdx.x < T) {
    int total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) total += lds.rsum[w][threadIdx.x];
    float m = lds.amax[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, lds.amax[w][threadIdx.x]);
    beta_x[t0 + threadIdx.x] = fmaxf(m, kEps);
    rowsum_x[t0 + threadIdx.x] = total;
  }
}

}  // namespace mote
