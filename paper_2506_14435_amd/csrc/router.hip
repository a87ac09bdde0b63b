// Router (gate softmax of Eq.3 + GShard-style top-k, Section 3.1) fused with the
// per-token absmax int8 quantiser Q_a(x) (Eq.8-10), and the dispatch plan that turns the
// top-k indices into an expert-major row permutation.
//
// router_quant_kernel (body in router_body.h): one workgroup owns TPW tokens, its four wavefronts split the channels.
// Each lane owns 8-channel chunks of the token rows (16-byte bf16 loads), multiplies them with the matching 8 rows of the
// bf16 router matrix and accumulates TPW x EMAX partial logits in fp64 (a bf16 x bf16
// product is exact, and fp64 accumulation makes the selected indices independent of the
// summation order).  A 6-step butterfly reduce-scatter leaves lane l with the finished
// logit (token l / EMAX, expert l % EMAX).  The token rows are then read a second time
// (L2 hits) to emit the int8 row, its absmax and its integer row sum.
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "router_body.h"

namespace mote {


template <int EMAX, int TPW, int NW>
__global__ __launch_bounds__(64 * NW) void router_quant_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w_router, const float* __restrict__ bias, int T,
    int d, int E, int k, int32_t* __restrict__ topk_idx, float* __restrict__ topk_p, int8_t* __restrict__ q_x,
    float* __restrict__ beta_x, int32_t* __restrict__ rowsum_x, float* __restrict__ gate_p) {
  // The grid is exact, ceil(T / TPW) workgroups: with a check in front the arguments are kept in spilled scalar registers
  // over the 64-expert body (d = 896, T = 64: 17.6 -> 19.0 us).
  __shared__ RouterScratch<TPW, NW> lds;
  router_quant_group<EMAX, TPW, NW, (EMAX > 16 ? 1 : 2)>(lds, blockIdx.x * TPW, x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x, beta_x,
                                                        rowsum_x, gate_p);
}

// ------------------------------------------------------------------------ many tokens, E <= 16
// The logits of 16 tokens x 16 experts are one accumulator tile of the fp64 matrix instruction
// (v_mfma_f64_16x16x4: the products of bf16 values are exact in fp64, the sums are fp64 as in the
// kernel above, one instruction where that kernel issues sixteen vector FMAs).  A workgroup of four
// wavefronts owns 16 tokens; wavefront w takes the channels 128 j + 32 w .. + 31 of every 128.  Lane
// (t = lane % 16, g = lane / 16) loads the 8 channels 128 j + 32 w + 8 g .. + 7 of token t (16 bytes) and
// keeps them in registers for the quantisation pass: element i of that chunk is this lane's A operand (row t,
// contraction slot g) of MFMA (j, i), whose B operand (slot g, expert lane % 16) is router row
// 128 j + 32 w + 8 g + i.  Every router row is used by one wavefront of the workgroup, so each wavefront
// turns its 32 rows of a step, converted to fp64, through LDS of its own ([i][lane], rows of 64 doubles padded by
// 16 bytes so that the writes of four rows at a time spread over the banks) and the steps need no barrier.  Tokens and
// rows are requested eight steps ahead in step order, the next step's rows are turned in front of a step's MFMAs.
// Bound by fp64 issue: an MFMA takes 29 - 33 ns per SIMD, a conversion to fp64 some 4 (T = 8192, d = 2048: 8.6 + 2 us
// of the 19.6 the kernel takes; 23.6 with the router in LDS blocks of the workgroup, two barriers each, behind all tokens'
// loads; with the counts, us, before -> after: T = 8192 at E = 16 31.0 -> 25.7, E = 12 33.5 -> 25.0, E = 6 32.0 -> 29.1,
// d = 3584 43.3 -> 34.6, T = 16384 79 -> 64).  Eight wavefronts per workgroup: d = 2048 -1 us, d = 3584 +2.5 (T = 8192).
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kRmTokens = 16;
// Above this many tokens, and for rows of up to 1024 channels above the batches of a workgroup per token.  us of the
// kernels above -> of this one: d = 2048, E = 16 T = 512 11.2 -> 11.4, T = 1024 11.7 -> 11.4, T = 2048 14.9 -> 11.6, T = 4000
// 23.7 -> 12.7; d = 896, E = 8 T = 512 9.1 -> 7.4, T = 2048 11.8 -> 7.8; d = 3584 T = 512 15.1 -> 17.1, T = 1024 15.8 -> 17.0,
// T = 1536 20.8 -> 17.0, T = 4000 37.9 -> 17.4.
constexpr int kRmMinTokens = 1024, kRmNarrow = 1024;
constexpr int kRmAhead = 8;   // steps of 128 channels on their way to each wavefront
constexpr int kRmRowBytes = 64 * 8 + 16;

// NGW: upper bound of the 128-channel steps (d / 128) the registers are sized for.  VEC: elements per load of a router row.
template <int NGW, int VEC>
__global__ __launch_bounds__(256) void router_mfma_kernel(
    const uint16_t* x, const uint16_t* w_router, const float* __restrict__ bias, int T,
    int d, int E, int k, int32_t* __restrict__ topk_idx, float* __restrict__ topk_p, int8_t* __restrict__ q_x,
    float* __restrict__ beta_x, int32_t* __restrict__ rowsum_x, float* __restrict__ gate_p) {
  __shared__ __attribute__((aligned(16))) unsigned char s_b[4][8 * kRmRowBytes];
  __shared__ double s_part[4][kRmTokens][16];
  __shared__ float s_amax[4][kRmTokens];
  __shared__ int s_rsum[4][kRmTokens];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = lane & 15, g = lane >> 4;
  const int t0 = blockIdx.x * kRmTokens;
  const int ngw = d >> 7;
  const uint16_t* const xrow = x + static_cast<int64_t>(min(t0 + t, T - 1)) * d + 32 * wave + 8 * g;
  // staging: this lane's router row of the 32 of a step, and its half of the experts (zero beyond E)
  const int sr = lane >> 1, se = 8 * (lane & 1);
  const uint16_t* const wrow = w_router + static_cast<int64_t>(32 * wave + sr) * E;
  const int64_t wstep = static_cast<int64_t>(128) * E;
  // eight elements as they come, addresses clamped to the row: what lies beyond E is zeroed when it is staged
  constexpr int kRaw = VEC == 1 ? 8 : 4;
  struct Raw { uint32_t v[kRaw]; };
  auto load_w = [&](int j) __attribute__((always_inline)) {
    Raw r;
    const uint16_t* const wr = wrow + j * wstep;
    if constexpr (VEC == 8) {
      const u4 p = *reinterpret_cast<const u4*>(wr + min(se, E - 8));
      r.v[0] = p.x; r.v[1] = p.y; r.v[2] = p.z; r.v[3] = p.w;
    } else if constexpr (VEC == 4) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint2 p = *reinterpret_cast<const uint2*>(wr + min(se + 4 * h, E - 4));
        r.v[2 * h] = p.x; r.v[2 * h + 1] = p.y;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) r.v[e] = wr[min(se + e, E - 1)];
    }
    return r;
  };
  auto weight = [&](const Raw& r, int e) __attribute__((always_inline)) {
    const uint32_t v = VEC == 1 ? r.v[e] << 16 : e & 1 ? r.v[e >> 1] & 0xFFFF0000u : r.v[e >> 1] << 16;
    return static_cast<double>(__uint_as_float(se + e < E ? v : 0u));
  };
  unsigned char* const s_dst = s_b[wave] + (sr & 7) * kRmRowBytes + (sr >> 3) * 128 + se * 8;
  const unsigned char* const s_src = s_b[wave] + lane * 8;

  u4 xk[NGW];
  Raw wk[kRmAhead];
#pragma unroll
  for (int j = 0; j < kRmAhead && j < NGW; ++j) {
    wk[j] = load_w(min(j, ngw - 1));
    xk[j] = *reinterpret_cast<const u4*>(xrow + 128 * min(j, ngw - 1));
    __builtin_amdgcn_sched_barrier(0);   // loads stay where they are issued: in step order, all in front of the work
  }
  // router rows of a step, as fp64, through this wavefront's own LDS (in order within a wavefront: no barrier)
  auto turn = [&](const Raw& wq, double (&b)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) *reinterpret_cast<double2*>(s_dst + e * 8) = make_double2(weight(wq, e), weight(wq, e + 1));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = *reinterpret_cast<const double*>(s_src + i * kRmRowBytes);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  v4d acc = {0.0, 0.0, 0.0, 0.0};
  float amax = 0.0f;
  double b[2][8];
  turn(wk[0], b[0]);
  // the steps nest (step j + 1 inside the condition of step j): each has one way in, so its wait counts the loads behind it
  auto step = [&](auto self, auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
    if (j >= ngw) return;
    if constexpr (j + kRmAhead < NGW) {   // the clamp keeps the loads of a step free of a branch of their own
      wk[j % kRmAhead] = load_w(min(j + kRmAhead, ngw - 1));
      xk[j + kRmAhead] = *reinterpret_cast<const u4*>(xrow + 128 * min(j + kRmAhead, ngw - 1));
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (j + 1 < NGW) turn(wk[(j + 1) % kRmAhead], b[(j + 1) & 1]);   // travels under the matrix instructions
    __builtin_amdgcn_sched_barrier(0);
    const u4 p = xk[j];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float xv = (i & 1) ? bf16_hi(p[i >> 1]) : bf16_lo(p[i >> 1]);
      amax = fmaxf(amax, fabsf(xv));
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(xv), b[j & 1][i], acc, 0, 0, 0);
    }
    if constexpr (j + 1 < NGW) self(self, std::integral_constant<int, j + 1>{});
  };
  step(step, std::integral_constant<int, 0>{});

  // accumulator element v of lane (t, g) is logit (token g + 4 v, expert t) over this wavefront's channels
#pragma unroll
  for (int v = 0; v < 4; ++v) s_part[wave][g + 4 * v][t] = acc[v];
  amax = fmaxf(amax, __shfl_xor(amax, 16, kWave));
  amax = fmaxf(amax, __shfl_xor(amax, 32, kWave));
  if (g == 0) s_amax[wave][t] = amax;
  __syncthreads();
  {   // wavefront w finishes tokens 4 w .. 4 w + 3: lane = 16 * (token % 4) + expert; fixed summation order
    const int tl = 4 * wave + (lane >> 4), e = lane & 15;
    const double l = ((s_part[0][tl][e] + s_part[1][tl][e]) + s_part[2][tl][e]) + s_part[3][tl][e];
    gate_topk<16>(l, e, t0 + tl < T, t0 + tl, bias, E, k, topk_idx, topk_p, gate_p);
  }
  if (q_x == nullptr) return;
  // Q_a(x): beta = max(absmax, 1e-5); s = 127 / beta (IEEE divide); q = clip(rne(x * s)).
  const float beta = fmaxf(fmaxf(fmaxf(s_amax[0][t], s_amax[1][t]), fmaxf(s_amax[2][t], s_amax[3][t])), kEps);
  const float scale = 127.0f / beta;
  int rs = 0;
  int8_t* const qrow = q_x + static_cast<int64_t>(t0 + t) * d + 32 * wave + 8 * g;
#pragma unroll
  for (int j = 0; j < NGW; ++j) {
    if (j < ngw) {
      const u4 p = xk[j];
      const int q0 = quant_i8(bf16_lo(p.x), scale), q1 = quant_i8(bf16_hi(p.x), scale);
      const int q2 = quant_i8(bf16_lo(p.y), scale), q3 = quant_i8(bf16_hi(p.y), scale);
      const int q4 = quant_i8(bf16_lo(p.z), scale), q5 = quant_i8(bf16_hi(p.z), scale);
      const int q6 = quant_i8(bf16_lo(p.w), scale), q7 = quant_i8(bf16_hi(p.w), scale);
      rs += q0 + q1 + q2 + q3 + q4 + q5 + q6 + q7;
      uint2 o;
      o.x = (q0 & 0xFF) | ((q1 & 0xFF) << 8) | ((q2 & 0xFF) << 16) | (static_cast<uint32_t>(q3 & 0xFF) << 24);
      o.y = (q4 & 0xFF) | ((q5 & 0xFF) << 8) | ((q6 & 0xFF) << 16) | (static_cast<uint32_t>(q7 & 0xFF) << 24);
      if (t0 + t < T) *reinterpret_cast<uint2*>(qrow + 128 * j) = o;
    }
  }
  rs += __shfl_xor(rs, 16, kWave);
  rs += __shfl_xor(rs, 32, kWave);
  if (g == 0) s_rsum[wave][t] = rs;
  __syncthreads();
  if (threadIdx.x < kRmTokens && t0 + threadIdx.x < T) {
    const int tt = threadIdx.x;
    beta_x[t0 + tt] = fmaxf(fmaxf(fmaxf(s_amax[0][tt], s_amax[1][tt]), fmaxf(s_amax[2][tt], s_amax[3][tt])), kEps);
    rowsum_x[t0 + tt] = s_rsum[0][tt] + s_rsum[1][tt] + s_rsum[2][tt] + s_rsum[3][tt];
  }
}

// Up to this many tokens every token gets a workgroup of its own.
static int router_token_blocks() { return knob(kKnobRouterTokenBlocks); }

hipError_t launch_router_quant(const uint16_t* x, const uint16_t* w_router, const float* bias, int T, int d,
                               int E, int k, int32_t* topk_idx, float* topk_p, int8_t* q_x, float* beta_x,
                               int32_t* rowsum_x, float* gate_p, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  // Few tokens: four wavefronts share a token group so that more of the chip takes part;
  // many tokens: one wavefront per group keeps the cross-lane reduction cost per token low.
  const bool coop = T <= 2048;
  if (E <= 16) {
    constexpr int kTpw = 4;
    const int blocks = (T + kTpw - 1) / kTpw;
    if (T <= router_token_blocks())   // a few tokens: one token per workgroup, a quarter of the arithmetic and of the reduction per lane
      router_quant_kernel<16, 1, 4><<<T, 256, 0, stream>>>(x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x, beta_x,
                                                           rowsum_x, gate_p);
    else if ((T > kRmMinTokens || d <= kRmNarrow) && d <= 4096) {   // 16 tokens per workgroup on the fp64 matrix instruction
      const int wgs = (T + kRmTokens - 1) / kRmTokens;
      const int vec = (E & 7) == 0 ? 8 : (E & 3) == 0 && (reinterpret_cast<uintptr_t>(w_router) & 7) == 0 ? 4 : 1;
#define MOTE_RM(NGW_, VEC_) router_mfma_kernel<NGW_, VEC_><<<wgs, 256, 0, stream>>>(x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x, beta_x, rowsum_x, gate_p)
#define MOTE_RM_VEC(NGW_) \
  if (vec == 8) MOTE_RM(NGW_, 8); else if (vec == 4) MOTE_RM(NGW_, 4); else MOTE_RM(NGW_, 1)
      if (d <= 1024) { MOTE_RM_VEC(8); }
      else if (d <= 2048) { MOTE_RM_VEC(16); }
      else { MOTE_RM_VEC(32); }
#undef MOTE_RM_VEC
#undef MOTE_RM
    }
    else if (coop)
      router_quant_kernel<16, kTpw, 4><<<blocks, 256, 0, stream>>>(x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x,
                                                                   beta_x, rowsum_x, gate_p);
    else
      router_quant_kernel<16, kTpw, 1><<<blocks, 64, 0, stream>>>(x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x,
                                                                   beta_x, rowsum_x, gate_p);
  } else {
    if (coop)
      router_quant_kernel<64, 1, 4><<<T, 256, 0, stream>>>(x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x, beta_x,
                                                           rowsum_x, gate_p);
    else
      router_quant_kernel<64, 1, 1><<<T, 64, 0, stream>>>(x, w_router, bias, T, d, E, k, topk_idx, topk_p, q_x, beta_x,
                                                           rowsum_x, gate_p);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------ dispatch plan
constexpr int kPlanThreads = 1024;

// One block per expert.  Every block histograms all R = T*k indices (so it knows every
// expert's count without a grid-wide dependency), then compacts the positions of its own
// expert in ascending flat order t*k + j: the dispatch order is deterministic and stable.
__global__ __launch_bounds__(kPlanThreads) void dispatch_plan_kernel(const int32_t* __restrict__ topk_idx, int R,
                                                                     int k, int E, int tile_m, DispatchPlan plan) {
  constexpr int kItems = 4;                       // indices per thread and pass: they stay in registers
  constexpr int kPass = kItems * kPlanThreads;
  constexpr int kPlanWaves = kPlanThreads / kWave;
  __shared__ int s_cnt[64];
  __shared__ int s_wave[kItems][kPlanWaves];
  __shared__ int s_off, s_tile_base;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e = blockIdx.x;
  if (tid < 64) s_cnt[tid] = 0;
  if (e == 0 && tid < 16 * kSchedStride) plan.sched[tid] = 0;
  __syncthreads();
  int first[kItems];                              // the first pass is kept for the compaction
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int i = j * kPlanThreads + tid;
    first[j] = i < R ? topk_idx[i] : -1;
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j)
    if (first[j] >= 0) atomicAdd(&s_cnt[first[j]], 1);
  for (int i = kPass + tid; i < R; i += kPlanThreads) atomicAdd(&s_cnt[topk_idx[i]], 1);
  __syncthreads();
  if (tid == 0) {
    int off = 0, tiles = 0;
    for (int j = 0; j < E; ++j) {
      if (j == e) { s_off = off; s_tile_base = tiles; }
      if (e == 0) { plan.counts[j] = s_cnt[j]; plan.offsets[j] = off; }
      off += s_cnt[j];
      tiles += (s_cnt[j] + tile_m - 1) / tile_m;
    }
    if (e == 0) { plan.offsets[E] = off; plan.n_tiles[0] = tiles; }
  }
  __syncthreads();
  const int my_off = s_off, my_cnt = s_cnt[e], tile_base = s_tile_base;
  for (int m = tid; m * tile_m < my_cnt; m += kPlanThreads) {
    plan.tile_expert[tile_base + m] = e;
    plan.tile_row0[tile_base + m] = my_off + m * tile_m;
    plan.tile_rows[tile_base + m] = min(tile_m, my_cnt - m * tile_m);
  }
  // Compaction, kItems * kPlanThreads indices per pass: index j * kPlanThreads + tid of the pass is
  // item j of this thread, so (item, wavefront, lane) order is ascending flat order.
  int running = 0;
  for (int base = 0; base < R; base += kPass) {
    bool flag[kItems];
    int prefix[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int i = base + j * kPlanThreads + tid;
      const int v = base == 0 ? first[j] : (i < R ? topk_idx[i] : -1);
      flag[j] = v == e;
      const uint64_t mask = __ballot(flag[j]);
      prefix[j] = __popcll(mask & ((1ull << lane) - 1ull));
      if (lane == 0) s_wave[j][wave] = __popcll(mask);
    }
    __syncthreads();
    int before[kItems], total = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      before[j] = total;
#pragma unroll
      for (int w = 0; w < kPlanWaves; ++w) {
        const int c = s_wave[j][w];
        if (w < wave) before[j] += c;
        total += c;
      }
    }
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (flag[j]) {
        const int i = base + j * kPlanThreads + tid;
        const int slot = my_off + running + before[j] + prefix[j];
        plan.row_of[i] = slot;
        plan.tok_of[slot] = i / k;
        plan.row_planes[slot] = 0;
      }
    }
    running += total;
    __syncthreads();
  }
}

// Histogram of the selected experts (mote_router_topk's optional output).
__global__ __launch_bounds__(kPlanThreads) void expert_counts_kernel(const int32_t* __restrict__ topk_idx, int R, int E,
                                                                     int32_t* __restrict__ counts) {
  __shared__ int s_cnt[64];
  if (threadIdx.x < 64) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < R; i += kPlanThreads) atomicAdd(&s_cnt[topk_idx[i]], 1);
  __syncthreads();
  if (threadIdx.x < E) counts[threadIdx.x] = s_cnt[threadIdx.x];
}

hipError_t launch_expert_counts(const int32_t* topk_idx, int R, int E, int32_t* counts, hipStream_t stream) {
  expert_counts_kernel<<<1, kPlanThreads, 0, stream>>>(topk_idx, R, E, counts);
  return hipGetLastError();
}

hipError_t launch_dispatch_plan(const int32_t* topk_idx, int T, int k, int E, int tile_m, const DispatchPlan& plan,
                                hipStream_t stream) {
  dispatch_plan_kernel<<<E, kPlanThreads, 0, stream>>>(topk_idx, T * k, k, E, tile_m, plan);
  return hipGetLastError();
}

}  // namespace mote
