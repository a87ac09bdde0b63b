// Shared expert FFN(x) of Eq.2: the dense checkpoint's full-precision SwiGLU FFN, active
// for every token.  bf16 operands on v_mfma_f32_16x16x32_bf16, fp32 accumulation.
//
//   gate-up mode : g = x W_gate^T, u = x W_up^T, h_s = bf16(u * SiLU(g))     [T, F]
//   down mode    : y_s = h_s W_down^T (fp32)                                 [T, d]
//
// Both operands are K-contiguous ([rows, K] row-major) and are loaded straight into LDS
// (buffer_load ... lds, 16 bytes per lane) in K chunks of 64 elements: a tile row is 128
// bytes = eight 16-byte chunks, chunk index XOR-swizzled with bits 1..3 of the row so that a
// ds_read_b128 of 16 consecutive rows touches every LDS bank once.  Two kernels: big_gemm (256 x 256
// tiles, bound by the matrix pipe and power) and mid_gemm (128-row tiles, bound by latency); gemm_choice
// says which takes a problem.
//
// MFMA operand mapping (16x16x32 bf16): first operand = weights (lane l: output channel
// l%16, 8 consecutive K elements of quarter l/16), second = activations (lane l: token row
// l%16); result register v of lane l is output channel 4*(l/16) + v of token row l%16.
//
// Why 16x16 and not 32x32 tiles: the chip is power-limited inside these GEMMs.  Register-only loops over random
// operands on all CUs sustain 2.00 PFLOP/s with v_mfma_f32_16x16x32_bf16 and 1.74 with v_mfma_f32_32x32x16_bf16
// (half as many accumulator registers read and written per flop), fed from LDS as here 1.75 and 1.55.
#include <stdlib.h>

#include <algorithm>

#include "common.h"
#include "launch.h"

namespace mote {

// Weights as 2-bit ternary codes (grouped GEMM of the straight-through gradients): blocks of 32 channels x 32
// K elements = 256 bytes, block (channel block, 32 K elements) row-major; in a block word 16Q + c holds the K elements
// 8Q .. 8Q+7 of channel c (pairs J = 0..3) and of channel 16 + c (J = 4..7), the operands of one lane for two
// fragments: pair J has its even element's "non-zero" at bit J and sign at bit 8+J, its odd element's at bits 16+J and 24+J.
// In each 16-bit half of
// word & (0x01010101 << J), multiplied by 127 << (7 - J), "non-zero" becomes 0x3F80 and the sign 0x8000 (modulo 2^16;
// 127 is odd): the pair as bf16 values 0, 1, -1 after one and and one packed 16-bit multiplication (a shift and an
// and give 0, 2, -2 instead, whose sums overflow from 2^127 on).  The codes are an eighth of the bytes of bf16 weights
// through L2 and LDS.
//
// Half h of the ternary word of a lane: eight K elements of fragment h as bf16 values 0, 1, -1.
__device__ __forceinline__ bf16x8 ternary_operand(uint32_t w, int h) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  uint32_t r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = 4 * h + i;
    const uint16_t c = static_cast<uint16_t>(127u << (7 - j));
    r[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, w & (0x01010101u << j)) * u16x2{c, c});
  }
  return __builtin_bit_cast(bf16x8, u4{r[0], r[1], r[2], r[3]});
}

struct SharedGemmArgs {
  const uint16_t* act;   // [M, K] bf16
  const uint16_t* w0;    // [N, K] bf16 (gate / down), or ternary blocks (Cfg::TERN)
  const uint16_t* w1;    // [N, K] bf16 (up)
  int M, N, K;
  uint16_t* h_out;       // gate-up: bf16 [M, N]
  float* y_out;          // down: fp32 [planes][M, N]
  int64_t plane_stride;  // elements between partial planes
  const float* scale0;   // optional fp32 [N]: the sums of w0 (w1) are multiplied by scale0 (scale1)
  const float* scale1;   // per output channel (RTN-quantised weights held as integer-valued bf16)
  float* y_split;        // row groups: where the planes of the row tiles from RowGroups::split_mt on go, counted like y_out
};

// Grouped rows: group e owns the rows row0[e] .. row0[e+1]-1 of act / the output and the row tiles
// tile0[e] .. tile0[e+1]-1 (ceil(rows / BM) of them, none for an empty group); its weights are matrix e
// of w0 ([n][N, K]) and its channel scales row e of scale0 ([n][N]).  A row tile that reaches beyond its
// group's last row loads the rows that follow (clamped to the last row of act) and stores only its own.
constexpr int kMaxRowGroups = 64;
struct RowGroups {
  int n;
  int split_mt;   // 256-row tiles: the row tiles below contract all of K in one plane

  int row0[kMaxRowGroups + 1];
  int tile0[kMaxRowGroups + 1];
};

// K ranges: plane p of the kplanes = rg->n planes contracts the K range row0[p] .. row0[p+1]-1 (multiples of 64
// elements; an empty range gives a plane of zeros).
//
// Tile order of all kernels here.  Persistent workgroups, dealt to the 8 XCDs round-robin by linear id: XCD x owns the
// (channel tile, K plane) pairs x, x+8, ... (the row tiles x, x+8, ... when there are fewer than 16 pairs); inside an XCD
// the tiles are ordered in bands of group_m row tiles, row tile fastest, so the resident workgroups share both
// activation tiles and weight slices in L2.  With kplanes > 1 the contraction is cut into planes of ktp K chunks; each
// plane writes its own partial output, added later in plane order.
//
// Loads: raw buffer loads written in assembly (the compiler has no exact model of outstanding direct-to-LDS loads across
// these loops).  Vector-memory operations complete in issue order, so waiting for "all but the N youngest" retires the
// chunk that is about to be contracted while later ones stay in flight; anything else issued since (stores of the
// previous epilogue) only makes that wait stricter.

// Large problems: 256 x 256 tiles (256 x (128+128) in gate-up mode), one workgroup of eight wavefronts per CU, each
// 64 rows x 128 channels.  K goes in chunks of 64 elements, so that a tile row in LDS is 128 bytes and a direct load
// brings eight rows x one whole cache line: on 64-byte rows a load needs twice the requests, and
// loads alone, without any MFMA, peak at 14 TB/s over the chip where 128-byte rows reach 25 - this kernel asks for 10
// to 13.
//
// LDS is a ring of five 32-KiB slots that take the operands in turn, A0 B0 A1 B1 A2 ...; chunk c is contracted out
// of two of them while the other three hold or receive A and B of chunk c+1 and A of chunk c+2.  A chunk is four
// quarters of 16 MFMAs per wavefront (half of the chunk's K x half of the weight fragments); every quarter reads the fragments of
// the next one between its MFMAs (an activation fragment as soon as its last MFMA has been issued), so the last
// quarter reads nothing of chunk c any more: in front of it stands the one barrier of the chunk, which publishes
// chunk c+1 and frees the two slots for B of chunk c+2 and A of chunk c+3 (requested in the last quarter and in the
// first one of chunk c+1: one and two chunks ahead of their use; spread evenly over all quarters, or all in the last one, the
// kernel is 2-3 % slower).  The wavefronts of the single workgroup of a CU are
// in step, so reads and loads in a block of their own would leave the matrix pipe idle on every SIMD at once: they
// go one by one between the MFMAs.
//
// Measured (random operands, start: the ring of four 32-element steps on 32x32x16 MFMAs): gate-up 8192 x 2048 x 11008
// 591 -> 511 us (1.44 PFLOP/s), down 314 -> 250 (1.48); 16384 x 3584 x 18944 3861 -> 3145, 1995 -> 1612.  What bounds it is
// power: with operands of zeros the first takes 374 us at 2.4 GHz, with random ones the chip clocks at 1.75 GHz.
//
// GROUPED: 0 plain, 1 row groups, 2 K ranges.
// TERN: weights as 2-bit codes in the blocks described above, unpacked in registers (eight vector instructions per
// four MFMAs).  The weights of a chunk are 4 KiB, so the ring is four whole stages (A, then weights) and the loads run
// three chunks ahead; the fragments of a half chunk are read during the half before it, into the other one of two
// register sets, and the barrier stands in the middle of the second half.
template <int MODE_, bool TERN_ = false>
struct BigCfg {
  static constexpr bool TERN = TERN_;
  static constexpr int MODE = MODE_;   // 0 gate-up, 1 down
  static constexpr int NMAT = MODE_ == 0 ? 2 : 1;
  static constexpr int BM = 256, BN = 256 / NMAT, WAVES = 8, THREADS = 512;
  static constexpr int A16 = 4, NB = 8, B16 = NB / NMAT, HB = NB / 2;   // 16-row and 16-channel fragments of a wavefront
  static constexpr int SLOT = 32768, STAGE = SLOT + 4096;   // STAGE: ternary weights
  static constexpr int LDS_BYTES = TERN_ ? 4 * STAGE : 5 * SLOT;
  static constexpr int OUT_BYTES = MODE_ == 0 ? 2 : 4;
  static constexpr int PATCH_ROW = 128 + 16, PATCH_BYTES = 32 * PATCH_ROW;   // epilogue: 32 rows of 128 bytes per wavefront
  static_assert(4 * PATCH_BYTES <= SLOT && 8 * PATCH_BYTES <= STAGE, "the patches fit two free slots / one free stage");
  static_assert(!TERN_ || MODE_ == 1, "ternary weights: one matrix");
};

template <typename Cfg, int GROUPED>
__device__ __forceinline__ void big_gemm_body(const SharedGemmArgs& a, const RowGroups* rg, int n_ntiles, int kplanes, int ktp, int group_m) {
  constexpr int NMAT = Cfg::NMAT, BM = Cfg::BM, BN = Cfg::BN, SLOT = Cfg::SLOT;
  constexpr int A16 = Cfg::A16, NB = Cfg::NB, B16 = Cfg::B16, HB = Cfg::HB;
  extern __shared__ __attribute__((aligned(16))) unsigned char s_lds[];
  const int M = a.M, N = a.N, K = a.K;
  const int KT = K >> 6;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave & 3, wn = wave >> 2;
  const int r16 = lane & 15, quart = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) unsigned char*)s_lds);
  // 128-byte rows of eight 16-byte chunks, chunk XOR-swizzled with row bits 1..3 (two rows span the banks once).  This
  // lane's 16 bytes of the wavefront's first fragment, K half 0; half 1 is at ^ 64
  const int frag = r16 * 128 + ((quart ^ (r16 >> 1)) << 4);
  const int a_lds = wm * 64 * 128 + frag, b_lds = wn * (BN / 2) * 128 + frag;

  // Tile order: as above; with row groups two such lists one after the other, the row tiles below
  // rg->split_mt with one plane and the others with kplanes.
  int n_mtiles = (M + BM - 1) / BM;
  if constexpr (GROUPED == 1) n_mtiles = rg->tile0[rg->n];
  const int mt1 = GROUPED == 1 ? rg->split_mt : 0;   // row tiles of the first list
  const int nk1 = n_ntiles, nk2 = n_ntiles * kplanes, mt2n = n_mtiles - mt1;
  const int xcd = blockIdx.x & 7;
  auto list_nt = [&](int nk) { return nk >= 16 ? (nk - xcd + 7) >> 3 : nk; };
  auto list_mt = [&](int nk, int mts) { return nk >= 16 ? mts : (mts - xcd + 7) >> 3; };
  const int work1 = GROUPED == 1 ? list_nt(nk1) * list_mt(nk1, mt1) : 0;
  const int xcd_work = work1 + list_nt(nk2) * list_mt(nk2, mt2n);
  const int stride = gridDim.x >> 3;
  int slot = blockIdx.x >> 3;
  if (slot >= xcd_work) return;

  constexpr int kBufferFlags = 0x00020000;   // raw buffer, 32-bit data format
  auto make_rsrc = [&](const void* base, int64_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    v4i r;
    r.x = static_cast<int>(static_cast<uint32_t>(p));
    r.y = static_cast<int>(static_cast<uint32_t>(p >> 32) & 0xFFFFu);
    r.z = static_cast<int>(bytes);
    r.w = kBufferFlags;
    return r;
  };
  const v4i rsrc_a = make_rsrc(a.act, static_cast<int64_t>(M) * K * 2);
  const v4i rsrc_b0 = make_rsrc(a.w0, Cfg::TERN ? static_cast<int64_t>(GROUPED == 1 ? rg->n : 1) * N * K / 4 : static_cast<int64_t>(N) * K * 2);
  const v4i rsrc_b1 = make_rsrc(NMAT == 2 ? a.w1 : a.w0, static_cast<int64_t>(N) * K * 2);
  // lane l of a load lands at byte 16*l of a 1-KiB block = tile row l/8, physical chunk l%8; pass p covers the tile
  // rows 64p + 8 * wavefront ..
  const int ld_row = wave_u * 8 + (lane >> 3);
  const uint32_t ld_chunk = static_cast<uint32_t>(((lane & 7) ^ ((ld_row >> 1) & 7)) << 4);
  uint32_t a_off[4], b_off[4];   // byte offsets of this lane's 16 bytes, chunk 0 of the plane
  int mt, nt, kc, ktl;
  int mrow, mend = M, grp = 0;   // first row of the tile, one past the last row it may store, its group (0 without groups)
  // slots of A, B of chunk c, A, B of chunk c+1, A of chunk c+2; ternary weights: stages of the chunks c .. c+3
  constexpr int PITCH = Cfg::TERN ? Cfg::STAGE : SLOT;
  int s0 = 0, s1 = PITCH, s2 = 2 * PITCH, s3 = 3 * PITCH, s4 = 4 * PITCH;

#define MOTE_DECODE(slot_, mt_, nt_, kc_, kl_)                                  \
  {                                                                             \
    const bool second_ = GROUPED != 1 || (slot_) >= work1;                      \
    const int nk_ = second_ ? nk2 : nk1, mts_ = second_ ? mt2n : mt1;           \
    const int kp_ = second_ ? kplanes : 1, s_ = second_ ? (slot_) - work1 : (slot_); \
    const bool split_n_ = nk_ >= 16;                                            \
    const int per_group_ = group_m * list_nt(nk_);                              \
    const int grp_ = s_ / per_group_;                                           \
    const int in_ = s_ - grp_ * per_group_;                                     \
    const int gsz_ = min(list_mt(nk_, mts_) - grp_ * group_m, group_m);         \
    const int ni_ = in_ / gsz_, mi_ = grp_ * group_m + (in_ - ni_ * gsz_);      \
    mt_ = (second_ ? mt1 : 0) + (split_n_ ? mi_ : xcd + 8 * mi_);               \
    const int ntk_ = split_n_ ? xcd + 8 * ni_ : ni_;                            \
    nt_ = ntk_ / kp_;                                                           \
    kc_ = ntk_ - nt_ * kp_;                                                     \
    kl_ = second_ ? ktp : KT;                                                   \
  }
  // byte offset of plane kc_ in an operand row and its chunks
#define MOTE_KRANGE(kc_, kl_, kb_, ktl_)                                        \
  {                                                                             \
    if constexpr (GROUPED == 2) {                                               \
      kb_ = static_cast<uint32_t>(rg->row0[kc_]) * 2u;                          \
      ktl_ = (rg->row0[(kc_) + 1] - rg->row0[kc_]) >> 6;                        \
    } else {                                                                    \
      kb_ = static_cast<uint32_t>((kc_) * (kl_)) * 128u;                        \
      ktl_ = min((kl_), KT - (kc_) * (kl_));                                    \
    }                                                                           \
  }
  // where row tile mt_ starts and ends (uniform; the group is found by walking the table)
#define MOTE_ROWS(mt_, mrow_, mend_, grp_)                                      \
  {                                                                             \
    if constexpr (GROUPED == 1) {                                               \
      int e_ = 0;                                                               \
      while (e_ + 1 < rg->n && rg->tile0[e_ + 1] <= (mt_)) ++e_;                \
      grp_ = e_;                                                                \
      mrow_ = rg->row0[e_] + ((mt_) - rg->tile0[e_]) * BM;                      \
      mend_ = rg->row0[e_ + 1];                                                 \
    } else {                                                                    \
      mrow_ = (mt_) * BM;                                                       \
    }                                                                           \
  }
#define MOTE_POINTERS(mrow_, grp_, nt_, kb_)                                                       \
  {                                                                                                \
    const uint32_t k0_ = (kb_) + ld_chunk;                                                         \
    _Pragma("unroll") for (int p = 0; p < 4; ++p) {                                                \
      a_off[p] = static_cast<uint32_t>(min((mrow_) + p * 64 + ld_row, M - 1)) * static_cast<uint32_t>(K) * 2u + k0_; \
      if constexpr (!Cfg::TERN)                                                                    \
        b_off[p] = static_cast<uint32_t>(min((nt_) * BN + (p * 64) % BN + ld_row, N - 1)) * static_cast<uint32_t>(K) * 2u + k0_; \
    }                                                                                              \
    if constexpr (Cfg::TERN) {                                                                     \
      const int blk_ = min((nt_) * (BN / 32) + wave_u, (N >> 5) - 1) + (grp_) * (N >> 5);          \
      b_off[0] = static_cast<uint32_t>(blk_) * static_cast<uint32_t>(K) * 8u + (kb_) * 4u + lane * 4u; \
    }                                                                                              \
  }
  // one 16-byte-per-lane direct load of pass p_ of chunk ks_ (M0: see ternary_gemm.hip)
#define MOTE_DMA(lds_, voff_, rsrc_, soff_)                                                        \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"           \
               :: "s"(lds_), "v"(voff_), "s"(rsrc_), "s"(soff_) : "memory")
#define MOTE_DMA_A(slot_, ks_, p_) MOTE_DMA(lds0 + (slot_) + ((p_) * 64 + wave_u * 8) * 128, a_off[p_], rsrc_a, (ks_) * 128)
#define MOTE_DMA_B(slot_, ks_, p_) \
  MOTE_DMA(lds0 + (slot_) + ((p_) * 64 + wave_u * 8) * 128, b_off[p_], (((p_) * 64) / BN == 0 ? rsrc_b0 : rsrc_b1), (ks_) * 128)
  // ternary: half h_ of the chunk of this wavefront's block of 32 channels
#define MOTE_DMA_W(stage_, ks_, h_)                                                                \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"             \
               :: "s"(lds0 + (stage_) + SLOT + (h_) * 2048 + wave_u * 256), "v"(b_off[0]), "s"(rsrc_b0), "s"((ks_) * 512 + (h_) * 256) : "memory")
#define MOTE_ISSUE_STAGE(stage_, ks_) { MOTE_ISSUE_A(stage_, ks_) MOTE_DMA_W(stage_, ks_, 0); MOTE_DMA_W(stage_, ks_, 1); }
  // the first loads of a tile of ktl_ chunks
#define MOTE_START(ktl_)                                                                           \
  if constexpr (Cfg::TERN) {                                                                       \
    if ((ktl_) > 0) MOTE_ISSUE_STAGE(s0, 0)                                                        \
    if ((ktl_) > 1) MOTE_ISSUE_STAGE(s1, 1)                                                        \
    if ((ktl_) > 2) MOTE_ISSUE_STAGE(s2, 2)                                                        \
  } else if ((ktl_) > 0) {                                                                         \
    MOTE_ISSUE_A(s0, 0);                                                                           \
    MOTE_ISSUE_B(s1, 0);                                                                           \
    if ((ktl_) > 1) MOTE_ISSUE_A(s2, 1);                                                           \
  }
#define MOTE_ISSUE_A(slot_, ks_) { _Pragma("unroll") for (int p = 0; p < 4; ++p) MOTE_DMA_A(slot_, ks_, p); }
#define MOTE_ISSUE_B(slot_, ks_) { _Pragma("unroll") for (int p = 0; p < 4; ++p) MOTE_DMA_B(slot_, ks_, p); }
#define MOTE_A_FRAG(slot_, h_, i_) *reinterpret_cast<const bf16x8*>(s_lds + (slot_) + (a_lds ^ ((h_) * 64)) + (i_) * 2048)
#define MOTE_B_FRAG(slot_, h_, b_) \
  *reinterpret_cast<const bf16x8*>(s_lds + (slot_) + (b_lds ^ ((h_) * 64)) + ((b_) / B16) * (BN * 128) + ((b_) % B16) * 2048)

  // ---- first tile ----
  int kl;
  MOTE_DECODE(slot, mt, nt, kc, kl);
  uint32_t kb;
  MOTE_KRANGE(kc, kl, kb, ktl);
  MOTE_ROWS(mt, mrow, mend, grp);
  MOTE_POINTERS(mrow, grp, nt, kb);
  MOTE_START(ktl)

  for (;;) {
    const int nslot = slot + stride;
    const bool has_next = nslot < xcd_work;
    int mt2 = mt, nt2 = nt, kc2 = kc, ktl2 = ktl, mrow2 = mrow, mend2 = mend, grp2 = grp;
    uint32_t kb2 = kb;
    if (has_next) {
      int kl2;
      MOTE_DECODE(nslot, mt2, nt2, kc2, kl2);
      MOTE_ROWS(mt2, mrow2, mend2, grp2);
      MOTE_KRANGE(kc2, kl2, kb2, ktl2);
    }
    // chunk 0 visible to every wavefront, the patches of the previous tile done
    if (Cfg::TERN && ktl > 2) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    else if (!Cfg::TERN && ktl > 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
    if (!Cfg::TERN && ktl > 1) MOTE_ISSUE_B(s3, 1);   // this slot held patches

    v4f acc[A16][NB];   // token rows 16i .., channels 16b .. of the wavefront's block (gate first, then up)
#pragma unroll
    for (int i = 0; i < A16; ++i)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[i][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (Cfg::TERN) {
      bf16x8 afx[A16], afy[A16];
      uint32_t wx[4], wy[4];
#define MOTE_TERN_READ(af_, w_, stage_, h_)                                                        \
      {                                                                                            \
        _Pragma("unroll") for (int i = 0; i < A16; ++i) af_[i] = MOTE_A_FRAG(stage_, h_, i);       \
        _Pragma("unroll") for (int f = 0; f < 4; ++f)                                              \
          w_[f] = *reinterpret_cast<const uint32_t*>(s_lds + (stage_) + SLOT + (h_) * 2048 + (wn * 4 + f) * 256 + lane * 4); \
      }
      // weight fragments b0_ .. of a half chunk with (af_, w_); the fragment behind the last one of w_ is the first of wn_;
      // behind the MFMAs of fragment b the statement side_(b)
#define MOTE_TERN_PART(b0_, b1_, af_, w_, wn_, side_)                                              \
      _Pragma("unroll") for (int b = b0_; b < b1_; ++b) {                                          \
        acc[0][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, af_[0], acc[0][b], 0, 0, 0);       \
        const bf16x8 wnext_ = b + 1 < NB ? ternary_operand(w_[((b + 1) % NB) / 2], (b + 1) & 1) : ternary_operand(wn_[0], 0); \
        _Pragma("unroll") for (int i = 1; i < A16; ++i)                                            \
          acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, af_[i], acc[i][b], 0, 0, 0);     \
        wf = wnext_;                                                                               \
        side_                                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                         \
      }
      // chunk c; PF_: with the requests of chunk c+3.  At the barrier chunk c+1 has landed (wait_), chunk c has been read
#define MOTE_TERN_CHUNK(PF_, wait_)                                                                \
      {                                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                                         \
        MOTE_TERN_PART(0, NB, afx, wx, wy, {                                                       \
          if (b == 0) MOTE_TERN_READ(afy, wy, s0, 1)                                               \
          if (PF_ && (b & 1) == 1) MOTE_DMA_A(s3, c + 3, b / 2);                                   \
        })                                                                                         \
        MOTE_TERN_PART(0, NB / 2, afy, wy, wx, {                                                   \
          if (PF_ && (b & 1) == 0) MOTE_DMA_W(s3, c + 3, b / 2);                                   \
        })                                                                                         \
        wait_                                                                                      \
        asm volatile("s_barrier" ::: "memory");                                                    \
        MOTE_TERN_PART(NB / 2, NB, afy, wy, wx, {                                                  \
          if (b == NB / 2) MOTE_TERN_READ(afx, wx, s1, 0)                                          \
        })                                                                                         \
        const int t0 = s0;                                                                         \
        s0 = s1; s1 = s2; s2 = s3; s3 = t0;                                                        \
      }
      MOTE_TERN_READ(afx, wx, s0, 0)
      bf16x8 wf = ternary_operand(wx[0], 0);
      int c = 0;
      for (; c + 3 < ktl; ++c) MOTE_TERN_CHUNK(true, asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");)
      for (; c < ktl; ++c) MOTE_TERN_CHUNK(false, {
        if (c + 2 < ktl) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      })
#undef MOTE_TERN_CHUNK
#undef MOTE_TERN_PART
#undef MOTE_TERN_READ
    } else {
    bf16x8 af[A16], bl[HB], bh[HB];
#pragma unroll
    for (int b = 0; b < HB; ++b) bl[b] = MOTE_B_FRAG(s1, 0, b);
#pragma unroll
    for (int i = 0; i < A16; ++i) af[i] = MOTE_A_FRAG(s0, 0, i);
    // a quarter: MFMAs of (af, b_) into the weight half o_; behind MFMA j the statement side_(i, b, j)
#define MOTE_QUARTER(b_, o_, side_)                                                                \
    _Pragma("unroll") for (int i = 0; i < A16; ++i)                                                \
      _Pragma("unroll") for (int b = 0; b < HB; ++b) {                                             \
        const int j = i * HB + b;                                                                  \
        acc[i][(o_) + b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b_[b], af[i], acc[i][(o_) + b], 0, 0, 0); \
        side_                                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                         \
      }
    // chunk c; PF_: with the requests of A and B of chunk c+2.  In front of the barrier chunk c+1 has landed (A of chunk
    // c+2 stays in flight) and this wavefront has read all of chunk c.  After the last chunk the last quarter's
    // reads are of slots nobody uses, and dropped.
#define MOTE_CHUNK(PF_)                                                                            \
    {                                                                                              \
      __builtin_amdgcn_sched_barrier(0);                                                           \
      MOTE_QUARTER(bl, 0, {                                                                        \
        if (j < HB) bh[j] = MOTE_B_FRAG(s1, 0, HB + j);                                            \
        if (PF_ && (j & 3) == 2) MOTE_DMA_A(s4, c + 2, j / 4);                                     \
      })                                                                                           \
      MOTE_QUARTER(bh, HB, {                                                                       \
        if (j < HB) bl[j] = MOTE_B_FRAG(s1, 1, j);                                                 \
        if (b == HB - 1) af[i] = MOTE_A_FRAG(s0, 1, i);                                            \
      })                                                                                           \
      MOTE_QUARTER(bl, 0, {                                                                        \
        if (j < HB) bh[j] = MOTE_B_FRAG(s1, 1, HB + j);                                            \
      })                                                                                           \
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(PF_ ? 4 : 0) : "memory");               \
      asm volatile("s_barrier" ::: "memory");                                                      \
      MOTE_QUARTER(bh, HB, {                                                                       \
        if (j < HB) bl[j] = MOTE_B_FRAG(s3, 0, j);                                                 \
        if (b == HB - 1) af[i] = MOTE_A_FRAG(s2, 0, i);                                            \
        if (PF_ && (j & 3) == 2) MOTE_DMA_B(s0, c + 2, j / 4);                                     \
      })                                                                                           \
      const int t0 = s0, t1 = s1;                                                                  \
      s0 = s2; s1 = s3; s2 = s4; s3 = t0; s4 = t1;                                                 \
    }
    // two loops rather than a test at every request: the branches between the MFMAs cost 4 %
    int c = 0;
    for (; c + 2 < ktl; ++c) MOTE_CHUNK(true)
    for (; c < ktl; ++c) MOTE_CHUNK(false)
#undef MOTE_CHUNK
#undef MOTE_QUARTER
    }

    // Start the next tile now: its first loads travel while this tile runs its epilogue in the two slots of the
    // last chunk.
    if (has_next) {
      MOTE_POINTERS(mrow2, grp2, nt2, kb2);
      MOTE_START(ktl2)
    }

    // ---- epilogue ----
    // In registers lane l owns token row r16 and four consecutive output channels of every fragment (4 * quart .. +3).
    // Each wavefront writes one 32-row block of 128 bytes per row into its private LDS patch and reads it back row-major,
    // 16 bytes per lane, so that a global store instruction covers whole 128-byte rows of the block.
    unsigned char* const patch = Cfg::TERN ? s_lds + s3 + wave * Cfg::PATCH_BYTES : s_lds + (wave < 4 ? s3 : s4) + (wave & 3) * Cfg::PATCH_BYTES;
    const int n_wave0 = nt * BN + wn * (BN / 2);
    const int rd_row = lane >> 3, rd_chunk = lane & 7;
    if (a.scale0 != nullptr) {   // row scales of quantised weights (uniform branch, not taken by the bf16 expert)
#pragma unroll
      for (int b = 0; b < B16; ++b) {
        const int ch = min(n_wave0 + b * 16 + 4 * quart, N - 4);
        const float4 s0_ = *reinterpret_cast<const float4*>(a.scale0 + static_cast<int64_t>(grp) * N + ch);
        float4 s1_ = s0_;
        if constexpr (NMAT == 2) s1_ = *reinterpret_cast<const float4*>(a.scale1 + ch);
#pragma unroll
        for (int i = 0; i < A16; ++i) {
          acc[i][b].x *= s0_.x; acc[i][b].y *= s0_.y; acc[i][b].z *= s0_.z; acc[i][b].w *= s0_.w;
          if constexpr (NMAT == 2) {
            v4f& au = acc[i][(NMAT - 1) * B16 + b];
            au.x *= s1_.x; au.y *= s1_.y; au.z *= s1_.z; au.w *= s1_.w;
          }
        }
      }
    }
    constexpr int PF = Cfg::MODE == 0 ? 4 : 2;   // fragments of a patch (128 bytes per row)
#pragma unroll
    for (int i = 0; i < A16; i += 2) {
#pragma unroll
      for (int f0 = 0; f0 < B16; f0 += PF) {
#pragma unroll
        for (int bb = 0; bb < PF; ++bb) {
          const int b = f0 + bb;
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const v4f v = acc[i + r][b];
            unsigned char* const dst = patch + (r * 16 + r16) * Cfg::PATCH_ROW + (bb * 16 + 4 * quart) * Cfg::OUT_BYTES;
            if constexpr (Cfg::MODE == 0) {
              const v4f u = acc[i + r][(NMAT - 1) * B16 + b];
              uint2 packed;
              packed.x = cvt_pk_bf16(u.x * silu_fast(v.x), u.y * silu_fast(v.y));
              packed.y = cvt_pk_bf16(u.z * silu_fast(v.z), u.w * silu_fast(v.w));
              *reinterpret_cast<uint2*>(dst) = packed;
            } else {
              *reinterpret_cast<float4*>(dst) = make_float4(v.x, v.y, v.z, v.w);
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int rd_n = n_wave0 + f0 * 16 + rd_chunk * (16 / Cfg::OUT_BYTES);   // first output channel of this lane's 16 bytes
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int pr = p * 8 + rd_row;
          const u4 v = *reinterpret_cast<const u4*>(patch + pr * Cfg::PATCH_ROW + rd_chunk * 16);
          const int orow = mrow + wm * 64 + i * 16 + pr;
          if (orow < mend && rd_n < N) {
            const int64_t o = static_cast<int64_t>(orow) * N + rd_n;
            if constexpr (Cfg::MODE == 0) *reinterpret_cast<u4*>(a.h_out + o) = v;
            else if (GROUPED == 1 && mt >= mt1) *reinterpret_cast<u4*>(a.y_split + static_cast<int64_t>(kc) * a.plane_stride + o) = v;
            else *reinterpret_cast<u4*>(a.y_out + static_cast<int64_t>(kc) * a.plane_stride + o) = v;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    if (!has_next) break;
    // No barrier here: the patches are private and their slots are not refilled before the next
    // tile's first barrier.
    slot = nslot; mt = mt2; nt = nt2; kc = kc2; ktl = ktl2; kb = kb2; mrow = mrow2; mend = mend2; grp = grp2;
  }
#undef MOTE_DECODE
#undef MOTE_KRANGE
#undef MOTE_POINTERS
#undef MOTE_DMA
#undef MOTE_DMA_A
#undef MOTE_DMA_B
#undef MOTE_ISSUE_A
#undef MOTE_ISSUE_B
#undef MOTE_ROWS
#undef MOTE_DMA_W
#undef MOTE_ISSUE_STAGE
#undef MOTE_START
#undef MOTE_A_FRAG
#undef MOTE_B_FRAG
}

template <typename Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 2) void big_gemm_kernel(SharedGemmArgs a, int n_ntiles, int kplanes, int ktp, int group_m) {
  big_gemm_body<Cfg, 0>(a, nullptr, n_ntiles, kplanes, ktp, group_m);
}
template <typename Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 2) void big_kgrouped_gemm_kernel(SharedGemmArgs a, RowGroups rg, int n_ntiles, int group_m) {
  big_gemm_body<Cfg, 2>(a, &rg, n_ntiles, rg.n, 0, group_m);
}

// ternary weights, groups of rows
__global__ __launch_bounds__(512, 2) void big_grouped_gemm_kernel(SharedGemmArgs a, RowGroups rg, int n_ntiles, int kplanes, int ktp, int group_m) {
  big_gemm_body<BigCfg<1, true>, 1>(a, &rg, n_ntiles, kplanes, ktp, group_m);
}


// Mid-size problems, where a CU has one or two tiles: 128-row tiles, one workgroup of eight wavefronts per CU, and a ring
// deep enough to cover the latency of a load by itself: K chunks of 64 elements (128-byte LDS rows, as above), the loads
// four (128 x 128) or two (128 x 256) chunks, some 2500 cycles, ahead.  A chunk is two halves of its K; the fragments of a
// half are read during the half before it, into the other one of two register sets.  The one barrier of a chunk stands
// between its halves: it publishes the next chunk and frees this one's stage, both its halves' fragments having been read.
// BNT: channels of a tile, both matrices together.  GROUPED: 0 plain, 1 row groups, 2 K ranges.  TERN: ternary weights, a
// half's fragments unpacked in front of its MFMAs: a wavefront has 64 rows x 32 channels of them (with 32 x 64 it unpacks twice as
// much: 16 groups of 6 rows, N = 2048, K = 10496: 101 -> 88 us).  Tiles of row groups with few rows: wavefronts without rows
// only load, and rows past the group's end are loads of its last row (88 -> 62; four wavefronts and two workgroups per CU, before: 80).
template <int MODE_, int BNT_, bool TERN_ = false>
struct MidCfg {
  static constexpr int MODE = MODE_;
  static constexpr int NMAT = MODE_ == 0 ? 2 : 1;
  static constexpr int BM = 128, BNT = BNT_, BN = BNT_ / NMAT, WAVES = 8, THREADS = 512;
  static constexpr int WAVES_M = BNT_ == 128 && !TERN_ ? 4 : 2, WAVES_N = 8 / WAVES_M;
  static constexpr int A16 = BM / WAVES_M / 16, NB = BNT_ / WAVES_N / 16, B16 = NB / NMAT;   // fragments of a wavefront
  static constexpr bool TERN = TERN_;
  static constexpr int A_BYTES = BM * 128, STAGE = A_BYTES + BNT_ * (TERN_ ? 16 : 128);
  static constexpr int STAGES = BNT_ == 128 ? 5 : 3, LDS_BYTES = STAGES * STAGE;
  static constexpr int A_LOADS = BM / 64, B_LOADS = TERN_ ? 1 : BNT_ / 64, NLOAD = A_LOADS + B_LOADS;   // per wavefront and chunk
  static constexpr int AHEAD = STAGES == 5 ? 3 : 2;   // chunks of the next tile requested in front of the epilogue; the patches have the other stages
  static constexpr int OUT_BYTES = MODE_ == 0 ? 2 : 4;
  static constexpr int PF = 2;                                        // fragments of a patch row
  static constexpr int PATCH_ROW = PF * 16 * OUT_BYTES + 16, PATCH_BYTES = 32 * PATCH_ROW;
  static_assert(B16 % PF == 0 && A16 % 2 == 0, "whole patches");
  static_assert(STAGES == 5 ? 4 * PATCH_BYTES <= STAGE : 8 * PATCH_BYTES <= STAGE, "the patches fit the free stages");
  static_assert(LDS_BYTES <= 163840 && (STAGES - 2) * NLOAD < 64, "LDS of a CU, vmcnt field");
  static_assert(A16 * NB >= NLOAD, "every load of a chunk finds an MFMA to follow");
  static_assert(!TERN_ || (MODE_ == 1 && BNT_ == 128), "ternary weights: four blocks of 32 channels, a wavefront brings one half of one");
};

template <typename Cfg, int GROUPED>
__device__ __forceinline__ void mid_gemm_body(const SharedGemmArgs& a, const RowGroups* rg, int n_ntiles, int kplanes, int ktp, int group_m) {
  constexpr int NMAT = Cfg::NMAT, BM = Cfg::BM, BN = Cfg::BN, STAGE = Cfg::STAGE, STAGES = Cfg::STAGES;
  constexpr int A16 = Cfg::A16, NB = Cfg::NB, B16 = Cfg::B16, NLOAD = Cfg::NLOAD;
  extern __shared__ __attribute__((aligned(16))) unsigned char s_lds[];
  const int M = a.M, N = a.N, K = a.K;
  const int KT = K >> 6;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  // TERN: the four wavefronts of 64 rows on different SIMDs
  const int wm = Cfg::TERN ? wave / Cfg::WAVES_N : wave % Cfg::WAVES_M, wn = Cfg::TERN ? wave % Cfg::WAVES_N : wave / Cfg::WAVES_M;
  const int r16 = lane & 15, quart = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) unsigned char*)s_lds);
  const int frag = r16 * 128 + ((quart ^ (r16 >> 1)) << 4);   // as in big_gemm_body; K half 1 at ^ 64
  const int a_lds = wm * A16 * 2048 + frag, b_lds = Cfg::A_BYTES + wn * B16 * 2048 + frag;

  n_ntiles *= kplanes;
  int n_mtiles = (M + BM - 1) / BM;
  if constexpr (GROUPED == 1) n_mtiles = rg->tile0[rg->n];
  const int xcd = blockIdx.x & 7;
  const bool split_n = n_ntiles >= 16;
  const int xcd_ntiles = split_n ? (n_ntiles - xcd + 7) >> 3 : n_ntiles;
  const int xcd_mtiles = split_n ? n_mtiles : (n_mtiles - xcd + 7) >> 3;
  const int xcd_work = xcd_ntiles * xcd_mtiles;
  const int per_group = group_m * xcd_ntiles;
  const int stride = gridDim.x >> 3;
  int slot = blockIdx.x >> 3;
  if (slot >= xcd_work) return;

  constexpr int kBufferFlags = 0x00020000;   // raw buffer, 32-bit data format
  auto make_rsrc = [&](const void* base, int64_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    v4i r;
    r.x = static_cast<int>(static_cast<uint32_t>(p));
    r.y = static_cast<int>(static_cast<uint32_t>(p >> 32) & 0xFFFFu);
    r.z = static_cast<int>(bytes);
    r.w = kBufferFlags;
    return r;
  };
  const v4i rsrc_a = make_rsrc(a.act, static_cast<int64_t>(M) * K * 2);
  const v4i rsrc_b0 = make_rsrc(a.w0, Cfg::TERN ? static_cast<int64_t>(GROUPED == 1 ? rg->n : 1) * N * K / 4 : static_cast<int64_t>(N) * K * 2);
  const v4i rsrc_b1 = make_rsrc(NMAT == 2 ? a.w1 : a.w0, static_cast<int64_t>(N) * K * 2);
  const int ld_row = wave_u * 8 + (lane >> 3);   // row of a 64-row loader pass, physical chunk l % 8
  const uint32_t ld_chunk = static_cast<uint32_t>(((lane & 7) ^ ((ld_row >> 1) & 7)) << 4);
  uint32_t a_off[Cfg::A_LOADS], b_off[Cfg::B_LOADS];
  int mt, nt, kc, ktl;
  int mrow, mend = M, grp = 0;   // first row of the tile, one past the last row it may store, its group (0 without groups)
  int st = 0;   // byte offset of the current chunk's stage; chunk c + i is at st + i stages, wrapped

#define MOTE_STAGE(i_) (st + (i_) * STAGE >= STAGES * STAGE ? st + (i_) * STAGE - STAGES * STAGE : st + (i_) * STAGE)
#define MOTE_DECODE(slot_, mt_, nt_, kc_)                                       \
  {                                                                             \
    const int grp_ = (slot_) / per_group;                                       \
    const int in_ = (slot_) - grp_ * per_group;                                 \
    const int gsz_ = min(xcd_mtiles - grp_ * group_m, group_m);                 \
    const int ni_ = in_ / gsz_, mi_ = grp_ * group_m + (in_ - ni_ * gsz_);      \
    mt_ = split_n ? mi_ : xcd + 8 * mi_;                                        \
    const int ntk_ = split_n ? xcd + 8 * ni_ : ni_;                             \
    nt_ = ntk_ / kplanes;                                                       \
    kc_ = ntk_ - nt_ * kplanes;                                                 \
  }
#define MOTE_KRANGE(kc_, kb_, ktl_)                                             \
  {                                                                             \
    if constexpr (GROUPED == 2) {                                               \
      kb_ = static_cast<uint32_t>(rg->row0[kc_]) * 2u;                          \
      ktl_ = (rg->row0[(kc_) + 1] - rg->row0[kc_]) >> 6;                        \
    } else {                                                                    \
      kb_ = static_cast<uint32_t>((kc_) * ktp) * 128u;                          \
      ktl_ = min(ktp, KT - (kc_) * ktp);                                        \
    }                                                                           \
  }
#define MOTE_ROWS(mt_, mrow_, mend_, grp_)                                      \
  {                                                                             \
    if constexpr (GROUPED == 1) {                                               \
      int e_ = 0;                                                               \
      while (e_ + 1 < rg->n && rg->tile0[e_ + 1] <= (mt_)) ++e_;                \
      grp_ = e_;                                                                \
      mrow_ = rg->row0[e_] + ((mt_) - rg->tile0[e_]) * BM;                      \
      mend_ = rg->row0[e_ + 1];                                                 \
    } else {                                                                    \
      mrow_ = (mt_) * BM;                                                       \
    }                                                                           \
  }
#define MOTE_POINTERS(mrow_, mlast_, grp_, nt_, kb_)                                                     \
  {                                                                                                \
    const uint32_t k0_ = (kb_) + ld_chunk;                                                         \
    _Pragma("unroll") for (int p = 0; p < Cfg::A_LOADS; ++p)                                       \
      a_off[p] = static_cast<uint32_t>(min((mrow_) + p * 64 + ld_row, (mlast_) - 1)) * static_cast<uint32_t>(K) * 2u + k0_; \
    if constexpr (Cfg::TERN) {                                                                     \
      const int blk_ = min((nt_) * (BN / 32) + (wave_u & 3), (N >> 5) - 1) + (grp_) * (N >> 5);    \
      b_off[0] = static_cast<uint32_t>(blk_) * static_cast<uint32_t>(K) * 8u + (kb_) * 4u + (wave_u >> 2) * 256u + lane * 4u; \
    } else _Pragma("unroll") for (int p = 0; p < Cfg::B_LOADS; ++p)                                \
      b_off[p] = static_cast<uint32_t>(min((nt_) * BN + (p * 64) % BN + ld_row, N - 1)) * static_cast<uint32_t>(K) * 2u + k0_; \
  }
  // load p_ of chunk ks_: the passes of A, then those of B (M0: see ternary_gemm.hip)
#define MOTE_DMA(stage_, ks_, p_)                                                                  \
  {                                                                                                \
    if (Cfg::TERN && (p_) == Cfg::A_LOADS)                                                         \
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"         \
                   :: "s"(lds0 + (stage_) + Cfg::A_BYTES + wave_u * 256), "v"(b_off[0]), "s"(rsrc_b0), "s"((ks_) * 512) : "memory"); \
    else                                                                                           \
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"       \
                   :: "s"(lds0 + (stage_) + ((p_) * 64 + wave_u * 8) * 128),                       \
                      "v"((p_) < Cfg::A_LOADS ? a_off[(p_) < Cfg::A_LOADS ? (p_) : 0] : b_off[(p_) < Cfg::A_LOADS ? 0 : (p_) - Cfg::A_LOADS]), \
                      "s"((p_) < Cfg::A_LOADS ? rsrc_a : (((p_) - Cfg::A_LOADS) * 64) / BN == 0 ? rsrc_b0 : rsrc_b1), "s"((ks_) * 128) : "memory"); \
  }
#define MOTE_ISSUE(stage_, ks_) { _Pragma("unroll") for (int p = 0; p < NLOAD; ++p) MOTE_DMA(stage_, ks_, p); }
#define MOTE_A_FRAG(stage_, h_, i_) *reinterpret_cast<const bf16x8*>(s_lds + (stage_) + (a_lds ^ ((h_) * 64)) + (i_) * 2048)
#define MOTE_B_FRAG(stage_, h_, b_) \
  *reinterpret_cast<const bf16x8*>(s_lds + (stage_) + (b_lds ^ ((h_) * 64)) + ((b_) / B16) * (BN * 128) + ((b_) % B16) * 2048)
  // fragment r_ of a half: the weights, then the activations
#define MOTE_READ(af_, b_, w_, stage_, h_, r_)                                                     \
  {                                                                                                \
    if (Cfg::TERN && (r_) < NB) {                                                                  \
      if (((r_) & 1) == 0)                                                                         \
        w_[(r_) < NB ? (r_) / 2 : 0] = *reinterpret_cast<const uint32_t*>(                         \
            s_lds + (stage_) + Cfg::A_BYTES + ((h_) * 4 + wn * (NB / 2) + ((r_) < NB ? (r_) / 2 : 0)) * 256 + lane * 4); \
    } else if ((r_) < NB) b_[(r_) < NB ? (r_) : 0] = MOTE_B_FRAG(stage_, h_, (r_) < NB ? (r_) : 0);       \
    else if ((r_) < NB + A16) af_[(r_) >= NB && (r_) < NB + A16 ? (r_) - NB : 0] = MOTE_A_FRAG(stage_, h_, (r_) >= NB && (r_) < NB + A16 ? (r_) - NB : 0); \
  }

  MOTE_DECODE(slot, mt, nt, kc);
  uint32_t kb;
  MOTE_KRANGE(kc, kb, ktl);
  MOTE_ROWS(mt, mrow, mend, grp);
  MOTE_POINTERS(mrow, mend, grp, nt, kb);
#pragma unroll
  for (int i = 0; i < Cfg::AHEAD; ++i)
    if (i < ktl) MOTE_ISSUE(MOTE_STAGE(i), i);

  for (;;) {
    const int nslot = slot + stride;
    const bool has_next = nslot < xcd_work;
    int mt2 = mt, nt2 = nt, kc2 = kc, ktl2 = ktl, mrow2 = mrow, mend2 = mend, grp2 = grp;
    uint32_t kb2 = kb;
    if (has_next) {
      MOTE_DECODE(nslot, mt2, nt2, kc2);
      MOTE_ROWS(mt2, mrow2, mend2, grp2);
      MOTE_KRANGE(kc2, kb2, ktl2);
    }
    // chunk 0 visible to every wavefront, the patches of the previous tile done
    if (ktl >= Cfg::AHEAD) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((Cfg::AHEAD - 1) * NLOAD) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int i = Cfg::AHEAD; i < STAGES; ++i)
      if (i < ktl) MOTE_ISSUE(MOTE_STAGE(i), i);

    v4f acc[A16][NB];
#pragma unroll
    for (int i = 0; i < A16; ++i)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[i][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 ax[A16], bx[NB], ay[A16], by[NB];
    uint32_t wx[NB / 2], wy[NB / 2];
    // a half: MFMAs of (af_, b_), behind MFMA j the statement side_(j)
#define MOTE_HALF(af_, b_, w_, side_)                                                              \
    if constexpr (Cfg::TERN) { _Pragma("unroll") for (int b = 0; b < NB; ++b) b_[b] = ternary_operand(w_[b / 2], b & 1); } \
    _Pragma("unroll") for (int i = 0; i < A16; ++i)                                                \
      _Pragma("unroll") for (int b = 0; b < NB; ++b) {                                             \
        const int j = i * NB + b;                                                                  \
        acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b_[b], af_[i], acc[i][b], 0, 0, 0);    \
        side_                                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                         \
      }
    // chunk c; PF_: with the requests of chunk c + STAGES into this chunk's stage.  After the last chunk the reads of the
    // second half are of a stage nobody uses, and dropped.
#define MOTE_CHUNK(PF_, wait_)                                                                     \
    {                                                                                              \
      const int nx = MOTE_STAGE(1);                                                                \
      __builtin_amdgcn_sched_barrier(0);                                                           \
      MOTE_HALF(ax, bx, wx, {                                                                          \
        if (j < (NB + A16 + 1) / 2) { MOTE_READ(ay, by, wy, st, 1, 2 * j) MOTE_READ(ay, by, wy, st, 1, 2 * j + 1) } \
      })                                                                                           \
      wait_                                                                                        \
      asm volatile("s_barrier" ::: "memory");                                                      \
      MOTE_HALF(ay, by, wy, {                                                                          \
        if (j < (NB + A16 + 1) / 2) { MOTE_READ(ax, bx, wx, nx, 0, 2 * j) MOTE_READ(ax, bx, wx, nx, 0, 2 * j + 1) } \
        if (PF_ && j >= A16 * NB - NLOAD) MOTE_DMA(st, c + STAGES, j >= A16 * NB - NLOAD ? j - (A16 * NB - NLOAD) : 0); \
      })                                                                                           \
      st = nx;                                                                                     \
    }
    // chunk c + 1 has landed: the `later` chunks behind it may be on their way
#define MOTE_WAIT_LAST(later_)                                                                     \
    {                                                                                              \
      if (STAGES > 4 && (later_) >= 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(3 * NLOAD) : "memory");  \
      else if (STAGES > 3 && (later_) >= 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(2 * NLOAD) : "memory"); \
      else if ((later_) >= 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(NLOAD) : "memory"); \
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");                             \
    }
    int c = 0;
    if (GROUPED == 1 && mrow + wave_u / Cfg::WAVES_N * A16 * 16 >= mend) {   // no rows for this wavefront: its share of the loads, and the barriers
      for (; c < ktl; ++c) {
        const int nx = MOTE_STAGE(1);
        if (c + STAGES < ktl) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((STAGES - 2) * NLOAD) : "memory");
        else MOTE_WAIT_LAST(ktl - 2 - c)
        asm volatile("s_barrier" ::: "memory");
        if (c + STAGES < ktl) MOTE_ISSUE(st, c + STAGES);
        st = nx;
      }
    } else {
#pragma unroll
      for (int r = 0; r < NB + A16; ++r) MOTE_READ(ax, bx, wx, st, 0, r)
      for (; c + STAGES < ktl; ++c)
        MOTE_CHUNK(true, asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((STAGES - 2) * NLOAD) : "memory");)
      for (; c < ktl; ++c) MOTE_CHUNK(false, MOTE_WAIT_LAST(ktl - 2 - c))
    }
#undef MOTE_WAIT_LAST
#undef MOTE_CHUNK
#undef MOTE_HALF

    if (has_next) {   // the next tile's first loads travel while this tile runs its epilogue in the stages behind them
      MOTE_POINTERS(mrow2, mend2, grp2, nt2, kb2);
#pragma unroll
      for (int i = 0; i < Cfg::AHEAD; ++i)
        if (i < ktl2) MOTE_ISSUE(MOTE_STAGE(i), i);
    }

    // ---- epilogue: as in big_gemm_body, patches of 32 rows x PF fragments ----
    constexpr int PF = Cfg::PF, LANES_PER_ROW = PF * 16 * Cfg::OUT_BYTES / 16, ROWS_PER_READ = 64 / LANES_PER_ROW;
    unsigned char* const patch = STAGES == 5 ? s_lds + (wave < 4 ? MOTE_STAGE(3) : MOTE_STAGE(4)) + (wave & 3) * Cfg::PATCH_BYTES
                                             : s_lds + MOTE_STAGE(2) + wave * Cfg::PATCH_BYTES;
    const int n_wave0 = nt * BN + wn * B16 * 16;
    const int rd_row = lane / LANES_PER_ROW, rd_chunk = lane % LANES_PER_ROW;
    if (a.scale0 != nullptr) {
#pragma unroll
      for (int b = 0; b < B16; ++b) {
        const int ch = min(n_wave0 + b * 16 + 4 * quart, N - 4);
        const float4 s0_ = *reinterpret_cast<const float4*>(a.scale0 + static_cast<int64_t>(grp) * N + ch);
        float4 s1_ = s0_;
        if constexpr (NMAT == 2) s1_ = *reinterpret_cast<const float4*>(a.scale1 + ch);
#pragma unroll
        for (int i = 0; i < A16; ++i) {
          acc[i][b].x *= s0_.x; acc[i][b].y *= s0_.y; acc[i][b].z *= s0_.z; acc[i][b].w *= s0_.w;
          if constexpr (NMAT == 2) {
            v4f& au = acc[i][(NMAT - 1) * B16 + b];
            au.x *= s1_.x; au.y *= s1_.y; au.z *= s1_.z; au.w *= s1_.w;
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < A16; i += 2) {
#pragma unroll
      for (int f0 = 0; f0 < B16; f0 += PF) {
#pragma unroll
        for (int bb = 0; bb < PF; ++bb) {
          const int b = f0 + bb;
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const v4f v = acc[i + r][b];
            unsigned char* const dst = patch + (r * 16 + r16) * Cfg::PATCH_ROW + (bb * 16 + 4 * quart) * Cfg::OUT_BYTES;
            if constexpr (Cfg::MODE == 0) {
              const v4f u = acc[i + r][(NMAT - 1) * B16 + b];
              uint2 packed;
              packed.x = cvt_pk_bf16(u.x * silu_fast(v.x), u.y * silu_fast(v.y));
              packed.y = cvt_pk_bf16(u.z * silu_fast(v.z), u.w * silu_fast(v.w));
              *reinterpret_cast<uint2*>(dst) = packed;
            } else {
              *reinterpret_cast<float4*>(dst) = make_float4(v.x, v.y, v.z, v.w);
            }
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int rd_n = n_wave0 + f0 * 16 + rd_chunk * (16 / Cfg::OUT_BYTES);
#pragma unroll
        for (int p = 0; p < 32 / ROWS_PER_READ; ++p) {
          const int pr = p * ROWS_PER_READ + rd_row;
          const u4 v = *reinterpret_cast<const u4*>(patch + pr * Cfg::PATCH_ROW + rd_chunk * 16);
          const int orow = mrow + wm * A16 * 16 + i * 16 + pr;
          if (orow < mend && rd_n < N) {
            const int64_t o = static_cast<int64_t>(orow) * N + rd_n;
            if constexpr (Cfg::MODE == 0) *reinterpret_cast<u4*>(a.h_out + o) = v;
            else *reinterpret_cast<u4*>(a.y_out + static_cast<int64_t>(kc) * a.plane_stride + o) = v;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    if (!has_next) break;
    slot = nslot; mt = mt2; nt = nt2; kc = kc2; ktl = ktl2; kb = kb2; mrow = mrow2; mend = mend2; grp = grp2;
  }
#undef MOTE_STAGE
#undef MOTE_DECODE
#undef MOTE_KRANGE
#undef MOTE_POINTERS
#undef MOTE_ROWS
#undef MOTE_DMA
#undef MOTE_ISSUE
#undef MOTE_A_FRAG
#undef MOTE_B_FRAG
#undef MOTE_READ
}

template <typename Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 2) void mid_gemm_kernel(SharedGemmArgs a, int n_ntiles, int kplanes, int ktp, int group_m) {
  mid_gemm_body<Cfg, 0>(a, nullptr, n_ntiles, kplanes, ktp, group_m);
}
template <typename Cfg>
__global__ __launch_bounds__(Cfg::THREADS, 2) void mid_kgrouped_gemm_kernel(SharedGemmArgs a, RowGroups rg, int n_ntiles, int group_m) {
  mid_gemm_body<Cfg, 2>(a, &rg, n_ntiles, rg.n, 0, group_m);
}
// ternary weights, groups of rows
__global__ __launch_bounds__(512, 2) void mid_grouped_gemm_kernel(SharedGemmArgs a, RowGroups rg, int n_ntiles, int kplanes, int ktp, int group_m) {
  mid_gemm_body<MidCfg<1, 128, true>, 1>(a, &rg, n_ntiles, kplanes, ktp, group_m);
}

static int shared_cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
  }
  return n;
}

static int shared_variant() { return knob(kKnobSharedVariant); }

constexpr int kBigBand = 4;   // row tiles per band, see launch_big_cfg

// Tiles of the XCD that owns most of them (see the tile order), i.e. eight times that many workgroups take them in one round.
static int64_t longest_list(int64_t mt, int64_t nk) { return nk >= 16 ? (nk + 7) / 8 * mt : (mt + 7) / 8 * nk; }
static unsigned gemm_blocks(int64_t longest) { return static_cast<unsigned>(std::min<int64_t>(shared_cu_count() / 8 * 8, longest * 8)); }

template <typename K>
static hipError_t allow_lds(K* kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// The plain kernels (rg == nullptr), or one plane per K range.
template <typename Cfg>
static hipError_t launch_big_cfg(const SharedGemmArgs& a, int kplanes, const RowGroups* rg, hipStream_t stream) {
  const int n_ntiles = (a.N + Cfg::BN - 1) / Cfg::BN, n_mtiles = (a.M + Cfg::BM - 1) / Cfg::BM;
  const int KT = a.K >> 6;
  const int ktp = (KT + kplanes - 1) / kplanes;   // chunks per plane
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = allow_lds(big_gemm_kernel<Cfg>, Cfg::LDS_BYTES);
    if constexpr (Cfg::MODE == 1) if (e == hipSuccess) e = allow_lds(big_kgrouped_gemm_kernel<Cfg>, Cfg::LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const unsigned blocks = gemm_blocks(longest_list(n_mtiles, static_cast<int64_t>(n_ntiles) * kplanes));
  // Band height: the 32 workgroups of an XCD share the least operand bytes as 4 x 8 tiles.  Weights that the memory-side cache
  // (256 MB) does not keep are read once per band: bands of eight (16384 x 3584 x 18944 gate-up: 3235 us of two, 3210 of four, 3145 of
  // eight; with 90 MB of weights all the same).  K ranges write more than they read; from eight ranges and eight channel
  // tiles on bands of three (us of bands of two / three / four: 16 ranges, 18944 x 3584, 200 rows in all 792 / 794 / 846, 4000 rows 1151 /
  // 1113 / 1337; 11008 x 2048, 4000 rows 452 / 364 / 387, 16384 rows 818 / 802 / 802; 3584 x 18944, 4000 rows 1272 / 1258 / 1329), but four below:
  // four ranges, 18944 x 3584, 4000 rows 514 / 520 / 487; 16 ranges, 8960 x 1536, 4000 rows 235 / 258 / 233.
  const int group_m = rg != nullptr ? (kplanes >= 8 && n_ntiles >= 8 ? 3 : kBigBand)
                                    : static_cast<int64_t>(Cfg::NMAT) * a.N * a.K * 2 > (int64_t{192} << 20) ? 8 : kBigBand;
  if constexpr (Cfg::MODE == 1) if (rg != nullptr) {
    big_kgrouped_gemm_kernel<Cfg><<<blocks, Cfg::THREADS, Cfg::LDS_BYTES, stream>>>(a, *rg, n_ntiles, group_m);
    return hipGetLastError();
  }
  big_gemm_kernel<Cfg><<<blocks, Cfg::THREADS, Cfg::LDS_BYTES, stream>>>(a, n_ntiles, kplanes, ktp, group_m);
  return hipGetLastError();
}

template <typename Cfg>
static hipError_t launch_mid_cfg(const SharedGemmArgs& a, int kplanes, const RowGroups* rg, hipStream_t stream) {
  const int n_ntiles = (a.N + Cfg::BN - 1) / Cfg::BN, n_mtiles = (a.M + Cfg::BM - 1) / Cfg::BM;
  const int KT = a.K >> 6;
  const int ktp = (KT + kplanes - 1) / kplanes;   // chunks per plane
  constexpr bool RANGES = Cfg::MODE == 1 && Cfg::BNT == 128;   // the tile that takes K ranges
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = allow_lds(mid_gemm_kernel<Cfg>, Cfg::LDS_BYTES);
    if constexpr (RANGES) if (e == hipSuccess) e = allow_lds(mid_kgrouped_gemm_kernel<Cfg>, Cfg::LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const unsigned blocks = gemm_blocks(longest_list(n_mtiles, static_cast<int64_t>(n_ntiles) * kplanes));
  if constexpr (RANGES) if (rg != nullptr) {
    mid_kgrouped_gemm_kernel<Cfg><<<blocks, Cfg::THREADS, Cfg::LDS_BYTES, stream>>>(a, *rg, n_ntiles, kBigBand);
    return hipGetLastError();
  }
  mid_gemm_kernel<Cfg><<<blocks, Cfg::THREADS, Cfg::LDS_BYTES, stream>>>(a, n_ntiles, kplanes, ktp, kBigBand);
  return hipGetLastError();
}

// Which tile takes a problem of M rows, N channels per matrix, K = 64 * KT, and in how many K planes (at most
// max_planes): the cheapest by a model of what a CU does, rounds of tiles of the busiest XCD x (chunks x time of a chunk +
// start and end of a tile) + reading a further plane back.  Measured per chunk at one workgroup per CU: 256 x 256
// 1.28 us, 128 x 256 0.74 us, 128 x 128 0.50 us.  Times of the kernels alone, us (256 x 256 / 128 x 256 / 128 x 128;
// before: 128-row tiles of four wavefronts on 64-byte rows):
//   gate-up  2048 x 896 x 4864 39 / 38 / 40 (43);  500 x 2048 x 11008 41 / 48 / 50 (79);  1024 x 2048 x 11008 80 / 84 / 98 (97)
//            300 x 1536 x 8960 29 / 21 / 25 (28);  130 x 3584 x 18944 75 / 84 / 78 (141);  600 x 896 x 4864 19 / - / 15 (23)
//   down     2048 x 4864 x 896 in 2 planes 44 / 28 / 22 (30);  500 x 11008 x 2048 in 4: 49 / 32 / 26 (40 in 5)
//            1024 x 11008 x 2048 in 4: 50 / 42 / 49 (57);  300 x 8960 x 1536 in 4: 40 / 25 / 17 (31 in 7)
//            2048 x 8960 x 1536 in 2: 75 / 56 / 65 (74)
// From four rounds of 256 x 256 tiles on those are taken in any case: the others move more operand bytes per flop.
// M counts in 128-row tiles and by max_planes only: the workspace has room for the planes, and mote_layer_workspace_bytes tries the
// last batch of every number of tiles (and the one in front of kSharedDownWideTokens).  Beside the shape the choice depends on
// the number of CUs and on the shared_variant knob.
enum GemmTile { kTileMid128 = 1, kTileMid256, kTileBig };
struct GemmChoice { GemmTile tile; int planes; };
static GemmChoice gemm_choice(int M, int N, int K, int nmat, int max_planes) {
  const int KT = K >> 6, cus8 = shared_cu_count() / 8;
  const int m128 = (M + 127) / 128, m256 = (M + 255) / 256;
  const struct { GemmTile tile; int mt, bn; double chunk, ends; } kinds[3] = {
      {kTileBig, m256, 256 / nmat, 1.28, 3.0}, {kTileMid256, m128, 256 / nmat, 0.74, 1.5}, {kTileMid128, m128, 128 / nmat, 0.50, 1.0}};
  const double plane_us = static_cast<double>(m128) * 128 * N * 4 / 5e6;
  const int forced = shared_variant();   // experiments: one of the three tiles
  GemmChoice best{kTileBig, 1};
  double best_us = 1e30;
  for (const auto& k : kinds) {
    const int64_t nt = (N + k.bn - 1) / k.bn;
    if (forced != 0 && forced != k.tile) continue;
    for (int p = 1; p <= max_planes; ++p) {
      const int ktp = (KT + p - 1) / p;
      if ((KT + ktp - 1) / ktp != p) continue;   // an empty plane
      const int64_t rounds = (longest_list(k.mt, nt * p) + cus8 - 1) / cus8;
      const double us = static_cast<double>(rounds) * (ktp * k.chunk + k.ends) + (p - 1) * plane_us;
      if (us < best_us) { best_us = us; best = {k.tile, p}; }
    }
    if (k.tile == kTileBig && k.mt * nt >= 4 * 8 * cus8) break;
  }
  return best;
}

double shared_gate_up_rounds(int T, int d, int F, int* tile_rows) {
  const GemmTile tile = gemm_choice(T, F, d, 2, 1).tile;
  *tile_rows = tile == kTileBig ? 256 : 128;
  if (tile == kTileMid128) return 0.0;
  return static_cast<double>((T + *tile_rows - 1) / *tile_rows) * ((F + 127) / 128) / shared_cu_count();
}

hipError_t launch_shared_gate_up(const uint16_t* x, const uint16_t* w_gate, const uint16_t* w_up, int T, int d,
                                 int F, uint16_t* h_s, hipStream_t stream) {
  return launch_shared_gate_up_scaled(x, w_gate, w_up, nullptr, nullptr, T, d, F, h_s, stream);
}

hipError_t launch_shared_gate_up_scaled(const uint16_t* x, const uint16_t* w_gate, const uint16_t* w_up,
                                        const float* s_gate, const float* s_up, int T, int d, int F, uint16_t* h_s,
                                        hipStream_t stream) {
  if (T == 0) return hipSuccess;
  SharedGemmArgs a{x, w_gate, w_up, T, F, d, h_s, nullptr, 0, s_gate, s_up, nullptr};
  switch (gemm_choice(T, F, d, 2, 1).tile) {
    case kTileMid128: return launch_mid_cfg<MidCfg<0, 128>>(a, 1, nullptr, stream);
    case kTileMid256: return launch_mid_cfg<MidCfg<0, 256>>(a, 1, nullptr, stream);
    default: return launch_big_cfg<BigCfg<0>>(a, 1, nullptr, stream);
  }
}

// K planes that the down projection may have: every further plane adds an fp32 partial output that is written by the GEMM
// and read back by the combine, and room for it in the scratch.  At most what two 128 x 128 tiles per CU or one
// plane of 2048 channels ask for, few tiles (small T, whose partial outputs are small) up to one tile per CU and planes of
// eight chunks; 48 to 64 tiles of 256 x 256 as many as fill the chip once, from kSharedDownWideTokens on (from
// 1409 = the first batch of as many row tiles 1 % slower: d = 2048, T = 1500, E = 16 430 -> 436 us per forward, T = 1472, E = 4, top-1 310 -> 314).
static int shared_down_max_planes(int T, int d, int F) {
  const int KT = F >> 6;
  const int64_t tiles256 = static_cast<int64_t>((T + 255) / 256) * ((d + 255) / 256);
  int planes = 0;
  if (T >= kSharedDownWideTokens && d >= 2048 && tiles256 <= 64) planes = std::min(static_cast<int>(256 / tiles256), F / 1024);
  if (planes < 2) {
    const int64_t tiles = static_cast<int64_t>((T + 127) / 128) * ((d + 127) / 128);
    planes = tiles > 0 ? static_cast<int>(512 / tiles) : 1;
    if (planes > F / 2048) planes = F / 2048;
    int fill = tiles > 0 ? static_cast<int>(256 / tiles) : 1;
    if (fill > KT / 8) fill = KT / 8;
    if (planes < fill) planes = fill;
    if (planes > 8) planes = 8;
  }
  if (planes < 1) planes = 1;
  const int ktp = (KT + planes - 1) / planes;
  return (KT + ktp - 1) / ktp;
}

int shared_down_planes(int T, int d, int F) { return gemm_choice(T, d, F, 1, shared_down_max_planes(T, d, F)).planes; }

hipError_t launch_shared_down(const uint16_t* h_s, const uint16_t* w_down, int T, int d, int F, float* y_s,
                              hipStream_t stream) {
  return launch_shared_down_scaled(h_s, w_down, nullptr, T, d, F, y_s, stream);
}

hipError_t launch_shared_down_scaled(const uint16_t* h_s, const uint16_t* w_down, const float* s_down, int T, int d,
                                     int F, float* y_s, hipStream_t stream) {
  if (T == 0) return hipSuccess;
  SharedGemmArgs a{h_s, w_down, nullptr, T, d, F, nullptr, y_s, static_cast<int64_t>(T) * d, s_down, nullptr, nullptr};
  const GemmChoice c = gemm_choice(T, d, F, 1, shared_down_max_planes(T, d, F));
  switch (c.tile) {
    case kTileMid128: return launch_mid_cfg<MidCfg<1, 128>>(a, c.planes, nullptr, stream);
    case kTileMid256: return launch_mid_cfg<MidCfg<1, 256>>(a, c.planes, nullptr, stream);
    default: return launch_big_cfg<BigCfg<1>>(a, c.planes, nullptr, stream);
  }
}

template <typename Cfg, typename Kernel>
static hipError_t launch_grouped_cfg(Kernel* kernel, const SharedGemmArgs& a, const int32_t* row0, int n_groups, int kplanes,
                                     int split_mt, hipStream_t stream) {
  RowGroups rg;
  rg.split_mt = split_mt;
  rg.n = n_groups;
  int tiles_m = 0;
  for (int e = 0; e < n_groups; ++e) {
    rg.row0[e] = row0[e] - row0[0];
    rg.tile0[e] = tiles_m;
    tiles_m += (row0[e + 1] - row0[e] + Cfg::BM - 1) / Cfg::BM;
  }
  rg.row0[n_groups] = row0[n_groups] - row0[0];
  rg.tile0[n_groups] = tiles_m;
  for (int e = n_groups + 1; e <= kMaxRowGroups; ++e) rg.row0[e] = rg.tile0[e] = 0;
  if (tiles_m == 0) return hipSuccess;
  const int n_ntiles = (a.N + Cfg::BN - 1) / Cfg::BN;
  const int KT = a.K >> 6;
  const int ktp = (KT + kplanes - 1) / kplanes;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = allow_lds(kernel, Cfg::LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const unsigned blocks = gemm_blocks(longest_list(split_mt, n_ntiles) + longest_list(tiles_m - split_mt, static_cast<int64_t>(n_ntiles) * kplanes));
  kernel<<<blocks, Cfg::THREADS, Cfg::LDS_BYTES, stream>>>(a, rg, n_ntiles, kplanes, ktp, kBigBand);
  return hipGetLastError();
}

// Row tiles a grouped launch has with tiles of bm rows.
static int64_t grouped_row_tiles(const int32_t* row0, int n_groups, int bm) {
  int64_t t = 0;
  for (int e = 0; e < n_groups; ++e) t += (row0[e + 1] - row0[e] + bm - 1) / bm;
  return t;
}

// How a grouped GEMM cuts its contraction (pure function of the group sizes and the shape, at most max_planes planes).
// 256 x 256 tiles: the row tiles that fill whole rounds of workgroups contract all of K, those of the last, partly
// empty round are cut into as many planes as fill it.  16 groups of about 1024 rows, N = 2048, K = 11008: 576 tiles on
// 256 CUs are two rounds of 512 and 64 tiles in four planes: 669 + 70 us (two planes for all rows, and their sum) -> 624 + 10.
// With fewer than 16 channel tiles the row tiles are dealt to the XCDs, so whole rounds are whole rounds of every XCD.
// Where no such cut exists: two planes for all rows when one plane leaves more than 15 % of the last round empty and two
// leave less.  Small problems (128 x 128 tiles, one workgroup per CU): by rounds of tiles, 0.36 - 0.44 us per chunk (tiles of up to
// 64 rows, more), and the launch that adds the planes.  16 groups of 6 rows, N = 2048, K = 10496: 256 tiles are one round and one
// plane (60 us; two planes 62 + 5); 16 of 125 rows, N = 1536, K = 8960: 300 tiles, two planes (98 + 3; one 122).
GemmSplit grouped_gemm_split(const int32_t* row0_host, int n_groups, int N, int K, int max_planes) {
  GemmSplit sp{1, 0, 0};
  const int cus = shared_cu_count();
  const int nt = (N + 255) / 256;
  const int mt = static_cast<int>(grouped_row_tiles(row0_host, n_groups, 256));
  const int64_t t256 = static_cast<int64_t>(mt) * nt;
  const int KT = K >> 6;
  if (t256 >= (3 * cus) / 4) {
    auto eff = [&](int p) {
      const int64_t rounds = (t256 * p + cus - 1) / cus;
      return static_cast<double>(t256 * p) / static_cast<double>(rounds * cus);
    };
    if (eff(1) >= 0.85 || max_planes < 2 || KT < 32) return sp;
    if (nt < 16 && cus % 8 == 0) {
      int whole = mt / 8 * 8;
      while (whole > 0 && (whole / 8 * nt) % (cus / 8) != 0) whole -= 8;
      const int left = mt - whole;
      int p = left > 0 ? cus / (left * nt) : 1;
      p = std::min(std::min(p, max_planes), KT / 16);
      if (whole > 0 && p >= 2) {
        sp.planes = (KT + (KT + p - 1) / p - 1) / ((KT + p - 1) / p);   // every plane non-empty
        sp.split_mt = whole;
        int e = 0, t = 0;   // first row of row tile `whole`
        for (; e < n_groups; ++e) {
          const int te = (row0_host[e + 1] - row0_host[e] + 255) / 256;
          if (t + te > whole) break;
          t += te;
        }
        sp.split_row = row0_host[e] - row0_host[0] + (whole - t) * 256;
        return sp;
      }
    }
    if (eff(2) > eff(1) + 0.05) sp.planes = 2;
    return sp;
  }
  // 128 x 128 tiles: the cheapest number of planes, of at least 16 chunks each, as in gemm_choice
  const int m128 = static_cast<int>(grouped_row_tiles(row0_host, n_groups, 128)), n128 = (N + 127) / 128, cus8 = cus / 8;
  const double plane_us = static_cast<double>(row0_host[n_groups] - row0_host[0]) * N * 4 / 5e6;
  double best_us = 1e30;
  for (int p = 1; p <= std::max(1, std::min(max_planes, KT / 16)); ++p) {
    const int ktp = (KT + p - 1) / p;
    if ((KT + ktp - 1) / ktp != p) continue;   // an empty plane
    const int64_t rounds = (longest_list(m128, static_cast<int64_t>(n128) * p) + cus8 - 1) / cus8;
    const double us = static_cast<double>(rounds) * (ktp * 0.40 + 2.0) + (p > 1 ? 5.0 + p * plane_us : 0.0);
    if (us < best_us) { best_us = us; sp.planes = p; }
  }
  return sp;
}

// Grouped GEMM for other callers: rows row0_host[e] .. row0_host[e+1]-1 of act (row0_host: n_groups + 1
// ascending HOST integers; act, out and the rows are counted from row0_host[0], which act and out point at)
// are contracted with matrix e of w ([n_groups] matrices of [N, K] ternary blocks) and scaled per
// channel by row e of scale ([n_groups][N]): out[r, n] = scale[e][n] * sum_k act[r, k] * t[e][n, k].  sp as given by
// grouped_gemm_split: the rows below sp.split_row go to out; with more than one plane, plane p of the others writes its
// partial sums to planes_out + p * (rows - split_row) * N (row split_row first) and the caller adds them.
// n_groups <= 64, n_groups * N * K / 4 bytes and rows * K * 2 bytes below 4 GiB, K a multiple of 64.
hipError_t launch_gemm_grouped_f32(const uint16_t* act, const uint32_t* w, const int32_t* row0_host, int n_groups, int N,
                                   int K, float* out, float* planes_out, const float* scale, const GemmSplit& sp, hipStream_t stream) {
  if (n_groups < 1 || n_groups > kMaxRowGroups) return hipErrorInvalidValue;
  const int M = row0_host[n_groups] - row0_host[0];
  if (M == 0 || N == 0) return hipSuccess;
  float* const y_split = sp.planes > 1 ? planes_out - static_cast<int64_t>(sp.split_row) * N : out;
  SharedGemmArgs a{act, reinterpret_cast<const uint16_t*>(w), nullptr, M, N, K, nullptr, out, static_cast<int64_t>(M - sp.split_row) * N, scale, nullptr, y_split};
  if (grouped_row_tiles(row0_host, n_groups, 256) * ((N + 255) / 256) >= (3 * shared_cu_count()) / 4)
    return launch_grouped_cfg<BigCfg<1, true>>(big_grouped_gemm_kernel, a, row0_host, n_groups, sp.planes, sp.split_mt, stream);   // 256 x 256
  a.y_out = y_split;
  return launch_grouped_cfg<MidCfg<1, 128, true>>(mid_grouped_gemm_kernel, a, row0_host, n_groups, sp.planes, 0, stream);   // 128 x 128
}

// Several contractions over consecutive K ranges of the same two operands in one launch: plane p,
// written to out + p * M * N, is sum over k0_host[p] <= k < k0_host[p+1] of act[m, k] * w[n, k] (operands
// [M, K] and [N, K] with K = k0_host[n_groups]; the offsets are HOST integers, multiples of 64, ascending from
// 0; an empty range gives zeros).  The caller's use: one problem per range, its operands side by side along K.
hipError_t launch_gemm_tn_f32_kgroups(const uint16_t* act, const uint16_t* w, int M, int N, const int32_t* k0_host,
                                      int n_groups, float* out, hipStream_t stream) {
  if (n_groups < 1 || n_groups > kMaxRowGroups) return hipErrorInvalidValue;
  if (M == 0 || N == 0) return hipSuccess;
  const int K = k0_host[n_groups];
  SharedGemmArgs a{act, w, nullptr, M, N, K, nullptr, out, static_cast<int64_t>(M) * N, nullptr, nullptr};
  RowGroups rg;
  rg.n = n_groups;
  rg.split_mt = 0;
  for (int e = 0; e <= kMaxRowGroups; ++e) {
    rg.row0[e] = k0_host[std::min(e, n_groups)];
    rg.tile0[e] = 0;
  }
  if (static_cast<int64_t>((M + 255) / 256) * ((N + 255) / 256) * n_groups >= 256)
    return launch_big_cfg<BigCfg<1>>(a, n_groups, &rg, stream);              // 256 x 256
  return launch_mid_cfg<MidCfg<1, 128>>(a, n_groups, &rg, stream);           // 128 x 128
}

}  // namespace mote
