// Block-sparse attention forward on gfx950 (Sec. 3.3: attention over C_i = T u K^curr u S_i,
// one kept-block list per query block serving both K and V).
//
// Work decomposition
//   * A unit is 256 query rows of one (batch, head): four query blocks of 64 rows or two of 128.
//     Query blocks are grouped by the first historical key block they keep (frame-causal calls may
//     put their frame before it, see plan_union_kernel), so that blocks which chose the same
//     context share a unit.  Its tiles are the 64-key sub-tiles of the union of its blocks' kept
//     lists, in ascending key order, each tagged with which of the unit's blocks kept it.
//   * A planner (two or three small kernels) computes the grouping, every unit's union list, the
//     schedule and one record per tile (first key, head, unit, ownership) in the tile sequence.
//     One persistent workgroup per CU runs, first, whole units handed out in rounds: in each
//     round the workgroups of one XCD start consecutive units of the same head together, so
//     they walk that head's shared chunk K/V in step and each K/V tile reaches the XCD's L2
//     about once per round; then an equal-work share of the remaining units (those past the
//     last full round and the longer ones), cut anywhere (stream-K).  A unit cut between two
//     shares leaves (O, m, l) partials that attn_combine merges with a log-sum-exp merge.  Heavy
//     query blocks therefore never bound the launch.
//
// The workgroup: 8 waves = two groups of four, one wave of each group per SIMD.  Each wave owns
// 32 query rows; the two waves of a SIMD own the two halves of the same query block, so both
// groups own the same tiles.  Per tile h the groups run two phases each, offset by one phase and
// separated by workgroup barriers:
//
//   phase    group 0                              group 1
//   A(h)     M(h): P.V of tile h-1, Q.K^T of h    V(h-1): softmax of tile h-1, then issues the
//                                                 loads of V(h+1)
//   B(h)     V(h): softmax of tile h, then        M(h): P.V of tile h-1, Q.K^T of tile h
//            issues the loads of K(h+2)
//
// so on every SIMD one wave feeds the matrix pipeline while the other does the softmax
// arithmetic.  K and V have three LDS stages each (tile h in stage h % 3).  The stage that K(h+2)
// overwrites in B(h) was last read in B(h-1), the one that V(h+1) overwrites in A(h) too; what a
// wave issues in iteration h it waits for at the end of iteration h+1, so the loads have a whole
// iteration to land.  They are asynchronous buffer-to-LDS loads, 16 bytes per lane, four per wave
// and tile; their buffer descriptors end at Lk, so the ragged last block reads zeros past the end.
//
// What bounds it: a wave issues at most one instruction every four cycles, scalar ones included,
// so a V phase lasts as long as its instruction count: 111 vector instructions (32 of them
// exponentials, 8 cycles each) and what the tile's record, masks and loads need.  Records, masks
// and load addresses are therefore kept to about 40 scalar instructions (150 and a 9th load in
// four of the waves, with all loads on group 1: 27 % more cycles).  Measured with every block kept
// (16 heads, 6240 x 43680, d 128, with 32x32x16 MFMAs, one card): 2039 -> 1844 us, on zeros 1607 ->
// 1271 us (1.76 PFLOP/s): on real data the kernel is bound by the card's power, not by its cycles (a
// large bf16 matrix product reaches 1.39 PFLOP/s on random data and 1.80 on zeros).
//
// Per wave and 64-key tile:
//   S^T (64 keys x 32 queries) = K_tile (64 x d) . Q^T        MFMA, bf16 in, fp32 out
//   online softmax over keys (fp32, base 2; the running max is only raised when weights over it
//   pass 2^8, so most tiles skip the rescale of O)
//   O^T (d x 32) += V^T (d x 64) . P^T (64 x 32)              MFMA
// S^T is computed transposed so that its accumulator layout is, 8 values at a time, directly the B
// operand of the P.V product.  The V^T operand is read with the LDS transpose load
// ds_read_b64_tr_b16 (two per operand).  The MFMA shape is 16x16x32 for d = 128 and 32x32x16 for
// d = 64.  On random operands the card sustains 2040 TFLOP/s of the first and 1725 of the second
// (power), but the first holds up the vector instructions of the other wave more (the softmax of a
// tile takes 1049 cycles beside it, 718 beside the second, 623 alone).  With d = 128 the power
// decides: 720P step 2283 -> 2205 us, 480P dense 1844 -> 1786 us (on zeros 1271 -> 1365); with d = 64
// a tile has the same softmax for half the products, and 16x16x32 was 2-3 % slower.
#include <math.h>

#include <type_traits>

#include "la_internal.h"

namespace la {
namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int KT = 64;          // keys per tile
constexpr int QW = 32;          // query rows per wave
constexpr int QR = 256;         // query rows per unit (workgroup)
constexpr int kMaxPersist = 256;        // persistent workgroups: one per CU, at most 256
// flags of a tile record (see TileRef)
constexpr int kFlFrom0 = 1 << 4, kFlToEnd = 1 << 5, kFlMask = 1 << 6, kFlLast = 1 << 7, kFlValid = 1 << 8;
// Bits 16..22 of a tile record's flags: keys at the end of the tile that are padding (0..64).
constexpr int kFlPadShift = 16;

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// Shape of the MFMAs for head dimension D (MR x MR x KC) and what follows from it: lane l is row or
// column l % MR of group l / MR; it holds AR accumulator values, of rows acc_row(i) + 4 (l / MR).
template <int D>
struct Mma {
  static constexpr int MR = D == 128 ? 16 : 32;
  static constexpr int NG = 64 / MR;         // lane groups
  static constexpr int KC = 8 * NG;          // contraction depth: 8 values per lane
  static constexpr int QT = 32 / MR;         // MFMA columns of a wave's 32 query rows
  static constexpr int AR = MR * MR / 64;
  typedef typename std::conditional<MR == 16, f32x4, f32x16>::type Acc;
  __device__ static constexpr int acc_row(int i) { return 8 * (i >> 2) + (i & 3); }
  __device__ static __forceinline__ Acc mma(bf16x8 a, bf16x8 b, Acc c) {
    if constexpr (MR == 16)
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    else
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
#define LDS_AS __attribute__((address_space(3)))

// Two floats -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32.
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2v f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2v));
}

// Workgroup barrier for waves with asynchronous tile loads in flight that they do not wait for
// here (an LDS release fence would wait for them: they write LDS).  The empty asm statements keep
// the compiler from moving memory accesses across the barrier; every LDS read of the wave has been
// consumed by then, and no wave writes LDS except by tile loads.
__device__ __forceinline__ void phase_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Waits until at most n of this wave's vector memory operations are outstanding (n < 16).
template <int n>
__device__ __forceinline__ void wait_vmem() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | n);   // vmcnt(n), expcnt and lgkmcnt left at their maximum
}

// LDS layout: K and V tiles of 64 key rows of D bf16, row-major and not padded, so that a tile is
// an even share of four loads for each of four waves.  In a K row the 16-byte slots are permuted
// (slot c of row r is stored at slot c ^ kswz(r)): an MFMA operand read touches 16 rows per LDS
// cycle at one c.  In a V row the chunks of 2 MR bytes are (chunk c at chunk c ^ vswz(r)): a
// transpose read touches, per half-wave, 8 consecutive rows x 32 bytes (MR = 16) or 4 x 64 (32).
// Both spread over all 64 banks.  Every K operand read is one of D/KC lane bases (base ^ 16 NG ks)
// plus a compile-time offset, every V read one of D/MR (base ^ 2 MR dt).
template <int D>
struct Tile {
  static constexpr int STRIDE = D * 2;                 // bytes per row
  static constexpr int SLOTS = STRIDE / 16;            // 16-byte slots per row
  static constexpr int BYTES = KT * STRIDE;
  static constexpr int PER = BYTES / 4096;             // 1 KiB loads per loading wave (four load a tile)
  // slot permutation of K row r: the 16 rows one LDS cycle of an operand read touches lie in
  // distinct 16-byte bank groups (D = 64: two rows share the 256 bytes of all banks)
  __device__ static constexpr int kswz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  // chunk permutation of V row r: eight 32-byte chunks (D = 128), or two of 64 bytes, with two rows
  // sharing the 256 bytes of all banks (D = 64)
  __device__ static constexpr int vswz(int r) { return D == 128 ? (r & 7) : ((r >> 1) & 1); }
};

// Global byte offset that lane `lane` of the i-th load of loading wave lw fetches, less the 1024 i
// of the instruction's immediate: LDS slot 64 i + lane of the wave's quarter of the tile holds
// slot s ^ kswz(row) of its row (K) or part w of chunk pc ^ vswz(row) (V).
template <int D, bool V>
__device__ inline uint32_t slot_offset(int lw, int i, int lane) {
  using T = Tile<D>;
  const int slot = 64 * i + lane;
  const int row = slot / T::SLOTS, sp = slot % T::SLOTS;
  constexpr int CS = Mma<D>::MR / 8;           // slots of a V chunk
  const int src = V ? ((sp / CS) ^ T::vswz(row)) * CS + sp % CS : (sp ^ T::kswz(row));
  return (uint32_t)(lw * (T::BYTES / 4) + row * T::STRIDE + src * 16 - 1024 * i);
}

// This wave's quarter of one tile of K or V (base: the tensor): a buffer descriptor that starts at
// the tile and ends at its head's Lk (rows past Lk read as zero; nrec 0 reads nothing).  The
// immediate offset of a load counts for both its addresses, so one LDS base (M0) serves all of
// them.  Written as one asm statement (the loads return nothing to registers): for the builtin the
// compiler waits for every load in flight before LDS reads whose stage it cannot tell apart.  M0 is
// an operand, so that the compiler writes it and knows what it holds.  The s_nop covers M0 and a
// descriptor word written just before by a VALU instruction (v_readlane).
template <int D>
__device__ __forceinline__ void issue_tile(unsigned char* dst, const uint16_t* base, uint64_t off, uint32_t nrec,
                                           const uint32_t* lane_off) {
  const uint64_t b = (uint64_t)(uintptr_t)base + off;
  const u32x4 rsrc = u32x4{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, nrec, 0x00020000u};
  const uint32_t m0 = (uint32_t)(uintptr_t)(LDS_AS unsigned char*)dst;
  if constexpr (Tile<D>::PER == 4)
    asm volatile("s_nop 4\n\t"
                 "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
                 ::"{m0}"(m0), "v"(lane_off[0]), "v"(lane_off[1]), "v"(lane_off[2]), "v"(lane_off[3]), "s"(rsrc)
                 : "memory");
  else
    asm volatile("s_nop 4\n\t"
                 "buffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds"
                 ::"{m0}"(m0), "v"(lane_off[0]), "v"(lane_off[1]), "s"(rsrc)
                 : "memory");
}

struct Geom {
  int Lq, Lk, block, NQ, NK, F, chunk0;
  int BH, U;          // heads and units of the plan (bounds for the fields read from it)
};

// Frame-causal chunks (F > 0): first key that query row t does not see, the end of its chunk frame.
// (One 32-bit division; with 64-bit ones the planner took 0.1 to 0.2 us more.)
__device__ __forceinline__ int row_key_limit(int t, int Lk, int F, int chunk0) {
  return (int)min((int64_t)Lk, (int64_t)chunk0 + (int64_t)((uint32_t)t / (uint32_t)F + 1u) * F);
}

// Per-wave constants of the tile loop (klimit changes with the unit).
struct WaveCtx {
  int klimit[2];             // keys >= klimit[qt] are invisible to this lane's query row of column qt
  int kbase, vbase;          // LDS read bases of this lane inside a K / V tile
  int g4;                    // 4 (lane / MR)
  float scale_log2;
};

// Scheduling-group masks of __builtin_amdgcn_sched_group_barrier.
constexpr int kSgMfma = 0x008;
constexpr int kSgDsRead = 0x100;

// S^T = K Q^T for one 64-key tile: accumulators [MR keys][MR queries].  The K operand reads run
// AHEAD operands ahead of their use, so LDS latency overlaps the matrix pipeline.
template <int D>
__device__ __forceinline__ void qk_tile(const unsigned char* __restrict__ kb,
                                        const bf16x8 (*qreg)[Mma<D>::QT],
                                        typename Mma<D>::Acc (*sacc)[Mma<D>::QT], int kbase) {
  using X = Mma<D>;
  constexpr int NT = KT / X::MR;                   // key groups
  constexpr int NO = NT * (D / X::KC);             // K operands per tile
  constexpr int AHEAD = X::MR == 16 ? 6 : 4;
  bf16x8 ka[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i)
    ka[i] = *(const bf16x8*)(kb + (kbase ^ (16 * X::NG * (i / NT))) + (i % NT) * X::MR * Tile<D>::STRIDE);
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int qt = 0; qt < X::QT; ++qt)
#pragma unroll
      for (int i = 0; i < X::AR; ++i) sacc[kt][qt][i] = 0.f;
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int qt = 0; qt < X::QT; ++qt) sacc[i % NT][qt] = X::mma(ka[i], qreg[i / NT][qt], sacc[i % NT][qt]);
  __builtin_amdgcn_sched_group_barrier(kSgDsRead, AHEAD, 0);
#pragma unroll
  for (int i = 0; i < NO - AHEAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(kSgMfma, X::QT, 0);
    __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(kSgMfma, X::QT * AHEAD, 0);
}

// O^T += V^T P^T for one 64-key tile (P: B operands [step of KC keys][MR queries]).  Slot e of lane
// group g of a step's contraction index is key 4 g + e (e < 4) or KC/2 + 4 g + e - 4 of the step,
// which is how the S accumulators lie; the two transpose reads of a V^T operand follow it.  They
// run AHEAD operands ahead of their use.
template <int D>
__device__ __forceinline__ void pv_tile(const unsigned char* __restrict__ vb, const bf16x8 (*pb)[Mma<D>::QT],
                                        typename Mma<D>::Acc (*oacc)[Mma<D>::QT], int vbase) {
  using X = Mma<D>;
  constexpr int DT = D / X::MR;
  constexpr int NO = (KT / X::KC) * DT;            // V^T operands per tile
  constexpr int AHEAD = X::MR == 16 ? 3 : 2;
  bf16x8 va[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const unsigned char* vp = vb + (vbase ^ (2 * X::MR * (i % DT))) + (X::KC * (i / DT)) * Tile<D>::STRIDE;
    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS v4i16*)(vp));
    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS v4i16*)(vp + X::KC / 2 * Tile<D>::STRIDE));
    const v8i16 a8 = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    va[i] = __builtin_bit_cast(bf16x8, a8);
  }
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int qt = 0; qt < X::QT; ++qt) oacc[i % DT][qt] = X::mma(va[i], pb[i / DT][qt], oacc[i % DT][qt]);
  __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2 * AHEAD, 0);
#pragma unroll
  for (int i = 0; i < NO - AHEAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(kSgMfma, X::QT, 0);
    __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2, 0);
  }
  __builtin_amdgcn_sched_group_barrier(kSgMfma, X::QT * AHEAD, 0);
}

// Masks of one tile (ragged tail, frame-causal pairs, padding at the end of the tile): invisible
// keys get -inf.  Lane holds keys key0 + MR kt + acc_row(i) + 4 (l / MR) of its query rows
// MR qt + l % MR; the NG lanes of one l % MR together hold a row's 64 keys.  The record's flag says
// that some row of the unit needs a mask; in a unit of several frames most waves do not (without
// the test the 78-of-1560 case of plan_union_kernel takes 564 instead of 515 us).
template <int D>
__device__ __forceinline__ void mask_tile(typename Mma<D>::Acc (*sacc)[Mma<D>::QT], int key0, int fl,
                                          const WaveCtx& w) {
  using X = Mma<D>;
  const int pad = (fl >> kFlPadShift) & 127;
  int vis[X::QT];                    // visible keys at the front of the tile
  bool need = false;
#pragma unroll
  for (int qt = 0; qt < X::QT; ++qt) {
    vis[qt] = min(w.klimit[qt] - key0, KT - pad);
    need = need || vis[qt] < KT;
  }
  if (!__any(need)) return;
#pragma unroll
  for (int qt = 0; qt < X::QT; ++qt) {
    const int lim = vis[qt] - w.g4;
#pragma unroll
    for (int kt = 0; kt < KT / X::MR; ++kt)
#pragma unroll
      for (int i = 0; i < X::AR; ++i)
        if (X::MR * kt + X::acc_row(i) >= lim) sacc[kt][qt][i] = -INFINITY;
  }
}

// P = 2^(S*scale - m) of the query column qt rounded to bf16 into the B operands of the P.V
// product; returns the sum of the lane's values (fp32, before rounding).
template <int D>
__device__ __forceinline__ float softmax_exp(const typename Mma<D>::Acc (*sacc)[Mma<D>::QT],
                                             bf16x8 (*pb)[Mma<D>::QT], int qt, float m_use, float scale_log2) {
  using X = Mma<D>;
  float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
  for (int s = 0; s < KT / X::KC; ++s) {
    u32x4 pw;
#pragma unroll
    for (int j2 = 0; j2 < 4; ++j2) {
      const int e = 8 * s + 2 * j2;
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[e / X::AR][qt][e % X::AR], scale_log2, -m_use));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[e / X::AR][qt][e % X::AR + 1], scale_log2, -m_use));
      pw[j2] = pack_bf16x2(p0, p1);
      rs0 += p0;
      rs1 += p1;
    }
    pb[s][qt] = __builtin_bit_cast(bf16x8, pw);
  }
  return rs0 + rs1;
}

// Max over the NG lanes that hold a query row's keys.
template <int D>
__device__ __forceinline__ float row_max(float x) {
  if constexpr (Mma<D>::NG == 4) {
    const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x),
                                                    false, false);
    x = fmaxf(__builtin_bit_cast(float, (uint32_t)s[0]), __builtin_bit_cast(float, (uint32_t)s[1]));
  }
  const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x),
                                                  false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)s[0]), __builtin_bit_cast(float, (uint32_t)s[1]));
}

// Softmax of one tile with a lazily raised running max (base 2).  P is first formed against the
// current max m_run, which is left alone while every sum of a row's values over half of the tile's
// keys stays within 2^8 (so no value exceeds 2^8 and the O accumulators keep their range); otherwise
// the row max of the tile is taken, m_run raised to it, O and l rescaled, and P formed again.  Most
// tiles thus skip both the row max and the rescale.  On the first tile of a piece m_run is -inf: the
// first pass then gives inf or NaN sums, which fail the test too.
// A raised max makes the largest P exactly 1, with no rounding to bf16, so the limit matters to the
// precision: with 2^8 over a lane's 16 values alone (d = 128) the error against 64 bits was up to
// 0.15 % larger, 0.0023393 instead of 0.0023358 at 720P.  A lane tests its own values first, at half
// the limit where it holds a quarter of the keys; the sums of the halves are taken where that fails
// (in every tile they cost 2 % of the call).
template <int D>
__device__ __forceinline__ void softmax_tile(typename Mma<D>::Acc (*sacc)[Mma<D>::QT], bf16x8 (*pb)[Mma<D>::QT],
                                             typename Mma<D>::Acc (*oacc)[Mma<D>::QT], float* m_run, float* l_run,
                                             float scale_log2) {
  using X = Mma<D>;
  float rs[X::QT];
  bool over = false;
#pragma unroll
  for (int qt = 0; qt < X::QT; ++qt) {
    rs[qt] = softmax_exp<D>(sacc, pb, qt, m_run[qt], scale_log2);
    over = over || !(rs[qt] <= (X::NG == 4 ? 128.f : 256.f));
  }
  if (__builtin_expect(__any(over), 0)) {
    if constexpr (X::NG == 4) {
      over = false;
#pragma unroll
      for (int qt = 0; qt < X::QT; ++qt) {
        const uint32_t r = __builtin_bit_cast(uint32_t, rs[qt]);
        const auto h = __builtin_amdgcn_permlane32_swap(r, r, false, false);      // lanes l and l ^ 32
        over = over || !(__builtin_bit_cast(float, (uint32_t)h[0]) + __builtin_bit_cast(float, (uint32_t)h[1]) <= 256.f);
      }
    }
    if (X::NG == 2 || __any(over)) {
#pragma unroll
      for (int qt = 0; qt < X::QT; ++qt) {
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < KT / X::MR; ++kt)
#pragma unroll
          for (int i = 0; i < X::AR; ++i) mx = fmaxf(mx, sacc[kt][qt][i]);
        const float mt = row_max<D>(mx) * scale_log2;
        if (mt > m_run[qt]) {
          const float alpha = __builtin_amdgcn_exp2f(m_run[qt] - mt);   // 0 while m_run is -inf
          m_run[qt] = mt;
          l_run[qt] *= alpha;
#pragma unroll
          for (int dt = 0; dt < D / X::MR; ++dt) oacc[dt][qt] *= alpha;
        }
        rs[qt] = softmax_exp<D>(sacc, pb, qt, m_run[qt] == -INFINITY ? 0.f : m_run[qt], scale_log2);
      }
    }
  }
#pragma unroll
  for (int qt = 0; qt < X::QT; ++qt) l_run[qt] += rs[qt];
}

// ---------------------------------------------------------------------------
// Work plan.  The query blocks of each (batch, head) bh are ordered by the first historical key
// block they keep and cut into groups of NL = 256 / block: unit u = (bh, g) holds query blocks
// qmap[u NL + L], L < NL (-1 past the last block).  Its tiles are the 64-key sub-tiles of the
// union of its lists in ascending block order, leaving out sub-tiles without a visible key (past
// Lk, or past the block's valid count); ulist[u NK (block / 64) + i] = block << 5 | sub-tile << 4
// | ownership bits (bit L: list L keeps the block), ucount[u] = sub-tiles.  The unit's tiles
// number max(1, ucount[u]): an empty unit gets one unowned tile, so that some workgroup writes
// its output.  The grouping only decides which rows share K/V tiles: any grouping gives the same
// result.

constexpr int kPlanThreads = 256;
constexpr int kMaxGroupNQ = 1024;   // heads with more query blocks keep the natural order

__device__ inline int block_excl_scan_i(int x, int* sh, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int incl = (int)wave_incl_scan((uint32_t)x);
  __syncthreads();
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  int base = 0, tot = 0;
  for (int wv = 0; wv < (int)(blockDim.x >> 6); ++wv) {
    if (wv < wave) base += sh[wv];
    tot += sh[wv];
  }
  *total = tot;
  return base + incl - x;
}

// 64-key sub-tiles of key block j that hold a visible key: the block's keys below Lk and, with
// kvalid, its first kvalid[j] keys (clamped to [0, block]); sub-tiles with none are left out of
// the plan (they would contribute nothing but masked MFMA work).
__device__ inline int block_subtiles(int j, int Lk, int block, const int32_t* __restrict__ kvalid) {
  int v = min(block, Lk - j * block);
  if (kvalid) v = min(v, min(max(kvalid[j], 0), block));
  return (v + KT - 1) / KT;
}

// Frame-causal chunks: first key that no row of query block qb sees (Lk without frames).  Keys from
// there on belong to frames later than the block's last row's.
__device__ inline int block_key_limit(int qb, int Lq, int Lk, int block, int F, int chunk0) {
  if (F <= 0) return Lk;
  return row_key_limit(min(Lq, (qb + 1) * block) - 1, Lk, F, chunk0);
}

// One workgroup per unit: its query blocks (rank by (key, block index) inside the head) and the
// union of their lists with ownership bits, expanded into the sub-tiles that hold visible keys.
// With frames inside the chunk a list owns a sub-tile only when some row of its query block sees
// it (block_key_limit).  The frames a query block cannot see are the later part of the chunk, 3/8
// of it with four frames, and a fully masked tile takes as long as a visible one: 24 heads, 14400
// queries in four frames, 117 of 563 blocks of 128 kept: 329508 -> 222102 tiles, 2658 -> 1777 us for
// the whole call with the attention loop of the time (1540 with the present one on the same card).
// The grouping key of a query block is its entry h0 (the first past the text blocks of an ascending
// list, as the selection writes them), or the first entry past the text blocks when entry h0 is
// none, when that is historical (below h1), NK otherwise.  Any other list order only changes the
// grouping.
// With frames, the blocks of one frame come first and the key decides inside a frame, unless the
// lists keep many historical blocks (frames_first below).  A unit of one frame walks no tile of a
// later one: on average 1 - (frames + 1) / (2 frames) of the chunk's blocks less than all of them.
// But a unit ordered by the key alone shares historical blocks, at the most NL - 1 of every block's
// own.  Frames come first where that is the smaller of the two, with a fifth added for partial
// frames and units, so that a plan walks no more tiles than one ordered by the key that walks the
// whole chunk.  Measured, whole calls: 16 heads, 6240 queries in four frames, 78 of 1560 historical
// blocks of 64 kept: 143990 tiles and 735 us by frames, 75891 and 511 us by the key.  24 heads,
// 14400 queries in four frames, 5 of 450 blocks of 128: 222102 tiles by frames, about 279000 by the
// key.
__global__ __launch_bounds__(kPlanThreads) void plan_union_kernel(const int32_t* __restrict__ counts,
                                                                  const int32_t* __restrict__ idx,
                                                                  const int32_t* __restrict__ kvalid, int NQ, int NK,
                                                                  int h0, int h1, int Lq, int Lk, int block, int F,
                                                                  int chunk0, int row_tiles,
                                                                  int32_t* __restrict__ qmap,
                                                                  int32_t* __restrict__ ulist,
                                                                  int32_t* __restrict__ ucount) {
  extern __shared__ __align__(16) uint32_t own[];     // 4 ownership bits per key block
  __shared__ int sh[kPlanThreads / 64];
  __shared__ int qsel[4];
  __shared__ int4 slim;               // block_key_limit of the unit's query blocks
  __shared__ __attribute__((aligned(16))) uint64_t skey[kMaxGroupNQ + 2];
  __shared__ int rank[kMaxGroupNQ];
  const int u = blockIdx.x;
  const int bh = u / row_tiles, g = u % row_tiles;
  const int tid = threadIdx.x;
  const int NL = QR / block;
  const int nsub = block / KT;
  const int nwords = (NK + 7) >> 3;
  for (int i = tid; i < nwords; i += kPlanThreads) own[i] = 0;
  if (tid < 4) qsel[tid] = -1;
  const bool grouped = NQ <= kMaxGroupNQ;
  const bool choose = grouped && F > 0 && F < Lq && NQ > NL;      // the order makes a difference
  int nhist = 0;                      // historical entries of this thread's lists (if choose)
  if (grouped)
    for (int i = tid; i < NQ; i += kPlanThreads) {
      const size_t row = (size_t)bh * NQ + i;
      const int32_t* lst = idx + row * NK;
      const int first = lst[min(h0, NK - 1)];      // loaded beside the count, not after it
      const int n = min(max(counts[row], 0), NK);
      int key = NK;
      if (n > h0 && first >= h0) {
        key = first < h1 ? first : NK;
      } else {
        for (int a = 0; a < n; ++a) {
          const int j = lst[a];
          if (j >= h0) {
            key = j < h1 ? j : NK;
            break;
          }
        }
      }
      // blocks of one frame first: the length of the visible chunk differs by whole frames; then the
      // key, then the block (NK, the block count of the limit and i are below 2^15, 2^15 and 2^10)
      const int lim = F > 0 ? ceil_div(block_key_limit(i, Lq, Lk, block, F, chunk0), block) : 0;
      skey[i] = ((uint64_t)lim << 32) | ((uint64_t)key << 16) | (uint64_t)i;
      rank[i] = 0;
      if (choose) {
        // of an ascending list that keeps the whole chunk, what lies before it, less the text blocks
        // when it keeps them; of any other list, all entries (more than there may be)
        const int tail = NK - h1;
        const bool chunk = tail > 0 && n >= tail && lst[n - tail] == h1;
        const bool text = n >= h0 && lst[max(h0 - 1, 0)] == h0 - 1;
        nhist += max(0, n - (chunk ? tail : 0) - (text ? h0 : 0));
      }
    }
  if (grouped && tid < 2) skey[NQ + tid] = ~0ull;      // padding of the pairs read below
  if (choose) {
    int hist;
    block_excl_scan_i(nhist, sh, &hist);
    const int64_t frames = ceil_div(Lq, F);
    const bool frames_first = 6 * (int64_t)(NL - 1) * hist * 2 * frames < 5 * (int64_t)NQ * NQ * (frames - 1);
    if (!frames_first)
      for (int i = tid; i < NQ; i += kPlanThreads) skey[i] = (uint32_t)skey[i];
  }
  __syncthreads();
  if (grouped) {
    // rank of every block among its head's keys, all different; the pairs of keys are counted by
    // kPlanThreads / (blocks rounded up to waves) threads per block (one thread per block and one
    // key per LDS read: a longer serial chain)
    const int rows = (NQ + 63) & ~63, parts = rows < kPlanThreads ? kPlanThreads / rows : 1;
    const int pairs = (NQ + 1) >> 1, per = (pairs + parts - 1) / parts;
    const ulonglong2* kp = (const ulonglong2*)skey;
    for (int e = tid; e < rows * parts; e += kPlanThreads) {
      const int i = e % rows, p0 = (e / rows) * per, p1 = min(p0 + per, pairs);
      if (i < NQ) {
        const uint64_t ki = skey[i];
        int r = 0;
#pragma unroll 8
        for (int j = p0; j < p1; ++j) {
          const ulonglong2 k2 = kp[j];
          r += (k2.x < ki) + (k2.y < ki);
        }
        if (parts == 1) rank[i] = r;
        else atomicAdd(&rank[i], r);
      }
    }
    __syncthreads();
    for (int i = tid; i < NQ; i += kPlanThreads) {
      const int r = rank[i];
      if (r >= g * NL && r < g * NL + NL) qsel[r - g * NL] = i;
    }
  } else if (tid < NL && g * NL + tid < NQ) {
    qsel[tid] = g * NL + tid;
  }
  __syncthreads();
  if (tid < NL) {
    qmap[(size_t)u * NL + tid] = qsel[tid];
    if (F > 0) ((int*)&slim)[tid] = block_key_limit(max(qsel[tid], 0), Lq, Lk, block, F, chunk0);
  }
  // all lists of the unit at once, kPlanThreads / NL threads each (one after another, every list
  // cost two more dependent loads; with the ranking above 10.4 -> 9.1 us at 400 units of four lists)
  {
    const int tpl = kPlanThreads / NL, L = tid / tpl;
    const int qb = qsel[L];
    if (qb >= 0) {
      const size_t row = (size_t)bh * NQ + qb;
      const int n = min(max(counts[row], 0), NK);
      const int32_t* lst = idx + row * NK;
      for (int i = tid % tpl; i < n; i += tpl) {
        const int j = lst[i];
        if ((unsigned)j < (unsigned)NK) atomicOr(&own[j >> 3], (1u << L) << ((j & 7) * 4));
      }
    }
  }
  __syncthreads();
  const int4 lim4 = slim;
  // the ownership bits of word wi (8 key blocks) whose lists see sub-tile `sub` of their block: with
  // frames, list L sees the first ones of the word (every sub-tile tested against every limit in LDS:
  // 15.3 instead of 10.8 us of planning for 16 heads, 64 queries, 4096 keys in blocks of 128, and of 10
  // without frames)
  auto seen = [&](uint32_t x, int wi, int sub) {
    uint32_t m = 0;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
      const int lim = L == 0 ? lim4.x : L == 1 ? lim4.y : L == 2 ? lim4.z : lim4.w;
      const int nv = min(max(lim - 8 * wi * block, 0), 8 * block);            // keys of the word it sees
      const int nb = ((nv + KT - 1) / KT - sub + nsub - 1) >> (nsub - 1);     // blocks
      m |= (nb >= 8 ? ~0u : (1u << (4 * nb)) - 1) & (0x11111111u << L);
    }
    return x & m;
  };
  const int per = (nwords + kPlanThreads - 1) / kPlanThreads;
  const int w0 = min(tid * per, nwords), w1 = min(w0 + per, nwords);
  // f(key block, sub-tile, owning lists) for every sub-tile of this thread's words
  auto subtiles = [&](auto f) {
    for (int wi = w0; wi < w1; ++wi) {
      const uint32_t x = own[wi];
      if (!x) continue;
      const uint32_t x0 = F > 0 ? seen(x, wi, 0) : x, x1 = F > 0 && nsub > 1 ? seen(x, wi, 1) : x;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t b0 = (x0 >> (4 * e)) & 15u, b1 = (x1 >> (4 * e)) & 15u;
        if (!b0) continue;                       // the first sub-tile is seen if the second is
        const int j = 8 * wi + e;
        const int ns = block_subtiles(j, Lk, block, kvalid);
        if (ns > 0) f(j, 0, b0);
        if (ns > 1 && b1) f(j, 1, b1);
      }
    }
  };
  int cnt = 0;
  auto count = [&](int, int, uint32_t) { ++cnt; };
  subtiles(count);
  int total;
  int pos = block_excl_scan_i(cnt, sh, &total);
  int32_t* out = ulist + (size_t)u * NK * nsub;
  auto emit = [&](int j, int sub, uint32_t b) { out[pos++] = (j << 5) | (sub << 4) | (int)b; };
  subtiles(emit);
  if (tid == 0) ucount[u] = total;
}

// Where every unit's tiles go in the tile sequence, and which tiles each persistent workgroup
// takes.  Units are handed out in two parts:
//   * rounds of whole units: round r gives workgroup lambda = x PX + c (x its XCD, PX = P / 8
//     workgroups per XCD) the unit x R PX + r PX + c, for r < R, unless that unit is longer than
//     thr = T / (P R) tiles.  The workgroups of one XCD thus start consecutive units, i.e. query
//     blocks of the same head, at the same time and walk the head's shared chunk K/V in step,
//     so each K/V tile reaches that XCD's L2 about once per round instead of once per unit.  A
//     workgroup's round units sit one after another at dp_start[lambda] .. dp_start[lambda + 1];
//     by the length limit they add up to at most T / P tiles.
//   * the other units (those past R P and the longer ones), concatenated in unit order after
//     all round units, are shared by stream-K: workgroup lambda takes [sk_start[lambda],
//     sk_start[lambda + 1]), sized so that its round tiles plus this share come as close as
//     possible to T / P.  Units cut at these boundaries are merged afterwards.
// R = (U - P / 4) / P leaves at least P / 4 units to the second part (when U >= P / 4), which
// absorbs the differences in unit length.  tstart[u] = first tile of unit u; tstart[U] = T.
// Computed by one whole workgroup of kPlanThreads >= P threads (sh: its scan scratch); with
// `all` it writes tstart, dp_start and sk_start, and in any case the placing thread writes the
// first tile of unit `me` to *me_start (read after the workgroup's next barrier).
__device__ void schedule_units(const int32_t* __restrict__ ucount, int U, int P, int me, bool all,
                               int32_t* __restrict__ tstart, int32_t* __restrict__ dp_start,
                               int32_t* __restrict__ sk_start, int* sh, int* me_start) {
  const int tid = threadIdx.x;
  const int PX = P >> 3;
  const int R = U > P / 4 ? (U - P / 4) / P : 0;
  const int U1 = R * P;                       // units considered for the rounds
  auto tiles = [&](int u) { return max(1, ucount[u]); };
  auto round_unit = [&](int lambda, int r) { return (lambda / PX) * R * PX + r * PX + lambda % PX; };
  // each thread takes a contiguous run of units, so its loads are independent of each other
  const int C = (U + kPlanThreads - 1) / kPlanThreads;
  const int u_lo = min(U, tid * C), u_hi = min(U, u_lo + C);
  int part = 0;
  for (int u = u_lo; u < u_hi; ++u) part += tiles(u);
  int T;
  block_excl_scan_i(part, sh, &T);
  const int thr = R > 0 ? max(1, (int)((int64_t)T / ((int64_t)P * R))) : 0;
  auto in_rounds = [&](int u) { return u < U1 && tiles(u) <= thr; };
  // round tiles of workgroup tid
  int dp = 0;
  if (tid < P)
#pragma unroll 4
    for (int r = 0; r < R; ++r) {
      const int u = round_unit(tid, r);
      if (in_rounds(u)) dp += tiles(u);
    }
  int Tdp;
  const int dpa = block_excl_scan_i(dp, sh, &Tdp);
  if (tid < P) {
    if (all) dp_start[tid] = dpa;
    int pos = dpa;
    for (int r = 0; r < R; ++r) {
      const int u = round_unit(tid, r);
      if (in_rounds(u)) {
        if (all) tstart[u] = pos;
        if (u == me) *me_start = pos;
        pos += tiles(u);
      }
    }
  }
  if (all && tid == 0) dp_start[P] = Tdp;
  // units of the second part, in unit order after the round units
  int skp = 0;
  for (int u = u_lo; u < u_hi; ++u)
    if (!in_rounds(u)) skp += tiles(u);
  int Tsk_sum;
  int pos = Tdp + block_excl_scan_i(skp, sh, &Tsk_sum);
  for (int u = u_lo; u < u_hi; ++u)
    if (!in_rounds(u)) {
      if (all) tstart[u] = pos;
      if (u == me) *me_start = pos;
      pos += tiles(u);
    }
  if (!all) return;
  const int Tsk = T - Tdp;
  if (tid == 0) tstart[U] = T;
  // second-part shares: quota q = max(0, ceil(T / P) - round tiles), scaled to the Tsk tiles
  // (sum q >= P ceil(T / P) - Tdp >= Tsk, so no share exceeds its quota)
  const int q = tid < P ? max(0, (int)(((int64_t)T + P - 1) / P) - dp) : 0;
  int Q;
  const int qa = block_excl_scan_i(q, sh, &Q);
  if (tid < P) sk_start[tid] = Tdp + (Q > 0 ? (int)((int64_t)Tsk * qa / Q) : 0);
  if (tid == 0) sk_start[P] = T;
}

// The schedule (above) as a launch of its own: one workgroup writes tstart, dp_start, sk_start.
__global__ __launch_bounds__(kPlanThreads) void plan_sched_kernel(const int32_t* __restrict__ ucount, int U, int P,
                                                                  int32_t* __restrict__ tstart,
                                                                  int32_t* __restrict__ dp_start,
                                                                  int32_t* __restrict__ sk_start) {
  __shared__ int sh[kPlanThreads / 64];
  __shared__ int unused;
  schedule_units(ucount, U, P, -1, true, tstart, dp_start, sk_start, sh, &unused);
}

// Units up to which every workgroup of plan_tiles_kernel computes the schedule itself (each reads
// all U unit counts, U^2 reads in all) instead of a launch of plan_sched_kernel before it.
constexpr int kFoldSchedUnits = 1024;

// Expands unit u's union list into one record per 64-key tile at its place in the tile
// sequence.  With fold, every workgroup computes the schedule (above) for its own unit and
// workgroup 0 also writes tstart, dp_start and sk_start for the run and the merge; otherwise the
// place is read from tstart, written by plan_sched_kernel.  With kvalid (valid keys at the front
// of each key block), a tile's padding keys are counted into its flags.
__global__ __launch_bounds__(kPlanThreads) void plan_tiles_kernel(const int32_t* __restrict__ ulist,
                                                                  const int32_t* __restrict__ ucount,
                                                                  const int32_t* __restrict__ kvalid, int U,
                                                                  int P, bool fold, int32_t* __restrict__ tstart,
                                                                  int32_t* __restrict__ dp_start,
                                                                  int32_t* __restrict__ sk_start, int NK,
                                                                  int Lk, int F, int chunk0,
                                                                  const int32_t* __restrict__ qmap, int block,
                                                                  int row_tiles, int4* __restrict__ trec) {
  __shared__ int sh[kPlanThreads / 64];
  __shared__ int first_tile;
  const int u = blockIdx.x;
  const int tid = threadIdx.x;
  if (fold) {
    if (tid == 0) first_tile = 0;
    schedule_units(ucount, U, P, u, u == 0, tstart, dp_start, sk_start, sh, &first_tile);
  } else if (tid == 0) {
    first_tile = tstart[u];
  }
  __syncthreads();
  const int nt = ucount[u], n = nt > 0 ? nt : 1;
  const int nsub = block / KT;
  const int bh = u / row_tiles;
  int4* out = trec + first_tile;
  // a tile that ends past the first key some row of the unit does not see needs the mask test
  int maskfrom = Lk;
  if (F > 0)
    for (int L = 0; L < QR / block; ++L) {
      const int qb = qmap[(size_t)u * (QR / block) + L];
      if (qb >= 0) maskfrom = min(maskfrom, row_key_limit(qb * block, Lk, F, chunk0));
    }
  const int32_t* ul = ulist + (size_t)u * NK * nsub;
  for (int a = tid; a < n; a += kPlanThreads) {
    int key0 = 0, bits = 0;
    if (nt > 0) {
      const int e = ul[a];
      const int j = e >> 5, sub = (e >> 4) & 1;
      key0 = j * block + sub * KT;
      bits = e & 15;
      if (kvalid) {
        const int kv = min(max(kvalid[j], 0), block) - sub * KT;
        bits |= (KT - min(max(kv, 0), KT)) << kFlPadShift;
      }
    }
    if (key0 + KT > maskfrom || (bits >> kFlPadShift)) bits |= kFlMask;
    out[a] = int4{key0, bh, u, bits | (a == 0 ? kFlFrom0 : 0) | (a == n - 1 ? kFlToEnd | kFlLast : 0)};
  }
}

// The tiles of one workgroup: n1 round tiles from a1, then its stream-K share from a2; its tile
// t (0 <= t < N) is tile at(t) of the sequence.
struct WgTiles {
  int a1, n1, a2, N;
  int Lk, BH, U;          // bounds of a record's first key, head and unit
  __device__ int at(int t) const { return t < n1 ? a1 + t : a2 + (t - n1); }
};

// One tile of a workgroup's work (wave-uniform).  Its record: x = first key, y = (batch, head),
// z = unit, w = ownership bits (0..3) | from0 | to_end and last (the unit's first / last tile) |
// mask (some key of it may be invisible to some row) | valid | padding; last is also set on the
// last tile of the workgroup.  fl is 0 past the end.
struct TileRef {
  int fl, key0;
};

// The record of the workgroup's tile t, read through the constant address space: the records
// are written by an earlier kernel and never during this one, so the loads can go through the
// scalar cache (s_load).  t is clamped to the last tile (N > 0).
typedef __attribute__((address_space(4))) const int cint32;
__device__ inline int4 load_tile(const int4* __restrict__ trec, int t, const WgTiles& g) {
  const cint32* r = (const cint32*)(trec + g.at(t < g.N ? t : g.N - 1));
  return int4{r[0], r[1], r[2], r[3]};
}

// The fields are clamped into range, so that even a plan the workspace no longer holds
// (overwritten by another call) reads and writes inside q, k, v, o and the workspace.
__device__ __forceinline__ TileRef decode_tile(const int4& e, int t, const WgTiles& g) {
  TileRef r;
  r.key0 = (int)min((uint32_t)e.x, (uint32_t)g.Lk);
  r.fl = t < g.N ? e.w | kFlValid | (t + 1 == g.N ? kFlLast : 0) : 0;
  return r;
}

// State of one wave's running unit piece.
template <int D>
struct WaveState {
  using X = Mma<D>;
  // [..][qt]: the wave's query rows MR qt .. MR qt + MR - 1
  typename X::Acc oacc[D / X::MR][X::QT];
  typename X::Acc sacc[KT / X::MR][X::QT];
  bf16x8 pb[KT / X::KC][X::QT];
  bf16x8 qreg[D / X::KC][X::QT];
  float m_run[X::QT], l_run[X::QT];
  int own;          // ownership bit of the wave's list, 0 when the wave's rows do not exist
  bool from0;       // the running piece starts at its unit's first tile
  int unit;
  int r0w;          // first query row of the wave in its (batch, head)
  int bh;
};

// Shared arguments of the phases.
struct KArgs {
  const uint16_t* q;
  uint16_t* o;
  float* lse;
  float* part_o;
  float* part_m;
  float* part_l;
  int32_t* cut;
  const int32_t* qmap;
  Geom gm;
  int lambda;
  int my_list;      // list of the unit (query block) the wave's rows belong to
  int r_sub;        // first row of the wave inside its query block
  int r_off;        // first row of the wave inside the unit: my_list * block + r_sub
  int c, g;         // lane % MR, lane / MR
};

// Starts a piece of the unit of tile t: zero O, reset the running max and sum, load the wave's
// Q rows.
template <int D>
__device__ __forceinline__ void start_piece(WaveState<D>& st, WaveCtx& w, const int4& e, const KArgs& ka) {
  using X = Mma<D>;
  const Geom& gm = ka.gm;
  st.bh = (int)min((uint32_t)e.y, (uint32_t)(gm.BH - 1));
  st.unit = (int)min((uint32_t)e.z, (uint32_t)(gm.U - 1));
  const int qb = ka.qmap[(size_t)st.unit * (QR / gm.block) + ka.my_list];
  st.r0w = __builtin_amdgcn_readfirstlane(qb >= 0 && qb < gm.NQ ? qb * gm.block + ka.r_sub : gm.Lq);
  st.own = st.r0w < gm.Lq ? 1 << ka.my_list : 0;
  st.from0 = e.w & kFlFrom0;
#pragma unroll
  for (int qt = 0; qt < X::QT; ++qt) {
    st.m_run[qt] = -INFINITY;
    st.l_run[qt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < D / X::MR; ++dt)
#pragma unroll
      for (int i = 0; i < X::AR; ++i) st.oacc[dt][qt][i] = 0.f;
    // Q^T operand: lane holds Q[row r0w + MR qt + l % MR][KC ks + 8 (l / MR) .. + 7]
    const int row = st.r0w + X::MR * qt + ka.c;
#pragma unroll
    for (int ks = 0; ks < D / X::KC; ++ks) {
      u32x4 qw = u32x4{0u, 0u, 0u, 0u};
      if (row < gm.Lq) qw = *(const u32x4*)(ka.q + ((size_t)st.bh * gm.Lq + row) * D + X::KC * ks + 8 * ka.g);
      st.qreg[ks][qt] = __builtin_bit_cast(bf16x8, qw);
    }
    // Key n is visible to query row t when n < Lk and, with frames of F tokens inside the chunk,
    // when its chunk frame is not later than t's: n < chunk0 + (t / F + 1) F (context keys,
    // n < chunk0, always pass).  One limit per lane and row replaces per-key frame arithmetic.
    w.klimit[qt] = gm.F > 0 ? row_key_limit(row, gm.Lk, gm.F, gm.chunk0) : gm.Lk;
  }
  // complete the Q loads here: left pending, they would make every later Q.K^T (reached also
  // without a piece start) wait for all vector memory traffic, the tile loads in flight included
  __builtin_amdgcn_s_waitcnt(0);
}

// Ends a piece: the normalised bf16 output (and lse) when the piece is the whole unit, else the
// fp32 partial (O unnormalised, running max m, sum l) in slot 2 lambda (the first piece of the
// workgroup's stream-K share, which continues an earlier share) or 2 lambda + 1 (its last,
// continued by a later share); cut[slot] names the unit (see CutMap).
// The stores are completed before returning (the tile-load waits count only tile loads).
template <int D>
__device__ __forceinline__ void end_piece(const WaveState<D>& st, bool to_end, const KArgs& ka) {
  using X = Mma<D>;
  const Geom& gm = ka.gm;
  if (!(st.from0 && to_end) && threadIdx.x == 0) ka.cut[2 * ka.lambda + (st.from0 ? 1 : 0)] = st.unit;
#pragma unroll
  for (int qt = 0; qt < X::QT; ++qt) {
    // lane holds O^T[MR dt + acc_row(i) + 4 g][query r0w + MR qt + l % MR]
    float l = st.l_run[qt];
    if constexpr (X::NG == 4) l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const int rw = X::MR * qt + ka.c, qrow = st.r0w + rw;
    if (qrow >= gm.Lq) {
    } else if (st.from0 && to_end) {
      const float inv = l > 0.f ? 1.0f / l : 0.f;
      uint16_t* orow = ka.o + ((size_t)st.bh * gm.Lq + qrow) * D + 4 * ka.g;
#pragma unroll
      for (int dt = 0; dt < D / X::MR; ++dt) {
        const typename X::Acc x = st.oacc[dt][qt] * inv;
#pragma unroll
        for (int i = 0; i < X::AR; i += 4)
          *(u32x2*)(orow + X::MR * dt + X::acc_row(i)) = u32x2{pack_bf16x2(x[i], x[i + 1]), pack_bf16x2(x[i + 2], x[i + 3])};
      }
      if (ka.lse && ka.g == 0)
        ka.lse[(size_t)st.bh * gm.Lq + qrow] = l > 0.f ? (st.m_run[qt] + log2f(l)) * 0.69314718055994531f : -INFINITY;
    } else {
      const int slot = 2 * ka.lambda + (st.from0 ? 1 : 0);
      const size_t prow = (size_t)slot * QR + ka.r_off + rw;
      float* po = ka.part_o + prow * D + 4 * ka.g;
#pragma unroll
      for (int dt = 0; dt < D / X::MR; ++dt) {
        const typename X::Acc x = st.oacc[dt][qt];
#pragma unroll
        for (int i = 0; i < X::AR; i += 4)
          *(f32x4*)(po + X::MR * dt + X::acc_row(i)) = f32x4{x[i], x[i + 1], x[i + 2], x[i + 3]};
      }
      if (ka.g == 0) {
        ka.part_m[prow] = st.m_run[qt];
        ka.part_l[prow] = l;
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
}

// M phase of tile t (cur; prev: tile t - 1): P.V of the previous tile, the change of piece after a
// last tile, Q.K^T of this one.
template <int D>
__device__ __forceinline__ void m_phase(WaveState<D>& st, WaveCtx& w, int prev_fl, int cur_fl, int t,
                                        const unsigned char* kcur, const unsigned char* vprev,
                                        const int4* __restrict__ trec, const WgTiles& g, const KArgs& ka) {
  if (prev_fl & st.own) pv_tile<D>(vprev, st.pb, st.oacc, w.vbase);
  if (__builtin_expect(prev_fl & kFlLast, 0)) {
    end_piece<D>(st, prev_fl & kFlToEnd, ka);
    if (cur_fl) start_piece<D>(st, w, load_tile(trec, t, g), ka);
  }
  if (cur_fl & st.own) qk_tile<D>(kcur, st.qreg, st.sacc, w.kbase);
}

// V phase of a tile: masks, softmax, P.
template <int D>
__device__ __forceinline__ void v_phase(WaveState<D>& st, const WaveCtx& w, const TileRef& t) {
  if (t.fl & st.own) {
    if (__builtin_expect(t.fl & kFlMask, 0)) mask_tile<D>(st.sacc, t.key0, t.fl, w);
    softmax_tile<D>(st.sacc, st.pb, st.oacc, st.m_run, st.l_run, w.scale_log2);
  }
}

template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_fwd_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int4* __restrict__ trec, const int32_t* __restrict__ dp_start, const int32_t* __restrict__ sk_start,
    const int32_t* __restrict__ qmap, uint16_t* __restrict__ o, float* __restrict__ lse, float* __restrict__ part_o,
    float* __restrict__ part_m, float* __restrict__ part_l, int32_t* __restrict__ cut, Geom gm, int Tcap,
    float scale_log2) {
  using T = Tile<D>;
  using X = Mma<D>;
  // stages of K, then of V (one array: the lane bases of the V reads include the offset of the V
  // stages, so that every stage is within reach of the 16-bit immediates)
  __shared__ __attribute__((aligned(1024))) unsigned char ring[6 * T::BYTES];

  // XCD-aware numbering: hardware places consecutive workgroup ids on consecutive XCDs (round
  // robin over 8); lambda = x PX + c numbers the workgroups of XCD x consecutively, which is
  // the numbering the plan hands out its units in.  P is a multiple of 8.
  const int P = gridDim.x;
  const int lambda = (blockIdx.x & 7) * (P >> 3) + (blockIdx.x >> 3);
  // the workgroup's tiles, clamped into the record array (Tcap records)
  WgTiles g;
  g.a1 = min(max(dp_start[lambda], 0), Tcap);
  g.n1 = min(max(dp_start[lambda + 1] - g.a1, 0), Tcap - g.a1);
  g.a2 = min(max(sk_start[lambda], 0), Tcap);
  g.N = g.n1 + min(max(sk_start[lambda + 1] - g.a2, 0), Tcap - g.a2);
  g.Lk = gm.Lk;
  g.BH = gm.BH;
  g.U = gm.U;
  if (threadIdx.x == 0) cut[2 * lambda] = cut[2 * lambda + 1] = -1;    // no piece in either slot yet
  if (g.N <= 0) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps tile-issue math scalar
  const bool g1 = wave >= 4;                                    // the lagging group
  const int lw = wave & 3;                                      // wave within its group

  KArgs ka;
  ka.q = q;
  ka.o = o;
  ka.lse = lse;
  ka.part_o = part_o;
  ka.part_m = part_m;
  ka.part_l = part_l;
  ka.cut = cut;
  ka.qmap = qmap;
  ka.gm = gm;
  ka.lambda = lambda;
  ka.c = lane % X::MR;
  ka.g = lane / X::MR;
  // the two waves of SIMD s (s and s + 4) own the two 32-row halves of one 64-row query block,
  // or (128-row blocks) waves {0, 1, 4, 5} and {2, 3, 6, 7} own the two blocks
  if (gm.block == 64) {
    ka.my_list = wave & 3;
    ka.r_sub = (wave >> 2) * QW;
    ka.r_off = ka.my_list * 64 + ka.r_sub;
  } else {
    ka.my_list = (wave & 3) >> 1;
    ka.r_sub = ((wave & 1) * 2 + (wave >> 2)) * QW;
    ka.r_off = ka.my_list * 128 + ka.r_sub;
  }

  WaveCtx w;
  w.kbase = ka.c * T::STRIDE + 16 * (ka.g ^ T::kswz(ka.c));
  {
    const int vrow = 4 * ka.g + ((lane & 15) >> 2);         // + multiples of KC / 2 rows in the immediates
    w.vbase = 3 * T::BYTES + vrow * T::STRIDE + 2 * X::MR * T::vswz(vrow) + (X::MR == 32 ? 2 * (lane & 16) : 0) +
              8 * (lane & 3);
  }
  w.g4 = 4 * ka.g;
  w.scale_log2 = scale_log2;

  WaveState<D> st;
  const int N = g.N;

  // Iteration t (phases A(t), B(t)); tile t lies in stage t % 3.  Group 0 loads K(t+2) in its V
  // phase B(t), group 1 V(t+1) in its V phase A(t); both wait at the end of B(t) for what they
  // issued in the iteration before.  The record of the tile to load is fetched (scalar load) at the
  // start of the V phase and decoded at its end, so that no scalar load is outstanding during an M
  // phase (it would force the LDS operand reads there to wait for all LDS traffic).  Three
  // iterations per trip, so that every stage is a compile-time choice.
  auto run = [&](auto G1) {
    constexpr bool IS_G1 = decltype(G1)::value;
    const uint16_t* const src = IS_G1 ? v : k;
    uint32_t off[T::PER];
#pragma unroll
    for (int i = 0; i < T::PER; ++i) off[i] = slot_offset<D, IS_G1>(lw, i, lane);
    unsigned char* const s0 = ring;
    unsigned char* const s1 = ring + T::BYTES;
    unsigned char* const s2 = ring + 2 * T::BYTES;
    constexpr int VOFF = 3 * T::BYTES;
    auto issue = [&](unsigned char* dst, const int4& e, const TileRef& r) {
      const uint32_t bh = min((uint32_t)e.y, (uint32_t)(g.BH - 1));
      const uint32_t nrec = r.fl ? (uint32_t)(g.Lk - r.key0) * (uint32_t)T::STRIDE : 0u;
      const uint64_t o64 = (uint64_t)bh * ((uint32_t)g.Lk * (uint32_t)T::STRIDE) + (uint32_t)r.key0 * (uint32_t)T::STRIDE;
      issue_tile<D>(dst + lw * (T::BYTES / 4), src, o64, nrec, off);
    };
    TileRef r0, r1, r2;        // tiles t with t % 3 = 0, 1, 2
    {
      const int4 e0 = load_tile(trec, 0, g), e1 = load_tile(trec, 1, g);
      r0 = decode_tile(e0, 0, g);
      r1 = decode_tile(e1, 1, g);
      r2 = TileRef{0, 0};
      start_piece<D>(st, w, e0, ka);
      issue(IS_G1 ? s0 + VOFF : s0, e0, r0);
      if constexpr (!IS_G1) {
        issue(s1, e1, r1);
        wait_vmem<T::PER>();
      }
    }
    phase_barrier();
    auto iteration = [&](int t, TileRef& rp, TileRef& rc, TileRef& rn, unsigned char* sc, unsigned char* sp,
                         unsigned char* sn) {
      if constexpr (!IS_G1) {
        m_phase<D>(st, w, rp.fl, rc.fl, t, sc, sp, trec, g, ka);
        phase_barrier();
        const int4 raw = load_tile(trec, t + 2, g);
        v_phase<D>(st, w, rc);
        rp = decode_tile(raw, t + 2, g);
        issue(sp, raw, rp);
      } else {
        const int4 raw = load_tile(trec, t + 1, g);
        v_phase<D>(st, w, rp);
        rn = decode_tile(raw, t + 1, g);
        issue(sn + VOFF, raw, rn);
        phase_barrier();
        m_phase<D>(st, w, rp.fl, rc.fl, t, sc, sp, trec, g, ka);
      }
      wait_vmem<T::PER>();
      phase_barrier();
    };
    for (int t = 0;; t += 3) {
      iteration(t, r2, r0, r1, s0, s2, s1);
      if (t + 1 > N) break;
      iteration(t + 1, r0, r1, r2, s1, s0, s2);
      if (t + 2 > N) break;
      iteration(t + 2, r1, r2, r0, s2, s1, s0);
      if (t + 3 > N) break;
    }
    wait_vmem<0>();            // no load may still write LDS when the workgroup ends
  };
  if (g1) run(std::true_type{});
  else run(std::false_type{});
}

// Merges the pieces of units that were split across the stream-K shares of the workgroups:
// O = sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s, over the pieces in share order
// (deterministic).  The attention kernel leaves in cut[slot] the unit whose piece a slot holds, -1
// for none; a unit that starts inside share lambda and continues past it has its first piece in
// slot 2 lambda + 1 and the others in the slots 2 lambda' of the shares that follow.  Workgroup
// (lambda, c) merges rows [16 c, 16 c + 16) of that unit, if there is one (32 rows: fewer registers
// free for loads in flight and half the workgroups: 17.0 instead of 14.8 us).  Units handed out in
// rounds are never split.  Latency bound: with the plan's records and unit tables instead of cut,
// two more loads in a row (18.7 instead of 17.7 us at 400 units, 53 MB of partials).
constexpr int kCombRows = 16;
constexpr int kCombThreads = 256;

template <int D>
__global__ __launch_bounds__(kCombThreads) void attn_combine_kernel(const int32_t* __restrict__ cut,
                                                                    const int32_t* __restrict__ qmap, int P, int U,
                                                                    int row_tiles, int Lq, int block,
                                                                    const float* __restrict__ part_o,
                                                                    const float* __restrict__ part_m,
                                                                    const float* __restrict__ part_l,
                                                                    uint16_t* __restrict__ o,
                                                                    float* __restrict__ lse) {
  constexpr int CG = D / 4;                    // 4-column groups per row
  constexpr int RSTEP = kCombThreads / CG;     // rows per pass
  constexpr int NI = kCombRows / RSTEP;        // rows per thread
  constexpr int BATCH = 4;                     // pieces whose loads are in flight together
  const int lam0 = blockIdx.x;
  const int lam = lam0 + 1 + threadIdx.x;
  const int piece = lam < P ? cut[2 * lam] : -1;
  const int u = cut[2 * lam0 + 1];
  if (u < 0 || u >= U) return;                 // (clamped, like every index read from the workspace)
  // The pieces of the unit, in share order; their slots are listed in LDS first, so that the loads
  // of several pieces can be in flight together.
  __shared__ int sh[kCombThreads / 64];
  __shared__ int pslot[kMaxPersist + 1];
  const int take = piece == u;
  int np;
  const int pos = block_excl_scan_i(take, sh, &np);
  if (take) pslot[1 + pos] = 2 * lam;
  if (threadIdx.x == 0) pslot[0] = 2 * lam0 + 1;
  __syncthreads();
  np += 1;
  const int bh = u / row_tiles;
  const int cg = threadIdx.x % CG, r0 = blockIdx.y * kCombRows + threadIdx.x / CG;
  float m[NI], l[NI];
  f32x4 acc[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    m[i] = -INFINITY;
    l[i] = 0.f;
    acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // batches of pieces: all loads of a batch first, then one rescale of the running (m, l, O) to
  // the batch's max and the pieces added with weights 2^(m_s - m) (0 for an empty piece or a
  // slot past the last piece); no branches, so the loads of a batch overlap
  for (int pc0 = 0; pc0 < np; pc0 += BATCH) {
    float bm[BATCH][NI], bl[BATCH][NI];
    f32x4 bo[BATCH][NI];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const bool ok = pc0 + j < np;
      const size_t pr0 = (size_t)pslot[ok ? pc0 + j : 0] * QR + r0;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const size_t pr = pr0 + RSTEP * i;
        bm[j][i] = ok ? part_m[pr] : -INFINITY;
        bl[j][i] = ok ? part_l[pr] : 0.f;
        bo[j][i] = ok ? *(const f32x4*)(part_o + pr * D + 4 * cg) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float mn = m[i];
#pragma unroll
      for (int j = 0; j < BATCH; ++j) mn = fmaxf(mn, bm[j][i]);
      const float mu = mn == -INFINITY ? 0.f : mn;
      const float a = exp2f(m[i] - mu);                // 0 while the running max is -inf
      l[i] *= a;
      acc[i] *= a;
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const float wgt = exp2f(bm[j][i] - mu);
        l[i] += wgt * bl[j][i];
        acc[i] += wgt * bo[j][i];
      }
      m[i] = mn;
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = r0 + RSTEP * i;                       // row inside the unit
    const int qb = qmap[(size_t)u * (QR / block) + r / block];
    const int qrow = qb * block + r % block;
    if (qb >= 0 && qb <= Lq / block && qrow < Lq) {
      const float inv = l[i] > 0.f ? 1.0f / l[i] : 0.f;
      u32x2 ow;
      ow[0] = pack_bf16x2(acc[i][0] * inv, acc[i][1] * inv);
      ow[1] = pack_bf16x2(acc[i][2] * inv, acc[i][3] * inv);
      *(u32x2*)(o + ((size_t)bh * Lq + qrow) * D + 4 * cg) = ow;
      if (lse && cg == 0)
        lse[(size_t)bh * Lq + qrow] = l[i] > 0.f ? (m[i] + log2f(l[i])) * 0.69314718055994531f : -INFINITY;
    }
  }
}

struct AttnWs {
  int4* trec;
  int32_t* qmap;
  int32_t* ulist;
  int32_t* ucount;
  int32_t* tstart;
  int32_t* dp_start;
  int32_t* sk_start;
  float* part_o;
  float* part_m;
  float* part_l;
  int32_t* cut;
  size_t bytes;
};

// Records the workspace holds: at most max(1, NK (block / 64)) tiles per unit.
size_t attn_tile_capacity(const Dims& dm) {
  return (size_t)dm.BH * ceil_div(dm.Lq, QR) * (size_t)dm.NK * (dm.block / KT);
}

AttnWs attn_ws_layout(const Dims& dm, void* base) {
  const int row_tiles = ceil_div(dm.Lq, QR);
  const size_t U = (size_t)dm.BH * row_tiles;
  const size_t slots = 2 * (size_t)kMaxPersist;
  size_t off = 0;
  AttnWs w;
  char* b = (char*)base;
  // at most max(1, NK * nsub) tiles per unit
  w.trec = (int4*)(b + off);
  off += align256(U * (size_t)dm.NK * (dm.block / KT) * sizeof(int4));
  w.qmap = (int32_t*)(b + off);
  off += align256(U * (size_t)(QR / dm.block) * sizeof(int32_t));
  w.ulist = (int32_t*)(b + off);
  off += align256(U * (size_t)dm.NK * (dm.block / KT) * sizeof(int32_t));
  w.ucount = (int32_t*)(b + off);
  off += align256(U * sizeof(int32_t));
  w.tstart = (int32_t*)(b + off);
  off += align256((U + 1) * sizeof(int32_t));
  w.dp_start = (int32_t*)(b + off);
  off += align256((kMaxPersist + 1) * sizeof(int32_t));
  w.sk_start = (int32_t*)(b + off);
  off += align256((kMaxPersist + 1) * sizeof(int32_t));
  w.part_o = (float*)(b + off);
  // slot 0 holds no piece (the first share continues none): its room holds cut [2 kMaxPersist]
  w.cut = (int32_t*)w.part_o;
  off += align256(slots * QR * dm.d * sizeof(float));
  w.part_m = (float*)(b + off);
  off += align256(slots * QR * sizeof(float));
  w.part_l = (float*)(b + off);
  off += align256(slots * QR * sizeof(float));
  w.bytes = off;
  return w;
}

// Persistent workgroups: one per CU of the current device, a multiple of 8 (XCD round robin),
// at most kMaxPersist (the partial slots of the workspace are sized for that many).
int persistent_workgroups() {
  int cus = device_cu_count();
  if (cus < 8) cus = 8;
  const int p = cus < kMaxPersist ? cus : kMaxPersist;
  return p & ~7;
}

}  // namespace

size_t attn_ws_bytes(const Dims& dm) { return attn_ws_layout(dm, nullptr).bytes; }

hipError_t launch_attn_plan(const Dims& dm, const int32_t* counts, const int32_t* idx, const int32_t* kvalid,
                            void* ws, hipStream_t st) {
  const int row_tiles = ceil_div(dm.Lq, QR);
  const int U = dm.BH * row_tiles;
  AttnWs w = attn_ws_layout(dm, ws);
  hipLaunchKernelGGL(plan_union_kernel, dim3(U), dim3(kPlanThreads), (size_t)((dm.NK + 7) / 8) * sizeof(uint32_t),
                     st, counts, idx, kvalid, dm.NQ, dm.NK, dm.h0, dm.h1, dm.Lq, dm.Lk, dm.block, dm.frame_tokens, dm.chunk0,
                     row_tiles, w.qmap, w.ulist, w.ucount);
  const int P = persistent_workgroups();
  const bool fold = U <= kFoldSchedUnits;
  if (!fold)
    hipLaunchKernelGGL(plan_sched_kernel, dim3(1), dim3(kPlanThreads), 0, st, w.ucount, U, P, w.tstart, w.dp_start,
                       w.sk_start);
  hipLaunchKernelGGL(plan_tiles_kernel, dim3(U), dim3(kPlanThreads), 0, st, w.ulist, w.ucount, kvalid, U, P, fold,
                     w.tstart, w.dp_start, w.sk_start, dm.NK, dm.Lk, dm.frame_tokens, dm.chunk0, w.qmap, dm.block, row_tiles,
                     w.trec);
  return hipGetLastError();
}

hipError_t launch_attn_run(const Dims& dm, const void* q, const void* k, const void* v, float scale, void* o,
                           float* lse, void* ws, hipStream_t st) {
  const int P = persistent_workgroups();
  AttnWs w = attn_ws_layout(dm, ws);
  const int Tcap = (int)attn_tile_capacity(dm);
  Geom gm{dm.Lq, dm.Lk, dm.block, dm.NQ, dm.NK, dm.frame_tokens, dm.chunk0, dm.BH, dm.BH * ceil_div(dm.Lq, QR)};
  const float scale_log2 = scale * 1.4426950408889634f;
  if (dm.d == 128)
    hipLaunchKernelGGL(attn_fwd_kernel<128>, dim3(P), dim3(kThreads), 0, st, (const uint16_t*)q,
                       (const uint16_t*)k, (const uint16_t*)v, w.trec, w.dp_start, w.sk_start, w.qmap,
                       (uint16_t*)o, lse, w.part_o, w.part_m, w.part_l, w.cut, gm, Tcap, scale_log2);
  else
    hipLaunchKernelGGL(attn_fwd_kernel<64>, dim3(P), dim3(kThreads), 0, st, (const uint16_t*)q,
                       (const uint16_t*)k, (const uint16_t*)v, w.trec, w.dp_start, w.sk_start, w.qmap,
                       (uint16_t*)o, lse, w.part_o, w.part_m, w.part_l, w.cut, gm, Tcap, scale_log2);
  return hipGetLastError();
}

hipError_t launch_attn_merge(const Dims& dm, void* o, float* lse, void* ws, hipStream_t st) {
  const int row_tiles = ceil_div(dm.Lq, QR);
  const int P = persistent_workgroups();
  AttnWs w = attn_ws_layout(dm, ws);
  const dim3 cgrid(P, QR / kCombRows);
  const int U = dm.BH * row_tiles;
  if (dm.d == 128)
    hipLaunchKernelGGL(attn_combine_kernel<128>, cgrid, dim3(kCombThreads), 0, st, w.cut, w.qmap, P, U, row_tiles,
                       dm.Lq, dm.block, w.part_o, w.part_m, w.part_l, (uint16_t*)o, lse);
  else
    hipLaunchKernelGGL(attn_combine_kernel<64>, cgrid, dim3(kCombThreads), 0, st, w.cut, w.qmap, P, U, row_tiles,
                       dm.Lq, dm.block, w.part_o, w.part_m, w.part_l, (uint16_t*)o, lse);
  return hipGetLastError();
}

hipError_t read_attn_schedule(const Dims& dm, const void* ws, int32_t* tstart, int32_t* ucount, int32_t* dp_start,
                              int32_t* sk_start, int* P, int* U, hipStream_t st) {
  const AttnWs w = attn_ws_layout(dm, const_cast<void*>(ws));
  *P = persistent_workgroups();
  *U = dm.BH * ceil_div(dm.Lq, QR);
  const struct {
    int32_t* dst;
    const int32_t* src;
    int n;
  } parts[4] = {{tstart, w.tstart, *U + 1}, {ucount, w.ucount, *U}, {dp_start, w.dp_start, *P + 1},
                {sk_start, w.sk_start, *P + 1}};
  for (const auto& c : parts) {
    if (!c.dst) continue;
    const hipError_t e = hipMemcpyAsync(c.dst, c.src, (size_t)c.n * sizeof(int32_t), hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace la
