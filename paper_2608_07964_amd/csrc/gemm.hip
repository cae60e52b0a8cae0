// Grouped expert GEMMs of one step: every (layer, expert) group of the step,
// from whatever layer, in one launch per GEMM (cross-layer workload
// combination, Section 4.1).  Groups are the contiguous row ranges
// offsets[key] .. offsets[key+1] of the grouped activations; the tile list
// (the group record of every row block) comes from the permutation scan.
//
//   gate/up:  h = dtype( SiLU(A Wgate^T) * (A Wup^T) )   A [P][H], W_gu[l][e] [2F][H]
//   down:     o = dtype( h Wdown^T )                     h [P][F], W_dn[l][e] [H][F]
//
// bf16 path: MFMA v_mfma_f32_32x32x16_bf16, up to 256x256 outputs per
// workgroup of 8 wavefronts, K stages of 64 in LDS rings filled by buffer
// loads straight into LDS (XOR-swizzled 16-byte chunks) several stages ahead
// of the MFMAs; persistent, XCD-aware work distribution.  The gate/up B tile
// interleaves the gate rows and the matching up rows per wavefront column,
// so each lane holds gate and up of the same (row, f) and SwiGLU runs in
// registers.  The expert weights are read in the packed layout that
// pack_bf16_kernel writes once (see there): every B stage of a tile is one
// contiguous 32 KB block holding exactly the bytes its LDS slot receives,
// and the blocks of one K stage of all of an expert's column tiles are
// adjacent, so concurrent items stream neighbouring blocks.
//
// Every output accumulates its K dimension in 16-wide MFMA steps in ascending
// order, whatever tile or group its row sits in: rows give the same bits
// whichever step (and schedule) they are computed in.
//
// fp32 path (fp32 stacks): the same item walk on fp32 MFMA, 64 x 128 outputs
// per item, same K-order guarantee.
#include "eb_internal.h"
#include "eb_numeric.h"

namespace eb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

enum { MODE_GATEUP = 0, MODE_DOWN = 1 };

// bf16 tiles.  Every tile is BM x 256 outputs on a workgroup of 8 wavefronts
// (two per SIMD) and K advances 64 at a time, so every 128-byte line of A and
// B is consumed whole by one stage; stages are filled by buffer loads straight
// into LDS.  The B tile (256 weight rows x 64 k) is the same in every shape;
// the shape of an m-tile follows the rows it holds:
//
//   BM 256 (> 128 rows): 2 x 4 wavefronts of 128 x 64 (4 x 2 MFMA blocks),
//          A ring of 2 stages (32 KB each), B ring of 3 stages (32 KB each);
//   BM 128 (65..128 rows): 2 x 4 wavefronts of 64 x 64, 3 stages of A and B;
//   BM 64  (<= 64 rows): 2 x 4 wavefronts of 32 x 64, 4 stages of A and B.
//
// Two wavefronts per SIMD keep each matrix core fed while the other one
// waits on a barrier or on LDS.  Groups that run few m-tiles are bound by
// streaming their expert's weights from HBM, which needs many bytes in flight
// per CU: every shape keeps at least two B stages in flight.  Fragments of the
// next k-step are read while the MFMAs of the current one run (every
// instruction's place in the k-step is fixed, see kstep), and the per-stage
// barrier sits before the last k-step's MFMAs.
constexpr int BN = 256, BK = 64;
constexpr int kWaves = 8;                        // two wavefronts per SIMD
constexpr int kThreads = 64 * kWaves;
constexpr int kKsteps = BK / 16;                 // MFMA k-steps per stage
constexpr int kBLoads = BN / (8 * kWaves);       // 8-row B blocks per wave per stage
constexpr int kBPart = kBLoads / (BK / 16);      // B loads issued per k-step
static_assert(kBPart * (BK / 16) == kBLoads, "B loads split evenly over the k-steps");
constexpr int kXcds = 8;

// Weights that one workgroup alone reads are loaded with the nt cache policy
// where a launch does little but stream them: they then leave the L2 and the
// memory-side cache alone, and HBM delivers 6.2 instead of 5.5 TB/s (64 tokens
// on 8 experts of H = 4096, F = 14336: step 495 -> 454 us).
constexpr int kNonTemporal = 2;  // bit nt of a buffer load's cache policy
// Most tokens at one layer (GroupedProblem::layer_tokens, a bound) for which a
// launch counts as such.  In steps of
// three micro-batches at three layers, 60 + 4 experts, H = 2048, F = 1408, nt
// loads for items of up to 64 rows take 4 to 5% off at 64 and 96 tokens,
// nothing at 128, and add 1 to 3% from 192 on; for longer items they gain
// nothing at any size.
constexpr int kNtTokens = 128;

template <int BM_, int WM_, int SA_, int SB_, bool NT_ = false>
struct TileCfg {
  static constexpr int B_POLICY = NT_ ? kNonTemporal : 0;  // cache policy of the weight loads
  static constexpr int BM = BM_;                 // tile rows
  static constexpr int WM = WM_, WN = kWaves / WM_;  // wavefront grid
  static constexpr int SA = SA_, SB = SB_;       // LDS stages of the A and B rings
  static constexpr int TM = BM / WM, TN = BN / WN;  // wavefront tile
  static constexpr int MB = TM / 32, NB = TN / 32;  // MFMA blocks per wavefront
  static constexpr int A_LOADS = BM / (8 * kWaves);  // 8-row A blocks per wave per stage
  static constexpr int A_ELEMS = BM * BK, B_ELEMS = BN * BK;  // one stage of each ring
  static constexpr int B_RING = SA * A_ELEMS;    // LDS element offset of the B ring
  static constexpr int LDS_ELEMS = SA * A_ELEMS + SB * B_ELEMS;
  static_assert(MB >= 1 && NB >= 2 && A_LOADS >= 1, "tile shape");
  static_assert(SA >= 2 && (SB == SA || SB == SA + 1), "ring depths");
};
using CfgBig = TileCfg<256, 2, 2, 3>;
using CfgMid = TileCfg<128, 2, 3, 3>;
using CfgSkinny = TileCfg<64, 2, 4, 4>;
using CfgSkinnyNt = TileCfg<64, 2, 4, 4, true>;
constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int kLdsElems = cmax(cmax(CfgBig::LDS_ELEMS, CfgMid::LDS_ELEMS), CfgSkinny::LDS_ELEMS);
static_assert(kLdsElems * 2 <= 160 * 1024, "LDS budget");
constexpr int BM = CfgBig::BM;                   // row-block granularity of the tile list

// 128-byte LDS rows hold eight 16-byte chunks; logical chunk c of row r sits
// at c ^ ((r >> 1) & 7).  A ds_read_b128 phase of 16 lanes reads 16
// consecutive rows at one logical chunk: two rows share each 256-byte bank
// window, and the XOR spreads the 8 rows of each parity over 8 chunks, so the
// 16 reads hit 16 distinct 16-byte groups of the 64 banks.
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// s_waitcnt immediates (gfx9 encoding: vmcnt bits 3:0 and 15:14, expcnt
// 6:4, lgkmcnt 11:8).  Issued through the builtin so that the compiler's own
// wait insertion sees them and does not add conservative waits of its own.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
constexpr int kWaitLgkm0 = 15 | (3 << 14) | (7 << 4);

// Bare workgroup barrier: this wave's outstanding buffer->LDS loads stay in
// flight across it (a fenced __syncthreads would drain them).
__device__ __forceinline__ void bar() {
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Barrier that orders LDS accesses only: a wave's LDS reads and writes are done
// when it arrives, its global stores need not be (__syncthreads would wait for
// an item's output stores, 3 to 6 us with every CU storing).
__device__ __forceinline__ void bar_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  bar();
}

// A wavefront-uniform pointer the compiler cannot prove uniform, in scalar
// registers (a buffer descriptor in vector registers costs a loop per load).
__device__ __forceinline__ const bf16_t* uniform(const bf16_t* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const bf16_t*)(((uint64_t)hi << 32) | lo);
}

// Raw buffer descriptor over [base, base + bytes) (bytes < 2^32); offsets
// past the end read zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// Load slots: in every stage wave w fills A rows (BM/4) w + 8 j + l/8
// (j < BM/32) of the tile, lane l at physical chunk l % 8, i.e. logical chunk
// (l % 8) ^ ((r >> 1) & 7), which is c0 for even j and c0 ^ 4 for odd j
// (every block base is a multiple of 16 rows).  An A load's byte offset is a
// per-lane part (row l/8 of the block and the chunk, by parity of j) plus a
// wave-uniform part (the block's first row and the stage's K offset) passed
// as soffset.  A rows past the buffer's end read zeros; rows past the group's
// end are loaded but their results are discarded.  B comes packed: wave w's
// load j of stage s copies the 1 KB at byte 4096 w + 1024 j of the stage's
// 32 KB block (LDS rows 32 w + 8 j .. + 7), lane l its 16 bytes at 16 l.
struct KLoop {
  bf16_t* smem;
  __amdgpu_buffer_rsrc_t ra, rb;   // buffer descriptors of the A tile and the expert's packed B
  int a_lane[2];                   // per-lane A byte offsets for even / odd j
  int b_lane;                      // per-lane B byte offset (16 l)
  int a_row0;                      // first A row (within the tile) of the wave's load blocks
  int b_tile;                      // byte offset of the wave's first B KB at the item's first stage
  int b_stage;                     // bytes from one K stage's blocks to the next one's
  int row_bytes;                   // K * 2
  int lds_a_load, lds_b_load;      // LDS element offsets of the wave's first A / B load rows
  int lds_a, lds_b;                // LDS element offsets of this lane's fragment rows (chunk-free)
  int sw;                          // this lane's fragment swizzle ((row >> 1) & 7)
  int nk, khalf;
};

template <class C>
struct Frags {
  bf16x8 a[C::MB], b[C::NB];
};

// Load j of the wave's A resp. B loads of stage s (K columns 64 s ..
// 64 s + 63) into A resp. B slot `slot`; issue_a issues all A loads of a stage,
// issue_b_part a quarter of the B loads.
template <int POLICY>
__device__ __forceinline__ void load16_lds(__amdgpu_buffer_rsrc_t r, bf16_t* lds, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, lds, 16, voff, soff, 0, POLICY);
}
template <class C>
__device__ __forceinline__ void load_a(const KLoop& L, int s, int slot, int j) {
  load16_lds<0>(L.ra, L.smem + slot * C::A_ELEMS + L.lds_a_load + j * 8 * BK, L.a_lane[j & 1],
             (L.a_row0 + 8 * j) * L.row_bytes + s * BK * 2);
}
template <class C>
__device__ __forceinline__ void load_b(const KLoop& L, int s, int slot, int j) {
  load16_lds<C::B_POLICY>(L.rb, L.smem + C::B_RING + slot * C::B_ELEMS + L.lds_b_load + j * 8 * BK, L.b_lane,
             L.b_tile + s * L.b_stage + j * 1024);
}
template <class C>
__device__ __forceinline__ void issue_a(const KLoop& L, int s, int slot) {
#pragma unroll
  for (int j = 0; j < C::A_LOADS; ++j) load_a<C>(L, s, slot, j);
}
// Part q (q < BK/16) of the B loads of stage s: loads j = q*kBPart .. +kBPart-1.
template <class C>
__device__ __forceinline__ void issue_b_part(const KLoop& L, int s, int slot, int q) {
#pragma unroll
  for (int i = 0; i < kBPart; ++i) load_b<C>(L, s, slot, q * kBPart + i);
}
template <class C>
__device__ __forceinline__ void issue_b(const KLoop& L, int s, int slot) {
#pragma unroll
  for (int q = 0; q < BK / 16; ++q) issue_b_part<C>(L, s, slot, q);
}

// Load order.  Stage t's A loads and the first quarter of its B loads are
// issued right after the barrier of step t-SA resp. t-SB, A first; the other
// three quarters of B(t) go out before the first three k-steps of the step
// after that, one quarter each, so no wave issues a burst of loads at once.
// The prologue issues stages 0 .. SB-1 in the same order as if the steps
// -SB .. -1 had run (the last three quarters of B(SB-1) go out in step 0).
// Every load is issued, also for stages past the item's last one: those load
// the last stage again into a slot that is never read, so the number of loads
// in flight at every wait is a constant.  Loads complete in issue order, so
// "A(t) and B(t) have landed" is "at most n loads are in flight", n = the
// loads issued after the later of the two.
template <class C>
struct LoadOrder {
  // loads after the last load of stage 0, when the prologue waits
  static constexpr int after_stage0() {
    int n = 0;
    bool after = false;
    for (int j = -C::SB; j < 0; ++j) {
      if (j + C::SA >= 0) {
        if (after) n += C::A_LOADS;
        if (j + C::SA == 0 && C::SB == C::SA + 1) after = true;  // A(0) comes after all of B(0)
      }
      if (j + C::SB >= 0) {
        if (after) n += kBPart;
        if (j + 1 < 0) {
          if (after) n += kBLoads - kBPart;
          if (j + C::SB == 0 && C::SB == C::SA) after = true;    // B(0) ends after A(0)
        }
      }
    }
    return n;
  }
  // loads after the last load of stage kt+1, when step kt waits
  static constexpr int after_next() {
    return C::SB == C::SA ? (C::SA - 2) * (C::A_LOADS + kBLoads)
                          : kBLoads + (C::SA - 2) * (C::A_LOADS + kBLoads);
  }
  static_assert(after_next() < 64 && after_stage0() < 64, "vmcnt range");
};

// Fragment rows of one lane: A rows wm*TM + mb*32 + lrow, B rows
// wn*TN + nb*32 + lrow; (row >> 1) & 7 = (lrow >> 1) & 7 for all of them, so
// one chunk term per k-step serves every block and the block offsets are
// immediates.
template <class C>
__device__ __forceinline__ const bf16_t* frag_base_a(const KLoop& L, int slot, int ks) {
  return L.smem + slot * C::A_ELEMS + ((ks * 2 + L.khalf) ^ L.sw) * 8 + L.lds_a;
}
template <class C>
__device__ __forceinline__ const bf16_t* frag_base_b(const KLoop& L, int slot, int ks) {
  return L.smem + C::B_RING + slot * C::B_ELEMS + ((ks * 2 + L.khalf) ^ L.sw) * 8 + L.lds_b;
}
template <class C, int NACT>
__device__ __forceinline__ void read_frags(const KLoop& L, int slot_a, int slot_b, int ks, Frags<C>& f) {
  const bf16_t* ba = frag_base_a<C>(L, slot_a, ks);
  const bf16_t* bb = frag_base_b<C>(L, slot_b, ks);
#pragma unroll
  for (int nb = 0; nb < C::NB; ++nb) f.b[nb] = *reinterpret_cast<const bf16x8*>(bb + nb * 32 * BK);
#pragma unroll
  for (int mb = 0; mb < NACT; ++mb) f.a[mb] = *reinterpret_cast<const bf16x8*>(ba + mb * 32 * BK);
}

// Buffer loads placed in one k-step: the first NA are A loads 0..NA-1 of
// stage a_s into A slot a_slot, the rest B loads b_j0, b_j0+1, ... of stage
// b_s into B slot b_slot.
struct StepLoads {
  int a_s, a_slot, b_s, b_slot, b_j0;
};
template <class C, int NA>
__device__ __forceinline__ void step_load(const KLoop& L, const StepLoads& ld, int j) {
  if (j < NA) load_a<C>(L, ld.a_s, ld.a_slot, j);
  else load_b<C>(L, ld.b_s, ld.b_slot, ld.b_j0 + j - NA);
}

// One k-step in a fixed issue order.  Its MFMAs run block row by block row
// (mb-major); the other work goes between them: first the fragment reads of
// the next k-step, B blocks then A blocks (the order in which that k-step's
// MFMAs consume them), then the V buffer loads of `ld`.  Op j of
// those R + V goes right after MFMA (j M) / (R + V), so every fragment is
// read at least M - R MFMAs before its first use and no wave issues a burst
// of loads.  Scheduling barriers fence each instruction group: the machine
// scheduler would otherwise move reads next to their consumers, which
// exposes the LDS latency.
// TR: the MFMA takes the weight fragment as its first operand, so the 32 x 32
// accumulator block is (weight row, token row): lane l holds token row
// l % 32 and weight rows 8 (v / 4) + 4 (l / 32) + v % 4, four consecutive
// output columns per group of four registers.  Otherwise the block is
// (token row, weight row): lane l holds output column l % 32 of token rows
// 8 (v / 4) + 4 (l / 32) + v % 4.  Either way every output is the same chain
// of MFMAs over K.
template <class C, int NACT, int NA, int V, bool TR>
__device__ __forceinline__ void kstep(const KLoop& L, const Frags<C>& cur, Frags<C>& nxt, int slot_a, int slot_b,
                                      int ks_next, floatx16 (&acc)[C::MB][C::NB], const StepLoads& ld) {
  constexpr int M = NACT * C::NB;
  constexpr int R = NACT > 0 ? C::NB + NACT : 0;
  constexpr int OPS = R + V;
  if constexpr (M == 0) {
#pragma unroll
    for (int j = 0; j < V; ++j) step_load<C, NA>(L, ld, j);
  } else {
    const bf16_t* ba = frag_base_a<C>(L, slot_a, ks_next);
    const bf16_t* bb = frag_base_b<C>(L, slot_b, ks_next);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const int mb = i / C::NB, nb = i % C::NB;
      if constexpr (TR)
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.b[nb], cur.a[mb], acc[mb][nb], 0, 0, 0);
      else
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[mb], cur.b[nb], acc[mb][nb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < OPS; ++j) {
        if ((j * M) / OPS == i) {
          if (j < C::NB)
            nxt.b[j] = *reinterpret_cast<const bf16x8*>(bb + j * 32 * BK);
          else if (j < R)
            nxt.a[j - C::NB] = *reinterpret_cast<const bf16x8*>(ba + (j - C::NB) * 32 * BK);
          else
            step_load<C, NA>(L, ld, j - R);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
}

// One item's K loop.  Stage s (K columns 64 s .. 64 s + 63) lives in A slot
// s % SA and B slot s % SB.  In step kt the four k-steps of stage kt run with
// the next k-step's fragments read ahead; before the MFMAs of the last k-step
// the wave waits for its reads of stage kt and its loads of stage kt+1, the
// barrier publishes stage kt+1 and frees the slots of stage kt, A(kt+SA) and
// B(kt+SB) are issued into them (see the load order above) and the first
// fragments of stage kt+1 are read.  NACT = active 32-row blocks of the wave's
// rows (inactive blocks of a ragged tile get neither LDS reads nor MFMAs).
template <class C, int NACT, bool TR>
__device__ __forceinline__ void k_loop(const KLoop& L, floatx16 (&acc)[C::MB][C::NB]) {
  const int nk = L.nk, last = nk - 1;
#pragma unroll
  for (int j = -C::SB; j < 0; ++j) {
    if (j + C::SA >= 0) issue_a<C>(L, min(j + C::SA, last), j + C::SA);
    if (j + C::SB >= 0) {
      issue_b_part<C>(L, min(j + C::SB, last), j + C::SB, 0);
      if (j + 1 < 0)
#pragma unroll
        for (int q = 1; q < BK / 16; ++q) issue_b_part<C>(L, min(j + C::SB, last), j + C::SB, q);
    }
  }
  int pb_s = min(C::SB - 1, last), pb_slot = C::SB - 1;  // B stage with quarters still to issue
  wait_vm<LoadOrder<C>::after_stage0()>();
  bar();
  Frags<C> f[2];
  if (NACT > 0) read_frags<C, NACT>(L, 0, 0, 0, f[0]);
  int ca = 0, cb = 0;  // slots of stage kt
  for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
    for (int ks = 0; ks < kKsteps - 1; ++ks) {
      const StepLoads ld{0, 0, pb_s, pb_slot, (ks + 1) * kBPart};
      kstep<C, NACT, 0, kBPart, TR>(L, f[ks & 1], f[(ks + 1) & 1], ca, cb, ks + 1, acc, ld);
    }
    // every fragment of stage kt is in registers, stage kt+1 has landed
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    wait_vm<LoadOrder<C>::after_next()>();
    bar();
    pb_s = min(kt + C::SB, last);
    pb_slot = cb;
    const StepLoads ld{min(kt + C::SA, last), ca, pb_s, pb_slot, 0};
    const int na = ca + 1 == C::SA ? 0 : ca + 1;
    const int nb = cb + 1 == C::SB ? 0 : cb + 1;
    kstep<C, NACT, C::A_LOADS, C::A_LOADS + kBPart, TR>(L, f[(kKsteps - 1) & 1], f[0], na, nb, 0, acc, ld);
    ca = na;
    cb = nb;
  }
  // the loads of the stages past the last one must land before the next
  // item's prologue writes the same LDS slots
  wait_vm<0>();
}

// K loop of the wave's nact active 32-row blocks (a compile-time count).
template <class C, bool TR>
__device__ __forceinline__ void k_loop_nact(const KLoop& kl, floatx16 (&acc)[C::MB][C::NB], int nact) {
  if constexpr (C::MB == 4) {
    switch (nact) {
      case 4: k_loop<C, 4, TR>(kl, acc); break;
      case 3: k_loop<C, 3, TR>(kl, acc); break;
      case 2: k_loop<C, 2, TR>(kl, acc); break;
      case 1: k_loop<C, 1, TR>(kl, acc); break;
      default: k_loop<C, 0, TR>(kl, acc); break;
    }
  } else if constexpr (C::MB == 2) {
    switch (nact) {
      case 2: k_loop<C, 2, TR>(kl, acc); break;
      case 1: k_loop<C, 1, TR>(kl, acc); break;
      default: k_loop<C, 0, TR>(kl, acc); break;
    }
  } else {
    static_assert(C::MB == 1, "tile shape");
    if (nact == 1) k_loop<C, 1, TR>(kl, acc); else k_loop<C, 0, TR>(kl, acc);
  }
}

// Float pair to packed bf16, round to nearest even (one hardware conversion).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}

// bf16 epilogue of transposed accumulators: acc[mb][nb][4 g + q] is token
// row r0w + mb*32 + lrow (r0w = the wavefront row's first row in the tile)
// and weight row wn*TN + nb*32 + 8 g + 4 khalf + q, i.e. four consecutive
// output columns per g.  Gate/up: blocks nb < NB/2 are gate rows and
// nb + NB/2 the up rows of the same f; h = bf16(SwiGLU(gate, up)).  Down:
// o = bf16(acc).  Blocks past nact were not computed (and may be another
// wavefront row's rows).
//
// The wavefront's tile goes through its own part of the LDS ring (free once
// every wavefront has left the K loop) so that each store instruction writes
// whole 128-byte (down) or 64-byte (gate/up) runs of a row; stored from the
// accumulators it would write 16 bytes of each of 32 rows.  Rows hold 16-byte
// chunks, XOR-swizzled by row against bank conflicts.  An item's time
// outside its K loop (2048-row groups, K = 1408, 256 columns: epilogue 4.1,
// then 5.7 us until the next item starts, beside 30 us of K loop) fell to 1.9
// and 1.8 us, with bar_lds instead of a barrier that waits for the stores.
template <class C, int MODE>
__device__ __forceinline__ void epilogue_tr(const GroupedProblem& p, const floatx16 (&acc)[C::MB][C::NB],
                                            bf16_t* smem, bf16_t* C_out, int row0, int row_end, int ni, int r0w,
                                            int wave, int wn, int nact, int lane) {
  constexpr int COLS = MODE == MODE_GATEUP ? C::TN / 2 : C::TN;  // output columns of the wavefront
  constexpr int CH = COLS / 8, ROWS = 64 / CH;                   // chunks of a row; rows of one store
  const int N = MODE == MODE_GATEUP ? p.F : p.H;
  const int lrow = lane & 31, khalf = lane >> 5;
  bf16_t* st = smem + wave * (C::TM * C::TN);
  auto chunk = [](int r, int c) { return c ^ (CH == 8 ? (r >> 1) & 7 : (r >> 2) & 3); };
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb) {
    if (mb >= nact) continue;
    const int r = mb * 32 + lrow;
#pragma unroll
    for (int nb = 0; nb < COLS / 32; ++nb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 v;
        if constexpr (MODE == MODE_GATEUP) {
          const floatx16 &gt = acc[mb][nb], &up = acc[mb][nb + C::NB / 2];
          v.x = pack_bf16x2(swiglu(gt[4 * g], up[4 * g]), swiglu(gt[4 * g + 1], up[4 * g + 1]));
          v.y = pack_bf16x2(swiglu(gt[4 * g + 2], up[4 * g + 2]), swiglu(gt[4 * g + 3], up[4 * g + 3]));
        } else {
          const floatx16& c = acc[mb][nb];
          v.x = pack_bf16x2(c[4 * g], c[4 * g + 1]);
          v.y = pack_bf16x2(c[4 * g + 2], c[4 * g + 3]);
        }
        *reinterpret_cast<uint2*>(st + r * COLS + chunk(r, nb * 4 + g) * 8 + khalf * 4) = v;
      }
  }
  asm volatile("" ::: "memory");  // the reads below are of the bytes written above, as another type
  // rows past the group's end are past the descriptor's end: not stored
  const int rows = max(0, min(nact * 32, row_end - row0 - r0w));
  const __amdgpu_buffer_rsrc_t rc = buffer_rsrc(uniform(C_out + (size_t)(row0 + r0w) * N), (uint32_t)(rows * N * 2));
  const int rl = lane / CH, c = lane % CH;
  int off = (rl * N + ni * (4 * COLS) + wn * COLS + c * 8) * 2;
#pragma unroll
  for (int i = 0; i < C::TM / ROWS; ++i) {
    if (i * ROWS < nact * 32) {
      const int r = i * ROWS + rl;
      typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
      __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(st + r * COLS + chunk(r, c) * 8), rc, off, 0, 0);
    }
    off += ROWS * N * 2;
  }
}

// One work item (m-tile row0.. of group rows ending at row_end, n-tile ni,
// K stages ks0 .. ks0+nks-1) in tile shape C.  part == nullptr: the item
// covers all of K and writes the output; else it writes its fp32 partial
// sums to part (row-major, N = H columns).
template <class C, int MODE>
__device__ __forceinline__ void run_item(const GroupedProblem& p, bf16_t* smem, const bf16_t* A,
                                         bf16_t* C_out, const bf16_t* Bbase, int row0, int row_end,
                                         int ni, int K, int ks0, int nks, float* part, int wave,
                                         int lane) {
  const int wm = wave / C::WN, wn = wave % C::WN;
  const int lrow = lane & 31, khalf = lane >> 5;
  // rows per wavefront row: the tile's rows split evenly over the WM
  // wavefront rows in whole 32-row blocks (a 150-row tile gives each of two
  // wavefront rows 96 rows, 3 blocks, instead of 128 + 22); the slowest
  // wavefront row sets the item's time
  const int tm = min(C::TM, 32 * ((row_end - row0 + 32 * C::WM - 1) / (32 * C::WM)));
  const int lr = lane >> 3, lp = lane & 7;
  const int k_off = ks0 * BK;  // first K column of the item
  const bf16_t* Atile = A + (size_t)row0 * K + k_off;
  const int a_rows = min(C::BM, p.P - row0);  // rows past it read zeros; their results are discarded

  KLoop kl;
  kl.smem = smem;
  kl.ra = buffer_rsrc(Atile, (uint32_t)(a_rows * K * 2 - k_off * 2));
  const int n_rows = MODE == MODE_GATEUP ? 2 * p.F : p.H;  // the expert matrix is n_rows x K
  kl.rb = buffer_rsrc(Bbase, (uint32_t)n_rows * (uint32_t)K * 2u);
  kl.row_bytes = K * 2;
  {
    // swizzle of the wave's first A load row; odd j flips bit 2
    const int ca = lp ^ ((((C::BM / kWaves) * wave + lr) >> 1) & 7);
    kl.a_lane[0] = lr * K * 2 + ca * 16;
    kl.a_lane[1] = lr * K * 2 + (ca ^ 4) * 16;
    kl.a_row0 = (C::BM / kWaves) * wave;
    kl.b_lane = lane * 16;
    kl.b_stage = (n_rows / BN) * (BN * BK * 2);
    kl.b_tile = ks0 * kl.b_stage + ni * (BN * BK * 2) + wave * (BN / kWaves) * BK * 2;
  }
  kl.lds_a_load = (C::BM / kWaves) * wave * BK;
  kl.lds_b_load = (BN / kWaves) * wave * BK;
  kl.lds_a = (wm * tm + lrow) * BK;
  kl.lds_b = (wn * C::TN + lrow) * BK;
  kl.sw = (lrow >> 1) & 7;
  kl.nk = nks;
  kl.khalf = khalf;

  floatx16 acc[C::MB][C::NB];
#pragma unroll
  for (int i = 0; i < C::MB; ++i)
#pragma unroll
    for (int j = 0; j < C::NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // 32-row blocks of this wave's TM rows that hold rows of the group
  const int nact = min(tm / 32, max(0, (row_end - (row0 + wm * tm) + 31) / 32));
  // bf16 outputs use the transposed accumulators (a lane holds four consecutive
  // columns, one 8-byte LDS write of epilogue_tr); fp32 partial sums the row
  // layout (32 lanes store a whole 128-byte line)
  if (MODE == MODE_GATEUP || part == nullptr) {
    k_loop_nact<C, true>(kl, acc, nact);
    bar_lds();  // every wave is done with the ring before it is written again
    epilogue_tr<C, MODE>(p, acc, smem, C_out, row0, row_end, ni, wm * tm, wave, wn, nact, lane);
  } else if constexpr (MODE == MODE_DOWN) {
    k_loop_nact<C, false>(kl, acc, nact);
    bar_lds();
    // acc[mb][nb][v]: output column wn*TN + nb*32 + lrow of token row
    // wm*tm + mb*32 + 8 (v / 4) + 4 khalf + v % 4
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) {
      if (mb >= nact) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = row0 + wm * tm + mb * 32 + 8 * (v >> 2) + 4 * khalf + (v & 3);
        if (row >= row_end) continue;
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb)
          part[(size_t)row * p.H + ni * BN + wn * C::TN + nb * 32 + lrow] = acc[mb][nb][v];
      }
    }
  }
}

// Persistent grouped GEMM.  Work item = (group, n-tile, m-tile); a group of
// R rows has ceil(R / 256) m-tiles sharing its rows evenly, enumerated group
// by group, then by blocks of kMBlock m-tiles, n-tile-major inside a block,
// m-tile fastest, so consecutive items share the weight tile and, running at
// the same pace, read each weight stage from L2 once (unequal m-tiles drift
// apart and fetch the weights again: 2.2-3.5x the weight bytes for two to
// three m-tiles).  The blocks bound how often a large group's activation rows
// are streamed: once per window of n-tiles rather than once per n-tile (with
// tens of m-tiles, 28 times over for a 7168-wide down projection).  Workgroup b runs on XCD b % 8 (round-robin
// dispatch) and takes items from its XCD's contiguous eighth of the list
// through that XCD's atomic counter, so items running together on one L2
// share weight and activation tiles and no workgroup idles while its XCD has
// work; once its XCD's range is drained it takes items from the other XCDs'
// ranges, then those set aside for the end (ItemQueue).  Every item is taken
// exactly once whichever workgroup takes it.
// The counter increment for the next item is issued at the start of the
// current one and its result used at its end.  Each item runs in the tile
// shape of the rows it holds; all shapes accumulate K in the same order, so a
// row's result does not depend on the shape or on which workgroup ran it.
// m-tiles per block of the item order (see grouped_gemm_bf16): a window of
// the 32 items one XCD runs at a time then spans 4 m-tiles x 8 n-tiles, so
// it streams 4 activation and 8 weight tiles instead of 32 and 1.
constexpr int kMBlock = 4;

// A group record by a scalar load (i uniform): it does not queue behind the
// vector loads in flight.  The records are written by an earlier launch.
__device__ __forceinline__ int4 scalar_record(const int4* p, int i) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 v = reinterpret_cast<const __attribute__((address_space(4))) i32x4*>((uintptr_t)p)[i];
  return make_int4(v.x, v.y, v.z, v.w);
}

// Position of an item inside its group's list: column tile and m-tile.
struct Tile2 {
  int ni, mi;
};
__device__ __forceinline__ Tile2 item_tile(int local, int mt, int n_ntiles) {
  const int mb = local / (kMBlock * n_ntiles);
  const int gm = min(kMBlock, mt - mb * kMBlock);
  const int rb = local - mb * kMBlock * n_ntiles;
  const int ni = rb / gm;
  return Tile2{ni, mb * kMBlock + (rb - ni * gm)};
}

// One thread's view of the item counters: the XCD whose range it draws from.
// Each XCD's counter has a cache line of its own, and another XCD's counter is
// read before it is drawn from: when every workgroup drew from all eight in
// one line on its way out, those 2000 atomics ran one after the other (gate/up
// at H = 2048, F = 1408: one token on 64 + 2 experts 37 -> 23 us, 80 tokens on
// three layers of 60 + 4 172 -> 165, 3072 tokens on five of 64 + 2 768 -> 764).
//
// The list's last n_tiles[0] - n_tiles[1] row blocks are small ones the scan
// set aside: their items are taken once the others are gone, so that the
// launch ends on short items.  They are split into eighths like the others
// (drawn by all XCDs from one counter, every XCD streamed from every expert:
// a launch of 256 items of K = 7168 took 220 instead of 158 us).
//
// A split-K launch has few, long items (32 per m-tile, of K = 7168, at
// H = 4096, F = 14336), and those of a small group, bound by streaming their
// weights, are hardly shorter than the others: they overlap better with the
// others' matrix work than with each other.  Setting them aside pays there only
// where the last round of items would leave most workgroups idle, or where all
// fit one round (every XCD then has some of them); else they stay in the queue.
// Down launch of 8 experts, 2 picks a token, in us, always set aside / by this
// rule / never: 2.0 rounds (128 tokens at each of two layers) 356 / 308 / 315;
// 4.0 rounds (64 at each of four) 646 / 583 / 603; 1.12 rounds (512 at one)
// 227 / 229 / 343; 2.25 rounds (384 at each of two) 437 / 438 / 480.
struct ItemQueue {
  int32_t* ctr;
  long long main;  // items before the ones set aside
  int total, xcd, victim, per_xcd;  // victim: XCD range drawn from, + kXcds for its set-aside range
  // Every item has a workgroup by number, nothing is drawn: the counters are
  // neither drawn from nor read (15 reads in turn on each workgroup's way out:
  // fp32 down launch of 774 tokens on three layers of 8 experts, H = 256,
  // F = 128, 14.2 -> 8.2 us).
  bool numbered;
  __device__ __forceinline__ ItemQueue(const GroupedProblem& p, int nsub)
      : ctr(p.work_ctr), total(p.n_tiles[0] * nsub), xcd(blockIdx.x % kXcds), victim(blockIdx.x % kXcds),
        per_xcd(gridDim.x / kXcds) {
    const int last = total % (int)gridDim.x;  // items of the last, partial round
    const bool aside = p.ksplit == 1 || total <= (int)gridDim.x || (last > 0 && 2 * last <= (int)gridDim.x);
    main = aside ? (long long)p.n_tiles[1] * nsub : total;
    numbered = main == total && total <= kXcds * per_xcd;
  }
  __device__ __forceinline__ int bound(int x) const {  // first item of range x; bound(2 kXcds) = total
    return x < kXcds ? (int)((x * main) / kXcds) : (int)(main + ((x - kXcds) * (total - main)) / kXcds);
  }
  __device__ __forceinline__ int32_t* counter() const {
    return ctr + (victim < kXcds ? victim * kWorkStride : (victim - kXcds) * kWorkStride + kWorkTail);
  }
  __device__ __forceinline__ int draw() const { return numbered ? 0 : atomicAdd(counter(), 1); }
  // The first items of an XCD's range go to its workgroups by number (drawn,
  // the first few to start would each hold a second item while others have
  // none), the rest through its counter.
  __device__ __forceinline__ int drawn(int got) const { return bound(victim) + got + (victim < kXcds ? per_xcd : 0); }
  // item index from a value drawn from victim's counter, or -1 once everything
  // is taken: the own range, the other XCDs', then the set-aside ones alike
  __device__ __forceinline__ int settle(int got) {
    if (numbered) return -1;
    int it = drawn(got);
    while (it >= bound(victim + 1)) {
      if (victim < kXcds) {
        victim = victim + 1 == kXcds ? 0 : victim + 1;
        if (victim == xcd) victim += kXcds;
      } else {
        victim = victim + 1 == 2 * kXcds ? kXcds : victim + 1;
        if (victim == xcd + kXcds) return -1;
      }
      it = drawn(__hip_atomic_load(counter(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (it < bound(victim + 1)) it = drawn(draw());
    }
    return it;
  }
  __device__ __forceinline__ int first() {
    const int it = bound(xcd) + (int)(blockIdx.x / kXcds);
    return it < bound(xcd + 1) ? it : settle(draw());
  }
};

template <int MODE>
__global__ __launch_bounds__(kThreads, 1) void grouped_gemm_bf16(GroupedProblem p, WeightTable wt,
                                                                 const bf16_t* __restrict__ A,
                                                                 bf16_t* __restrict__ C,
                                                                 int n_ntiles) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[kLdsElems];
  // the next item index is broadcast through the first word of the ring, which
  // no load writes between an item's last K stage and the next prologue (and
  // only wavefront 0's own output tile passes through)
  int* s_next = reinterpret_cast<int*>(smem);
  // the LDS ring is written by global->LDS loads the compiler does not see
  asm volatile("" ::"v"(smem) : "memory");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ksplit = MODE == MODE_DOWN ? p.ksplit : 1;
  const int nsub = n_ntiles * ksplit;  // items per m-tile
  ItemQueue q(p, nsub);  // used by thread 0 only
  const int K = MODE == MODE_GATEUP ? p.H : p.F;
  const int ES = p.E + p.S;

  if (tid == 0) *s_next = q.first();
  __syncthreads();
  int it = __builtin_amdgcn_readfirstlane(*s_next);
  __syncthreads();

  while (it >= 0) {
    int got = 0;
    if (tid == 0) got = q.draw();
    // group of this item: a group's items it * nsub .. (it + mt) * nsub - 1
    // cover its m-tiles it .. it + mt - 1, so item / nsub is one of them
    const int4 gd = scalar_record(p.tiles, it / nsub);  // key, first row, rows, first m-tile
    const int mt = (gd.z + BM - 1) / BM;
    // within the group: K part slowest, then blocks of kMBlock m-tiles, then
    // n-tile, m-tile fastest (the last block holds the mt % kMBlock rest)
    const int local = it - gd.w * nsub;
    const int kh = local / (mt * n_ntiles);
    const Tile2 tile = item_tile(local - kh * mt * n_ntiles, mt, n_ntiles);
    const int ni = tile.ni, mi = tile.mi;
    const int nks = K / BK / ksplit, ks0 = kh * nks;
    float* part = ksplit > 1 ? p.partial + (size_t)kh * p.P * p.H : nullptr;
    // the group's mt m-tiles share its rows evenly (whole 32-row blocks), so
    // they run at the same pace and meet the same weight stages in L2
    const int rpt = 32 * ((gd.z + 32 * mt - 1) / (32 * mt));
    const int row0 = gd.y + mi * rpt, row_end = min(gd.y + gd.z, row0 + rpt);
    const int layer = gd.x / ES, e = gd.x - layer * ES;
    const bf16_t* Bbase = MODE == MODE_GATEUP
        ? static_cast<const bf16_t*>(wt.gu[layer]) + (size_t)e * 2 * p.F * p.H
        : static_cast<const bf16_t*>(wt.dn[layer]) + (size_t)e * p.H * p.F;
    const int rows = row_end - row0;
    if (rows > CfgMid::BM)
      run_item<CfgBig, MODE>(p, smem, A, C, Bbase, row0, row_end, ni, K, ks0, nks, part, wave, lane);
    else if (rows > CfgSkinny::BM)
      run_item<CfgMid, MODE>(p, smem, A, C, Bbase, row0, row_end, ni, K, ks0, nks, part, wave, lane);
    else if (p.layer_tokens <= kNtTokens)
      run_item<CfgSkinnyNt, MODE>(p, smem, A, C, Bbase, row0, row_end, ni, K, ks0, nks, part, wave, lane);
    else
      run_item<CfgSkinny, MODE>(p, smem, A, C, Bbase, row0, row_end, ni, K, ks0, nks, part, wave, lane);
    if (tid == 0) *s_next = q.settle(got);
    bar_lds();
    it = __builtin_amdgcn_readfirstlane(*s_next);
    bar_lds();  // every thread has read it before the next prologue refills the ring
  }
}

// ---------------------------------------------------------------------------
// Decode launches (bf16): every group has a few rows, so the launch does
// nothing but stream the experts' weights once.  Each wavefront is a stream of
// its own: a workgroup is one wavefront with a 40 KB LDS ring (four per CU)
// and no barrier anywhere.  A unit is one 64-weight-row column of a 256-row
// column tile (a contiguous 8 KB of every packed block) for up to 8 NA token
// rows; each stage's ring slot holds the unit's A rows (NA KB) and B rows
// (8 KB).  The stages of consecutive units form one sequence: while a unit's
// last stages are multiplied, the first stages of the wavefront's next unit
// are already being loaded, so a unit's end costs its stores and nothing else.
// Each output is the same chain of MFMAs as in grouped_gemm_bf16, bit for bit.
//
// Bound by HBM: 74 groups of 2 to 31 rows at H = 2048, F = 1408 stream their
// weights at 6.4 (gate/up, 133 us) and 6.0 TB/s (down, 69 us), 149 and 76 us
// without the nt policy, against 162 and 87 us in 256-column items on whole-CU
// workgroups; one token with 8 expert slots 16 and 12 against 28 and 21 us
// (four times the units, so every CU has some).  Five wavefronts of 32 KB per
// CU, three of 53 KB or two of 80 KB measured 0 to 5% slower.
constexpr int kStreamLds = 40 * 1024, kStreamPerCu = 4;
template <int NA>
struct StreamCfg {
  static constexpr int SLOT = (NA + 8) * 512;       // elements of one stage (A rows, then B rows)
  static constexpr int FIT = kStreamLds / (2 * SLOT), R = FIT > 4 ? 4 : FIT;  // ring slots
  static constexpr int LOADS = NA + 8;              // 1 KB loads of one stage
  static_assert(R >= 3 && (R - 2) * LOADS < 64, "ring");
};
constexpr int kStreamMinStages = 4;                 // K stages a unit needs for the look-ahead (R - 1, plus one)

// What a stream loads next: the unit's descriptors and its next K stage.
struct StreamUnit {
  int tile_row0, rows;             // token rows of the unit's chunk
  int row_end;                     // end of the m-tile's rows (chunks follow while rows remain)
  int col;                         // 64-weight-row column of the expert matrix
  int kh;                          // K part
  const bf16_t* B;                 // expert matrix
};

template <int MODE, int NA>
__global__ __launch_bounds__(64, 1) void stream_gemm_bf16(GroupedProblem p, WeightTable wt,
                                                          const bf16_t* __restrict__ A, bf16_t* __restrict__ C) {
  using Cfg = StreamCfg<NA>;
  constexpr int R = Cfg::R, LOADS = Cfg::LOADS;
  __shared__ __attribute__((aligned(1024))) bf16_t smem[kStreamLds / 2];
  // the ring is written by global->LDS loads the compiler does not see
  asm volatile("" ::"v"(smem) : "memory");
  const int lane = threadIdx.x, lrow = lane & 31, khalf = lane >> 5;
  const int K = MODE == MODE_GATEUP ? p.H : p.F;
  const int n_rows = MODE == MODE_GATEUP ? 2 * p.F : p.H;
  const int ksplit = MODE == MODE_DOWN ? p.ksplit : 1;
  const int n_cols = n_rows / 64, nsub = n_cols * ksplit, nk = K / BK / ksplit;
  const int ES = p.E + p.S;
  const int b_stage = (n_rows / BN) * (BN * BK * 2);  // bytes from one K stage's blocks to the next one's

  // Units: XCD x owns a contiguous eighth of the list and its wavefronts take
  // every per_xcd-th unit of it.  Units all cost the same, so a counter would
  // balance nothing (counters were measured only with all of them in one cache
  // line, which took a thousand wavefronts 60 us).
  const long long total = (long long)(*p.n_tiles) * nsub;
  const int xcd = blockIdx.x % kXcds, per_xcd = gridDim.x / kXcds;
  const int u_end = (int)(((xcd + 1) * total) / kXcds);

  auto decode = [&](int unit) {
    StreamUnit d;
    const int u = __builtin_amdgcn_readfirstlane(unit);
    const int4 gd = scalar_record(p.tiles, u / nsub);  // key, first row, rows, first m-tile
    const int mt = (gd.z + BM - 1) / BM;
    const int local = u - gd.w * nsub;           // K part, then column, m-tile fastest
    d.kh = local / (mt * n_cols);
    const int rem = local - d.kh * mt * n_cols;
    d.col = rem / mt;
    const int rpt = 32 * ((gd.z + 32 * mt - 1) / (32 * mt));
    d.tile_row0 = gd.y + (rem - d.col * mt) * rpt;
    d.row_end = min(gd.y + gd.z, d.tile_row0 + rpt);
    d.rows = min(8 * NA, d.row_end - d.tile_row0);
    const int layer = gd.x / ES, e = gd.x - layer * ES;
    d.B = (MODE == MODE_GATEUP ? static_cast<const bf16_t*>(wt.gu[layer]) : static_cast<const bf16_t*>(wt.dn[layer])) +
          (size_t)e * n_rows * K;
    return d;
  };

  // load cursor
  __amdgpu_buffer_rsrc_t ra, rb;
  int a_soff = 0, b_voff = 0;  // next stage's A byte offset (uniform) and this lane's B byte offset
  const int lr = lane >> 3, c_even = (lane & 7) ^ (lr >> 1);
  const int a_even = lr * K * 2 + c_even * 16, a_odd = lr * K * 2 + (c_even ^ 4) * 16;
  auto aim = [&](const StreamUnit& d, bool any) {  // any false: no next unit, loads of an empty buffer
    // rows past the chunk read zeros
    ra = buffer_rsrc(uniform(A + (size_t)d.tile_row0 * K + (size_t)d.kh * nk * BK),
                     __builtin_amdgcn_readfirstlane(any ? d.rows * K * 2 - d.kh * nk * BK * 2 : 0));
    rb = buffer_rsrc(uniform(d.B + (size_t)d.kh * nk * (b_stage / 2) + (size_t)(d.col >> 2) * (BN * BK) +
                             (d.col & 3) * (64 * BK)),
                     __builtin_amdgcn_readfirstlane(any ? (nk - 1) * b_stage + 64 * BK * 2 : 0));
    a_soff = 0;
    b_voff = lane * 16;
  };
  auto issue = [&](int slot) {
    bf16_t* st = smem + slot * Cfg::SLOT;
#pragma unroll
    for (int j = 0; j < NA; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, st + j * 512, 16, 8 * j * K * 2 + ((j & 1) ? a_odd : a_even), a_soff,
                                               0, 0);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, st + (NA + j) * 512, 16, b_voff + j * 1024, 0, 0,
                                               kNonTemporal);
    a_soff += BK * 2;
    b_voff += b_stage;
  };

  int u = (int)((xcd * total) / kXcds) + (int)(blockIdx.x / kXcds);
  if (u >= u_end) return;
  StreamUnit cur = decode(u);
  aim(cur, true);
#pragma unroll
  for (int s = 0; s < R - 1; ++s) issue(s);
  int slot = 0;
  floatx16 acc[2];
  const int sw = (lrow >> 1) & 7;
  // one stage: its loads have landed, the slot of the stage before is free
  // (its fragment reads are done), the load cursor's next stage goes there
  auto step = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    wait_vm<(R - 2) * LOADS>();
    asm volatile("" ::: "memory");
    issue(slot == 0 ? R - 1 : slot - 1);
    const bf16_t* sa = smem + slot * Cfg::SLOT + lrow * BK;  // rows past 8 NA: other rows, results discarded
    const bf16_t* sb = smem + slot * Cfg::SLOT + NA * 512 + lrow * BK;
    bf16x8 a[4], b[2][4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int ch = ((2 * ks + khalf) ^ sw) * 8;
      a[ks] = *reinterpret_cast<const bf16x8*>(sa + ch);
      b[0][ks] = *reinterpret_cast<const bf16x8*>(sb + ch);
      b[1][ks] = *reinterpret_cast<const bf16x8*>(sb + 32 * BK + ch);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[nb][ks], a[ks], acc[nb], 0, 0, 0);
    slot = slot == R - 1 ? 0 : slot + 1;
  };

  for (;;) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nb][v] = 0.f;
    for (int s = 0; s < nk - (R - 1); ++s) step();
    // the load cursor moves on to the wavefront's next unit; a group with more
    // rows than the launch was sized for (a caller's token that picks an
    // expert twice) first goes on with its next rows
    StreamUnit nxt = cur;
    bool more = true;
    if (cur.tile_row0 + 8 * NA < cur.row_end) {
      nxt.tile_row0 += 8 * NA;
      nxt.rows = min(8 * NA, cur.row_end - nxt.tile_row0);
    } else {
      u += per_xcd;
      more = u < u_end;
      if (more) nxt = decode(u);
    }
    aim(nxt, more);
#pragma unroll
    for (int s = 0; s < R - 1; ++s) step();
    // acc[nb][4 g + q]: token row lrow, weight row 32 nb + 8 g + 4 khalf + q of the column
    if (lrow < cur.rows) {
      const size_t row = cur.tile_row0 + lrow;
      if constexpr (MODE == MODE_GATEUP) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          uint2 v;
          v.x = pack_bf16x2(swiglu(acc[0][4 * g], acc[1][4 * g]), swiglu(acc[0][4 * g + 1], acc[1][4 * g + 1]));
          v.y = pack_bf16x2(swiglu(acc[0][4 * g + 2], acc[1][4 * g + 2]), swiglu(acc[0][4 * g + 3], acc[1][4 * g + 3]));
          *reinterpret_cast<uint2*>(C + row * p.F + cur.col * 32 + 8 * g + 4 * khalf) = v;
        }
      } else {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const floatx16& c = acc[nb];
            const int n = cur.col * 64 + nb * 32 + 8 * g + 4 * khalf;
            if (ksplit > 1) {
              *reinterpret_cast<float4*>(p.partial + ((size_t)cur.kh * p.P + row) * p.H + n) =
                  make_float4(c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]);
            } else {
              uint2 v;
              v.x = pack_bf16x2(c[4 * g], c[4 * g + 1]);
              v.y = pack_bf16x2(c[4 * g + 2], c[4 * g + 3]);
              *reinterpret_cast<uint2*>(C + row * p.H + n) = v;
            }
          }
      }
    }
    if (!more) break;
    cur = nxt;

  }
  wait_vm<0>();  // no load may write LDS after the wavefront has ended
}

// ---------------------------------------------------------------------------
// fp32 path: the same grouped, persistent item walk on
// v_mfma_f32_16x16x4_f32.  An item is 64 rows x 128 weight rows on a workgroup
// of 8 wavefronts; wavefront w owns weight rows 16 w .. + 15 of the tile
// (gate/up: 8 gate rows and the matching 8 up rows) for all 64 token rows, so
// every SIMD works however few rows the item has, and rows are padded to 16
// only.  K advances 32 per stage (one 128-byte line of each row) through a
// 3-stage LDS ring filled by buffer loads straight into LDS; 72 KB of LDS, so
// two workgroups share a CU and cover each other's waits.
//
// Bound by the fp32 matrix rate on large groups and by streaming the weights
// on small ones; a launch takes about the sum of the two.  Measured, H = 1024,
// F = 2816: one 4096-row group 111 (gate/up) and 95 TFLOP/s (down); 42 groups
// of one or two rows 5.5 TB/s of weights; a two-layer step of 34 groups and
// 2400 rows 1125 -> 530 us against the 64 x 64 VALU tiles this replaces.
// 64 weight rows per item (with the K of a stage split over two sets of
// wavefronts, or three workgroups per CU) measured 5 to 15% slower.
constexpr int FBM = 64, FBN = 128, FBK = 32, FST = 3;
constexpr int kF32Waves = 8, kF32PerCu = 2;       // wavefronts; workgroups per CU
constexpr int kF32Stage = (FBM + FBN) * FBK;      // floats of one stage
constexpr int kF32Loads = (FBM + FBN) / 8 / kF32Waves;  // 8-row loads of one wavefront and stage
static_assert(FBM / 8 == kF32Waves && FBN / 16 == kF32Waves, "one A load and one 16-row column per wavefront");
static_assert(kF32Stage * 4 * FST * kF32PerCu + 1024 <= 160 * 1024, "LDS budget");
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct F32Loop {
  float* smem;
  __amdgpu_buffer_rsrc_t ra, rb[2];  // A rows of the item; the wavefront's first / second 8 weight rows
  int a_off, b_off[2];               // per-lane byte offset of a load's row and chunk
  int wave, lrow, quarter, nk;
};

// Loads of stage s (K columns 32 s .. 32 s + 31) into ring slot `slot`:
// wavefront w fills A rows 8 w .. + 7 and its own weight rows.  A row holds
// eight 16-byte chunks, logical chunk c at c ^ ((row >> 1) & 7).
template <bool NT>
__device__ __forceinline__ void f32_issue(const F32Loop& L, int s, int slot) {
  float* st = L.smem + slot * kF32Stage;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(L.ra, st + 8 * L.wave * FBK, 16, L.a_off, s * FBK * 4, 0, 0);
#pragma unroll
  for (int j = 0; j < 2; ++j)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(L.rb[j], st + (FBM + 16 * L.wave + 8 * j) * FBK, 16, L.b_off[j],
                                             s * FBK * 4, 0, NT ? kNonTemporal : 0);
}

// K loop over NACT active 16-row blocks.  Lane l reads 16-byte chunk
// 4 kc + l / 16 of row l % 16 of each block, and element i of the chunks goes
// to MFMA i: every MFMA sums K columns 16 kc + i + {0, 4, 8, 12}, the same
// order for every row of every item.  The weights are the first operand, so
// a lane holds four consecutive output columns of one token row.
template <int NACT, bool NT>
__device__ __forceinline__ void f32_k_loop(const F32Loop& L, floatx4 (&acc)[FBM / 16]) {
#pragma unroll
  for (int s = 0; s < FST - 1; ++s) f32_issue<NT>(L, s, s);  // nk >= 4 (K is a multiple of 128)
  const int sw = swz(L.lrow, 0), last = L.nk - 1;
  int slot = 0;
  for (int s = 0; s < L.nk; ++s) {
    // this wavefront's loads of stage s have landed and its reads of stage
    // s-1 are done before the barrier publishes the one and frees the other;
    // past the last stage that one is loaded again into a slot nobody reads,
    // so the count in flight is a constant
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    wait_vm<(FST - 2) * kF32Loads>();
    bar();
    f32_issue<NT>(L, min(s + FST - 1, last), slot == 0 ? FST - 1 : slot - 1);
    const float* st = L.smem + slot * kF32Stage + L.lrow * FBK;
#pragma unroll
    for (int kc = 0; kc < FBK / 16; ++kc) {
      const int ch = ((4 * kc + L.quarter) ^ sw) * 4;
      floatx4 a[NACT];
      const floatx4 b = *reinterpret_cast<const floatx4*>(st + (FBM + 16 * L.wave) * FBK + ch);
#pragma unroll
      for (int mb = 0; mb < NACT; ++mb) a[mb] = *reinterpret_cast<const floatx4*>(st + 16 * mb * FBK + ch);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int mb = 0; mb < NACT; ++mb)
          acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[i], a[mb][i], acc[mb], 0, 0, 0);
    }
    slot = slot == FST - 1 ? 0 : slot + 1;
  }
  wait_vm<0>();  // the reloads past the last stage, before the ring is written again
}

template <int MODE>
__global__ __launch_bounds__(64 * kF32Waves, kF32Waves * kF32PerCu / 4) void grouped_gemm_f32(
    GroupedProblem p, WeightTable wt, const float* __restrict__ A, float* __restrict__ C, int n_ntiles) {
  // One array for the ring and the next item's index: with two LDS variables
  // the compiler tells their accesses apart and then guards every fragment
  // read with a wait for all loads into the ring.
  __shared__ __attribute__((aligned(1024))) float smem[FST * kF32Stage + 4];
  int* s_next = reinterpret_cast<int*>(smem + FST * kF32Stage);
  // the ring is written by global->LDS loads the compiler does not see
  asm volatile("" ::"v"(smem) : "memory");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 15, quarter = lane >> 4;
  const int K = MODE == MODE_GATEUP ? p.H : p.F;
  const int ES = p.E + p.S;
  ItemQueue q(p, n_ntiles);
  if (tid == 0) *s_next = q.first();
  __syncthreads();
  int it = __builtin_amdgcn_readfirstlane(*s_next);

  while (it >= 0) {
    int got = 0;
    if (tid == 0) got = q.draw();
    const int4 gd = scalar_record(p.tiles, it / n_ntiles);  // key, first row, rows, first m-tile
    const int mt = (gd.z + FBM - 1) / FBM;
    const Tile2 tile = item_tile(it - gd.w * n_ntiles, mt, n_ntiles);
    // the group's m-tiles share its rows evenly in whole 16-row blocks
    const int rpt = 16 * ((gd.z + 16 * mt - 1) / (16 * mt));
    const int row0 = gd.y + tile.mi * rpt, rows = min(gd.y + gd.z - row0, rpt);
    const int layer = gd.x / ES, e = gd.x - layer * ES;
    // the wavefront's 16 weight rows: two runs of 8
    const float* B0;
    const float* B1;
    if (MODE == MODE_GATEUP) {
      B0 = static_cast<const float*>(wt.gu[layer]) + ((size_t)e * 2 * p.F + tile.ni * (FBN / 2) + 8 * wave) * K;
      B1 = B0 + (size_t)p.F * K;
    } else {
      B0 = static_cast<const float*>(wt.dn[layer]) + ((size_t)e * p.H + tile.ni * FBN + 16 * wave) * K;
      B1 = B0 + (size_t)8 * K;
    }
    F32Loop L;
    L.smem = smem;
    L.ra = buffer_rsrc(A + (size_t)row0 * K, (uint32_t)(rows * K * 4));  // rows past the item's read zeros
    L.rb[0] = buffer_rsrc(B0, (uint32_t)(8 * K * 4));
    L.rb[1] = buffer_rsrc(B1, (uint32_t)(8 * K * 4));
    {
      const int lr = lane >> 3, c = (lane & 7) ^ (lr >> 1);  // chunk in an even 8-row block; odd ones flip bit 2
      L.a_off = (8 * wave + lr) * K * 4 + (c ^ ((wave & 1) * 4)) * 16;
      L.b_off[0] = lr * K * 4 + c * 16;
      L.b_off[1] = lr * K * 4 + (c ^ 4) * 16;
    }
    L.wave = wave;
    L.lrow = lrow;
    L.quarter = quarter;
    L.nk = K / FBK;
    floatx4 acc[FBM / 16];
#pragma unroll
    for (int mb = 0; mb < FBM / 16; ++mb) acc[mb] = (floatx4){0.f, 0.f, 0.f, 0.f};
    const int nact = (rows + 15) >> 4;
    switch (nact) {
      case 1:
        if (p.layer_tokens <= kNtTokens) f32_k_loop<1, true>(L, acc);
        else f32_k_loop<1, false>(L, acc);
        break;
      case 2: f32_k_loop<2, false>(L, acc); break;
      case 3: f32_k_loop<3, false>(L, acc); break;
      default: f32_k_loop<4, false>(L, acc); break;
    }
    // acc[mb][v]: token row 16 mb + lane % 16, weight row 4 (lane / 16) + v.
    // Gate/up: the upper 32 lanes hold the up rows of the lower lanes' gate
    // rows; the lower lanes finish even row blocks, the upper ones odd blocks.
    const bool hi = quarter >= 2;
#pragma unroll
    for (int mb = 0; mb < FBM / 16; ++mb) {
      if (mb >= nact) continue;
      if constexpr (MODE == MODE_GATEUP) {
        if (mb & 1) continue;
        floatx4 g, u;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float x = __shfl_xor(hi ? acc[mb][v] : acc[mb + 1][v], 32, 64);
          g[v] = hi ? x : acc[mb][v];
          u[v] = hi ? acc[mb + 1][v] : x;
        }
        const int r = 16 * (mb + hi) + lrow;
        if (r < rows)
          *reinterpret_cast<float4*>(C + (size_t)(row0 + r) * p.F + tile.ni * (FBN / 2) + 8 * wave +
                                     4 * (quarter & 1)) =
              make_float4(swiglu(g[0], u[0]), swiglu(g[1], u[1]), swiglu(g[2], u[2]), swiglu(g[3], u[3]));
      } else {
        const int r = 16 * mb + lrow;
        if (r < rows)
          *reinterpret_cast<float4*>(C + (size_t)(row0 + r) * p.H + tile.ni * FBN + 16 * wave + 4 * quarter) =
              make_float4(acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]);
      }
    }
    if (tid == 0) *s_next = q.settle(got);
    bar_lds();  // every wavefront is done with the ring; the next item is published
    it = __builtin_amdgcn_readfirstlane(*s_next);
    bar_lds();  // and read, before the next one overwrites it
  }
}

// o = dtype(p0 + p1) for the K halves of a split down GEMM, 4 elements per
// thread over the live rows *P_live (H is a multiple of 256); the second
// half starts `stride` floats after the first.
__global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ part, long long stride,
                                                        const int32_t* __restrict__ P_live, int H,
                                                        bf16_t* __restrict__ o) {
  const long long i = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= (long long)(*P_live) * H) return;
  const float4 a = *reinterpret_cast<const float4*>(part + i);
  const float4 b = *reinterpret_cast<const float4*>(part + stride + i);
  uint2 u;
  u.x = (uint32_t)f32_to_bf16(a.x + b.x) | ((uint32_t)f32_to_bf16(a.y + b.y) << 16);
  u.y = (uint32_t)f32_to_bf16(a.z + b.z) | ((uint32_t)f32_to_bf16(a.w + b.w) << 16);
  *reinterpret_cast<uint2*>(o + i) = u;
}

// Packed bf16 expert weights.  An expert matrix W [N][K] (gate/up: N = 2F
// rows, gate rows f then up rows F + f, K = H; down: N = H, K = F) becomes
// (K / 64) x (N / 256) blocks of 256 x 64 elements (32 KB), block (s, t) at
// index s * (N / 256) + t holding K columns 64 s .. 64 s + 63 of column tile
// t.  Block row r is weight row
//   down:     256 t + r
//   gate/up:  128 t + 32 (r / 64) + (r % 64 < 32 ? r % 64 : r % 64 - 32 + F)
// (the 64 rows of wavefront column r / 64 are 32 gate rows and the matching
// 32 up rows), and its 16-byte chunk at position c holds the 8 K columns
// 64 s + 8 (c ^ ((r >> 1) & 7)) .. + 7 (the LDS swizzle of the ring).
// One thread per 16-byte chunk of dst; n matrices back to back.
__global__ __launch_bounds__(256) void pack_bf16_kernel(const uint4* __restrict__ src,
                                                        uint4* __restrict__ dst, long long chunks,
                                                        int N, int K, int F, int gateup) {
  const long long per_mat = (long long)N * K / 8;
  const int ntiles = N / BN;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < chunks;
       i += (long long)gridDim.x * blockDim.x) {
    const long long mat = i / per_mat;
    const int rem = (int)(i - mat * per_mat);
    const int blk = rem / (BN * BK / 8), in = rem - blk * (BN * BK / 8);
    const int r = in >> 3, c = in & 7;
    const int st = blk / ntiles, t = blk - st * ntiles;
    int row;
    if (gateup) {
      const int q = r & 63;
      row = t * (BN / 2) + (r >> 6) * 32 + (q < 32 ? q : q - 32 + F);
    } else {
      row = t * BN + r;
    }
    const int col = st * BK + 8 * swz(r, c);
    dst[i] = src[mat * per_mat + ((long long)row * K + col) / 8];
  }
}

}  // namespace

int gemm_bm(int dtype) { return dtype == EB_DTYPE_BF16 ? BM : FBM; }

// Row blocks to set aside for the end of a launch (see ItemQueue): one and a
// half gate/up items per workgroup (the down launch has the same list: 1.1
// items at H = 2048, F = 1408, 2.6 at H = 7168, F = 2048), from groups of up to
// half a tile, whose items take half as long as a full tile's.  Without them
// the workgroups ended up to one long item apart: gate/up of 8192 tokens on
// 256 experts of H = 7168, F = 2048 4050 -> 3990 us (its down launch gains
// nothing from them), of three 512-token micro-batches on 8 experts of
// H = 4096, F = 14336 940 -> 920 us.  fp32 items are short as they are (no
// gain).  Where the down launch splits K, only groups of the 64-row tile shape:
// a 65- to 128-row item of K = 7168 is nearly as long as a full tile's, and ends
// the launch late (768 tokens on those 8 experts, down launch 363 us with
// them, 346 without; a whole pass of that stack, its nine down launches 4.93
// ms, 4.66 with the rule of ItemQueue as well).
TailRule gemm_tail(int dtype, int F) {
  if (dtype != EB_DTYPE_BF16) return TailRule{0, 0};
  const int nsub = F / (BN / 2);
  return TailRule{(384 + nsub - 1) / nsub, down_ksplit(dtype, F) > 1 ? CfgSkinny::BM : BM / 2};
}

hipError_t launch_pack_weights(int dtype, int gateup, int n, int N, int K, int F, const void* src,
                               void* dst, hipStream_t s) {
  const size_t elem = dtype == EB_DTYPE_BF16 ? 2 : 4;
  const size_t bytes = (size_t)n * N * K * elem;
  if (bytes == 0) return hipSuccess;
  if (dtype != EB_DTYPE_BF16) return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s);
  const long long chunks = (long long)(bytes / 16);
  const long long want = (chunks + 255) / 256;
  const unsigned grid = (unsigned)(want < 65536 ? want : 65536);
  hipLaunchKernelGGL(pack_bf16_kernel, dim3(grid), dim3(256), 0, s, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), chunks, N, K, F, gateup);
  return hipGetLastError();
}

static int persistent_grid() {
  static int grid = 0;
  if (grid == 0) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    grid = (cus + kXcds - 1) / kXcds * kXcds;
  }
  return grid;
}

// Whether a launch's groups are so small that it only streams weights: at
// most 32 tokens at any layer by the bound the host has (one MFMA block of
// rows), and K long enough for the streams' look-ahead.  Up to 64 tokens (two blocks, 16 KB ring slots) the
// 256-column items measured the same or faster.
static bool stream_launch(const GroupedProblem& p) {
  return p.layer_tokens <= 32 && p.H / BK >= kStreamMinStages && p.F / BK / p.ksplit >= kStreamMinStages;
}

template <int MODE, int NA>
static void launch_stream_na(const GroupedProblem& p, const WeightTable& wt, const bf16_t* A, bf16_t* C, hipStream_t s) {
  hipLaunchKernelGGL((stream_gemm_bf16<MODE, NA>), dim3(kStreamPerCu * persistent_grid()), dim3(64), 0, s, p, wt, A, C);
}
template <int MODE>
static void launch_stream(const GroupedProblem& p, const WeightTable& wt, const bf16_t* A, bf16_t* C, hipStream_t s) {
  if (p.layer_tokens <= 8) launch_stream_na<MODE, 1>(p, wt, A, C, s);
  else if (p.layer_tokens <= 16) launch_stream_na<MODE, 2>(p, wt, A, C, s);
  else launch_stream_na<MODE, 4>(p, wt, A, C, s);
}

hipError_t launch_gateup(int dtype, const GroupedProblem& p, const WeightTable& wt,
                         const void* a_perm, void* h, hipStream_t s) {
  prof_start(EB_K_GATEUP, s);
  if (dtype == EB_DTYPE_BF16 && stream_launch(p)) {
    launch_stream<MODE_GATEUP>(p, wt, static_cast<const bf16_t*>(a_perm), static_cast<bf16_t*>(h), s);
  } else if (dtype == EB_DTYPE_BF16) {
    hipLaunchKernelGGL(grouped_gemm_bf16<MODE_GATEUP>, dim3(persistent_grid()), dim3(kThreads), 0, s,
                       p, wt, static_cast<const bf16_t*>(a_perm), static_cast<bf16_t*>(h),
                       p.F / (BN / 2));
  } else {
    hipLaunchKernelGGL(grouped_gemm_f32<MODE_GATEUP>, dim3(kF32PerCu * persistent_grid()), dim3(64 * kF32Waves), 0,
                       s, p, wt, static_cast<const float*>(a_perm), static_cast<float*>(h), p.F / (FBN / 2));
  }
  prof_stop(EB_K_GATEUP, s);
  return hipGetLastError();
}

hipError_t launch_down(int dtype, const GroupedProblem& p, const WeightTable& wt, const void* h,
                       void* o, hipStream_t s, bool sum_halves) {
  prof_start(EB_K_DOWN, s);
  if (dtype == EB_DTYPE_BF16) {
    if (stream_launch(p))
      launch_stream<MODE_DOWN>(p, wt, static_cast<const bf16_t*>(h), static_cast<bf16_t*>(o), s);
    else
      hipLaunchKernelGGL(grouped_gemm_bf16<MODE_DOWN>, dim3(persistent_grid()), dim3(kThreads), 0, s,
                         p, wt, static_cast<const bf16_t*>(h), static_cast<bf16_t*>(o), p.H / BN);
    if (p.ksplit > 1 && sum_halves) {
      const long long n = (long long)p.P * p.H;
      hipLaunchKernelGGL(split_sum_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s,
                         p.partial, n, p.P_live, p.H, static_cast<bf16_t*>(o));
    }
  } else {
    hipLaunchKernelGGL(grouped_gemm_f32<MODE_DOWN>, dim3(kF32PerCu * persistent_grid()), dim3(64 * kF32Waves), 0, s,
                       p, wt, static_cast<const float*>(h), static_cast<float*>(o), p.H / FBN);
  }
  prof_stop(EB_K_DOWN, s);
  return hipGetLastError();
}

}  // namespace eb
