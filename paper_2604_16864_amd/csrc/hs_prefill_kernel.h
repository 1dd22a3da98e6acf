// Prefill attention: Algorithm 1 (Trans-Both: S^T = K Q^T, O^T = V^T P^T with K and V^T as
// the first, possibly 2:4-sparse, operand of the matrix instruction) with the mixed
// dense/sparse dispatch of Sec. III-C-2, online softmax, and tile skipping.
//
// Work decomposition: a "slab" is 16 NB consecutive query positions of one query head (NB = 2: 32 positions; NB = 1 where
// these would leave compute units idle, hs_prefill.hip); a wave owns one slab, keeps Q^T (B operand of GEMM1), the running softmax
// state and O^T (128 x 16 NB fp32) in registers for the whole kernel.  The 4 waves of a
// workgroup take 4 consecutive slabs in (position-tile, head-in-group) order, so for a GQA
// group of 4 they are the 4 query heads of one position tile and share every KV tile, which is
// copied once per workgroup into an LDS ring by direct global->LDS loads issued up to 2 tiles
// ahead.  Pools are stored in operand order, so LDS reads are conflict-free 16-byte-per-lane
// reads and GEMM1's accumulators become GEMM2's B operand in place (no re-layout step).
#pragma once
#include <type_traits>

#include "hs_common.h"

// Wave priority per phase.  Two waves share a SIMD; letting the one that is in its vector-ALU
// (softmax) phase issue first measured ~5 % faster than equal priorities or the opposite choice.
#ifndef HS_PRIO_MFMA
#define HS_PRIO_MFMA 0
#define HS_PRIO_VALU 1
#endif


namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  bf2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

// p0, p1 -> hi = packed bf16 pair (round to nearest even) and lo = packed bf16 pair of the
// remainders p - hi, so that hi + lo reproduces p to ~16 bits.  The remainder is taken with the
// packed dot product hi . (-1, 0) + p0 (resp. (0, -1) + p1): one instruction per element, and
// exact, because bf16 products are exact in fp32 and p - hi is representable.
// The two selector pairs (-1, 0) and (0, -1) are handed in as opaque register values: written
// as literals the compiler folds the first into the inline constant -1.0, which the
// instruction does not read as the bf16 pair (-1, 0).
struct SplitConsts { uint32_t neg_lo, neg_hi; };
__device__ __forceinline__ SplitConsts split_consts() {
  SplitConsts c;
  asm volatile("s_mov_b32 %0, 0x0000bf80\n\ts_mov_b32 %1, 0xbf800000" : "=s"(c.neg_lo), "=s"(c.neg_hi));
  return c;
}
__device__ __forceinline__ void split_hi_lo(float p0, float p1, const SplitConsts& sc, uint32_t& hi, uint32_t& lo) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  hi = pack_bf16(p0, p1);
  const bf2 h = __builtin_bit_cast(bf2, hi);
  const float r0 = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf2, sc.neg_lo), p0, false);
  const float r1 = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf2, sc.neg_hi), p1, false);
  lo = pack_bf16(r0, r1);
}

// LDS staging ring.  One stage holds one tile: a K region then a V region, each 9 KiB (8 KiB of
// values + 1 KiB of metadata) when every tile of that tensor is 2:4 and 16 KiB otherwise.  Two
// workgroups share a compute unit's 160 KiB, so a ring may take 80 KiB: 3 stages when at least one
// tensor is all 2:4, 2 otherwise.  With 3 stages a tile is requested two tiles ahead: with the barrier in mid-iteration (MID
// below) one iteration before it is waited for, and nothing else is in flight then; with the barrier at the end nearly two,
// and the tile behind it stays in flight.  A fourth stage would fit when both tensors are 2:4: a 2K prompt takes 43.4 us with
// it and 41.7 with 3, one of 8K 357 and 352 (one tile less to wait for before the first is worked on, less state per tile);
// longer ones differ by less than two runs of one side.
template <int KM> constexpr int region_bytes() { return KM == 0 ? 9216 : 16384; }
template <int KM, int VM> constexpr int stage_bytes() { return region_bytes<KM>() + region_bytes<VM>(); }
#ifndef HS_MAX_STAGES
#define HS_MAX_STAGES 3  // at most 4: stage_wait leaves up to two tiles in flight
#endif
template <int KM, int VM> constexpr int n_stages() {
  constexpr int fit = 81920 / stage_bytes<KM, VM>();
  return fit < HS_MAX_STAGES ? fit : HS_MAX_STAGES;
}
// fewest direct-to-LDS loads any of the 4 waves issues for one tile (chunks / 4; the metadata
// chunks go to waves 0 and 1 on top of that)
template <int KM, int VM> constexpr int min_loads_per_tile() { return (KM == 1 ? 4 : 2) + (VM == 1 ? 4 : 2); }

typedef __attribute__((address_space(3))) void* lptr_t;

// One direct global->LDS load of 64 lanes x 16 B: lane l's bytes come from gbase + voff (voff = 16 l
// plus the tile's offset in its pool) and land at LDS address lds_addr + IMM + 16 l.  Written as
// inline assembly on purpose: the compiler treats the built-in form as a vector-memory write to LDS
// that any later LDS read may alias, and puts a full vmcnt(0) wait in front of the first such read,
// i.e. right after the prefetch is issued.  Completion is tracked by hand instead (stage_wait +
// workgroup barrier before a stage is read).  gbase and lds_addr are wave-uniform.
template <int IMM>
__device__ __forceinline__ void lds_dma16(uint32_t lds_addr, const uint8_t* gbase, uint32_t voff) {
  asm volatile("s_add_i32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
               :
               : "s"(lds_addr), "i"(IMM), "v"(voff), "s"((uint64_t)gbase)
               : "memory", "m0", "scc");
}

__device__ __forceinline__ const uint8_t* uniform_ptr(const uint8_t* p) {
  const uint64_t g = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)g);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(g >> 32));
  return (const uint8_t*)(((uint64_t)hi << 32) | lo);
}

// Where a wave's copies of a tile come from: the pools of the workgroup's (batch, kv head) row with the
// wave's share of the 1 KiB chunks folded in (value chunk c of a tile goes to wave c % 4), one
// pointer per chunk, so that a tile costs one shift-add for its offset in the pool and nothing
// else per copy.  The per-tile scalar work counts: it is issued by every wave for every tile.
struct TileSrc {
  const uint8_t *k_sp[2], *k_meta, *k_dn[4], *v_sp[2], *v_meta, *v_dn[4];
};
template <int KM, int VM>
__device__ __forceinline__ TileSrc tile_src(const hs_kv_dev& kv, int64_t row, int w) {
  TileSrc s = {};
  if (KM != 1) {
    const uint8_t* b = kv.k_nnz + row * kv.cap_sparse_k * (int64_t)HS_TILE_NNZ_BYTES + w * 1024;
    s.k_sp[0] = uniform_ptr(b);
    s.k_sp[1] = uniform_ptr(b + 4096);
    s.k_meta = uniform_ptr(kv.k_meta + row * kv.cap_sparse_k * (int64_t)HS_TILE_META_BYTES);
  }
  if (KM != 0) {
    const uint8_t* b = kv.k_dense + row * kv.cap_dense_k * (int64_t)HS_TILE_DENSE_BYTES + w * 1024;
#pragma unroll
    for (int i = 0; i < 4; i++) s.k_dn[i] = uniform_ptr(b + 4096 * i);
  }
  if (VM != 1) {
    const uint8_t* b = kv.v_nnz + row * kv.cap_sparse_v * (int64_t)HS_TILE_NNZ_BYTES + w * 1024;
    s.v_sp[0] = uniform_ptr(b);
    s.v_sp[1] = uniform_ptr(b + 4096);
    s.v_meta = uniform_ptr(kv.v_meta + row * kv.cap_sparse_v * (int64_t)HS_TILE_META_BYTES);
  }
  if (VM != 0) {
    const uint8_t* b = kv.v_dense + row * kv.cap_dense_v * (int64_t)HS_TILE_DENSE_BYTES + w * 1024;
#pragma unroll
    for (int i = 0; i < 4; i++) s.v_dn[i] = uniform_ptr(b + 4096 * i);
  }
  return s;
}

// Copy one tile (K and V operands) from its pool slots into an LDS stage: a chunk is 64 lanes x 16 B =
// 1 KiB, stored in the pools in the order the lanes consume it.  The 4 waves share the chunks
// round-robin.  2:4 tile: 8 value chunks + 1 metadata chunk per tensor (value chunks at 0..8 KiB,
// metadata at 8 KiB of the tensor's region); dense: 16 chunks.  stage_w = LDS address of the stage
// + 1024 w.  Offsets inside a row's pool are 32-bit (the launcher checks the pool sizes).
template <int KM, int VM>
__device__ __forceinline__ void stage_issue(uint32_t stage_w, const TileSrc& src, int mk, int mv, int w,
                                            uint32_t lane_off) {
  const bool k_sparse = KM == 0 || (KM == 2 && mk < 0);
  const bool v_sparse = VM == 0 || (VM == 2 && mv < 0);
  constexpr int voff = region_bytes<KM>();
  if (k_sparse) {
    const uint32_t slot = (uint32_t)~mk;  // -mk - 1
    const uint32_t off = lane_off + slot * (uint32_t)HS_TILE_NNZ_BYTES;
    lds_dma16<0>(stage_w, src.k_sp[0], off);
    lds_dma16<4096>(stage_w, src.k_sp[1], off);
    if (w == 0) lds_dma16<8192>(stage_w, src.k_meta, lane_off + slot * (uint32_t)HS_TILE_META_BYTES);
  } else {
    const uint32_t off = lane_off + (uint32_t)(mk - 1) * (uint32_t)HS_TILE_DENSE_BYTES;
    lds_dma16<0>(stage_w, src.k_dn[0], off);
    lds_dma16<4096>(stage_w, src.k_dn[1], off);
    lds_dma16<8192>(stage_w, src.k_dn[2], off);
    lds_dma16<12288>(stage_w, src.k_dn[3], off);
  }
  if (v_sparse) {
    const uint32_t slot = ((uint32_t)(-mv) & 0x3fffffffu) - 1u;  // -mv = slot + 1 (+ the encoding bit)
    const uint32_t off = lane_off + slot * (uint32_t)HS_TILE_NNZ_BYTES;
    lds_dma16<voff>(stage_w, src.v_sp[0], off);
    lds_dma16<voff + 4096>(stage_w, src.v_sp[1], off);
    // wave 1's metadata chunk lands at the region's 8 KiB: stage_w already carries its 1024
    if (w == 1) lds_dma16<voff + 8192 - 1024>(stage_w, src.v_meta, lane_off + slot * (uint32_t)HS_TILE_META_BYTES);
  } else {
    const uint32_t off = lane_off + ((uint32_t)hs_map_plain(mv) - 1u) * (uint32_t)HS_TILE_DENSE_BYTES;
    lds_dma16<voff>(stage_w, src.v_dn[0], off);
    lds_dma16<voff + 4096>(stage_w, src.v_dn[1], off);
    lds_dma16<voff + 8192>(stage_w, src.v_dn[2], off);
    lds_dma16<voff + 12288>(stage_w, src.v_dn[3], off);
  }
}

// Wait until all but the newest `tiles_in_flight` tiles' worth of this wave's direct-to-LDS loads
// have landed (loads complete in order).  PER = loads per tile that every wave issues at least.  Two
// tiles are left in flight by a ring of 4 stages only; without that case the loops of bf16 caches come out
// up to 0.8 % slower (16K prompt 1326 against 1337 us).
// Immediate: vmcnt in bits 3..0 and 15..14, the other counters left at their maxima.
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }
template <int PER>
__device__ __forceinline__ void stage_wait(int tiles_in_flight) {
  static_assert(2 * PER <= 63, "vmcnt range");
  switch (tiles_in_flight) {
    case 0: __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); break;
    case 1: __builtin_amdgcn_s_waitcnt(vmcnt_imm(PER)); break;
    default: __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * PER)); break;
  }
}

// stage_wait with this wave's own load count per tile: waves 0 and 1 also fetch the metadata chunk of a
// 2:4 K resp. V tile.  (Waiting by the smallest count of any wave made those two wait for the first
// load of a tile requested only one iteration ago, and the workgroup with them at the barrier.)  Mixed
// tensors: the count varies per tile, the smallest is used.
template <int KM, int VM>
__device__ __forceinline__ void stage_wait_wave(int tiles_in_flight, int w) {
  constexpr int base = min_loads_per_tile<KM, VM>();
  if ((KM == 0 && w == 0) || (VM == 0 && w == 1)) stage_wait<base + 1>(tiles_in_flight);
  else stage_wait<base>(tiles_in_flight);
}

union B16 {  // one B operand of the 16x16x64 sparse instruction = two of the dense 16x16x32 one
  uint4 q[2];
  uint32_t u[8];
};

// KM / VM (per tensor): 0 = every tile 2:4 or skipped, 1 = every tile dense or skipped, 2 = any mix
// (the specialised all-dense / all-sparse kernels of Sec. IV-C-3, chosen per tensor so that the
// keys-dense / values-2:4 setting of Sec. V-A carries no dynamic dispatch).
// NB: column blocks (of 16 queries) per wave: a wave owns a slab of 16*NB query positions of one
// head.  NB = 2 fits 2 waves per SIMD (NB = 4, 1 wave per SIMD, measured 1.3-1.4x slower; NB = 3 at 2 waves spills: 16K prompt
// 1346 -> 1529 us); NB = 1 takes three quarters of its time for half of the work.
// F16: element type of the cache (hs_elem).  A V tile of a bf16 cache may be stored in fp16 encoding
// (HS_MAP_F16 in its map entry).  Against fp16 V the numerators have 11 significant bits and enter
// GEMM2 as one fp16 term; against bf16 V they enter as two bf16 terms.  The reference is kept
// kShift binades under the running maximum and renewed before a numerator can reach the fp16
// maximum (constants below).
// TEAMS (2 with NB = 1 and without SPLIT only): two teams of 4 waves share the workgroup's slabs and take its tiles in turn, each with a ring of its own, and
// combine through LDS at the end.  A wave alone on its SIMD leaves it idle most of a tile's time (1500 clocks, ~220 instructions
// and 16 products), so where a call has no second workgroup for a compute unit, 512 threads take two tiles in the time that 256
// take for 1.3; what bounds the pair is the LDS (90 KB read and written a tile, 720 clocks) and the barrier all 8 waves meet at.
// Slabs of 32 spill and lose (64 queries on 32768 tokens 39 / 39, 512 on 2048 36 / 33 against 22 with slabs of 16).
// SPLIT: the tiles a workgroup may look at are cut into gridDim.y ranges, one workgroup per range; each
// writes a normalised fp32 partial output and its log-sum-exp (ws_o [row][split][128], ws_l
// [row][split], row = (b, query head, query)) for the merge kernel instead of O and LSE.
template <int KM, int VM, int NB, int TEAMS, bool F16, bool SPLIT>
__global__ __launch_bounds__(256 * TEAMS, 2) void prefill_kernel(int Hq, int Hkv, int T, int Lq, int off,
                                                                      float scale_log2, int causal,
                                                                      const uint16_t* __restrict__ Q, hs_kv_dev kv,
                                                                      uint16_t* __restrict__ O,
                                                                      float* __restrict__ LSE, float* __restrict__ ws_o,
                                                                      float* __restrict__ ws_l) {
  static_assert(TEAMS == 1 || (NB == 1 && !SPLIT), "two teams: slabs of 16 in one range");
  typedef hs_elem<F16> E;
  typedef hs_elem<true> E16;
  // Reference = running maximum - kShift at the time it was last renewed; it is renewed when a lane's
  // partial row sum passes kRedo, i.e. before a numerator can pass 2^15 (fp16 holds 65504).  A new
  // score may thus exceed the maximum seen so far by 15 - kShift = 11 binades before the tile has
  // to be redone; with 8 / 2^14 (6 binades) keys with large channels redid 5 % of the work.
  // What fp16 flushes to zero lies 24 + kShift binades under the largest numerator: a context of
  // 2^17 tokens loses < 2^-11 of a row sum even if every other token sits just under that level.
  constexpr float kShift = 4.f;
  constexpr float kRedo = 0x1p15f;
  // FLAG: "a column has no reference yet" is kept as one scalar flag, tested once in front of the softmax, instead of a
  // comparison and a select per column in it; LITERAL: the causal mask compares with literals instead of with 16 constants
  // held in registers.  us with neither / both: all 2:4, 16K prompt 1318 / 1305, 16 prompts of 1K 157 / 150; bf16 with mixed values
  // (2:4 with dense ends) 8K 404 / 375, 192 queries on 25728 tokens 83.1 / 76.5.  With a tensor all dense the flag costs registers
  // that are not there (keys dense, 8K 409 / 433; both dense 486 / 490).  Other mixed tensors in slabs of 32 lose by both: fp16
  // with dense ends 356.5 / 352.2 at 8K, but 158.1 / 163.3 for 1408 queries on 9024 tokens and 85.3 / 87.7 for 192 on 25728; half of
  // the keys dense, 128 queries on 6912 tokens 31.4 / 32.2, fp16, 16 x 512 on 3776 88.7 / 90.4, 8K 399.6 / 401.2.
  constexpr bool MIXED = KM == 2 || VM == 2;
  constexpr bool FLAG = (KM == 0 && VM == 0) || (MIXED && (NB == 1 || (VM == 2 && !F16)));
  constexpr bool LITERAL = FLAG || !MIXED;
  constexpr int QS = 16 * NB;  // query positions per slab
  constexpr int NS = n_stages<KM, VM>(), D = NS - 1;  // ring size, prefetch distance in tiles
  // MID: the per-tile barrier sits between softmax and GEMM2 instead of at the end of the
  // iteration, so that the next tile's K operands can be fetched from LDS while GEMM2 runs.  Needs
  // the next tile requested an iteration before that barrier (NS >= 3: at least one tensor all 2:4).
  // It is used where every V tile the workgroup meets takes one fp16 term of P (fp16 caches; rows
  // of a bf16 cache whose V tiles are all in fp16 encoding): with both GEMM2 forms in the loop,
  // or mixed V, no registers are left for the K prefetch.
  constexpr bool MID_OK = KM != 2 && VM != 2 && NS >= 3;
  constexpr int kStage = stage_bytes<KM, VM>();
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[TEAMS * NS * kStage];
  const int tid = threadIdx.x, l = tid & 63, a = l >> 4, c = l & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, scalar: branches on it stay scalar
  const int w = TEAMS == 1 ? wave : wave & 3, team = TEAMS == 1 ? 0 : wave >> 2;
  uint8_t* const lds = lds_all + team * (NS * kStage);
  const int G = Hq / Hkv;
  // kv head = block index mod Hkv: workgroups go round-robin over the 8 XCDs, so with 8 kv heads (or a
  // divisor of 8) each XCD's L2 streams the tiles of its own heads only (measured 1-2.5 % faster)
  const int hkv = blockIdx.x % Hkv, b = blockIdx.z;
  const int n_slabs = (Lq / QS) * G;
  // heavy (late) query positions first: causal work grows with the position
  const int grp = (int)(gridDim.x / Hkv) - 1 - (int)(blockIdx.x / Hkv);
  const int slab = 4 * grp + w;
  const bool valid = slab < n_slabs;
  const int qpos = valid ? (slab / G) * QS : 0, hg = valid ? slab % G : 0;
  const int hq = hkv * G + hg;
  const int64_t row = (int64_t)b * Hkv + hkv;
  const int32_t* km = kv.k_map + row * T;
  const int32_t* vm = kv.v_map + row * T;
  const TileSrc src = tile_src<KM, VM>(kv, row, w);
  // query i (absolute position i + off) sees token j iff j <= i + off; last KV tile this wave /
  // the workgroup may look at, and first tile that needs masking inside
  const int jmax_w = causal ? (qpos + QS - 1 + off) / HS_BT : T - 1;
  const int last_slab = min(4 * grp + 3, n_slabs - 1);
  const int jmax_wg = causal ? min(T - 1, ((last_slab / G) * QS + QS - 1 + off) / HS_BT) : T - 1;
  // tiles t_lo .. t_last are this workgroup's: all it may look at, or its share of them (an inclusive end: with jmax_wg + 1
  // as an exclusive one the unsplit bf16 kernels spill more or schedule worse: keys dense / values 2:4 22 registers
  // instead of 11, 32768 tokens 6350 against 6312 us; mixed tensors, 1024 queries on 2048 tokens 42.3 against 41.3 us)
  const int n_splits = SPLIT ? (int)gridDim.y : 1, split = SPLIT ? (int)blockIdx.y : 0;
  const int t_lo = SPLIT ? (int)((int64_t)(jmax_wg + 1) * split / n_splits) : 0;
  const int t_last = SPLIT ? (int)((int64_t)(jmax_wg + 1) * (split + 1) / n_splits) - 1 : jmax_wg;

  // Q^T (B operand): column block nb, 64-channel block kb: query qpos+16nb+c, channels
  // 64kb + 32h + 8a + e for element 8h+e
  B16 qb[NB][2];
  {
    const uint16_t* qp = Q + (((int64_t)b * Hq + hq) * Lq + qpos + c) * HS_D + 8 * a;
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int h = 0; h < 2; h++)
          qb[nb][kb].q[h] = valid ? *reinterpret_cast<const uint4*>(qp + (int64_t)(16 * nb) * HS_D + 64 * kb + 32 * h)
                                  : make_uint4(0, 0, 0, 0);
  }

  f32x4_t o[8][NB];
#pragma unroll
  for (int mb = 0; mb < 8; mb++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) o[mb][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run[NB], l_run[NB];
  const SplitConsts sc = split_consts();
  bool no_ref = FLAG;  // a query column of this wave has no reference yet
#pragma unroll
  for (int nb = 0; nb < NB; nb++) { m_run[nb] = -INFINITY; l_run[nb] = 0.f; }

  // Map entries steer branches around matrix instructions, which ignore the EXEC mask: they are
  // forced into scalar registers so that those branches are scalar too.
  // tj[i]: the i-th visible tile from the current one on (-1: none), tk / tv: its map entries;
  // tile tj[i] sits in (or is on its way to) stage (st + i) % NS.
  int tj[NS], tk[NS], tv[NS];
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lptr_t)lds) + 1024 * w;
  const uint32_t lane_off = 16 * l;
  // The maps are read 64 tiles at a time, lane t of the window holding the entries of tile
  // wbase + t; entries are picked out with readlane and the next tile is found on a ballot.
  // This keeps map reads (vector loads, which complete in order with the tile loads and would
  // otherwise have to wait for them) off the per-tile path.
  // Order of the tiles: up to three groups, one after the other over the whole range, ascending
  // inside a group: V tile in fp16 encoding and 2:4 (or of the tensor's only kind); in fp16 encoding
  // and dense (mixed V tensors); V tile in bf16 encoding (bf16 caches: tiles with a value that fp16
  // does not hold, e.g. ~5 % of dense N(0,1) tiles, which contain a number under 2^-17).  Softmax
  // does not care about the order and the causal mask goes by the tile's index.  The loop below
  // exists once per GEMM2 form; with this order a workgroup changes form at most twice.  (A change
  // is not cheap: the loops hold the accumulators in different registers, and the spill reloads
  // the compiler puts on the way wait for the tile loads in flight as well.)
  int wbase = 0, wgroup = 0;
  int32_t wk = 0, wv = 0;
  uint64_t wrem = 0;  // tiles of the window still to hand out
  auto window_load = [&](int base) {
    const int t = base + l;
    wk = t <= t_last ? km[t] : 0;
    wv = t <= t_last ? vm[t] : 0;
    const bool g2 = !F16 && !hs_map_f16(wv);
    const bool g1 = !g2 && VM == 2 && wv > 0;
    const int grp = g2 ? 2 : (g1 ? 1 : 0);
    wrem = __ballot(wk != 0 && grp == wgroup);
    wbase = base;
  };
  auto next_of_all = [&]() -> int {  // next tile (<= t_last, not skipped) in the order above, or -1
    for (;;) {
      if (wrem != 0) {
        const int t = __builtin_ctzll(wrem);
        wrem &= wrem - 1;
        return wbase + t;
      }
      if (wbase + 64 <= t_last) {
        window_load(wbase + 64);
        continue;
      }
      do wgroup++;
      while ((wgroup == 1 && VM != 2) || (wgroup == 2 && F16));  // groups this kernel cannot meet
      if (wgroup > 2) return -1;
      window_load(t_lo);
    }
  };
  // Two teams take the tiles in turn; each walks the whole order and passes over the other's.
  bool pass_over = TEAMS > 1 && team != 0, unpaired = false;  // unpaired: the last tile of team 0 has none beside it
  auto next_tile = [&]() -> int {
    if (TEAMS == 1) return next_of_all();
    if (pass_over && next_of_all() < 0) return -1;
    const bool after_other = pass_over && team != 0;
    pass_over = true;
    const int t = next_of_all();
    unpaired = after_other && t < 0;
    return t;
  };
  int st = 0;
  window_load(t_lo);
#pragma unroll
  for (int i = 0; i < D; i++) {
    tj[i] = i == 0 || tj[i - 1] >= 0 ? next_tile() : -1;
    tk[i] = tv[i] = 0;
    if (tj[i] >= 0) {
      tk[i] = __builtin_amdgcn_readlane(wk, tj[i] - wbase); tv[i] = __builtin_amdgcn_readlane(wv, tj[i] - wbase);
      stage_issue<KM, VM>(lds_wave + i * kStage, src, tk[i], tv[i], w, lane_off);
    }
  }
  stage_wait<1>(0);
  __syncthreads();
  // 2:4 operands of the sparse instruction are fetched from LDS a phase ahead of their use:
  // V of the current tile before the softmax, K of the next tile before GEMM2 (MID mode).
  uint4 ak[8], kix, av[8], vix;
  auto k_fetch = [&](int stage) {
    const uint4* kl = reinterpret_cast<const uint4*>(lds + stage * kStage);
#pragma unroll
    for (int i = 0; i < 8; i++) ak[i] = kl[i * 64 + l];  // a 2:4 tile in full; the first two row blocks of a dense one
    if (KM != 1) kix = kl[512 + l];
  };
  auto request = [&]() {  // look up the tile D ahead and start its copy into the stage D ahead
    tj[D] = tj[D - 1] >= 0 ? next_tile() : -1;
    tk[D] = tv[D] = 0;
    if (tj[D] >= 0) {
      tk[D] = __builtin_amdgcn_readlane(wk, tj[D] - wbase); tv[D] = __builtin_amdgcn_readlane(wv, tj[D] - wbase);
      int sd = st + D;
      if (sd >= NS) sd -= NS;
      stage_issue<KM, VM>(lds_wave + sd * kStage, src, tk[D], tv[D], w, lane_off);
    }
  };
  // mid_tag: MID mode; only16_tag: every V tile ahead is known to be in fp16 encoding
  auto main_loop = [&](auto mid_tag, auto only16_tag) {
    constexpr bool MID = decltype(mid_tag)::value, ONLY16 = F16 || decltype(only16_tag)::value;
    // 2:4 V operands are fetched from LDS before the softmax, unless the K prefetch of MID mode already holds the registers (both
    // together spill; measured no gain there), which leaves fp16 caches with mixed keys.  us without / with it, half of the keys dense, slabs
    // of 16: one team 512 tokens 11.49 / 11.07, two teams 512 queries on 2048 23.6 / 22.8, in ranges 128 on 4096 24.5 / 23.7.
    constexpr bool V_EARLY = F16 && VM == 0 && !MID;
    // Whole rows of 2:4 tiles, slabs of 16: the score accumulators of the next tile are cleared among the products of GEMM2,
    // where the vector ALU is idle, instead of in front of GEMM1 (the sparse instruction accumulates in place): 512 tokens
    // 10.94 -> 10.70 us, 1024 tokens 18.9 -> 18.4.  Elsewhere the registers or the scheduling it costs are worth more (slabs of
    // 32: 16K prompt, fp16, 1 % slower, bf16 spills; ranges 3 %, mixed keys 3 % slower).
    constexpr bool CLEARED = NB == 1 && KM == 0 && VM == 0 && !SPLIT;
    typedef f32x4_t Scores[4][NB];
    auto clear = [](Scores& x) {
#pragma unroll
      for (int m = 0; m < 4; m++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++) x[m][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    Scores s_kept;
    if (CLEARED) clear(s_kept);
    // One iteration = one tile.  The loop exists once per GEMM2 form (V tile dense or 2:4, one fp16
    // term of P or two bf16 terms), so that each copy is straight-line code around its matrix
    // instructions and keeps the accumulators where they are (a per-tile branch around GEMM2 made
    // the compiler move all 64 accumulator registers in and out of the branch).  The form is
    // scalar: map entries come through v_readlane.
    // enc: 0 = V tile in bf16 encoding, 1 = in fp16 encoding; vkind: 0 = V tile 2:4, 1 = dense,
    // 2 = look at the tile (the tensor has one kind, or the rare bf16-encoded tiles of a mixed one)
    auto iteration = [&](auto enc, auto vkind) {
      constexpr int kEnc = decltype(enc)::value;
      const int j = tj[0], mk = tk[0], mv = tv[0];
      // END mode: request the tile D ahead now; its stage held the tile of the previous iteration,
      // which every wave has left behind (barrier at the end of that iteration)
      if (!MID) request();
      const bool ok = valid && j <= jmax_w;
      const bool k_sparse = KM == 0 || (KM == 2 && mk < 0);
      constexpr int kVK = decltype(vkind)::value;
      const bool v_sparse = kVK == 2 ? (VM == 0 || (VM == 2 && mv < 0)) : kVK == 0;
      constexpr bool v_f16 = kEnc == 1;
      const uint4* kl = reinterpret_cast<const uint4*>(lds + st * kStage);
      const uint4* vl = reinterpret_cast<const uint4*>(lds + st * kStage + region_bytes<KM>());
      B16 ph[NB], pl[NB];
      // V_TOP (slabs of 16, 2:4 V beside K of one kind): V's operands are requested first of all, so that they are there when the
      // softmax ends.  Two teams: 512 queries on 2048 tokens 22.8 -> 21.9 us, 192 on 896 13.1 -> 12.6; one team, all 2:4, fp16: 192 on 896
      // 13.8 -> 13.4, 1024 tokens 18.1 -> 17.8.  One team of a bf16 cache, whose registers it fills, loses (1344 queries on 2560 tokens 35.3 -> 36.6), and so does one beside dense keys (16 x 320 on 448 13.1 -> 13.5).
      constexpr bool V_TOP = NB == 1 && VM == 0 && KM != 2 && (TEAMS == 2 || (F16 && KM == 0));
      if (V_TOP && ok) {
        if (!MID) k_fetch(st);
#pragma unroll
        for (int i = 0; i < 8; i++) av[i] = vl[i * 64 + l];
        vix = vl[512 + l];
        __builtin_amdgcn_sched_barrier(0);
      }
      if (ok) {
        // ---------------- GEMM1: S^T[64 tokens x 16 NB queries] ----------------
        __builtin_amdgcn_s_setprio(HS_PRIO_MFMA);
        Scores s_tile;
        Scores& s = CLEARED ? s_kept : s_tile;
        if (!CLEARED) clear(s);
        if (k_sparse) {
          if (!MID && !V_TOP) k_fetch(st);
          const int kidx[4] = {(int)kix.x, (int)kix.y, (int)kix.z, (int)kix.w};
          // 4 NB independent accumulators between the two instructions that share one
#pragma unroll
          for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int m = 0; m < 4; m++)
              s[m][nb] = E::template smma<0>(ak[2 * m], qb[nb][0].q[0], qb[nb][0].q[1], s[m][nb], kidx[m]);
#pragma unroll
          for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int m = 0; m < 4; m++)
              s[m][nb] = E::template smma<1>(ak[2 * m + 1], qb[nb][1].q[0], qb[nb][1].q[1], s[m][nb], kidx[m]);
        } else {
          if (KM == 1) {
            // Row blocks 2 and 3 take the registers of 0 and 1 and are requested while the block between is multiplied: a block
            // read just in front of its products leaves the wave waiting for the LDS four times a tile (both tensors dense,
            // 8K prompt 516 -> 498 us).  Not where the kind is looked at per tile: the two arms then want different registers
            // for the operands and the loop spills (2:4 values, half of the keys dense, 398 -> 437).
            if (!MID && !V_TOP) {
#pragma unroll
              for (int i = 0; i < 8; i++) ak[i] = kl[i * 64 + l];
            }
#pragma unroll
            for (int m = 0; m < 4; m++) {
#pragma unroll
              for (int st = 0; st < 4; st++)
#pragma unroll
                for (int nb = 0; nb < NB; nb++)
                  s[m][nb] = E::mma(ak[4 * (m & 1) + st], qb[nb][st >> 1].q[st & 1], s[m][nb]);
              if (m < 2) {
#pragma unroll
                for (int st = 0; st < 4; st++) ak[4 * m + st] = kl[(4 * (m + 2) + st) * 64 + l];
                __builtin_amdgcn_sched_barrier(0);
              }
            }
          } else {
#pragma unroll
            for (int m = 0; m < 4; m++) {
              uint4 a4[4];
#pragma unroll
              for (int st = 0; st < 4; st++) a4[st] = kl[(4 * m + st) * 64 + l];
#pragma unroll
              for (int st = 0; st < 4; st++)
#pragma unroll
                for (int nb = 0; nb < NB; nb++)
                  s[m][nb] = E::mma(a4[st], qb[nb][st >> 1].q[st & 1], s[m][nb]);
            }
          }
        }
        if (V_EARLY) {  // V operands: on their way while the softmax runs
#pragma unroll
          for (int i = 0; i < 8; i++) av[i] = vl[i * 64 + l];
          vix = vl[512 + l];
          __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(HS_PRIO_VALU);
        // causal mask inside a tile that reaches past the slab's first query
        if (causal && HS_BT * j + HS_BT - 1 > qpos + off) {
          // query 16nb+c sees in-tile token 16m+4a+i iff 16m+4a+i <= lim + 16nb
          const int lim = qpos + off - HS_BT * j + c, lim_a = lim - 4 * a;
#pragma unroll
          for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int m = 0; m < 4; m++)
#pragma unroll
              for (int i = 0; i < 4; i++)
                if (LITERAL ? 16 * m + i - 16 * nb > lim_a : 16 * m + 4 * a + i > lim + 16 * nb) s[m][nb][i] = -INFINITY;
        }
        // ---------------- P = exp2(S*scale - m_run), reference m_run updated lazily ----------------
        // P is first computed against the current reference of each query column, with no look at
        // the tile's maximum.  Only if a partial row sum comes out huge (or the column has no
        // reference yet) is the exact running maximum taken, O and l rescaled, and P recomputed.
        // With a stale reference P merely holds larger numbers (harmless in fp32 / bf16); the final
        // O / l and LSE = m_run + log2(l) do not depend on which reference was used.
        // P goes through the matrix unit as two bf16 terms (hi + remainder): a single bf16 P alone
        // costs ~1.3e-3 mean relative error on the output, on top of the bf16 rounding of O itself.
        float psum[NB];
        auto softmax_as = [&](auto enc, auto safe) {  // enc: std::true_type = fp16 numerators, one term
          constexpr bool kF16 = decltype(enc)::value;
#pragma unroll
          for (int nb = 0; nb < NB; nb++) {
            float acc = 0.f;
            const float mref = decltype(safe)::value && !(m_run[nb] > -INFINITY) ? 0.f : m_run[nb];
#pragma unroll
            for (int m = 0; m < 4; m++) {
              float p[4];
#pragma unroll
              for (int i = 0; i < 4; i++) {
                p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[m][nb][i], scale_log2, -mref));
                acc += p[i];
              }
              if (kF16) {
                ph[nb].u[2 * m] = E16::pack2(p[0], p[1]);
                ph[nb].u[2 * m + 1] = E16::pack2(p[2], p[3]);
              } else {
                split_hi_lo(p[0], p[1], sc, ph[nb].u[2 * m], pl[nb].u[2 * m]);
                split_hi_lo(p[2], p[3], sc, ph[nb].u[2 * m + 1], pl[nb].u[2 * m + 1]);
              }
            }
            psum[nb] = acc;
          }
        };
        auto softmax_tile = [&](auto safe) { softmax_as(std::integral_constant<bool, v_f16>{}, safe); };
        bool redo = no_ref;
        if (!no_ref) {
          softmax_tile(std::integral_constant<bool, !FLAG>{});
          bool big = false;
#pragma unroll
          for (int nb = 0; nb < NB; nb++) big = big || !(psum[nb] <= kRedo) || (!FLAG && !(m_run[nb] > -INFINITY));
          redo = __any(big);
        }
        if (redo) {
          bool none = false;
#pragma unroll
          for (int nb = 0; nb < NB; nb++) {
            float mx = s[0][nb][0];
#pragma unroll
            for (int m = 0; m < 4; m++)
#pragma unroll
              for (int i = 0; i < 4; i++) mx = fmaxf(mx, s[m][nb][i]);
            mx = mx * scale_log2 - kShift;
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // a column with nothing visible in this tile keeps its reference
            const float m_new = fmaxf(m_run[nb], mx);
            const float alpha = m_new > -INFINITY ? __builtin_amdgcn_exp2f(m_run[nb] - m_new) : 1.0f;
            m_run[nb] = m_new;
            none = none || !(m_new > -INFINITY);
            l_run[nb] *= alpha;
#pragma unroll
            for (int mb = 0; mb < 8; mb++) o[mb][nb] *= alpha;
          }
          if (FLAG) no_ref = __any(none);
          softmax_tile(std::true_type{});
        }
#pragma unroll
        for (int nb = 0; nb < NB; nb++) l_run[nb] += psum[nb];
      }
      if (MID) {
        // The next tile must have landed in full (own loads, then everybody's: barrier) before its K
        // operands are fetched; with a ring of 3 it is the newest one requested.  The stage of the
        // previous tile is free from here on (all of its reads precede this barrier).
        int later = 0;
#pragma unroll
        for (int i = 2; i < D; i++) later += tj[i] >= 0;
        stage_wait_wave<KM, VM>(later, w);
        __syncthreads();
        request();
        if (valid && tj[1] >= 0) {
          k_fetch(st + 1 == NS ? 0 : st + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (ok) {
        __builtin_amdgcn_s_setprio(HS_PRIO_MFMA);
        if (v_sparse) {
          if (!V_EARLY && !V_TOP) {
#pragma unroll
            for (int i = 0; i < 8; i++) av[i] = vl[i * 64 + l];
            vix = vl[512 + l];
          }
          const int vidx[4] = {(int)vix.x, (int)vix.y, (int)vix.z, (int)vix.w};
          if (v_f16) {  // one fp16 term
#pragma unroll
            for (int nb = 0; nb < NB; nb++)
#pragma unroll
              for (int mb = 0; mb < 8; mb++) {
                if (mb & 1)
                  o[mb][nb] = E16::template smma<1>(av[mb], ph[nb].q[0], ph[nb].q[1], o[mb][nb], vidx[mb >> 1]);
                else
                  o[mb][nb] = E16::template smma<0>(av[mb], ph[nb].q[0], ph[nb].q[1], o[mb][nb], vidx[mb >> 1]);
                if (CLEARED && (mb & 1)) {  // accumulator (mb / 2, nb) of the next tile's scores
                  s_kept[mb >> 1][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                  asm volatile("" : "+v"(s_kept[mb >> 1][nb]));
                }
              }
          } else {
            if (CLEARED) clear(s_kept);
#pragma unroll
            for (int t2 = 0; t2 < 2; t2++)  // first the upper-half term of every block, then the remainder
#pragma unroll
              for (int nb = 0; nb < NB; nb++)
#pragma unroll
                for (int mb = 0; mb < 8; mb++) {
                  const B16& bp = t2 == 0 ? ph[nb] : pl[nb];
                  if (mb & 1)
                    o[mb][nb] = E::template smma<1>(av[mb], bp.q[0], bp.q[1], o[mb][nb], vidx[mb >> 1]);
                  else
                    o[mb][nb] = E::template smma<0>(av[mb], bp.q[0], bp.q[1], o[mb][nb], vidx[mb >> 1]);
                }
          }
        } else {
          // V of one kind: four row blocks are in flight, and the registers of a block are requested anew while the next one is
          // multiplied (read block by block, as mixed tensors do for want of registers, each of the eight waits for the LDS: both
          // tensors dense, 8K prompt 498 -> 485 us, 2:4 keys with dense values 432 -> 418).
          constexpr bool PIPE = VM == 1;
          if (PIPE) {
#pragma unroll
            for (int i = 0; i < 8; i++) av[i] = vl[i * 64 + l];
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int mb = 0; mb < 8; mb++) {
            const uint4 a0 = PIPE ? av[2 * (mb & 3)] : vl[(2 * mb) * 64 + l], a1 = PIPE ? av[2 * (mb & 3) + 1] : vl[(2 * mb + 1) * 64 + l];
            if (v_f16) {
#pragma unroll
              for (int h = 0; h < 2; h++)
#pragma unroll
                for (int nb = 0; nb < NB; nb++) o[mb][nb] = E16::mma(h == 0 ? a0 : a1, ph[nb].q[h], o[mb][nb]);
            } else {
#pragma unroll
              for (int t2 = 0; t2 < 2; t2++)
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                  for (int nb = 0; nb < NB; nb++)
                    o[mb][nb] = E::mma(h == 0 ? a0 : a1, t2 == 0 ? ph[nb].q[h] : pl[nb].q[h], o[mb][nb]);
            }
            if (PIPE) {
              if (mb >= 1 && mb < 5) {
#pragma unroll
                for (int h = 0; h < 2; h++) av[2 * ((mb - 1) & 3) + h] = vl[(2 * (mb + 3) + h) * 64 + l];
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
      __builtin_amdgcn_s_setprio(HS_PRIO_VALU);
      if (!MID) {
        // the next tile must have landed; the ones requested after it may still be in flight
        int later = 0;
#pragma unroll
        for (int i = 2; i <= D; i++) later += tj[i] >= 0;
        stage_wait_wave<KM, VM>(later, w);
        __syncthreads();
      }
#pragma unroll
      for (int i = 0; i < D; i++) { tj[i] = tj[i + 1]; tk[i] = tk[i + 1]; tv[i] = tv[i + 1]; }
      st = st + 1 == NS ? 0 : st + 1;
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    if (MID && valid && tj[0] >= 0) k_fetch(0);
    while (tj[0] >= 0) {
      // one loop per GEMM2 form, each run over consecutive tiles of its form (a branch around GEMM2
      // inside one loop makes the compiler move all 64 accumulators per tile; going from one loop
      // to another costs that move once per change, which the tile order keeps rare)
      if (!ONLY16 && !hs_map_f16(tv[0])) {  // V tile in bf16 encoding: two terms of P; kind looked at per tile
        do iteration(I0{}, I2{});
        while (tj[0] >= 0 && !hs_map_f16(tv[0]));
      } else if (VM == 2 && tv[0] > 0) {
        do iteration(I1{}, I1{});
        while (tj[0] >= 0 && tv[0] > 0 && (ONLY16 || hs_map_f16(tv[0])));
      } else if (VM == 2) {
        do iteration(I1{}, I0{});
        while (tj[0] >= 0 && tv[0] < 0 && (ONLY16 || hs_map_f16(tv[0])));
      } else {
        do iteration(I1{}, I2{});
        while (tj[0] >= 0 && (ONLY16 || hs_map_f16(tv[0])));
      }
    }
  };
  if constexpr (F16) {
    main_loop(std::integral_constant<bool, MID_OK>{}, std::true_type{});
  } else if constexpr (MID_OK) {
    // bf16 cache: are all V tiles this workgroup can meet in fp16 encoding?  (every wave scans the
    // same entries, so the workgroup agrees; the answer is scalar)
    bool all16 = true;
    for (int base = t_lo; base <= t_last; base += 64) {
      const int t = base + l;
      const int32_t m = t <= t_last ? vm[t] : 0;
      all16 = all16 && !__any(m != 0 && !hs_map_f16(m));
    }
    if (all16) main_loop(std::integral_constant<bool, MID_OK>{}, std::true_type{});
    else main_loop(std::false_type{}, std::false_type{});
  } else {
    main_loop(std::false_type{}, std::false_type{});
  }

  if constexpr (TEAMS > 1) {
    // The teams have met at a barrier per tile; the one with a tile less makes up for it.  Then each hands half of its O^T (and all
    // of its references and sums, lane by lane) to its counterpart of the same slab through LDS and finishes the other half.
    if (unpaired) __syncthreads();
    __syncthreads();
    float4* const ex = reinterpret_cast<float4*>(lds_all);
    constexpr int kVec = 4 * NB * 64;  // float4 per wave
    float* const exl = reinterpret_cast<float*>(ex + 8 * kVec);
    auto give = [&](auto from) {
#pragma unroll
      for (int mb = 0; mb < 4; mb++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
          const f32x4_t x = o[decltype(from)::value + mb][nb];
          ex[wave * kVec + (mb * NB + nb) * 64 + l] = make_float4(x[0], x[1], x[2], x[3]);
        }
    };
    if (team == 0) give(std::integral_constant<int, 4>{});
    else give(std::integral_constant<int, 0>{});
#pragma unroll
    for (int nb = 0; nb < NB; nb++) {
      exl[((wave * NB + nb) * 2) * 64 + l] = m_run[nb];
      exl[((wave * NB + nb) * 2 + 1) * 64 + l] = l_run[nb];
    }
    __syncthreads();
    if (!valid) return;
    const int other = wave ^ 4;
    auto finish = [&](auto from) {
      constexpr int kFrom = decltype(from)::value;
#pragma unroll
      for (int nb = 0; nb < NB; nb++) {
        const float m_other = exl[((other * NB + nb) * 2) * 64 + l], l_other = exl[((other * NB + nb) * 2 + 1) * 64 + l];
        // a team without a reference has seen nothing (l and O are 0) or only NaN scores (l is NaN)
        const float m = fmaxf(m_run[nb], m_other), ref = m > -INFINITY ? m : 0.f;
        const float f = __builtin_amdgcn_exp2f(m_run[nb] - ref), fo = __builtin_amdgcn_exp2f(m_other - ref);
        float lt = l_run[nb] * f + l_other * fo;
        lt += __shfl_xor(lt, 16);
        lt += __shfl_xor(lt, 32);
        const float inv = lt == 0.f ? 0.f : 1.f / lt;
        const float lse = lt == 0.f ? -INFINITY : (m + __builtin_amdgcn_logf(lt)) * kLn2;
        const int64_t qrow = ((int64_t)b * Hq + hq) * Lq + qpos + 16 * nb + c;
        const float g = f * inv, go = fo * inv;
#pragma unroll
        for (int mb = 0; mb < 4; mb++) {
          const float4 y = ex[other * kVec + (mb * NB + nb) * 64 + l];
          const f32x4_t x = o[kFrom + mb][nb];
          const float r0 = x[0] * g + y.x * go, r1 = x[1] * g + y.y * go, r2 = x[2] * g + y.z * go, r3 = x[3] * g + y.w * go;
          *reinterpret_cast<uint2*>(O + qrow * HS_D + 4 * a + 16 * (kFrom + mb)) = make_uint2(E::pack2(r0, r1), E::pack2(r2, r3));
        }
        if (LSE != nullptr && a == 0 && kFrom == 0) LSE[qrow] = lse;
      }
    };
    if (team == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, 4>{});
    return;
  }
  // ---------------- epilogue: O = O^T / l, LSE ----------------
  if (!valid) return;
#pragma unroll
  for (int nb = 0; nb < NB; nb++) {
    float lt = l_run[nb];
    lt += __shfl_xor(lt, 16);
    lt += __shfl_xor(lt, 32);
    const float inv = lt == 0.f ? 0.f : 1.f / lt;  // 0: no token seen; a NaN score makes l NaN, and O and LSE with it
    const float lse = lt == 0.f ? -INFINITY : (m_run[nb] + __builtin_amdgcn_logf(lt)) * kLn2;
    const int64_t qrow = ((int64_t)b * Hq + hq) * Lq + qpos + 16 * nb + c;
    if constexpr (SPLIT) {
      float* op = ws_o + (qrow * n_splits + split) * HS_D + 4 * a;
#pragma unroll
      for (int mb = 0; mb < 8; mb++)
        *reinterpret_cast<float4*>(op + 16 * mb) =
            make_float4(o[mb][nb][0] * inv, o[mb][nb][1] * inv, o[mb][nb][2] * inv, o[mb][nb][3] * inv);
      if (a == 0) ws_l[qrow * n_splits + split] = lse;
      continue;
    }
    uint16_t* op = O + qrow * HS_D + 4 * a;
#pragma unroll
    for (int mb = 0; mb < 8; mb++) {
      const uint2 v = make_uint2(E::pack2(o[mb][nb][0] * inv, o[mb][nb][1] * inv),
                                 E::pack2(o[mb][nb][2] * inv, o[mb][nb][3] * inv));
      *reinterpret_cast<uint2*>(op + 16 * mb) = v;
    }
    if (LSE != nullptr && a == 0) LSE[qrow] = lse;
  }
}

}  // namespace

template <int KM, int VM, int NB, int TEAMS = 1>
static hipError_t launch_prefill(int B, int Hq, int Hkv, int T, int Lq, int q_start, float sl2, int causal, const uint16_t* Q,
                                 const hs_kv_dev& kv, uint16_t* O, float* LSE, hipStream_t st, bool f16, int n_splits, float* ws_o,
                                 float* ws_l) {
  const int G = Hq / Hkv;
  const int n_groups = ((Lq / (16 * NB)) * G + 3) / 4;
  const dim3 grid(n_groups * Hkv, n_splits, B);
#define HS_LAUNCH(F16_, SPLIT_)                                                                                            \
  hipLaunchKernelGGL((prefill_kernel<KM, VM, NB, TEAMS, F16_, SPLIT_>), grid, dim3(256 * TEAMS), 0, st, Hq, Hkv, T, Lq, q_start, sl2, causal, \
                     Q, kv, O, LSE, ws_o, ws_l)
  if (n_splits > 1) {
    if constexpr (TEAMS == 1) {
      if (f16) HS_LAUNCH(true, true); else HS_LAUNCH(false, true);
    } else {
      return hipErrorInvalidValue;
    }
  } else {
    if (f16) HS_LAUNCH(true, false); else HS_LAUNCH(false, false);
  }
#undef HS_LAUNCH
  return hipGetLastError();
}
// slabs of 16 queries, by one team of waves or by two
template <int KM, int VM, class... Args>
static hipError_t launch_prefill_narrow(int teams, Args... args) {
  return teams == 2 ? launch_prefill<KM, VM, 1, 2>(args...) : launch_prefill<KM, VM, 1, 1>(args...);
}
