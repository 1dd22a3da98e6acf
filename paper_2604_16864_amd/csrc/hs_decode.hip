// Decode attention: split-KV kernel + merge kernel (Sec. IV-C: each workgroup handles a
// subset of the KV blocks and emits a partial output with its log-sum-exp; a light
// post-processing kernel combines them; the query heads that share a KV head are folded
// into the N dimension of the matrix instruction).
//
// The kernel is HBM-bound: every byte of the packed cache is read exactly once, straight
// from global memory into matrix-core operand registers (the pools are stored in operand
// order), so there is no LDS staging and no cross-lane shuffle in the main loop.  The
// sparse matrix instruction is used as the decompressor: it consumes the 2-bit metadata
// natively, so no vector-ALU work is spent on selecting operands.
#include <mutex>
#include <type_traits>

#include "hs_common.h"

#ifndef HS_DEC_DEPTH
#define HS_DEC_DEPTH 2
#endif
#ifndef HS_DEC_BYCOUNT_MIN_PER
#define HS_DEC_BYCOUNT_MIN_PER 128  /* tiles per split from which the kept tiles are handed out by count */
#endif
#ifndef HS_DEC_EARLY
#define HS_DEC_EARLY 1  /* uniform caches: the first round of a wave guesses its tiles' form and loads them at once */
#endif
#ifndef HS_DEC_OCC
#define HS_DEC_OCC (NW == 8 || (KM == 0 && VM == 0) || KM == 2 || VM == 2 ? 2 : 1)  /* a dense tensor at depth 2 needs > 256 registers */
#endif

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;


// streaming (non-temporal) 16-byte load: the packed cache is read once per call
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream(const uint4* p) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p)));
}



// four consecutive 16-bit outputs; O is the caller's and need not be aligned to more than its elements
__device__ __forceinline__ void store4(uint16_t* p, uint32_t lo, uint32_t hi, bool aligned8) {
  if (aligned8) {
    *reinterpret_cast<uint2*>(p) = make_uint2(lo, hi);
  } else {
    p[0] = (uint16_t)lo; p[1] = (uint16_t)(lo >> 16); p[2] = (uint16_t)hi; p[3] = (uint16_t)(hi >> 16);
  }
}

// Operand registers of one tile (K and V), filled by tile_load and consumed by tile_compute.
// KM / VM: kind of the K / V tile, 0 = 2:4, 1 = dense (the kernel sorts its tiles by kind first).
template <int KM, int VM>
struct TileRegs {
  static_assert((KM == 0 || KM == 1) && (VM == 0 || VM == 1), "one kind per operand");
  static constexpr int kNK = KM == 0 ? 8 : 16;  // 16-byte chunks per lane: 2:4 tile 8, dense tile 16
  static constexpr int kNV = VM == 0 ? 8 : 16;
  uint4 k[kNK];
  uint4 v[kNV];
  uint4 km, vm;  // the lane's four 32-bit index words of the K / V tile
};

template <int KM, int VM>
__device__ __forceinline__ void tile_load(TileRegs<KM, VM>& r, const hs_kv_dev& kv, int64_t row, int mk, int mv, int l) {  // mk, mv: wave-uniform
  mv = hs_map_plain(mv);
  r.km = make_uint4(0, 0, 0, 0);  // only 2:4 tiles carry index words
  r.vm = make_uint4(0, 0, 0, 0);
  constexpr bool k_sparse = KM == 0, v_sparse = VM == 0;
  if (k_sparse) {
    const int64_t slot = row * kv.cap_sparse_k + (-mk - 1);
    const uint4* p = reinterpret_cast<const uint4*>(kv.k_nnz + slot * (int64_t)HS_TILE_NNZ_BYTES) + l;
#pragma unroll
    for (int i = 0; i < 8; i++) r.k[i] = ld_stream(p + 64 * i);
    r.km = ld_stream(reinterpret_cast<const uint4*>(kv.k_meta + slot * (int64_t)HS_TILE_META_BYTES) + l);
  } else {
    const int64_t slot = row * kv.cap_dense_k + (mk - 1);
    const uint4* p = reinterpret_cast<const uint4*>(kv.k_dense + slot * (int64_t)HS_TILE_DENSE_BYTES) + l;
#pragma unroll
    for (int i = 0; i < 16; i++) r.k[i % TileRegs<KM, VM>::kNK] = ld_stream(p + 64 * i);
  }
  if (v_sparse) {
    const int64_t slot = row * kv.cap_sparse_v + (-mv - 1);
    const uint4* p = reinterpret_cast<const uint4*>(kv.v_nnz + slot * (int64_t)HS_TILE_NNZ_BYTES) + l;
#pragma unroll
    for (int i = 0; i < 8; i++) r.v[i] = ld_stream(p + 64 * i);
    r.vm = ld_stream(reinterpret_cast<const uint4*>(kv.v_meta + slot * (int64_t)HS_TILE_META_BYTES) + l);
  } else {
    const int64_t slot = row * kv.cap_dense_v + (mv - 1);
    const uint4* p = reinterpret_cast<const uint4*>(kv.v_dense + slot * (int64_t)HS_TILE_DENSE_BYTES) + l;
#pragma unroll
    for (int i = 0; i < 16; i++) r.v[i % TileRegs<KM, VM>::kNV] = ld_stream(p + 64 * i);
  }
}

// One tile: GEMM1 (S^T = K Q^T), online softmax, GEMM2 (O^T += V^T P^T).
// F16: element type of the cache (hs_elem).  A V tile of a bf16 cache may be stored in fp16
// encoding (HS_MAP_F16 in its map entry); the numerators then go into GEMM2 as fp16 too.  The
// running reference sits kShift = 8 binades under the running maximum, so that numerators reach
// 2^8 and what fp16 flushes to zero is below 2^-32 of the largest one (a context of 2^17 tokens
// then loses < 2^-15 of the sum).
// ENC: 0 = V tile in bf16, 1 = in fp16 (encoding bit, or an fp16 cache).
template <int KM, int VM, bool F16, int ENC>
__device__ __forceinline__ void tile_compute(const TileRegs<KM, VM>& r, const uint4 (&qb)[4], float scale_log2, int c,
                                             f32x4_t (&o)[8], float& m_run, float& l_run) {
  constexpr bool k_sparse = KM == 0, v_sparse = VM == 0;
  constexpr int kNK = TileRegs<KM, VM>::kNK, kNV = TileRegs<KM, VM>::kNV;
  typedef hs_elem<F16> E;
  typedef hs_elem<true> E16;
  constexpr float kShift = 8.f;
  constexpr bool v_f16 = ENC == 1;
  f32x4_t s[4];
  const int kidx[4] = {(int)r.km.x, (int)r.km.y, (int)r.km.z, (int)r.km.w};
  const int vidx[4] = {(int)r.vm.x, (int)r.vm.y, (int)r.vm.z, (int)r.vm.w};
#pragma unroll
  for (int m = 0; m < 4; m++) s[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (k_sparse) {  // the 4 row blocks are independent chains
#pragma unroll
    for (int m = 0; m < 4; m++)
      s[m] = E::template smma<0>(r.k[2 * m], qb[0], qb[1], s[m], kidx[m]);
#pragma unroll
    for (int m = 0; m < 4; m++)
      s[m] = E::template smma<1>(r.k[2 * m + 1], qb[2], qb[3], s[m], kidx[m]);
  }
#pragma unroll
  for (int m = 0; m < 4; m++) {
    if (!k_sparse) {
#pragma unroll
      for (int st = 0; st < 4; st++)
        s[m] = E::mma(r.k[(4 * m + st) % kNK], qb[st], s[m]);
    }
  }
  // online softmax for column c (log2 domain)
  const float m_prev = m_run;
  float mx = -INFINITY;
#pragma unroll
  for (int m = 0; m < 4; m++)
#pragma unroll
    for (int i = 0; i < 4; i++) mx = fmaxf(mx, s[m][i]);
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  m_run = fmaxf(m_prev, mx * scale_log2 - kShift);
  const float m_ref = m_run > -INFINITY ? m_run : 0.f;  // every score -inf so far: weights 0, not exp2(-inf + inf)
  const float alpha = __builtin_amdgcn_exp2f(m_prev - m_ref);  // 0 on the first tile
  float psum = 0.f;
  // P^T as the B operand: element 8h+4u+i of lane group a <- token 16(2h+u)+4a+i.
  // Columns < 8 carry bf16(p), columns >= 8 carry bf16(p - bf16(p)), so that the sum of
  // the two accumulator columns sees p to ~16 bits although the operand type is bf16.
  float p[4][4];
#pragma unroll
  for (int m = 0; m < 4; m++)
#pragma unroll
    for (int i = 0; i < 4; i++) {
      p[m][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[m][i], scale_log2, -m_ref));
      psum += p[m][i];
    }
  uint32_t pb[8];
  auto pack_as = [&](auto enc) {
    typedef hs_elem<decltype(enc)::value> EP;
#pragma unroll
    for (int m = 0; m < 4; m++) {
      const uint32_t hi0 = EP::pack2(p[m][0], p[m][1]), hi1 = EP::pack2(p[m][2], p[m][3]);
      const uint32_t lo0 = EP::pack2(p[m][0] - EP::lo_f32(hi0), p[m][1] - EP::hi_f32(hi0));
      const uint32_t lo1 = EP::pack2(p[m][2] - EP::lo_f32(hi1), p[m][3] - EP::hi_f32(hi1));
      pb[2 * m] = c < 8 ? hi0 : lo0;
      pb[2 * m + 1] = c < 8 ? hi1 : lo1;
    }
  };
  if (v_f16) pack_as(std::true_type{});
  else pack_as(std::false_type{});
  l_run = l_run * alpha + psum;
#pragma unroll
  for (int i = 0; i < 8; i++) o[i] *= alpha;
  const uint4 pb_lo = make_uint4(pb[0], pb[1], pb[2], pb[3]);  // dense step h = 0
  const uint4 pb_hi = make_uint4(pb[4], pb[5], pb[6], pb[7]);  // dense step h = 1
  if (v_f16) {
#pragma unroll
    for (int mb = 0; mb < 8; mb++) {
      if (v_sparse) {
        if (mb & 1) o[mb] = E16::template smma<1>(r.v[mb], pb_lo, pb_hi, o[mb], vidx[mb >> 1]);
        else o[mb] = E16::template smma<0>(r.v[mb], pb_lo, pb_hi, o[mb], vidx[mb >> 1]);
      } else {
        o[mb] = E16::mma(r.v[(2 * mb) % kNV], pb_lo, o[mb]);
        o[mb] = E16::mma(r.v[(2 * mb + 1) % kNV], pb_hi, o[mb]);
      }
    }
  } else {
#pragma unroll
    for (int mb = 0; mb < 8; mb++) {
      if (v_sparse) {
        if (mb & 1) o[mb] = E::template smma<1>(r.v[mb], pb_lo, pb_hi, o[mb], vidx[mb >> 1]);
        else o[mb] = E::template smma<0>(r.v[mb], pb_lo, pb_hi, o[mb], vidx[mb >> 1]);
      } else {
        o[mb] = E::mma(r.v[(2 * mb) % kNV], pb_lo, o[mb]);
        o[mb] = E::mma(r.v[(2 * mb + 1) % kNV], pb_hi, o[mb]);
      }
    }
  }
}

// Which tile forms (bit 0 K dense, bit 1 V dense, bit 2 V in bf16 encoding) a kernel instantiation can meet:
// KM / VM 0 = every tile 2:4, 1 = every tile dense, 2 = any mix; an fp16 cache has no bf16-encoded tiles.
template <int KM, int VM, bool F16>
__host__ __device__ constexpr bool form_allowed(int f) {
  return ((f & 1) ? KM != 0 : KM != 1) && ((f & 2) ? VM != 0 : VM != 1) && ((f & 4) ? !F16 : true);
}
// fn(std::integral_constant<int, f>) for every allowed form f except SKIP_FORM, in ascending order
template <int KM, int VM, bool F16, int SKIP_FORM, int F = 0, typename Fn>
__device__ __forceinline__ void static_for_forms(Fn&& fn) {
  if constexpr (F < 8) {
    if constexpr (F != SKIP_FORM && form_allowed<KM, VM, F16>(F)) fn(std::integral_constant<int, F>{});
    static_for_forms<KM, VM, F16, SKIP_FORM, F + 1>(fn);
  }
}

// The dense tail (at most one tile of not yet compressed tokens) as seen by the split kernel: `len` < 0 = the call has
// none; `lens` (device, [B], or NULL) replaces `len` per batch row, kept inside the tail buffer.
struct TailArgs {
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* lens;
  int len;
};

// Q^T of one (batch, kv head) row as the B operand: columns 0..G-1 and 8..8+G-1 both hold head column % 8 of the group
// (GEMM2 over the tiles gives the second copy the low-order half of P).  hq0: the group's first query head.
__device__ __forceinline__ void load_q(const uint16_t* __restrict__ Q, int64_t hq0, int G, int a, int c, uint4 (&qb)[4]) {
  const int head = c & 7;
  const bool valid = head < G;
  const uint16_t* q = Q + (hq0 + (valid ? head : 0)) * HS_D + 8 * a;
#pragma unroll
  for (int s = 0; s < 4; s++) qb[s] = valid ? *reinterpret_cast<const uint4*>(q + 32 * s) : make_uint4(0, 0, 0, 0);
}

// A wave's share of the dense tail of one row: tokens 16 q .. 16 q + 15 of the tail buffer, all query heads of the group, into the
// combine's slots (reference, sum, unnormalised O^T per column).  Everything it reads is requested at once; the scores come from
// the 16-bit matrix instruction like those of a dense tile, O^T from the 32-bit one, so that P keeps its 32 bits:
// its k is a lane group's token i (the accumulators of the scores are its B operand as they stand), its row r of block mb is channel
// 8 r + mb, so that a lane reads 8 consecutive channels of 4 tokens.  Tokens from tail_len on are not read.
// Latency-bound, one chain of load, products, exponentials, products.  The same on the vector ALU, with q and P in LDS, read
// the LDS once more per head and was the last to end: us a call, then / now, 8 rows of 256 tiles with a tail, 4 heads a row
// 14.1 / 12.5, 8 heads 16.1 / 12.8; 128 rows of 16 tiles 13.7 / 12.4, 15.9 / 12.8; 8 rows of 32 tiles 8.3 / 7.6, 10.1 / 7.6; with one
// head a row the same.
// AHEAD: the caller has raised the wave's priority, until its loads are requested.
template <bool F16, bool AHEAD>
__device__ __forceinline__ void tail_piece(const TailArgs& tail, int tail_len, int64_t row, int q, const uint4 (&qb)[4], float scale_log2,
                                           int l, float (&sm_o)[8][HS_D], float (&sm_m)[8], float (&sm_l)[8]) {
  typedef hs_elem<F16> E;
  const int a = l >> 4, c = l & 15, left = tail_len - 16 * q;  // left: wave-uniform
  float m = -INFINITY, sum = 0.f;
  f32x4_t o[8];
#pragma unroll
  for (int mb = 0; mb < 8; mb++) o[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (left > 0) {
    const uint16_t* tk = tail.k + (row * HS_BT + 16 * q + c) * HS_D + 8 * a;
    const uint16_t* tv = tail.v + (row * HS_BT + 16 * q + 4 * a) * HS_D + 8 * c;
    uint4 kk[4], vv[4];
#pragma unroll
    for (int s = 0; s < 4; s++) kk[s] = c < left ? *reinterpret_cast<const uint4*>(tk + 32 * s) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; i++) vv[i] = 4 * a + i < left ? *reinterpret_cast<const uint4*>(tv + i * HS_D) : make_uint4(0, 0, 0, 0);
    if constexpr (AHEAD) { __builtin_amdgcn_sched_barrier(0); __builtin_amdgcn_s_setprio(0); }
    f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 4; st++) s = E::mma(kk[st], qb[st], s);
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if (4 * a + i >= left) s[i] = -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    m = mx * scale_log2;
    const float ref = m > -INFINITY ? m : 0.f;  // every score -inf: weights 0, not exp2(-inf + inf)
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
      p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], scale_log2, -ref));
      sum += p[i];
    }
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const uint32_t d[4] = {vv[i].x, vv[i].y, vv[i].z, vv[i].w};
#pragma unroll
      for (int mb = 0; mb < 8; mb++)
        o[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(mb & 1 ? E::hi_f32(d[mb >> 1]) : E::lo_f32(d[mb >> 1]), p[i], o[mb], 0, 0, 0);
    }
  }
  if (c < 8) {
    if (a == 0) { sm_m[c] = m; sm_l[c] = sum; }
#pragma unroll
    for (int i = 0; i < 4; i++) {
      float4* d = reinterpret_cast<float4*>(&sm_o[c][8 * (4 * a + i)]);
      d[0] = make_float4(o[0][i], o[1][i], o[2][i], o[3][i]);
      d[1] = make_float4(o[4][i], o[5][i], o[6][i], o[7][i]);
    }
  }
}

// Combines the N parts that the waves have left in LDS (and, with_tail, the tail's four behind them) and writes the row's partial of split
// `slot`, or (DIRECT) its O and LSE.  Thread = (head tid / 32, 4 channels).  part_m, part_l, part_o: 8 heads a part.
template <bool F16, bool DIRECT, int N>
__device__ __forceinline__ void combine_parts(int tid, bool with_tail, int G, int64_t hq0, const float (*part_m)[8], const float (*part_l)[8],
                                              const float (*part_o)[8][HS_D], int n_splits, int slot, float* __restrict__ ws_o,
                                              float* __restrict__ ws_l) {
  const int g = tid >> 5, ch = (tid & 31) * 4;
  if (g >= G) return;
  const int64_t hq = hq0 + g;
  float mstar = -INFINITY;
#pragma unroll
  for (int k = 0; k < N; k++) mstar = fmaxf(mstar, part_m[k][g]);
  if (DIRECT && with_tail) {
#pragma unroll
    for (int k = N; k < N + 4; k++) mstar = fmaxf(mstar, part_m[k][g]);
  }
  // a part without a reference has seen nothing (l and O are 0) or only NaN scores (l is NaN): neither is left out,
  // and only l == 0 is an empty split, so that a NaN reaches O and LSE however the tiles are divided
  const float mref = mstar > -INFINITY ? mstar : 0.f;
  float lsum = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
  auto add = [&](int k) {
    const float f = __builtin_amdgcn_exp2f(part_m[k][g] - mref);
    lsum += f * part_l[k][g];
#pragma unroll
    for (int i = 0; i < 4; i++) acc[i] += f * part_o[k][g][ch + i];
  };
#pragma unroll
  for (int k = 0; k < N; k++) add(k);
  if (DIRECT && with_tail) {
#pragma unroll
    for (int k = N; k < N + 4; k++) add(k);
  }
  const float inv = lsum == 0.f ? 0.f : 1.f / lsum;
  const float lse = lsum == 0.f ? -INFINITY : (mstar + __builtin_amdgcn_logf(lsum)) * kLn2;
  if constexpr (DIRECT) {
    typedef hs_elem<F16> E;
    uint16_t* po = reinterpret_cast<uint16_t*>(ws_o) + hq * HS_D + ch;
    store4(po, E::pack2(acc[0] * inv, acc[1] * inv), E::pack2(acc[2] * inv, acc[3] * inv), ((uintptr_t)ws_o & 7) == 0);
    if (ws_l != nullptr && (tid & 31) == 0) ws_l[hq] = lse;
  } else {
    float* po = ws_o + (hq * n_splits + slot) * HS_D + ch;
    *reinterpret_cast<float4*>(po) = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    if ((tid & 31) == 0) ws_l[hq * n_splits + slot] = lse;
  }
}

// Split-KV kernel.  grid = (n_work, Hkv, B); with a dense tail the B * Hkv tail workgroups follow as further
// planes of the grid, behind all others: as one more workgroup of every row they pushed whole splits onto compute
// units that already had one (16 rows x 8 heads, 2 splits: 99 instead of 66 us).  workgroup = 4 waves; split s owns tiles
// [s*per, (s+1)*per); wave w takes every 4th tile of them.  Each wave preloads the map
// entries of its tiles with one vector load, drops the skipped ones, and streams the rest
// with a two-deep register pipeline (the loads of tile i+1 are in flight while tile i is
// being multiplied).
// Each workgroup emits a normalised partial output and its log-sum-exp per query head.
//
// MODE (how the tiles of a row are handed out):
//   kByRange    split s owns tiles [s*per, (s+1)*per), wave w every 4th of them; skipped tiles are dropped
//               as they are met, so a split or a wave may end up with fewer tiles than its neighbours.
//   kUniform    as kByRange, for a cache the caller promises to be uniform (no tile skipped, one kind per
//               tensor, slot == tile): the K map is not read at all.
//   kByCount    the kept (not skipped) tiles of the row are numbered in tile order, split s owns the numbers
//               [n*s/S, n*(s+1)/S) and wave w every 4th of them: every wave of the grid gets the same number
//               of tiles to within one, whatever the skip pattern.  Costs two passes over the row's maps
//               at kernel start (count, then list through LDS), so the host picks it for long rows only.
enum { kByRange = 0, kUniform = 1, kByCount = 2 };
constexpr int kListCap = 2048;  // tiles listed in LDS at a time (kByCount); longer shares take several passes
constexpr int kScanBatch = 2048;  // tiles of the row looked at per scan step: 8 per thread

// NW: waves per workgroup.  4: the partial of a split goes to ws_o / ws_l.  8: the workgroup has the whole row (one
// split, and the row's dense tail) and writes O and LSE itself (handed in as ws_o, ws_l): no merge launch.
// waves_per_eu: what the registers allow, as the most too: the scheduler otherwise goes by what the LDS would allow, and orders the loads
// of a mixed tensor's tiles worse (4 sequences of 32K tokens, half of the keys dense, 58.7 / 58.3 us).
template <int KM, int VM, int MODE, bool F16, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(HS_DEC_OCC, HS_DEC_OCC)))
void decode_split_kernel(int B, int z0, int turn, int Hq, int Hkv, int T, float scale_log2, int n_splits, int per,
                         const uint16_t* __restrict__ Q, hs_kv_dev kv, TailArgs tail, float* __restrict__ ws_o, float* __restrict__ ws_l) {
  const int hkv = blockIdx.y, b = blockIdx.z + z0;
  // Workgroups go round-robin over the 8 XCDs by their index: with an even number of splits the same splits of every row
  // meet on an XCD (with 8 of them, split s on XCD s), and where rows differ in length the XCDs of the late splits have little to
  // do.  So every 8 / gcd(splits, 8) rows the splits start one further on (turn - 1 = log2 of that).  us, before / after: 16 sequences of 4K to 16K
  // tokens, 2 splits 67.5 / 66.5; 8 of 8K to 32K, 4 splits 67.8 / 64.4; 4 of them, 8 splits 43.6 / 37.0; 2 of 2K to 8K 12.3 / 11.8.  Rows of
  // one length are 1 to 2 % faster without (32K tokens with dense ends 12.9 / 13.1), so the launcher asks for it (turn > 0)
  // where rows may differ.
  int split = blockIdx.x;
  if (MODE == kByRange && NW == 4 && turn > 0) split = (split + ((b * Hkv + hkv) >> (turn - 1))) % (int)gridDim.x;
  const int tid = threadIdx.x, l = tid & 63, a = l >> 4, c = l & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, scalar: branches on it stay scalar
  const int G = Hq / Hkv;
  constexpr bool DIRECT = NW == 8;
  constexpr int kParts = DIRECT ? NW + 4 : NW;  // the waves', and the dense tail's where it does not have a workgroup of its own
  __shared__ __attribute__((aligned(16))) float sm_o[kParts][8][HS_D];
  __shared__ float sm_m[kParts][8], sm_l[kParts][8];
  const int n_work = gridDim.x;  // partial slots of the cache's tiles; the tail's is the next one
  auto tail_length = [&](int of) -> int {
    return __builtin_amdgcn_readfirstlane(tail.lens != nullptr ? min(max(tail.lens[of], 0), HS_BT) : tail.len);
  };
  // Where the results go, in registers from the start: left to itself the compiler reads the two pointers from the kernel's arguments
  // in front of the last stores, and the launch ends 0.3 to 0.5 us later (16 sequences of 4K to 16K tokens with tails 66.0 / 66.5 us,
  // 128 rows of 49 tiles 17.3 / 17.6).
  typedef __attribute__((address_space(1))) float* global_t;
  global_t to_o = (global_t)ws_o, to_l = (global_t)ws_l;
  asm volatile("" : "+s"(to_o), "+s"(to_l));
  // the row, its group's first query head, and the partial slot that this workgroup writes
  int64_t row = (int64_t)b * Hkv + hkv, hq0 = (int64_t)b * Hq + hkv * G;
  int slot = split;
  if (!DIRECT && __builtin_expect(b >= B, 0)) {  // the whole workgroup: the dense tail of a row
    row = ((int64_t)(b - B) * Hkv + hkv) * n_work + split;
    if (row >= (int64_t)B * Hkv) return;
    // One short chain beside waves that stream: last, it would be what the launch ends with, so its loads are requested ahead of theirs.  Its
    // arithmetic is not put first: it takes issue slots from splits of few tiles.  us, no priority / all the way / until the loads are
    // requested: 128 rows of 2K tokens, one head a row, 17.5 / 16.8 / 16.8, 4 heads 17.5 / 17.2 / 17.1; 128 rows that keep 9 tiles of 36 11.04 / 11.33 / 11.05.
    __builtin_amdgcn_s_setprio(3);
    const int tb = (int)(row / Hkv);
    hq0 = (int64_t)tb * Hq + (row - (int64_t)tb * Hkv) * G;
    slot = n_work;
    uint4 qt[4];
    load_q(Q, hq0, G, a, c, qt);
    tail_piece<F16, true>(tail, tail_length(tb), row, w, qt, scale_log2, l, sm_o[w], sm_m[w], sm_l[w]);
  } else {
    const int t_begin = split * per, t_end = min(T, t_begin + per);

    uint4 qb[4];  // dense k-steps s = 0..3 (channels 32s + 8a + e); sparse kb uses steps 2kb, 2kb+1
    load_q(Q, hq0, G, a, c, qb);

    f32x4_t o[8];
#pragma unroll
    for (int i = 0; i < 8; i++) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    // A tile's form: bit 0 = K tile dense, bit 1 = V tile dense, bit 2 = V tile stored in bf16 encoding (bf16
    // caches only; a V tile of a bf16 cache is normally stored in fp16 encoding, HS_MAP_F16).  The tiles are
    // worked through one form at a time ("sweeps"): the loads and matrix instructions of a sweep are all of one
    // type, no branch sits between them, and each sweep keeps as many tiles in flight as its operands leave
    // registers for.  The softmax recurrence does not care in which order tiles arrive.
    auto form_of = [](int mk, int mv) -> int { return (mk > 0 ? 1 : 0) | (mv > 0 ? 2 : 0) | ((!F16 && !hs_map_f16(mv)) ? 4 : 0); };
    constexpr bool kMixed = KM == 2 || VM == 2;
    constexpr int kFirstForm = (KM == 1 ? 1 : 0) | (VM == 1 ? 2 : 0);  // swept first: it also notes which other forms occur
    // One sweep.  The tiles come as a sequence of map entry pairs numbered [first, last): `entry(i, mk, mv)` yields
    // pair i; wave w takes every NW-th pair starting at first + w.  Returns (COLLECT) the set of forms among them.
    // SPEC (uniform caches, first sweep): where the wave's first tiles sit is known without the maps (slot ==
    // tile), only their form is not (the encoding bit of the V map of a bf16 cache), so the first round is a
    // straight-line copy of its own that issues their loads at once, behind the map read instead of after it
    // and with no ballot or branch in front of them (4-6 % of the kernel at the 32K-context shape, fp16 caches,
    // which have no map to wait for, included).  If one of the tiles turns out to be of another form (a V tile
    // that fp16 cannot hold) the sweep returns kGuessFailed before it has touched the accumulators, and is run
    // again without guessing.
    constexpr unsigned kGuessFailed = 1u << 31;
    auto sweep = [&](auto form_c, auto collect_c, auto spec_c, int first, int last, auto entry) -> unsigned {
      constexpr int kForm = decltype(form_c)::value;
      constexpr bool COLLECT = decltype(collect_c)::value;
      constexpr bool SPEC = decltype(spec_c)::value;
      constexpr int KK = kForm & 1, VK = (kForm >> 1) & 1, kEnc = (kForm & 4) ? 0 : 1;
      // Tiles in flight per wave.  Measured on the 32K-context shape: depth 1, 2, 3 and 4 (the deeper ones at
      // 1 wave per SIMD) all land within run-to-run noise, and even a variant with the arithmetic removed is only
      // ~10 % faster: the kernel is bound by the load stream.  A kernel for mixed tensors runs at 2 waves per
      // SIMD, where only two 2:4 tiles (or one tile with a dense operand) fit.
      constexpr int DEPTH = kMixed || NW == 8 ? ((KK == 0 && VK == 0) ? 2 : 1) : HS_DEC_DEPTH;
      TileRegs<KK, VK> ring[DEPTH];
      unsigned seen = 0;
      // what the two copies of a round below share: the form ballots, and the loop that consumes the tiles in
      // flight and refills their ring slots from `act`
#define HS_ROUND_BALLOTS                                                                                              \
    const int form_v = form_of(mk_v, mv_v);                                                                             \
    unsigned long long act = __ballot(mk_v != 0 && form_v == kForm);                                                    \
    if (COLLECT) {                                                                                                      \
      _Pragma("unroll") for (int f = 0; f < 8; f++)                                                                     \
        if (f != kForm && form_allowed<KM, VM, F16>(f)) seen |= (__ballot(mk_v != 0 && form_v == f) != 0ull ? 1u : 0u) << f; \
    }
#define HS_ROUND_CONSUME                                                                                              \
    bool go = have[0];                                                                                                  \
    while (go) {                                                                                                        \
      _Pragma("unroll") for (int d = 0; d < DEPTH; d++) {                                                               \
        if (go && have[d]) { /* tiles are consumed in issue order: the first empty slot ends the round */               \
          tile_compute<KK, VK, F16, kEnc>(ring[d], qb, scale_log2, c, o, m_run, l_run);                                 \
          have[d] = act != 0ull;                                                                                        \
          if (have[d]) {                                                                                                \
            const int i = __builtin_ctzll(act);                                                                         \
            act &= act - 1;                                                                                             \
            tile_load<KK, VK>(ring[d], kv, row, __builtin_amdgcn_readlane(mk_v, i), __builtin_amdgcn_readlane(mv_v, i), l); \
          }                                                                                                             \
        } else {                                                                                                        \
          go = false;                                                                                                   \
        }                                                                                                               \
      }                                                                                                                 \
    }
      int base = first + w;
      if constexpr (SPEC) {
        if (base < last) {  // first round, tiles guessed
          const int i_mine = base + NW * l;
          int mk_v = 0, mv_v = 0;
          if (i_mine < last) entry(i_mine, mk_v, mv_v);
          bool have[DEPTH];
          unsigned long long guessed = 0ull;
#pragma unroll
          for (int d = 0; d < DEPTH; d++) {
            const int t = base + NW * d;
            have[d] = t < last;
            if (have[d]) {
              guessed |= 1ull << d;
              tile_load<KK, VK>(ring[d], kv, row, KK == 0 ? -(t + 1) : t + 1, VK == 0 ? -(t + 1) : t + 1, l);
            }
          }
          HS_ROUND_BALLOTS
          if constexpr (!F16)  // an fp16 cache has one encoding: nothing to guess wrong
            if ((act & ((1ull << DEPTH) - 1ull)) != guessed) return kGuessFailed;
          act &= ~guessed;
          HS_ROUND_CONSUME
          base += 64 * NW;
        }
      }
      for (; base < last; base += 64 * NW) {  // up to 64 tiles of this wave per round
        const int i_mine = base + NW * l;
        int mk_v = 0, mv_v = 0;
        if (i_mine < last) entry(i_mine, mk_v, mv_v);
        // Tile kinds must reach the branches below as scalar (wave-uniform) values: matrix
        // instructions ignore the EXEC mask, so a branch the compiler treats as divergent would run
        // both the dense and the 2:4 instruction on every tile.  Lane values are therefore read
        // with v_readlane, never with a lane shuffle.
        HS_ROUND_BALLOTS
        bool have[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; d++) {
          have[d] = act != 0ull;
          if (have[d]) {
            const int i = __builtin_ctzll(act);
            act &= act - 1;
            tile_load<KK, VK>(ring[d], kv, row, __builtin_amdgcn_readlane(mk_v, i), __builtin_amdgcn_readlane(mv_v, i), l);
          }
        }
        HS_ROUND_CONSUME
      }
#undef HS_ROUND_BALLOTS
#undef HS_ROUND_CONSUME
      return seen;
    };
    auto all_sweeps = [&](int first, int last, auto entry) {
      constexpr bool kGuess = HS_DEC_EARLY && MODE == kUniform;
      unsigned seen = sweep(std::integral_constant<int, kFirstForm>{}, std::true_type{}, std::integral_constant<bool, kGuess>{},
                            first, last, entry);
      if (kGuess && !F16 && seen == kGuessFailed)
        seen = sweep(std::integral_constant<int, kFirstForm>{}, std::true_type{}, std::false_type{}, first, last, entry);
      static_for_forms<KM, VM, F16, kFirstForm>([&](auto form_c) {
        if ((seen >> decltype(form_c)::value) & 1u) sweep(form_c, std::false_type{}, std::false_type{}, first, last, entry);
      });
    };
    auto from_map = [&](int t, int& mk, int& mv) {
      if (MODE == kUniform) {  // promised by the caller: no tile skipped, one kind per tensor, slot == tile
        mk = KM == 0 ? -(t + 1) : t + 1;
        mv = F16 ? (VM == 0 ? -(t + 1) : t + 1) : kv.v_map[row * T + t];  // bf16: encoding bit
      } else {
        mk = kv.k_map[row * T + t];
        mv = kv.v_map[row * T + t];
      }
    };
    if constexpr (MODE != kByCount) {
      all_sweeps(t_begin, t_end, from_map);
    } else {
      __shared__ int2 sm_list[kListCap];  // (k_map, v_map) entries of this workgroup's tiles, in tile order
      __shared__ int sm_cnt[36];          // [0..3] kept tiles per wave (count pass); [4 + 4 j + w] per scan segment
      const int* kmap = kv.k_map + row * T;
      const int* vmap = kv.v_map + row * T;
      const unsigned long long lanes_below = (1ull << l) - 1ull;
      // pass 1: kept tiles of the row
      int mine_cnt = 0;
      for (int b0 = 0; b0 < T; b0 += kScanBatch) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int t = b0 + 256 * j + tid;
          const int mk = t < T ? kmap[t] : 0;
          const int mv = t < T ? vmap[t] : 0;  // not needed yet: fetched so that pass 2 finds both maps in the L2
          asm volatile("" ::"v"(mv));
          mine_cnt += __builtin_popcountll(__ballot(mk != 0));
        }
      }
      if (l == 0) sm_cnt[w] = mine_cnt;
      __syncthreads();
      const int n_kept = sm_cnt[0] + sm_cnt[1] + sm_cnt[2] + sm_cnt[3];
      const int lo = (int)((int64_t)n_kept * split / n_work), hi = (int)((int64_t)n_kept * (split + 1) / n_work);
      if (n_kept == T) {  // nothing skipped: a tile's number is its index, no list needed
        all_sweeps(lo, hi, from_map);
      } else
      for (int r0 = lo; r0 < hi; r0 += kListCap) {  // workgroup-uniform bounds: every thread takes the same trips
        const int r1 = min(hi, r0 + kListCap);
        // pass 2: list the tiles numbered [r0, r1)
        int carried = 0;  // kept tiles before the scan step
        for (int b0 = 0; b0 < T && carried < r1; b0 += kScanBatch) {
          int mk8[8], mv8[8];  // read again in every pass (from L2 by now) rather than held across the tile loop
#pragma unroll
          for (int j = 0; j < 8; j++) {
            const int t = b0 + 256 * j + tid;
            mk8[j] = t < T ? kmap[t] : 0;
            mv8[j] = t < T ? vmap[t] : 0;
          }
          unsigned long long kept[8];
#pragma unroll
          for (int j = 0; j < 8; j++) {
            kept[j] = __ballot(mk8[j] != 0);
            if (l == 0) sm_cnt[4 + 4 * j + w] = __builtin_popcountll(kept[j]);
          }
          __syncthreads();
          int run = carried;  // tile t = b0 + 256 j + 64 w + l: segments in (j, w) order are in tile order
#pragma unroll
          for (int j = 0; j < 8; j++) {
            int before = run;
#pragma unroll
            for (int ww = 0; ww < 4; ww++) {
              const int c_seg = sm_cnt[4 + 4 * j + ww];
              if (ww < w) before += c_seg;
              run += c_seg;
            }
            const int number = before + __builtin_popcountll(kept[j] & lanes_below);
            if (mk8[j] != 0 && number >= r0 && number < r1) sm_list[number - r0] = make_int2(mk8[j], mv8[j]);
          }
          carried = run;
          __syncthreads();  // the counts are rewritten by the next scan step
        }
        const int n_list = r1 - r0;
        // the same sweeps, over the list: pair i goes to wave i % 4
        auto from_list = [&](int i, int& mk, int& mv) {
          const int2 e = sm_list[i];
          mk = e.x;
          mv = e.y;
        };
        all_sweeps(0, n_list, from_list);
        __syncthreads();  // the list is rewritten by the next pass
      }
    }

    // ---------------- combine: lane groups, hi/lo columns, then the 4 waves ----------------
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
#pragma unroll
    for (int i = 0; i < 8; i++)
#pragma unroll
      for (int j = 0; j < 4; j++) {  // column c + column c^8 (rotate by 8 inside the 16-lane row)
        const int other = __builtin_amdgcn_mov_dpp(__float_as_int(o[i][j]), 0x128, 0xf, 0xf, true);
        o[i][j] += __int_as_float(other);
      }

    if (c < 8) {
      if (a == 0) { sm_m[w][c] = m_run; sm_l[w][c] = l_run; }
#pragma unroll
      for (int mb = 0; mb < 8; mb++)
        *reinterpret_cast<float4*>(&sm_o[w][c][16 * mb + 4 * a]) = make_float4(o[mb][0], o[mb][1], o[mb][2], o[mb][3]);
    }
    if constexpr (DIRECT) {
      if (tail.len >= 0) {  // by the waves that have no tile where the row has few
        const int q = NW - 1 - w;
        if (q < 4) tail_piece<F16, false>(tail, tail_length(b), row, q, qb, scale_log2, l, sm_o[NW + q], sm_m[NW + q], sm_l[NW + q]);
      }
    }
  }
  __syncthreads();
  combine_parts<F16, DIRECT, NW>(tid, tail.len >= 0, G, hq0, sm_m, sm_l, sm_o, n_splits, slot, (float*)to_o, (float*)to_l);
}

// Merge of the split partials (Sec. IV-C "lightweight post-processing kernel"):
// O = sum_s e^{LSE_s - M} O_s / sum_s e^{LSE_s - M}, M = max_s LSE_s, done in one pass with a
// running reference per thread.  A partial of LSE -inf is empty (its O is 0) and weighs nothing; one of LSE NaN makes
// the row NaN.  A row (one query of one head) is merged by SL split lanes of 32
// threads (4 channels each), which are combined in LDS; a workgroup takes R rows.  A thread requests U partials before
// it looks at the first (a test per partial in front of its use made them wait for each other: 4.0 -> 3.2 us at 32 rows
// x 32 splits, 16 -> 4.2 us at 256 splits).
// A separate launch on purpose: folding it into the split kernel ("last workgroup to arrive
// merges") needs device-scope visibility between workgroups on different XCDs, and both ways
// of getting it (a device-wide fence per workgroup, or write-through stores and L2-bypassing
// loads) measured slower than this launch.
template <bool F16, int SL, int R, int U>
__global__ __launch_bounds__(32 * SL * R) void merge_kernel(int64_t rows, int n_splits, const float* __restrict__ ws_o,
                                                            const float* __restrict__ ws_l, uint16_t* __restrict__ O,
                                                            float* __restrict__ LSE) {
  __shared__ __attribute__((aligned(16))) float sm_acc[R][SL][HS_D];
  __shared__ float sm_ml[R][SL][2];
  const int tid = threadIdx.x, r = tid / (32 * SL), sl = tid / 32 % SL, ch = (tid & 31) * 4;
  const int64_t row = (int64_t)blockIdx.x * R + r;
  const bool valid = R == 1 || row < rows;
  const float* po = ws_o + (valid ? row : 0) * n_splits * HS_D + ch;
  const float* pl = ws_l + (valid ? row : 0) * n_splits;
  float M = -INFINITY, den = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = sl; s0 < n_splits; s0 += SL * U) {  // U partials requested at once
    float lse[U];
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int s = s0 + SL * u;
      lse[u] = s < n_splits ? pl[s] : -INFINITY;
      v[u] = s < n_splits ? *reinterpret_cast<const float4*>(po + (int64_t)s * HS_D) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < U; u++) Mn = fmaxf(Mn, lse[u]);
    const float ref = Mn > -INFINITY ? Mn : 0.f;
    const float fo = __expf(M - ref);  // 0 while M is still -inf
    den *= fo;
#pragma unroll
    for (int i = 0; i < 4; i++) acc[i] *= fo;
#pragma unroll
    for (int u = 0; u < U; u++) {
      const float fn = __expf(lse[u] - ref);  // 0 for a split that saw nothing
      den += fn;
      acc[0] += fn * v[u].x; acc[1] += fn * v[u].y; acc[2] += fn * v[u].z; acc[3] += fn * v[u].w;
    }
    M = Mn;
  }
  if (SL > 1) {
    if ((tid & 31) == 0) { sm_ml[r][sl][0] = M; sm_ml[r][sl][1] = den; }
    *reinterpret_cast<float4*>(&sm_acc[r][sl][ch]) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    __syncthreads();
    if (sl != 0) return;
    float Mt = -INFINITY;
#pragma unroll
    for (int k = 0; k < SL; k++) Mt = fmaxf(Mt, sm_ml[r][k][0]);
    den = 0.f;
#pragma unroll
    for (int i = 0; i < 4; i++) acc[i] = 0.f;
    const float ref = Mt > -INFINITY ? Mt : 0.f;
#pragma unroll
    for (int k = 0; k < SL; k++) {
      const float f = __expf(sm_ml[r][k][0] - ref);  // 0 for a split lane that saw nothing
      const float4 v = *reinterpret_cast<const float4*>(&sm_acc[r][k][ch]);
      den += f * sm_ml[r][k][1];
      acc[0] += f * v.x; acc[1] += f * v.y; acc[2] += f * v.z; acc[3] += f * v.w;
    }
    M = Mt;
  }
  if (!valid) return;
#pragma unroll
  for (int i = 0; i < 4; i++) acc[i] = den == 0.f ? 0.f : acc[i] / den;
  store4(O + row * HS_D + ch, hs_elem<F16>::pack2(acc[0], acc[1]), hs_elem<F16>::pack2(acc[2], acc[3]), ((uintptr_t)O & 7) == 0);
  if (LSE != nullptr && (tid & 31) == 0) LSE[row] = den == 0.f ? -INFINITY : M + __logf(den);
}


}  // namespace

// Split partials of hs_decode_attn_static: a fixed array in device memory, one copy per GPU the
// library is loaded on, held until the process ends.  In host code the name `scratch` is only a
// handle for hipGetSymbolAddress; the address kernels and copies use is the one looked up below.
static __device__ __align__(256) unsigned char scratch[HS_STATIC_SCRATCH_BYTES];

hipError_t hs_static_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* per_device[kMaxDevices] = {};  // each GPU has its own copy of the array at its own address
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (per_device[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // for the current device
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  *bytes = HS_STATIC_SCRATCH_BYTES;
  return hipSuccess;
}

// Workspace: [partial O (normalised) [B*Hq][n_splits][128] fp32][partial LSE [B*Hq][n_splits] fp32].
template <int KM, int VM, int MODE, int NW>
static hipError_t launch_split(dim3 grid, hipStream_t st, int B, int turn, int Hq, int Hkv, int T, float sl2, int n_splits, int per,
                               const uint16_t* Q, const hs_kv_dev& kv, const TailArgs& tail, float* wo, float* wl, bool f16) {
  // planes B .. grid.z - 1 are the tail's; a grid has at most 65535, so batches of more than half of that take a second launch
  const unsigned all = grid.z;
  for (unsigned z0 = 0; z0 < all; z0 += grid.z) {
    grid.z = all - z0 > 65535u ? (unsigned)B : all - z0;
    if (f16)
      hipLaunchKernelGGL((decode_split_kernel<KM, VM, MODE, true, NW>), grid, dim3(64 * NW), 0, st, B, (int)z0, turn, Hq, Hkv, T, sl2,
                         n_splits, per, Q, kv, tail, wo, wl);
    else
      hipLaunchKernelGGL((decode_split_kernel<KM, VM, MODE, false, NW>), grid, dim3(64 * NW), 0, st, B, (int)z0, turn, Hq, Hkv, T, sl2,
                         n_splits, per, Q, kv, tail, wo, wl);
  }
  return hipGetLastError();
}

// Splits per row for n_splits == 0: at most `most` (what the workspace has room for).  Time relative to the best, against
// the number of workgroups (1 per compute unit is 256), measured on caches of 0.3 to 2.4 GB: 100 1.30, 128 1.14, 160
// 1.035, 192 to 224 1.00, 256 1.03 (all-2:4 caches 50.7 us at 256 and 48.7 us at 192, dense 86.7 and 83.8 us, 8 x 128K
// tokens with half of the tiles skipped 185 and 178 us), and a second, partly filled round costs: 264 1.36 (24 rows of 512
// 2:4 tiles: 51.7 us with 11 splits, 38.0 with 10, 37.4 with the 8 it takes), 320 1.21, 384 1.075, 512 1.05.  A split whose
// tiles do not divide among its waves costs about a quarter of what it wastes.  Small caches (fewer than 8 tiles per wave) do
// not gain from fewer than 256 workgroups unless all tiles are dense, and rows with skipped tiles that are split by range want as
// many as fit.  So do rows whose fill the host does not know (hs_kept_by_pools): where they differ, the longest one's splits
// are the last to end (mixed tensors with room for every tile, filled to 25 to 100 %: 64 rows of 512 tiles 71.0 us with 3 splits,
// 64.6 with 4; 24 rows 33.3 with 8, 28.4 with 10; all filled to 40 %, 8 rows of 1024: 23.0 with 24, 19.8 with 32).
static int pick_splits(int64_t rows, int T, int most, bool dense, hs_kept kept, int bycount_per) {
  static const struct { double wgs, g; } kCurve[] = {{100, 1.30}, {128, 1.14}, {160, 1.035}, {192, 1.0}, {224, 1.005}, {256, 1.03},
                                                     {257, 1.36}, {320, 1.21}, {384, 1.075}, {512, 1.05}};
  const bool prefer_fewer = dense || rows * T >= 8192;
  int best = most;
  double best_cost = 0.0;
  for (int n = most; n >= 1 && rows * n >= 96; n--) {  // below 96 workgroups fewer is never better
    const double w = (double)(rows * n);
    if (w > 512) continue;
    double g = 1.30;
    for (int i = 0; i + 1 < 10; i++)
      if (w >= kCurve[i].wgs && w <= kCurve[i + 1].wgs)
        g = kCurve[i].g + (kCurve[i + 1].g - kCurve[i].g) * (w - kCurve[i].wgs) / (kCurve[i + 1].wgs - kCurve[i].wgs);
    const int per = (T + n - 1) / n;
    const bool by_count = per >= bycount_per;
    if (w >= 192 && w <= 256 && (!prefer_fewer || kept == HS_KEPT_UNKNOWN || (kept == HS_KEPT_FEWER && !by_count)))
      g = 1.0 + (256 - w) * 1e-4;
    const double waste = by_count ? 0.0 : (double)((per + 3) / 4) * 4 * n / T - 1.0;
    const double cost = g * (1.0 + 0.25 * waste);
    if (best_cost == 0.0 || cost < best_cost) { best = n; best_cost = cost; }
  }
  return best;
}

hipError_t hs_launch_decode(int B, int Hq, int Hkv, int T, float scale, int n_work, int auto_splits, const uint16_t* Q, hs_kv_dev kv,
                            const uint16_t* tail_k, const uint16_t* tail_v, int tail_len, const int32_t* tail_lens,
                            uint16_t* O, float* LSE, float* ws, hipStream_t st, int phases, int dtype) {
  const int km = kv.cap_dense_k == 0 ? 0 : (kv.cap_sparse_k == 0 ? 1 : 2);
  const int vm = kv.cap_dense_v == 0 ? 0 : (kv.cap_sparse_v == 0 ? 1 : 2);
  // Tiles by count on long splits only: the two passes over the maps at kernel start cost about 3 us, which the even
  // shares win back (3-7 % of the kernel when tiles are skipped) from 128 tiles per split for all-2:4 tensors and from 256
  // otherwise.  us, by range / by count, 64 rows of 640 2:4 tiles in 4 splits: half skipped 67.6 / 65.7, three quarters
  // 40.2 / 37.9, all but every eighth 29.1 / 22.8 (by range the skip pattern decides how even the waves' shares are), rows
  // filled to 25 to 100 % 79.2 / 84.7.
  const hs_kept kept = hs_kept_by_pools(kv, T);
  const int bycount_per = km == 0 && vm == 0 && !kv.uniform ? HS_DEC_BYCOUNT_MIN_PER : 2 * HS_DEC_BYCOUNT_MIN_PER;
  if (auto_splits) n_work = pick_splits((int64_t)B * Hkv, T, n_work, km == 1 && vm == 1, kept, bycount_per);
  // One workgroup of 8 waves per row and no merge launch, where that is faster than split + merge: very short rows (one
  // compute unit reads about 42 GB/s; us, split + merge / direct, 2:4: 1 row of 4 / 8 / 16 tiles 6.1 / 4.1, 6.0 / 5.4, 6.2 /
  // 8.2; dense, 4 / 8 tiles 6.3 / 5.4, 6.8 / 7.6), and rows numerous enough to fill the chip (256 rows of 8 / 32 / 96 tiles
  // 11.7 / 8.8, 27.5 / 25.4, 69.9 / 67.7; 200 rows of 192 tiles, half of them skipped, 60.2 by count / 58.6; 128 rows of
  // 16 / 32 tiles 11.6 / 10.2, 17.4 / 17.4).  Longer rows are split or handed out by count; so are those of 128 tiles or more
  // that may have any pattern of skipped tiles (200 rows of 160, all but every eighth skipped: 19.1 by count / 25.7).
  // A dense tail goes to the waves that have no tile, so it costs little up to 6 tiles (us with the caller's buffers, split + merge /
  // direct, 8 rows of 5 / 6 / 7 tiles 6.5 / 5.7, 6.5 / 6.3, 6.5 / 6.4, 32 rows 7.6 / 7.1, 7.7 / 7.7, 7.7 / 8.0; 4 tiles, dense 8.5 / 7.8, dense
  // keys 7.7 / 7.2, dense ends 8.5 / 7.7; 256 rows of 8 / 32 / 96 tiles 12.9 / 11.0, 29.1 / 28.8, 74.2 / 71.4, 200 rows of 64 tiles 40.4 / 40.6).
  const int short_row = km == 0 && vm == 0 ? (tail_len < 0 ? 8 : 6) : 4;
  const bool direct = auto_splits && phases == 3 &&
                      (T <= short_row || (n_work == 1 && T < (kept == HS_KEPT_UNKNOWN ? bycount_per : 2 * HS_DEC_BYCOUNT_MIN_PER)) || ((int64_t)B * Hkv >= 128 && T <= 16));
  if (direct) n_work = 1;
  const TailArgs tail{tail_k, tail_v, tail_lens, tail_len};
  const dim3 grid(n_work, Hkv, B + (tail_len >= 0 && !direct ? (B + n_work - 1) / n_work : 0));
  const bool f16 = dtype == HS_FP16;
  const float sl2 = scale * kLog2e;
  const int per = (T + n_work - 1) / n_work;
  // partial slots per query head: the n_work cache splits, then one for the dense tail if there is
  // one (the kernels take the slot count as their stride)
  const int n_splits = n_work + (tail_len >= 0 ? 1 : 0);
  float* wo = direct ? reinterpret_cast<float*>(O) : ws;
  float* wl = direct ? LSE : wo + (size_t)B * Hq * n_splits * HS_D;
  hipError_t e = hipSuccess;
  if (phases & 1) {
  const int turn = kept == HS_KEPT_UNKNOWN && n_work % 2 == 0 ? (n_work % 8 == 0 ? 1 : (n_work % 4 == 0 ? 2 : 3)) : 0;
  const bool by_count = per >= bycount_per;
#define HS_SPLIT(KM_, VM_, MODE_, NW_) \
  launch_split<KM_, VM_, MODE_, NW_>(grid, st, B, turn, Hq, Hkv, T, sl2, n_splits, per, Q, kv, tail, wo, wl, f16)
#define HS_GO_DYN(KM_, VM_)                                                                                            \
  e = direct ? HS_SPLIT(KM_, VM_, kByRange, 8)                                                                         \
             : (by_count ? HS_SPLIT(KM_, VM_, kByCount, 4) : HS_SPLIT(KM_, VM_, kByRange, 4));                         \
  break
#define HS_GO(KM_, VM_)                                                                                       \
  if (kv.uniform) {                                                                                           \
    e = direct ? HS_SPLIT(KM_, VM_, kUniform, 8) : HS_SPLIT(KM_, VM_, kUniform, 4);                           \
    break;                                                                                                    \
  }                                                                                                           \
  HS_GO_DYN(KM_, VM_)
  switch (km * 3 + vm) {
    case 0: HS_GO(0, 0);
    case 1: HS_GO(0, 1);
    case 2: HS_GO_DYN(0, 2);
    case 3: HS_GO(1, 0);
    case 4: HS_GO(1, 1);
    case 5: HS_GO_DYN(1, 2);
    case 6: HS_GO_DYN(2, 0);
    case 7: HS_GO_DYN(2, 1);
    default: HS_GO_DYN(2, 2);
  }
#undef HS_GO
#undef HS_GO_DYN
#undef HS_SPLIT
  }
  if (e != hipSuccess || direct || !(phases & 2)) return e;
  return hs_launch_merge((int64_t)B * Hq, n_splits, wo, wl, O, LSE, st, dtype);
}

hipError_t hs_launch_merge(int64_t rows, int n_splits, const float* ws_o, const float* ws_l, uint16_t* O, float* LSE,
                           hipStream_t st, int dtype) {
#define HS_MERGE(SL_, R_, U_)                                                                                              \
  do {                                                                                                                     \
    const dim3 grid((unsigned)((rows + R_ - 1) / R_)), block(32 * SL_ * R_);                                               \
    if (dtype == HS_FP16) hipLaunchKernelGGL((merge_kernel<true, SL_, R_, U_>), grid, block, 0, st, rows, n_splits, ws_o, ws_l, O, LSE); \
    else hipLaunchKernelGGL((merge_kernel<false, SL_, R_, U_>), grid, block, 0, st, rows, n_splits, ws_o, ws_l, O, LSE);   \
  } while (0)
  // Latency decides: few splits want no exchange between lanes, many want them requested side by side.  Kernel times in us
  // of <1, 8, 4> / <8, 1, 4> / <16, 1, 4>: 32 rows x 8 splits 2.7 / 3.0 / 3.3, 8192 x 8 4.4 / 9.4 / 12.1, 32768 x 2 7.8 /
  // 19.7 / 34; 32 x 32 4.7 / 3.2 / 3.4, 2048 x 32 7.2 / 4.8 / 6.3; 32 x 128 13.3 / 4.3 / 4.0, 4 x 256 23.7 / 5.4 / 4.2.
  if (n_splits <= 8) HS_MERGE(1, 8, 4);
  else if (n_splits <= 64) HS_MERGE(8, 1, 4);
  else HS_MERGE(16, 1, 4);
#undef HS_MERGE
  return hipGetLastError();
}
