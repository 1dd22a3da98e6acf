// Compress path: tile scoring, tile selection, fused 2:4 prune + pack, and unpack.
// Paper: hierarchical pruner Sec. III-A (Eq. 2a-d), cache compressor Sec. III-B,
// fused magnitude compressor Sec. IV-B.
#include "hs_common.h"

namespace {

constexpr int kVStride = 132;  // LDS row stride (elements) of a staged V tile: 8-byte aligned rows, shifted banks

// 16-byte global accesses of the compressor.  Every input byte is read once and every output byte
// written once per call, so the pool bytes of 2:4 tiles are written with non-temporal stores, and
// their inputs read non-temporally when the tensors are large (pack_kernel); for tiles that stay
// dense, where as many bytes are written as read, the plain forms measured faster and are kept.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ uint4 ld16(const void* p) {
  if (NT) return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p)));
  return *reinterpret_cast<const uint4*>(p);
}
template <bool NT>
__device__ __forceinline__ void st16(void* p, uint4 v) {
  if (NT) __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t*>(p));
  else *reinterpret_cast<uint4*>(p) = v;
}

// Top-2-of-4 by magnitude (Eq. 2a-b with an exact count of two): x0..x3 are bf16 bit
// patterns; element j outranks element i if |x_j| > |x_i|, or |x_j| == |x_i| and j < i.
// Returns the 4-bit keep mask (exactly two bits set).
// rule != 0 (input already masked): the key is "non-zero" instead of the magnitude, so the
// non-zero entries win and ties (zeros) go to the lower position.
__device__ __forceinline__ uint32_t top2_mask(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, int rule) {
  uint32_t k0 = x0 & 0x7fffu, k1 = x1 & 0x7fffu, k2 = x2 & 0x7fffu, k3 = x3 & 0x7fffu;
  if (rule != 0) { k0 = k0 != 0; k1 = k1 != 0; k2 = k2 != 0; k3 = k3 != 0; }
  const uint32_t g01 = k0 >= k1, g02 = k0 >= k2, g03 = k0 >= k3, g12 = k1 >= k2, g13 = k1 >= k3, g23 = k2 >= k3;
  const uint32_t c0 = 3u - g01 - g02 - g03;        // how many outrank element 0
  const uint32_t c1 = g01 + 2u - g12 - g13;
  const uint32_t c2 = g02 + g12 + 1u - g23;
  const uint32_t c3 = g03 + g13 + g23;
  return (c0 < 2u) | ((c1 < 2u) << 1) | ((c2 < 2u) << 2) | ((c3 < 2u) << 3);
}

// From the keep mask: the two kept values packed (lower position in the low half) and
// the metadata nibble i0 | i1 << 2 (Sec. IV-B: 2-bit position of each kept element).
__device__ __forceinline__ void top2_emit(uint32_t mask, uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                          uint32_t& vals, uint32_t& nib) {
  const uint32_t i0 = (uint32_t)__builtin_ctz(mask);
  const uint32_t i1 = 31u - (uint32_t)__builtin_clz(mask);
  const uint32_t v0 = (mask & 1u) ? x0 : ((mask & 2u) ? x1 : x2);
  const uint32_t v1 = (mask & 8u) ? x3 : ((mask & 4u) ? x2 : x1);
  vals = (v0 & 0xffffu) | (v1 << 16);
  nib = i0 | (i1 << 2);
}

template <bool F16> __device__ __forceinline__ double elem_val(uint32_t bits) { return (double)hs_elem<F16>::to_f32(bits); }

// ----------------------------------------------------------------------------------
// Staging of one V tile [64 tokens][128 ch] into LDS with coalesced 16-byte loads.
// ----------------------------------------------------------------------------------
template <bool NT = false>
__device__ __forceinline__ void stage_v_tile(const uint16_t* vt, int64_t tok_stride, uint16_t* lds) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int q = tid + 256 * i;
    const int tok = q >> 4, c8 = q & 15;
    const uint4 d = ld16<NT>(vt + tok * tok_stride + 8 * c8);
    uint2* dst = reinterpret_cast<uint2*>(lds + tok * kVStride + 8 * c8);
    dst[0] = make_uint2(d.x, d.y);
    dst[1] = make_uint2(d.z, d.w);
  }
}

// ----------------------------------------------------------------------------------
// Tile scores: energy = sum K^2 + sum V^2 (skip ranking), loss_x = L1 norm of what the
// 2:4 mask removes (Eq. 2c).  fp64 (every term exact), fixed reduction order.
// scores = [3][rows][T].  WHAT: bit 0 = the policy ranks by energy, bit 1 = by the losses; a
// plane that is not asked for is written as zeros (the selection then falls back to tile order
// there, which is all it needs when a count is 0 or everything).
// ----------------------------------------------------------------------------------
template <bool F16> __device__ __forceinline__ double add_sq8(double e, uint4 d) {  // e + the squares of 8 elements
  const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const double f0 = (double)hs_elem<F16>::lo_f32(w[i]), f1 = (double)hs_elem<F16>::hi_f32(w[i]);
    e = fma(f0, f0, e);
    e = fma(f1, f1, e);
  }
  return e;
}

// sum of the magnitudes of the two elements of a group that the 2:4 mask drops, any rule
template <bool F16>
__device__ __forceinline__ double dropped_l1(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, int rule) {
  const uint32_t drop = ~top2_mask(x0, x1, x2, x3, rule) & 15u;
  uint32_t pair, nib;
  top2_emit(drop, x0, x1, x2, x3, pair, nib);
  return fabs(elem_val<F16>(pair & 0xffffu)) + fabs(elem_val<F16>(pair >> 16));
}

// The same by magnitude needs no mask: the sum of the two smallest of four magnitudes (which of several equal
// ones is dropped does not matter to the sum).  Bit patterns without the sign order like the magnitudes, so a network
// of packed 16-bit minima and maxima finds them, two groups at a time.
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}
// a group = four channels in two words: (x0, x1), (x2, x3)
template <bool F16> __device__ __forceinline__ double add_dropped_row(double s, uint32_t x01, uint32_t x23, int rule) {
  if (rule != 0) return s + dropped_l1<F16>(x01 & 0xffffu, x01 >> 16, x23 & 0xffffu, x23 >> 16, rule);
  const uint32_t a = x01 & 0x7fff7fffu, b = x23 & 0x7fff7fffu;
  const uint32_t lo = pk_min(a, b), hi = pk_max(a, b);
  const uint32_t lo_r = __builtin_amdgcn_alignbit(lo, lo, 16), hi_r = __builtin_amdgcn_alignbit(hi, hi, 16);
  const uint32_t s1 = pk_min(lo, lo_r), s2 = pk_min(pk_max(lo, lo_r), pk_min(hi, hi_r));
  return s + ((double)hs_elem<F16>::lo_f32(s1) + (double)hs_elem<F16>::lo_f32(s2));
}
// two groups = two channels of four tokens, a word per token
template <bool F16>
__device__ __forceinline__ double add_dropped_col(double s, uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3, int rule) {
  if (rule != 0)
    return s + (dropped_l1<F16>(r0 & 0xffffu, r1 & 0xffffu, r2 & 0xffffu, r3 & 0xffffu, rule) +
                dropped_l1<F16>(r0 >> 16, r1 >> 16, r2 >> 16, r3 >> 16, rule));
  const uint32_t m0 = r0 & 0x7fff7fffu, m1 = r1 & 0x7fff7fffu, m2 = r2 & 0x7fff7fffu, m3 = r3 & 0x7fff7fffu;
  const uint32_t lo0 = pk_min(m0, m1), hi0 = pk_max(m0, m1), lo1 = pk_min(m2, m3), hi1 = pk_max(m2, m3);
  const uint32_t s1 = pk_min(lo0, lo1), s2 = pk_min(pk_max(lo0, lo1), pk_min(hi0, hi1));
  return s + (((double)hs_elem<F16>::lo_f32(s1) + (double)hs_elem<F16>::lo_f32(s2)) +
              ((double)hs_elem<F16>::hi_f32(s1) + (double)hs_elem<F16>::hi_f32(s2)));
}

// Data-parallel-primitive moves (a few cycles against the ~100 of a lane shuffle through LDS): lanes without a source
// read `id`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_mov(int v, int id) { return __builtin_amdgcn_update_dpp(id, v, CTRL, ROW_MASK, 0xf, false); }
template <int CTRL, int ROW_MASK> __device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)dpp_mov<CTRL, ROW_MASK>((int)b, 0), hi = (unsigned)dpp_mov<CTRL, ROW_MASK>((int)(b >> 32), 0);
  return v + __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
__device__ __forceinline__ double wave_sum_last(double v) {  // lane 63: the sum of the wave, fixed order
  v = dpp_add<0x111, 0xf>(v);  // row_shr:1
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
}

// One workgroup per tile.  Bound by the read of K and V; what could keep it from that is arithmetic, so: no LDS staging
// (a thread reads the same 8 channels of a whole token group of V), no element masks (above), one fma per square.
// All three planes at 8 rows of 512 tiles (134 MB): 44.8 -> 29.0 us = 4.6 TB/s (a large copy reaches 5.1 here).
// NT: non-temporal reads.  They pay when K and V exceed the last-level cache (energy alone, B 8 x L 131072: 1.32 -> 1.26 ms
// for score + select + pack) and cost when they fit, because the pack kernel's second read of the kept tiles then no
// longer hits that cache (L 32768: 56 -> 60 us).
template <bool F16, int WHAT, bool NT>
__global__ __launch_bounds__(256) void score_kernel(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                                                    int64_t sb, int64_t sh, int64_t st, int Hkv, int T, int rule,
                                                    double* __restrict__ scores) {
  constexpr bool ENERGY = (WHAT & 1) != 0, LOSS = (WHAT & 2) != 0;
  __shared__ double red[3][4];
  const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const uint16_t* kt = K + b * sb + h * sh + (int64_t)t * HS_BT * st + 8 * (tid & 15);
  const uint16_t* vt = V + b * sb + h * sh + (int64_t)t * HS_BT * st + 8 * (tid & 15);
  uint4 kd[4], vd[4];  // K: tokens tid / 16 + 16 i; V: tokens 4 (tid / 16) + i; channels 8 (tid % 16) .. +7
#pragma unroll
  for (int i = 0; i < 4; i++) kd[i] = ld16<NT>(kt + ((tid >> 4) + 16 * i) * st);
#pragma unroll
  for (int i = 0; i < 4; i++) vd[i] = ld16<NT>(vt + (4 * (tid >> 4) + i) * st);
  double e = 0.0, lk = 0.0, lv = 0.0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (ENERGY) e = add_sq8<F16>(e, kd[i]);
    if (LOSS) {
      lk = add_dropped_row<F16>(lk, kd[i].x, kd[i].y, rule);
      lk = add_dropped_row<F16>(lk, kd[i].z, kd[i].w, rule);
    }
  }
  if (ENERGY) {
    double ev = 0.0;
#pragma unroll
    for (int i = 0; i < 4; i++) ev = add_sq8<F16>(ev, vd[i]);
    e += ev;
  }
  if (LOSS) {
    lv = add_dropped_col<F16>(lv, vd[0].x, vd[1].x, vd[2].x, vd[3].x, rule);
    lv = add_dropped_col<F16>(lv, vd[0].y, vd[1].y, vd[2].y, vd[3].y, rule);
    lv = add_dropped_col<F16>(lv, vd[0].z, vd[1].z, vd[2].z, vd[3].z, rule);
    lv = add_dropped_col<F16>(lv, vd[0].w, vd[1].w, vd[2].w, vd[3].w, rule);
  }
  // wave sums, then 4 partials in LDS
  if (ENERGY) e = wave_sum_last(e);
  if (LOSS) {
    lk = wave_sum_last(lk);
    lv = wave_sum_last(lv);
  }
  if (l == 63) { red[0][w] = e; red[1][w] = lk; red[2][w] = lv; }
  __syncthreads();
  if (tid < 3) {
    const int64_t rows = (int64_t)gridDim.z * Hkv;
    const int64_t row = (int64_t)b * Hkv + h;
    scores[(tid * rows + row) * T + t] = (red[tid][0] + red[tid][1]) + (red[tid][2] + red[tid][3]);
  }
}

// ----------------------------------------------------------------------------------
// Tile selection per (b, kv head) row (Eq. 2d + the skip extension) and slot assignment (the two
// sequential counters of Sec. III-B, done as an exclusive prefix count), one workgroup per row.
// "The n tiles with the lowest (score, tile index)" is found by radix selection instead of by
// ranking every tile: scores are non-negative doubles, whose bit patterns order like unsigned
// integers.  The kernel is a chain of barriers on a handful of workgroups, so the chain is kept short:
// the bits in which the row's scores do not differ at all are skipped (scores of one row share their exponent and
// often more), one 256-bin histogram over the next eight bits usually leaves a bin with a few tiles, and up to 64
// of those are ranked by one wave at once; only rows with many (nearly) equal scores need further histograms.
// 8 rows of 512 tiles, skip + one ranked loss: 20.9 us with eight histograms of fixed bytes, 10.0 us now.
// Every thread owns a contiguous run of tiles, so "ascending tile index" is thread order, and a thread only
// re-reads map entries it wrote itself.
// ----------------------------------------------------------------------------------
// inclusive scan over the 64 lanes; `id` is the operation's neutral element
template <class Op>
__device__ __forceinline__ int wave_scan(int v, int id, Op op) {
  v = op(v, dpp_mov<0x111, 0xf>(v, id));  // row_shr:1
  v = op(v, dpp_mov<0x112, 0xf>(v, id));
  v = op(v, dpp_mov<0x114, 0xf>(v, id));
  v = op(v, dpp_mov<0x118, 0xf>(v, id));
  v = op(v, dpp_mov<0x142, 0xa>(v, id));  // row_bcast:15 into rows 1 and 3
  v = op(v, dpp_mov<0x143, 0xc>(v, id));  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ int wave_scan_sum(int v) { return wave_scan(v, 0, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ unsigned long long wave_and(unsigned long long k) {
  auto f = [](int a, int b) { return a & b; };
  const int lo = wave_scan((int)k, -1, f), hi = wave_scan((int)(k >> 32), -1, f);
  return (unsigned)__builtin_amdgcn_readlane(lo, 63) | (unsigned long long)(unsigned)__builtin_amdgcn_readlane(hi, 63) << 32;
}

constexpr int kFewTiles = 64;  // candidates one wave ranks directly
struct SelectShared {
  __attribute__((aligned(16))) int hist[256];
  int wsum[4][4];
  unsigned long long wand[4], wor[4];
  unsigned long long cand[kFewTiles], thr;
  int cand_t[kFewTiles], thr_t;
  int bin, want, count, n_cand;
};

template <int N>
__device__ __forceinline__ void block_exclusive_scan(int (&v)[N], int (*wsum)[4], int tid) {  // 256 threads; contains barriers
  const int l = tid & 63, w = tid >> 6;
  int incl[N];
#pragma unroll
  for (int i = 0; i < N; i++) incl[i] = wave_scan_sum(v[i]);
  __syncthreads();  // wsum may still be read from the previous call
#pragma unroll
  for (int i = 0; i < N; i++)
    if (l == 63) wsum[i][w] = incl[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; i++) {
    int base = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) base += j < w ? wsum[i][j] : 0;
    v[i] = base + incl[i] - v[i];
  }
}

// The keys of this thread's tiles [t0, t1), held in registers when the run is short (at most CACHE tiles), else (CACHE
// 0) re-read from memory on every pass.
template <int CACHE>
struct TileKeys {
  const double* keys;
  int t0, t1;
  unsigned long long k[CACHE > 0 ? CACHE : 1];
};

template <int CACHE>
__device__ __forceinline__ TileKeys<CACHE> load_keys(const double* __restrict__ keys, int t0, int t1, bool wanted) {
  TileKeys<CACHE> tk;
  tk.keys = keys; tk.t0 = t0; tk.t1 = t1;
#pragma unroll
  for (int i = 0; i < CACHE; i++)
    tk.k[i] = wanted && t0 + i < t1 ? (unsigned long long)__double_as_longlong(keys[t0 + i]) : 0ull;
  return tk;
}

// f(t, key) for every eligible tile of the thread, ascending t
template <int CACHE, class Eligible, class F>
__device__ __forceinline__ void for_each_key(const TileKeys<CACHE>& tk, Eligible eligible, F f) {
  if (CACHE > 0) {
#pragma unroll
    for (int i = 0; i < CACHE; i++)
      if (tk.t0 + i < tk.t1 && eligible(tk.t0 + i)) f(tk.t0 + i, tk.k[i]);
  } else {
    for (int t = tk.t0; t < tk.t1; t++)
      if (eligible(t)) f(t, (unsigned long long)__double_as_longlong(tk.keys[t]));
  }
}

// Marks the n eligible tiles with the lowest (key, tile index); there are at least n.
template <int CACHE, class Eligible, class Mark>
__device__ __forceinline__ void mark_lowest(const TileKeys<CACHE>& tk, Eligible eligible, int n, SelectShared& sm, int tid, Mark mark) {
  if (n <= 0) return;  // uniform: nobody is in the set
  const int w = tid >> 6, l = tid & 63;
  unsigned long long all = ~0ull, any = 0ull;  // AND and OR of the keys
  for_each_key(tk, eligible, [&](int, unsigned long long k) { all &= k; any |= k; });
  all = wave_and(all);
  any = ~wave_and(~any);
  sm.hist[tid] = 0;
  if (l == 0) { sm.wand[w] = all; sm.wor[w] = any; }
  if (tid == 0) sm.n_cand = 0;
  __syncthreads();
  all = (sm.wand[0] & sm.wand[1]) & (sm.wand[2] & sm.wand[3]);
  any = (sm.wor[0] | sm.wor[1]) | (sm.wor[2] | sm.wor[3]);
  // Invariant: the n-th lowest key is among the eligible keys with k >> done == prefix (done == 64: all of them), `want`
  // of these belong to the set, and so does every key below them.  The first histogram starts at the highest bit in which
  // keys differ.
  const unsigned long long differ = any & ~all;
  int done = differ == 0 ? 0 : 64 - __builtin_clzll(differ);
  unsigned long long prefix = done == 64 ? 0ull : all >> done;
  int want = n, count = -1;  // count of keys under the prefix; not known before the first histogram
  auto under = [&](unsigned long long k) { return done == 64 || (k >> done) == prefix; };
  while (done > 0) {
    const int sh = done > 8 ? done - 8 : 0;
    const int bits = done - sh;
    for_each_key(tk, eligible, [&](int, unsigned long long k) {
      if (under(k)) atomicAdd(&sm.hist[(int)(k >> sh) & ((1 << bits) - 1)], 1);
    });
    __syncthreads();
    if (w == 0) {  // one wave looks for the bin, four bins per lane
      const int4 h = *reinterpret_cast<const int4*>(&sm.hist[4 * l]);
      *reinterpret_cast<int4*>(&sm.hist[4 * l]) = make_int4(0, 0, 0, 0);
      const int mine = h.x + h.y + h.z + h.w;
      int before = wave_scan_sum(mine) - mine;
      if (before < want && want <= before + mine) {
        int j = 0, c = h.x;
        if (want > before + c) { before += c; j = 1; c = h.y; }
        if (j == 1 && want > before + c) { before += c; j = 2; c = h.z; }
        if (j == 2 && want > before + c) { before += c; j = 3; c = h.w; }
        sm.bin = 4 * l + j; sm.want = want - before; sm.count = c;
      }
    }
    __syncthreads();
    prefix = (done == 64 ? 0ull : prefix << bits) | (unsigned long long)sm.bin;
    want = sm.want;
    count = sm.count;
    done = sh;
    if (count == want || count <= kFewTiles) break;
    __syncthreads();  // bin, want, count are rewritten by the next round
  }
  if (count == want) {  // everything under the prefix belongs to the set
    for_each_key(tk, eligible, [&](int t, unsigned long long k) {
      if ((k >> done) <= prefix) mark(t);
    });
  } else if (done > 0) {  // a few keys: ranked by one wave, one key per lane
    for_each_key(tk, eligible, [&](int t, unsigned long long k) {
      if (under(k)) {
        const int i = atomicAdd(&sm.n_cand, 1);
        sm.cand[i] = k;
        sm.cand_t[i] = t;
      }
    });
    __syncthreads();
    if (w == 0) {
      const unsigned long long k = l < count ? sm.cand[l] : ~0ull;
      const int t = l < count ? sm.cand_t[l] : 0x7fffffff;
      int rank = 0;
      for (int j = 0; j < count; j++) {
        const unsigned long long kj = (unsigned)__builtin_amdgcn_readlane((int)k, j) |
                                      (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(k >> 32), j) << 32;
        rank += kj < k || (kj == k && __builtin_amdgcn_readlane(t, j) < t);
      }
      if (l < count && rank == want - 1) { sm.thr = k; sm.thr_t = t; }
    }
    __syncthreads();
    const unsigned long long thr = sm.thr;
    const int thr_t = sm.thr_t;
    for_each_key(tk, eligible, [&](int t, unsigned long long k) {
      if (k < thr || (k == thr && t <= thr_t)) mark(t);
    });
  } else {  // equal keys: the first `want` of them by tile index
    int ties[1] = {0};
    for_each_key(tk, eligible, [&](int, unsigned long long k) { ties[0] += k == prefix; });
    block_exclusive_scan(ties, sm.wsum, tid);
    int tie_rank = ties[0];
    for_each_key(tk, eligible, [&](int t, unsigned long long k) {
      if (k < prefix || (k == prefix && tie_rank++ < want)) mark(t);
    });
  }
}

// Tiles t < n_first or t >= T - n_last are protected: always kept dense, outside both rankings.
// Tile states live in registers while the selection runs (2 bits per tile) when a thread's run is
// short, else in the map arrays themselves; the maps are written once, at the end.
// CACHE: tiles per thread that the registers hold (0: any number).
template <int CACHE>
__global__ __launch_bounds__(256) void select_kernel(const double* __restrict__ scores, int rows, int T, int n_skip,
                                                     int n_sparse_k, int n_sparse_v, int n_first, int n_last,
                                                     int32_t* __restrict__ k_map, int32_t* __restrict__ v_map) {
  __shared__ SelectShared sm;
  const int row = blockIdx.x, tid = threadIdx.x;
  const double* en = scores + (int64_t)row * T;                // plane 0 = energy
  const double* lk = scores + ((int64_t)1 * rows + row) * T;   // planes 1, 2 = pruning losses
  const double* lv = scores + ((int64_t)2 * rows + row) * T;
  int32_t* km = k_map + (int64_t)row * T;
  int32_t* vm = v_map + (int64_t)row * T;
  const int per = (T + 255) / 256;
  const int t0 = min(tid * per, T), t1 = min(t0 + per, T);
  constexpr bool in_regs = CACHE > 0;
  unsigned rk = 0x5555u, rv = 0x5555u;  // HS_DENSE everywhere
  static_assert(HS_DENSE == 1 && 2 * CACHE <= 32, "packed tile states");
  auto state_k = [&](int t) -> int { return in_regs ? (rk >> (2 * (t - t0))) & 3u : km[t]; };
  auto state_v = [&](int t) -> int { return in_regs ? (rv >> (2 * (t - t0))) & 3u : vm[t]; };
  auto set_k = [&](int t, int v) {
    if (in_regs) rk = (rk & ~(3u << (2 * (t - t0)))) | ((unsigned)v << (2 * (t - t0)));
    else km[t] = v;
  };
  auto set_v = [&](int t, int v) {
    if (in_regs) rv = (rv & ~(3u << (2 * (t - t0)))) | ((unsigned)v << (2 * (t - t0)));
    else vm[t] = v;
  };
  auto is_protected = [&](int t) { return t < n_first || t >= T - n_last; };
  // the scores of all rankings are requested at once
  const int n_keep = T - n_first - n_last - n_skip;
  const TileKeys<CACHE> by_energy = load_keys<CACHE>(en, t0, t1, n_skip > 0);
  const TileKeys<CACHE> by_loss_k = load_keys<CACHE>(lk, t0, t1, n_sparse_k > 0 && n_sparse_k < n_keep);
  const TileKeys<CACHE> by_loss_v = load_keys<CACHE>(lv, t0, t1, n_sparse_v > 0 && n_sparse_v < n_keep);
  if (!in_regs)
    for (int t = t0; t < t1; t++) km[t] = vm[t] = HS_DENSE;
  // the n_skip lowest-energy tiles are skipped
  mark_lowest(by_energy, [&](int t) { return !is_protected(t); }, n_skip, sm, tid,
              [&](int t) { set_k(t, HS_SKIP); set_v(t, HS_SKIP); });
  // of the kept ones, the n_sparse_x with the lowest pruning loss are 2:4 (all of them: no ranking)
  auto kept = [&](int t) { return !is_protected(t) && state_k(t) != HS_SKIP; };
  if (n_sparse_k >= n_keep) {
    for (int t = t0; t < t1; t++) if (kept(t)) set_k(t, HS_SPARSE24);
  } else {
    mark_lowest(by_loss_k, kept, n_sparse_k, sm, tid, [&](int t) { set_k(t, HS_SPARSE24); });
  }
  if (n_sparse_v >= n_keep) {
    for (int t = t0; t < t1; t++) if (kept(t)) set_v(t, HS_SPARSE24);
  } else {
    mark_lowest(by_loss_v, kept, n_sparse_v, sm, tid, [&](int t) { set_v(t, HS_SPARSE24); });
  }
  // slots in ascending tile order
  int n[4] = {0, 0, 0, 0};  // dense K, 2:4 K, dense V, 2:4 V
  for (int t = t0; t < t1; t++) {
    const int sk = state_k(t), sv = state_v(t);
    n[0] += sk == HS_DENSE; n[1] += sk == HS_SPARSE24; n[2] += sv == HS_DENSE; n[3] += sv == HS_SPARSE24;
  }
  block_exclusive_scan(n, sm.wsum, tid);
  for (int t = t0; t < t1; t++) {
    const int sk = state_k(t), sv = state_v(t);
    km[t] = sk == HS_DENSE ? ++n[0] : (sk == HS_SPARSE24 ? -(++n[1]) : 0);
    vm[t] = sv == HS_DENSE ? ++n[2] : (sv == HS_SPARSE24 ? -(++n[3]) : 0);
  }
}

// ----------------------------------------------------------------------------------
// Slot assignment for one row from known tile states (the two sequential counters per tensor of
// Sec. III-B): tile t in state (sk, sv) = state(t) takes the next slot of the pool each state names.
// A tile is stored only if both of its pools still have a free slot when its turn comes; otherwise
// it is left out of K and V alike, takes no slot in either pool (so the used slots of a pool are
// always 0 .. count-1 with no holes, which is what appending relies on), and bit 0 of *flag is set.
// state(t) must return a consistent pair (both SKIP or neither).  emit(t, mk, mv) receives the map
// entries +-(slot + 1) or 0.  One workgroup of 256 threads per row; each thread owns a contiguous
// run of tiles.  When everything fits (the totals say so) the slots are prefix counts; a row that
// overflows is walked again by one thread, in order, so that which tiles survive is exactly what a
// sequential walk gives.
// ----------------------------------------------------------------------------------
struct SlotShared {
  int wsum[4][4];
  int total[4];
};

template <class State, class Emit>
__device__ __forceinline__ void assign_slots_row(int T, int tid, int cap_dk, int cap_sk, int cap_dv, int cap_sv,
                                                 SlotShared& sm, int32_t* flag, State state, Emit emit) {
  const int per = (T + 255) / 256;
  const int t0 = min(tid * per, T), t1 = min(t0 + per, T);
  int n[4] = {0, 0, 0, 0};  // dense K, 2:4 K, dense V, 2:4 V
  for (int t = t0; t < t1; t++) {
    int sk, sv;
    state(t, sk, sv);
    n[0] += sk == HS_DENSE; n[1] += sk == HS_SPARSE24; n[2] += sv == HS_DENSE; n[3] += sv == HS_SPARSE24;
  }
  int base[4] = {n[0], n[1], n[2], n[3]};
  block_exclusive_scan(base, sm.wsum, tid);
#pragma unroll
  for (int i = 0; i < 4; i++)
    if (tid == 255) sm.total[i] = base[i] + n[i];
  __syncthreads();
  const bool all_fit = sm.total[0] <= cap_dk && sm.total[1] <= cap_sk && sm.total[2] <= cap_dv && sm.total[3] <= cap_sv;
  if (all_fit) {
    for (int t = t0; t < t1; t++) {
      int sk, sv;
      state(t, sk, sv);
      const int mk = sk == HS_DENSE ? ++base[0] : (sk == HS_SPARSE24 ? -(++base[1]) : 0);
      const int mv = sv == HS_DENSE ? ++base[2] : (sv == HS_SPARSE24 ? -(++base[3]) : 0);
      emit(t, mk, mv);
    }
  } else if (tid == 0) {
    int c[4] = {0, 0, 0, 0};
    bool dropped = false;
    for (int t = 0; t < T; t++) {
      int sk, sv;
      state(t, sk, sv);
      int mk = 0, mv = 0;
      if (sk != HS_SKIP) {
        const bool room_k = sk == HS_DENSE ? c[0] < cap_dk : c[1] < cap_sk;
        const bool room_v = sv == HS_DENSE ? c[2] < cap_dv : c[3] < cap_sv;
        if (room_k && room_v) {
          mk = sk == HS_DENSE ? ++c[0] : -(++c[1]);
          mv = sv == HS_DENSE ? ++c[2] : -(++c[3]);
        } else {
          dropped = true;
        }
      }
      emit(t, mk, mv);
    }
    if (dropped && flag != nullptr) atomicOr(flag, 1);
  }
}

// Explicit per-tile states (device int8 [rows, T], the block-level masks a pruner hands over:
// Sec. III-A, "agnostic to the pruning algorithms") -> signed index maps (Sec. III-B).  A pair of
// states that is not valid (a value outside SKIP / DENSE / SPARSE24, or a tile skipped in only one
// of K and V) is stored as SKIP in both tensors and sets bit 1 of *flag.
__global__ __launch_bounds__(256) void states_to_maps_kernel(const int8_t* __restrict__ state_k,
                                                             const int8_t* __restrict__ state_v, int T, int cap_dk,
                                                             int cap_sk, int cap_dv, int cap_sv,
                                                             int32_t* __restrict__ k_map, int32_t* __restrict__ v_map,
                                                             int32_t* flag) {
  __shared__ SlotShared sm;
  const int row = blockIdx.x, tid = threadIdx.x;
  const int8_t* sk_row = state_k + (int64_t)row * T;
  const int8_t* sv_row = state_v + (int64_t)row * T;
  int32_t* km = k_map + (int64_t)row * T;
  int32_t* vm = v_map + (int64_t)row * T;
  bool invalid = false;
  assign_slots_row(
      T, tid, cap_dk, cap_sk, cap_dv, cap_sv, sm, flag,
      [&](int t, int& sk, int& sv) {
        sk = sk_row[t];
        sv = sv_row[t];
        if (sk < 0 || sk > 2 || sv < 0 || sv > 2 || (sk == HS_SKIP) != (sv == HS_SKIP)) {
          invalid = true;
          sk = sv = HS_SKIP;
        }
      },
      [&](int t, int mk, int mv) { km[t] = mk; vm[t] = mv; });
  if (invalid && flag != nullptr) atomicOr(flag, 2);
}

// Appending (Sec. III-B counters): map entries of tiles [tile, tile + n_tiles) of every row = the
// next slots of the pool their state names, counted from how many tiles of that kind the row
// holds; tiles for which a pool has no slot left stay skipped and raise *overflow.  One workgroup
// per row.
__global__ __launch_bounds__(256) void append_slots_kernel(int T, int tile, int n_tiles, int state_k, int state_v,
                                                           hs_kv_dev kv, int32_t* overflow) {
  __shared__ int part[4][4];
  const int row = blockIdx.x, tid = threadIdx.x;
  int32_t* km = const_cast<int32_t*>(kv.k_map) + (int64_t)row * T;
  int32_t* vm = const_cast<int32_t*>(kv.v_map) + (int64_t)row * T;
  int n[4] = {0, 0, 0, 0};  // dense K, 2:4 K, dense V, 2:4 V
  for (int t = tid; t < T; t += 256) {
    if (t >= tile && t < tile + n_tiles) continue;
    const int a = km[t], c = vm[t];
    n[0] += a > 0; n[1] += a < 0; n[2] += c > 0; n[3] += c < 0;
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n[i] += __shfl_xor(n[i], off);
    if ((tid & 63) == 0) part[i][tid >> 6] = n[i];
  }
  __syncthreads();
  int c[4];
#pragma unroll
  for (int i = 0; i < 4; i++) c[i] = part[i][0] + part[i][1] + part[i][2] + part[i][3];
  const int ck = state_k == HS_DENSE ? c[0] : c[1], cv = state_v == HS_DENSE ? c[2] : c[3];
  const int room_k = (state_k == HS_DENSE ? kv.cap_dense_k : kv.cap_sparse_k) - ck;
  const int room_v = (state_v == HS_DENSE ? kv.cap_dense_v : kv.cap_sparse_v) - cv;
  for (int i = tid; i < n_tiles; i += 256) {  // the i-th appended tile takes the i-th free slot of each pool
    const bool fits = i < room_k && i < room_v;
    km[tile + i] = !fits ? 0 : (state_k == HS_DENSE ? ck + i + 1 : -(ck + i + 1));
    vm[tile + i] = !fits ? 0 : (state_v == HS_DENSE ? cv + i + 1 : -(cv + i + 1));
    if (!fits && overflow != nullptr) *overflow = 1;
  }
}

// V tiles of a bf16 cache in fp16 encoding.  A bf16 pair is converted (round to nearest) and read
// back: equal values mean the pair survives the round trip (NaN never does, infinities do).
__device__ __forceinline__ bool pair_to_f16(uint32_t bf_pair, uint32_t& f16_pair) {
  const float f0 = hs_elem<false>::lo_f32(bf_pair), f1 = hs_elem<false>::hi_f32(bf_pair);
  f16_pair = hs_elem<true>::pack2(f0, f1);
  return hs_elem<true>::lo_f32(f16_pair) == f0 && hs_elem<true>::hi_f32(f16_pair) == f1;
}
__device__ __forceinline__ uint32_t pair_to_bf16(uint32_t f16_pair) {  // exact for what pair_to_f16 accepted
  const uint32_t lo = __float_as_uint(hs_elem<true>::lo_f32(f16_pair)), hi = __float_as_uint(hs_elem<true>::hi_f32(f16_pair));
  return (lo >> 16) | (hi & 0xffff0000u);
}

// ----------------------------------------------------------------------------------
// Tile writers shared by the compress, append and re-compress kernels.  Workgroup of 4 waves;
// wave w, lane l = 16a + r.
// ----------------------------------------------------------------------------------
// 2:4 K tile.  Lane (w, a, r) prunes token 16w + r, channels 64kb + 16a .. +16 for kb = 0, 1;
// load(kb, half) returns the 8 channels 64kb + 16a + 8 half .. +8 of that token.
template <class Load>
__device__ __forceinline__ void k_sparse_store(uint8_t* nnz, uint8_t* meta, int w, int l, int rule, Load load) {
  uint32_t idx = 0;
#pragma unroll
  for (int kb = 0; kb < 2; kb++) {
    const uint4 d0 = load(kb, 0);
    const uint4 d1 = load(kb, 1);
    const uint32_t wds[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
    uint32_t out[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const uint32_t x0 = wds[2 * q] & 0xffffu, x1 = wds[2 * q] >> 16, x2 = wds[2 * q + 1] & 0xffffu, x3 = wds[2 * q + 1] >> 16;
      uint32_t nib;
      top2_emit(top2_mask(x0, x1, x2, x3, rule), x0, x1, x2, x3, out[q], nib);
      idx |= nib << (16 * kb + 4 * q);
    }
    st16<true>(nnz + ((w * 2 + kb) * 64 + l) * 16, make_uint4(out[0], out[1], out[2], out[3]));
  }
  *reinterpret_cast<uint32_t*>(meta + (l * 4 + w) * 4) = idx;
}

// V tile (dense if mv > 0, 2:4 if mv < 0; mv = +-(slot + 1), workgroup-uniform, != 0) from the
// tile staged in LDS as vl[token][channel] (row stride kVStride); the caller has synchronised.
// The words to store are built first.  v_f16 (bf16 cache): if every value the tile stores is
// exact in fp16 (workgroup vote), the tile is written in fp16 encoding and *map_entry, which the
// caller has set to mv, gets HS_MAP_F16, so that the attention kernels can feed the softmax
// numerators as one fp16 term.  256 threads call this, tid = 0 .. 255; vote(bad) tells each whether any of them is bad.  It is called
// exactly once if v_f16 is set and not at all otherwise, and there is no other barrier here: append_kernel's other waves count on it.
template <class Vote>
__device__ __forceinline__ void v_tile_store(const uint16_t* vl, int mv, int32_t* map_entry, const hs_kv_dev& kv,
                                             int64_t row, int rule, int v_f16, int tid, Vote vote) {
  const int w = tid >> 6, l = tid & 63, a = l >> 4, r = l & 15;
  uint32_t words[4][4];
  const int n_chunks = mv > 0 ? 4 : 2;  // 16-byte chunks this lane stores
  uint32_t idx = 0;
  if (mv > 0) {
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int ch = 4 * w + j, mb = ch >> 1, hh = ch & 1;
      const int c = 16 * mb + r;
#pragma unroll
      for (int p = 0; p < 4; p++) {
        const int e0 = 2 * p, e1 = 2 * p + 1;
        const int tok0 = 16 * (2 * hh + (e0 >> 2)) + 4 * a + (e0 & 3);
        const int tok1 = 16 * (2 * hh + (e1 >> 2)) + 4 * a + (e1 & 3);
        words[j][p] = (uint32_t)vl[tok0 * kVStride + c] | ((uint32_t)vl[tok1 * kVStride + c] << 16);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int mb = 2 * w + j, c = 16 * mb + r;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int g = hs_v_group(a, q);
        const uint32_t x0 = vl[(4 * g + 0) * kVStride + c], x1 = vl[(4 * g + 1) * kVStride + c];
        const uint32_t x2 = vl[(4 * g + 2) * kVStride + c], x3 = vl[(4 * g + 3) * kVStride + c];
        uint32_t nib;
        top2_emit(top2_mask(x0, x1, x2, x3, rule), x0, x1, x2, x3, words[j][q], nib);
        idx |= nib << (16 * j + 4 * q);
      }
    }
  }
  if (v_f16) {  // workgroup-uniform
    uint32_t conv[4][4];
    int bad = 0;
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int p = 0; p < 4; p++)
        if (j < n_chunks) bad |= !pair_to_f16(words[j][p], conv[j][p]);
    if (!vote(bad)) {
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int p = 0; p < 4; p++)
          if (j < n_chunks) words[j][p] = conv[j][p];
      if (tid == 0) *map_entry = mv > 0 ? (mv | HS_MAP_F16) : -(-mv | HS_MAP_F16);
    }
  }
  if (mv > 0) {
    uint8_t* dst = const_cast<uint8_t*>(kv.v_dense) + (row * kv.cap_dense_v + (mv - 1)) * (int64_t)HS_TILE_DENSE_BYTES;
#pragma unroll
    for (int j = 0; j < 4; j++)
      st16<false>(dst + ((4 * w + j) * 64 + l) * 16, make_uint4(words[j][0], words[j][1], words[j][2], words[j][3]));
  } else {
    const int64_t slot = row * kv.cap_sparse_v + (-mv - 1);
    uint8_t* nnz = const_cast<uint8_t*>(kv.v_nnz) + slot * (int64_t)HS_TILE_NNZ_BYTES;
    uint8_t* meta = const_cast<uint8_t*>(kv.v_meta) + slot * (int64_t)HS_TILE_META_BYTES;
#pragma unroll
    for (int j = 0; j < 2; j++)
      st16<true>(nnz + ((2 * w + j) * 64 + l) * 16, make_uint4(words[j][0], words[j][1], words[j][2], words[j][3]));
    *reinterpret_cast<uint32_t*>(meta + (l * 4 + w) * 4) = idx;
  }
}

__device__ __forceinline__ void v_tile_store(const uint16_t* vl, int mv, int32_t* map_entry, const hs_kv_dev& kv,
                                             int64_t row, int rule, int v_f16, int tid) {  // by the whole workgroup
  v_tile_store(vl, mv, map_entry, kv, row, rule, v_f16, tid, [](int bad) { return __syncthreads_or(bad) != 0; });
}

// Dense V tile in pool order -> vl[token][channel], as bf16 patterns when the tile is held in fp16
// encoding (is_f16); the caller synchronises afterwards.
__device__ __forceinline__ void v_dense_to_lds(const uint8_t* src, bool is_f16, uint16_t* vl, int tid) {
  const int w = tid >> 6, l = tid & 63, a = l >> 4, r = l & 15;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const int ch = 4 * w + j, mb = ch >> 1, hh = ch & 1, c = 16 * mb + r;
    const uint4 d = *reinterpret_cast<const uint4*>(src + (ch * 64 + l) * 16);
    uint32_t vals[4] = {d.x, d.y, d.z, d.w};
    if (is_f16) {
#pragma unroll
      for (int i = 0; i < 4; i++) vals[i] = pair_to_bf16(vals[i]);
    }
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const int tok = 16 * (2 * hh + (e >> 2)) + 4 * a + (e & 3);
      vl[tok * kVStride + c] = (uint16_t)((vals[e >> 1] >> (16 * (e & 1))) & 0xffffu);
    }
  }
}

// ----------------------------------------------------------------------------------
// Fused prune + pack (Sec. IV-B): one workgroup per tile, K then V.
// ----------------------------------------------------------------------------------
// uni_k / uni_v: 0 = read the tile's map entries (written by an earlier launch); HS_DENSE or
// HS_SPARSE24 = every tile of that tensor is of this kind, but for the n_first first and n_last last
// ones of a row, which are dense: the entry follows from the tile's index and this kernel writes it
// (saves the separate map-fill launch of the unranked policies: 8 rows of 64 / 512 tiles with protected
// ends 11.5 -> 7.5 / 41.3 -> 36.3 us).
// NTL: the inputs of tiles that become 2:4 are read non-temporally.  That pays when K and V exceed the
// last-level cache (B 8 x L 131072: 1.20 -> 1.08 ms) and costs a little when they fit (L 32768: 38.7 -> 40.3 us;
// the two 16-byte reads a lane makes of one K line then both go to L2), so the launcher decides by size.
// APPEND: the tile is new in its row, in states uni_k / uni_v: this kernel counts the row's tiles of these kinds itself
// (next slot of each pool, Sec. III-B) while the tile's first loads are under way, writes the entries, and raises
// *overflow where a pool has no slot left.  Counting in every workgroup saves the launch of append_slots_kernel.
// RANKED: the tile's entries follow from the scores of its row of at most 64 tiles, which every wave ranks for itself, a tile per lane, while
// the tile's V is on its way: no select_kernel and no barrier (8 rows of 16 tiles 14.7 -> 12.0 us a call).
struct RankBy {
  const double* scores;  // [3][rows][T] of score_kernel; counts as for select_kernel
  int n_skip, n_sparse_k, n_sparse_v;
};
// of the lanes in `among` (wave-uniform), those that hold the n lowest (key, lane); there are at least n
__device__ __forceinline__ unsigned long long lowest_lanes(unsigned long long key, unsigned long long among, int n, int l) {
  if (n <= 0) return 0ull;
  int rank = 0;
  for (unsigned long long left = among; left != 0ull; left &= left - 1) {
    const int j = __builtin_ctzll(left);
    const unsigned long long kj = (unsigned)__builtin_amdgcn_readlane((int)key, j) |
                                  (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(key >> 32), j) << 32;
    rank += kj < key || (kj == key && j < l);
  }
  return __ballot(rank < n) & among;
}
// the map entries of tile t of a row: as select_kernel gives them
__device__ __forceinline__ void ranked_entries(const RankBy& by, int64_t rows, int64_t row, int T, int t, int n_first, int n_last, int l, int& mk,
                                               int& mv) {
  const int n_keep = T - n_first - n_last - by.n_skip;
  const bool rank_k = by.n_sparse_k > 0 && by.n_sparse_k < n_keep, rank_v = by.n_sparse_v > 0 && by.n_sparse_v < n_keep;
  unsigned long long key[3];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    const bool wanted = i == 0 ? by.n_skip > 0 : (i == 1 ? rank_k : rank_v);
    key[i] = wanted && l < T ? (unsigned long long)__double_as_longlong(by.scores[(i * rows + row) * T + l]) : 0ull;
  }
  const unsigned long long all = T >= 64 ? ~0ull : (1ull << T) - 1, middle = __ballot(l >= n_first && l < T - n_last);
  const unsigned long long skip = lowest_lanes(key[0], middle, by.n_skip, l), kept = middle & ~skip;
  const unsigned long long sk = by.n_sparse_k >= n_keep ? kept : lowest_lanes(key[1], kept, rank_k ? by.n_sparse_k : 0, l);
  const unsigned long long sv = by.n_sparse_v >= n_keep ? kept : lowest_lanes(key[2], kept, rank_v ? by.n_sparse_v : 0, l);
  const unsigned long long below = (1ull << t) - 1;
  auto entry = [&](unsigned long long sparse) {
    if ((skip >> t) & 1) return 0;
    const bool is_sparse = (sparse >> t) & 1;
    const int slot = __builtin_popcountll((is_sparse ? sparse : all & ~skip & ~sparse) & below);
    return is_sparse ? -(slot + 1) : slot + 1;
  };
  mk = entry(sk);
  mv = entry(sv);
}

template <bool NTL, bool APPEND, bool RANKED = false>
__global__ __launch_bounds__(256) void pack_kernel(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                                                   int64_t sb, int64_t sh, int64_t st, int Hkv, int T, hs_kv_dev kv,
                                                   int uni_k, int uni_v, int n_first, int n_last, int rule, int t0, int v_f16,
                                                   const int32_t* __restrict__ t0_rows, int32_t* overflow, RankBy by) {
  __shared__ uint16_t vl[HS_BT * kVStride];
  // source tile blockIdx.x of K, V goes to tile t of the cache (t0 = 0 except when appending;
  // t0_rows: one t0 per batch row, entries that are not a tile index leave the row out)
  const int ts = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  if (t0_rows != nullptr) {
    t0 = t0_rows[b];
    if (t0 < 0 || t0 >= T) return;  // the whole workgroup
  }
  const int t = ts + t0;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, a = l >> 4, r = l & 15;
  const int64_t row = (int64_t)b * Hkv + h;
  const uint16_t* kt = K + b * sb + h * sh + (int64_t)ts * HS_BT * st;
  const uint16_t* vt = V + b * sb + h * sh + (int64_t)ts * HS_BT * st;
  int mk, mv;
  if constexpr (APPEND) {
    __shared__ int part[2][4];
    int32_t* km = const_cast<int32_t*>(kv.k_map) + row * T;
    int32_t* vm = const_cast<int32_t*>(kv.v_map) + row * T;
    if (uni_v == HS_SPARSE24) stage_v_tile<NTL>(vt, st, vl);
    else stage_v_tile<false>(vt, st, vl);
    int nk = 0, nv = 0;  // entries [t0, t0 + gridDim.x) are being written by this launch and do not count
#pragma unroll 4
    for (int i = tid; i < T; i += 256) {
      const bool old = i < t0 || i >= t0 + (int)gridDim.x;
      const int a_ = old ? km[i] : 0, c_ = old ? vm[i] : 0;
      nk += uni_k == HS_DENSE ? a_ > 0 : a_ < 0;
      nv += uni_v == HS_DENSE ? c_ > 0 : c_ < 0;
    }
    nk = wave_scan_sum(nk);
    nv = wave_scan_sum(nv);
    if (l == 63) { part[0][w] = nk; part[1][w] = nv; }
    __syncthreads();
    const int sk = part[0][0] + part[0][1] + part[0][2] + part[0][3] + ts, sv = part[1][0] + part[1][1] + part[1][2] + part[1][3] + ts;
    const bool fits = sk < (uni_k == HS_DENSE ? kv.cap_dense_k : kv.cap_sparse_k) && sv < (uni_v == HS_DENSE ? kv.cap_dense_v : kv.cap_sparse_v);
    mk = !fits ? 0 : (uni_k == HS_DENSE ? sk + 1 : -(sk + 1));
    mv = !fits ? 0 : (uni_v == HS_DENSE ? sv + 1 : -(sv + 1));
    if (tid == 0) {
      km[t] = mk;
      vm[t] = mv;
      if (!fits && overflow != nullptr) *overflow = 1;
    }
    if (!fits) return;  // the whole workgroup
  } else if constexpr (RANKED) {
    stage_v_tile<NTL>(vt, st, vl);
    ranked_entries(by, (int64_t)gridDim.z * Hkv, row, T, t, n_first, n_last, l, mk, mv);
    if (tid == 0) {
      const_cast<int32_t*>(kv.k_map)[row * T + t] = mk;
      const_cast<int32_t*>(kv.v_map)[row * T + t] = mv;
    }
  } else if (uni_k != 0) {
    // slots in tile order, one counter per pool: of a 2:4 tensor, the protected tiles are the dense pool
    const bool end = t >= T - n_last, prot = t < n_first || end;
    const int dense_slot = end ? t - (T - n_last) + n_first : t;
    mk = uni_k == HS_DENSE ? t + 1 : (prot ? dense_slot + 1 : -(t - n_first + 1));
    mv = uni_v == HS_DENSE ? t + 1 : (prot ? dense_slot + 1 : -(t - n_first + 1));
    if (tid == 0) {
      const_cast<int32_t*>(kv.k_map)[row * T + t] = mk;
      const_cast<int32_t*>(kv.v_map)[row * T + t] = mv;
    }
  } else {
    mk = kv.k_map[row * T + t];
    mv = kv.v_map[row * T + t];
  }
  if (!APPEND && !RANKED) {
    if (mv < 0) stage_v_tile<NTL>(vt, st, vl);
    else if (mv > 0) stage_v_tile<false>(vt, st, vl);
  }

  // ---- K ----
  if (mk > 0) {  // dense: permuted copy into operand order
    uint8_t* dst = const_cast<uint8_t*>(kv.k_dense) + (row * kv.cap_dense_k + (mk - 1)) * (int64_t)HS_TILE_DENSE_BYTES;
    const uint16_t* src = kt + (int64_t)(16 * w + r) * st + 8 * a;
#pragma unroll
    for (int s = 0; s < 4; s++) {
      st16<false>(dst + ((w * 4 + s) * 64 + l) * 16, ld16<false>(src + 32 * s));
    }
  } else if (mk < 0) {
    const int64_t slot = row * kv.cap_sparse_k + (-mk - 1);
    const uint16_t* src = kt + (int64_t)(16 * w + r) * st + 16 * a;
    k_sparse_store(const_cast<uint8_t*>(kv.k_nnz) + slot * (int64_t)HS_TILE_NNZ_BYTES,
                   const_cast<uint8_t*>(kv.k_meta) + slot * (int64_t)HS_TILE_META_BYTES, w, l, rule,
                   [&](int kb, int half) { return ld16<NTL>(src + 64 * kb + 8 * half); });
  }

  // ---- V ----
  if (mv == 0) return;
  __syncthreads();
  v_tile_store(vl, mv, const_cast<int32_t*>(kv.v_map) + row * T + t, kv, row, rule, v_f16, tid);
}

// Appends tile blockIdx.x of K, V to its row as tile t0 + blockIdx.x (t0_rows: one t0 per batch row, entries that are not a tile index
// leave the row out), in states uni_k / uni_v: what pack_kernel does with APPEND, for few tiles.  There the call is one chain of
// latencies (place, tile, maps, stores), so 4 waves take K and 4 take V: either half requests its tile and counts its map at once, and
// both prune at the same time.  us, by 4 waves one after the other / by 8: 8 rows of 128 tiles, one tile 6.0 / 5.0, fp16 5.1 / 4.5; 128 rows
// 6.2 / 5.3; 8 rows of 2048 6.6 / 5.5; 8 tiles in each of 8 rows 6.2 / 5.3.
__global__ __launch_bounds__(512) void append_kernel(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                                                     int64_t sb, int64_t sh, int64_t st, int T, hs_kv_dev kv, int uni_k, int uni_v,
                                                     int rule, int t0, int v_f16, const int32_t* __restrict__ t0_rows, int32_t* overflow) {
  __shared__ uint16_t vl[HS_BT * kVStride];
  __shared__ int part[2][4], bad_waves[4];
  const int ts = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  if (t0_rows != nullptr) {
    t0 = t0_rows[b];
    if (t0 < 0 || t0 >= T) return;  // the whole workgroup
  }
  const int t = ts + t0;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool for_v = wave >= 4;  // wave-uniform
  const int tid = threadIdx.x & 255, w = wave & 3, l = tid & 63, a = l >> 4, r = l & 15;
  const int64_t row = (int64_t)b * gridDim.y + h;
  const int64_t from = b * sb + h * sh + (int64_t)ts * HS_BT * st;
  // K: what the thread stores (dense: channels 32 i + 8 a .. +7 of its token; 2:4: 64 (i / 2) + 16 a + 8 (i % 2) .. +7); V: its part of the rows
  const uint16_t* src = for_v ? V + from + (tid >> 4) * st + 8 * (tid & 15) : K + from + (16 * w + r) * st + (uni_k == HS_DENSE ? 8 : 16) * a;
  uint4 d[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int64_t step = for_v ? 16 * i * st : (uni_k == HS_DENSE ? 32 * i : 64 * (i >> 1) + 8 * (i & 1));
    d[i] = ld16<false>(src + step);
  }
  int32_t* const map = const_cast<int32_t*>(for_v ? kv.v_map : kv.k_map) + row * T;
  const bool dense = (for_v ? uni_v : uni_k) == HS_DENSE;
  int n = 0;  // entries [t0, t0 + gridDim.x) are being written by this launch and do not count
#pragma unroll 4
  for (int i = tid; i < T; i += 256) {
    const bool old = i < t0 || i >= t0 + (int)gridDim.x;
    const int e = old ? map[i] : 0;
    n += dense ? e > 0 : e < 0;
  }
  n = wave_scan_sum(n);
  if (l == 63) part[for_v][w] = n;
  if (for_v) {
#pragma unroll
    for (int i = 0; i < 4; i++) {  // as stage_v_tile
      uint2* dst = reinterpret_cast<uint2*>(vl + ((tid >> 4) + 16 * i) * kVStride + 8 * (tid & 15));
      dst[0] = make_uint2(d[i].x, d[i].y);
      dst[1] = make_uint2(d[i].z, d[i].w);
    }
  }
  __syncthreads();
  const int sk = part[0][0] + part[0][1] + part[0][2] + part[0][3] + ts, sv = part[1][0] + part[1][1] + part[1][2] + part[1][3] + ts;
  const bool fits = sk < (uni_k == HS_DENSE ? kv.cap_dense_k : kv.cap_sparse_k) && sv < (uni_v == HS_DENSE ? kv.cap_dense_v : kv.cap_sparse_v);
  const int slot = for_v ? sv : sk, entry = !fits ? 0 : (dense ? slot + 1 : -(slot + 1));
  if (tid == 0) {
    map[t] = entry;
    if (!fits && overflow != nullptr) *overflow = 1;
  }
  if (!fits) return;  // the whole workgroup
  if (!for_v) {
    if (dense) {
      uint8_t* dst = const_cast<uint8_t*>(kv.k_dense) + (row * kv.cap_dense_k + slot) * (int64_t)HS_TILE_DENSE_BYTES;
#pragma unroll
      for (int i = 0; i < 4; i++) st16<false>(dst + ((w * 4 + i) * 64 + l) * 16, d[i]);
    } else {
      const int64_t at = row * kv.cap_sparse_k + slot;
      k_sparse_store(const_cast<uint8_t*>(kv.k_nnz) + at * (int64_t)HS_TILE_NNZ_BYTES,
                     const_cast<uint8_t*>(kv.k_meta) + at * (int64_t)HS_TILE_META_BYTES, w, l, rule,
                     [&](int kb, int half) { return d[2 * kb + half]; });
    }
    // The vote that v_tile_store calls once if v_f16 is set.  (One barrier that both halves reach, between building V's words and storing
    // them, is slower: fp16 4.33 -> 4.45 us, bf16 of one head 4.49 -> 4.55.)
    if (v_f16) __syncthreads();
  } else {
    v_tile_store(vl, entry, map + t, kv, row, rule, v_f16, tid, [&](int bad) {
      const bool any = __any(bad);
      if (l == 0) bad_waves[w] = any;
      __syncthreads();
      return (bad_waves[0] | bad_waves[1] | bad_waves[2] | bad_waves[3]) != 0;
    });
  }
}

// ----------------------------------------------------------------------------------
// Further pruning of a packed cache (Sec. III, overview: after the prefill phase the dense pool
// can be pruned and compressed again, so that decode runs at another sparsity than prefill).
// ----------------------------------------------------------------------------------
// New state of a tile = the sparser of its current state and its target (DENSE < 2:4 < SKIP).
__device__ __forceinline__ int sparser_state(int map_entry, int target) {
  const int cur = map_entry > 0 ? HS_DENSE : (map_entry < 0 ? HS_SPARSE24 : HS_SKIP);
  const int rc = cur == HS_SKIP ? 2 : cur - 1, rt = target == HS_SKIP ? 2 : target - 1;
  const int rn = rc > rt ? rc : rt;
  return rn == 2 ? HS_SKIP : rn + 1;
}

// Target states of a re-compression: tgt_k / tgt_v (device int8 [rows, T]) when given -- a pair that is not valid
// leaves the tile as it is --; else the sign of map_k / map_v (maps the selection kernel wrote for a ranked target:
// > 0 dense, < 0 2:4, 0 skipped) when given; else DENSE for the n_first first and n_last last tiles of the row and
// frac_k / frac_v in between.
struct RestateTarget {
  const int8_t* tgt_k;
  const int8_t* tgt_v;
  const int32_t* map_k;
  const int32_t* map_v;
  int frac_k, frac_v, n_first, n_last;
};
// new states of tile t of a row; returns false if its explicit target pair is not valid
__device__ __forceinline__ bool restate_tile(const RestateTarget& tg, const hs_kv_dev& src, int64_t row, int T, int t, int& sk, int& sv) {
  const int64_t i = row * T + t;
  bool ok = true;
  int tk, tv;
  if (tg.tgt_k != nullptr) {
    tk = tg.tgt_k[i];
    tv = tg.tgt_v[i];
    if (tk < 0 || tk > 2 || tv < 0 || tv > 2 || (tk == HS_SKIP) != (tv == HS_SKIP)) {
      ok = false;
      tk = tv = HS_DENSE;  // no further pruning of this tile
    }
  } else if (tg.map_k != nullptr) {
    const int a = tg.map_k[i], c = tg.map_v[i];
    tk = a > 0 ? HS_DENSE : (a < 0 ? HS_SPARSE24 : HS_SKIP);
    tv = c > 0 ? HS_DENSE : (c < 0 ? HS_SPARSE24 : HS_SKIP);
  } else {
    const bool prot = t < tg.n_first || t >= T - tg.n_last;
    tk = prot ? HS_DENSE : tg.frac_k;
    tv = prot ? HS_DENSE : tg.frac_v;
  }
  sk = sparser_state(src.k_map[i], tk);
  sv = sparser_state(src.v_map[i], tv);
  if (sk == HS_SKIP || sv == HS_SKIP) sk = sv = HS_SKIP;  // a tile leaves K and V together
  return ok;
}
// a V tile that keeps its kind keeps its encoding bit
__device__ __forceinline__ int keep_encoding(int mv, int mv_old) {
  if (mv != 0 && (mv > 0) == (mv_old > 0) && hs_map_f16(mv_old)) mv = mv > 0 ? (mv | HS_MAP_F16) : -(-mv | HS_MAP_F16);
  return mv;
}

// Maps of the re-compressed cache: slots in ascending tile order with one counter per pool
// (Sec. III-B); a tile that keeps its kind keeps its encoding bit.  A tile for which a pool of dst
// has no slot left is left out of both tensors, takes no slot, and bit 0 of *overflow is raised
// (assign_slots_row); an explicit pair that is not valid raises bit 1.  One workgroup per row.
__global__ __launch_bounds__(256) void restate_kernel(int T, hs_kv_dev src, RestateTarget tg, hs_kv_dev dst, int32_t* overflow) {
  __shared__ SlotShared sm;
  const int row = blockIdx.x, tid = threadIdx.x;
  const int32_t* svm = src.v_map + (int64_t)row * T;
  int32_t* km = const_cast<int32_t*>(dst.k_map) + (int64_t)row * T;
  int32_t* vm = const_cast<int32_t*>(dst.v_map) + (int64_t)row * T;
  bool invalid = false;
  assign_slots_row(
      T, tid, dst.cap_dense_k, dst.cap_sparse_k, dst.cap_dense_v, dst.cap_sparse_v, sm, overflow,
      [&](int t, int& sk, int& sv) { invalid |= !restate_tile(tg, src, row, T, t, sk, sv); },
      [&](int t, int mk, int mv) {
        km[t] = mk;
        vm[t] = keep_encoding(mv, svm[t]);
      });
  if (invalid && overflow != nullptr) atomicOr(overflow, 2);
}

// One workgroup per tile: tiles that keep their kind are copied slot to slot; a dense tile that
// became 2:4 is read from its dense slot (pool order) and pruned with the writers above.
// COUNT: the maps of dst are not written yet: the workgroup counts the row's new states itself, takes its tile's slots as
// restate_kernel would hand them out and writes the tile's entries, which saves that launch.
constexpr int kCountEntries = 2 << 20;  // map entries that all workgroups of a launch may read to count: rows of up to 1448 tiles
template <bool COUNT>
__global__ __launch_bounds__(256) void repack_kernel(int Hkv, int T, hs_kv_dev src, RestateTarget tg, hs_kv_dev dst, int rule, int v_f16,
                                                     int32_t* overflow) {
  __shared__ __attribute__((aligned(16))) uint16_t vl[HS_BT * kVStride];
  static_assert((int64_t)sizeof(vl) * sizeof(vl) >= kCountEntries, "a byte of vl per tile of the row");
  const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, a = l >> 4, r = l & 15;
  const int64_t row = (int64_t)b * Hkv + h;
  const int mk_old = src.k_map[row * T + t], mv_old_raw = src.v_map[row * T + t];
  int mk, mv_raw;
  if constexpr (COUNT) {
    __shared__ int part[8][4], entry[2];
    uint8_t* const states = reinterpret_cast<uint8_t*>(vl);
    int n[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // dense K, 2:4 K, dense V, 2:4 V: of the row; of the tiles before this one
    for (int i = tid; i < T; i += 256) {
      int sk, sv;
      const bool ok = restate_tile(tg, src, row, T, i, sk, sv);
      if (!ok && i == t && overflow != nullptr) atomicOr(overflow, 2);
      states[i] = (uint8_t)(sk | sv << 2);
      const int c[4] = {sk == HS_DENSE, sk == HS_SPARSE24, sv == HS_DENSE, sv == HS_SPARSE24};
#pragma unroll
      for (int j = 0; j < 4; j++) {
        n[j] += c[j];
        n[4 + j] += i < t ? c[j] : 0;
      }
    }
#pragma unroll
    for (int j = 0; j < 8; j++) {
      const int s_ = wave_scan_sum(n[j]);
      if (l == 63) part[j][w] = s_;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; j++) n[j] = part[j][0] + part[j][1] + part[j][2] + part[j][3];
    const int sk = states[t] & 3, sv = states[t] >> 2;
    if (n[0] <= dst.cap_dense_k && n[1] <= dst.cap_sparse_k && n[2] <= dst.cap_dense_v && n[3] <= dst.cap_sparse_v) {
      mk = sk == HS_DENSE ? n[4] + 1 : (sk == HS_SPARSE24 ? -(n[5] + 1) : 0);
      mv_raw = sv == HS_DENSE ? n[6] + 1 : (sv == HS_SPARSE24 ? -(n[7] + 1) : 0);
    } else {  // some tile of the row finds a pool full: walked in order, as assign_slots_row does
      if (tid == 0) {
        int c[4] = {0, 0, 0, 0}, ek = 0, ev = 0;
        for (int i = 0; i <= t; i++) {
          const int a_ = states[i] & 3, b_ = states[i] >> 2;
          ek = ev = 0;
          if (a_ == HS_SKIP) continue;
          const bool room_k = a_ == HS_DENSE ? c[0] < dst.cap_dense_k : c[1] < dst.cap_sparse_k;
          const bool room_v = b_ == HS_DENSE ? c[2] < dst.cap_dense_v : c[3] < dst.cap_sparse_v;
          if (room_k && room_v) {
            ek = a_ == HS_DENSE ? ++c[0] : -(++c[1]);
            ev = b_ == HS_DENSE ? ++c[2] : -(++c[3]);
          } else if (i == t && overflow != nullptr) {
            atomicOr(overflow, 1);
          }
        }
        entry[0] = ek;
        entry[1] = ev;
      }
      __syncthreads();
      mk = entry[0];
      mv_raw = entry[1];
    }
    mv_raw = keep_encoding(mv_raw, mv_old_raw);
    if (tid == 0) {
      const_cast<int32_t*>(dst.k_map)[row * T + t] = mk;
      const_cast<int32_t*>(dst.v_map)[row * T + t] = mv_raw;
    }
    __syncthreads();  // vl holds the V tile from here on
  } else {
    mk = dst.k_map[row * T + t];
    mv_raw = dst.v_map[row * T + t];
  }
  if (mk == 0 || mv_raw == 0) return;  // dropped (both tensors together)
  const int mv_old = hs_map_plain(mv_old_raw), mv = hs_map_plain(mv_raw);
  // ---- K ----
  if (mk > 0) {
    const uint4* s4 = reinterpret_cast<const uint4*>(src.k_dense + (row * src.cap_dense_k + (mk_old - 1)) * (int64_t)HS_TILE_DENSE_BYTES);
    uint4* d4 = reinterpret_cast<uint4*>(const_cast<uint8_t*>(dst.k_dense) + (row * dst.cap_dense_k + (mk - 1)) * (int64_t)HS_TILE_DENSE_BYTES);
#pragma unroll
    for (int i = 0; i < 4; i++) d4[i * 256 + tid] = s4[i * 256 + tid];
  } else {
    const int64_t slot = row * dst.cap_sparse_k + (-mk - 1);
    uint8_t* nnz = const_cast<uint8_t*>(dst.k_nnz) + slot * (int64_t)HS_TILE_NNZ_BYTES;
    uint8_t* meta = const_cast<uint8_t*>(dst.k_meta) + slot * (int64_t)HS_TILE_META_BYTES;
    if (mk_old < 0) {
      const int64_t so = row * src.cap_sparse_k + (-mk_old - 1);
      const uint4* s4 = reinterpret_cast<const uint4*>(src.k_nnz + so * (int64_t)HS_TILE_NNZ_BYTES);
      uint4* d4 = reinterpret_cast<uint4*>(nnz);
#pragma unroll
      for (int i = 0; i < 2; i++) d4[i * 256 + tid] = s4[i * 256 + tid];
      if (tid < 64)
        reinterpret_cast<uint4*>(meta)[tid] = reinterpret_cast<const uint4*>(src.k_meta + so * (int64_t)HS_TILE_META_BYTES)[tid];
    } else {
      // dense pool order: chunk 4w + s of lane (a', r) = token 16w + r, channels 32s + 8a' .. +8
      const uint8_t* sd = src.k_dense + (row * src.cap_dense_k + (mk_old - 1)) * (int64_t)HS_TILE_DENSE_BYTES;
      k_sparse_store(nnz, meta, w, l, rule, [&](int kb, int half) {
        const int s = 2 * kb + (a >> 1), a2 = 2 * (a & 1) + half;
        return *reinterpret_cast<const uint4*>(sd + ((w * 4 + s) * 64 + 16 * a2 + r) * 16);
      });
    }
  }
  // ---- V ---- (branches are workgroup-uniform)
  if (mv > 0) {
    const uint4* s4 = reinterpret_cast<const uint4*>(src.v_dense + (row * src.cap_dense_v + (mv_old - 1)) * (int64_t)HS_TILE_DENSE_BYTES);
    uint4* d4 = reinterpret_cast<uint4*>(const_cast<uint8_t*>(dst.v_dense) + (row * dst.cap_dense_v + (mv - 1)) * (int64_t)HS_TILE_DENSE_BYTES);
#pragma unroll
    for (int i = 0; i < 4; i++) d4[i * 256 + tid] = s4[i * 256 + tid];
  } else if (mv_old < 0) {
    const int64_t so = row * src.cap_sparse_v + (-mv_old - 1), sn = row * dst.cap_sparse_v + (-mv - 1);
    const uint4* s4 = reinterpret_cast<const uint4*>(src.v_nnz + so * (int64_t)HS_TILE_NNZ_BYTES);
    uint4* d4 = reinterpret_cast<uint4*>(const_cast<uint8_t*>(dst.v_nnz) + sn * (int64_t)HS_TILE_NNZ_BYTES);
#pragma unroll
    for (int i = 0; i < 2; i++) d4[i * 256 + tid] = s4[i * 256 + tid];
    if (tid < 64)
      reinterpret_cast<uint4*>(const_cast<uint8_t*>(dst.v_meta) + sn * (int64_t)HS_TILE_META_BYTES)[tid] =
          reinterpret_cast<const uint4*>(src.v_meta + so * (int64_t)HS_TILE_META_BYTES)[tid];
  } else {
    v_dense_to_lds(src.v_dense + (row * src.cap_dense_v + (mv_old - 1)) * (int64_t)HS_TILE_DENSE_BYTES,
                   hs_map_f16(mv_old_raw), vl, tid);
    __syncthreads();
    v_tile_store(vl, mv, const_cast<int32_t*>(dst.v_map) + row * T + t, dst, row, rule, v_f16, tid);
  }
}

// ----------------------------------------------------------------------------------
// Unpack (tests / debugging): packed -> dense bf16 [B, Hkv, L, D], zeros where pruned
// or skipped.
// ----------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void unpack_kernel(int Hkv, int T, hs_kv_dev kv, uint16_t* __restrict__ K_out,
                                                     uint16_t* __restrict__ V_out) {
  __shared__ uint16_t vl[HS_BT * kVStride];
  const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, a = l >> 4, r = l & 15;
  const int64_t row = (int64_t)b * Hkv + h;
  const int mk = kv.k_map[row * T + t], mv_raw = kv.v_map[row * T + t];
  const bool v_is_f16 = hs_map_f16(mv_raw);
  const int mv = hs_map_plain(mv_raw);  // +-(slot + 1)
  uint16_t* ko = K_out + (row * T + t) * (int64_t)(HS_BT * HS_D);
  uint16_t* vo = V_out + (row * T + t) * (int64_t)(HS_BT * HS_D);
  {  // K: token 16w+r
    uint16_t* dst = ko + (16 * w + r) * HS_D;
    if (mk > 0) {
      const uint8_t* src = kv.k_dense + (row * kv.cap_dense_k + (mk - 1)) * (int64_t)HS_TILE_DENSE_BYTES;
#pragma unroll
      for (int s = 0; s < 4; s++)
        *reinterpret_cast<uint4*>(dst + 32 * s + 8 * a) = *reinterpret_cast<const uint4*>(src + ((w * 4 + s) * 64 + l) * 16);
    } else if (mk < 0) {
      const int64_t slot = row * kv.cap_sparse_k + (-mk - 1);
      const uint8_t* nnz = kv.k_nnz + slot * (int64_t)HS_TILE_NNZ_BYTES;
      const uint32_t idx = *reinterpret_cast<const uint32_t*>(kv.k_meta + slot * (int64_t)HS_TILE_META_BYTES + (l * 4 + w) * 4);
#pragma unroll
      for (int kb = 0; kb < 2; kb++) {
        const uint4 d = *reinterpret_cast<const uint4*>(nnz + ((w * 2 + kb) * 64 + l) * 16);
        const uint32_t vals[4] = {d.x, d.y, d.z, d.w};
        uint16_t o[16];
#pragma unroll
        for (int i = 0; i < 16; i++) o[i] = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const uint32_t nib = (idx >> (16 * kb + 4 * q)) & 0xfu;
          const uint32_t i0 = nib & 3u, i1 = nib >> 2;
#pragma unroll
          for (int p = 0; p < 4; p++) {
            if (i0 == (uint32_t)p) o[4 * q + p] = (uint16_t)(vals[q] & 0xffffu);
            if (i1 == (uint32_t)p) o[4 * q + p] = (uint16_t)(vals[q] >> 16);
          }
        }
        uint32_t pk[8];
#pragma unroll
        for (int i = 0; i < 8; i++) pk[i] = (uint32_t)o[2 * i] | ((uint32_t)o[2 * i + 1] << 16);
        uint4* d4 = reinterpret_cast<uint4*>(dst + 64 * kb + 16 * a);
        d4[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        d4[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; s++) *reinterpret_cast<uint4*>(dst + 32 * s + 8 * a) = make_uint4(0, 0, 0, 0);
    }
  }
  // V: rebuild the tile in LDS in [token][channel] order, then store it coalesced
  if (mv > 0) {
    v_dense_to_lds(kv.v_dense + (row * kv.cap_dense_v + (mv - 1)) * (int64_t)HS_TILE_DENSE_BYTES, v_is_f16, vl, tid);
  } else if (mv < 0) {
    const int64_t slot = row * kv.cap_sparse_v + (-mv - 1);
    const uint8_t* nnz = kv.v_nnz + slot * (int64_t)HS_TILE_NNZ_BYTES;
    const uint32_t idx = *reinterpret_cast<const uint32_t*>(kv.v_meta + slot * (int64_t)HS_TILE_META_BYTES + (l * 4 + w) * 4);
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int mb = 2 * w + j, c = 16 * mb + r;
      const uint4 d = *reinterpret_cast<const uint4*>(nnz + (mb * 64 + l) * 16);
      uint32_t vals[4] = {d.x, d.y, d.z, d.w};
      if (v_is_f16) {
#pragma unroll
        for (int i = 0; i < 4; i++) vals[i] = pair_to_bf16(vals[i]);
      }
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int g = hs_v_group(a, q);
        const uint32_t nib = (idx >> (16 * j + 4 * q)) & 0xfu;
        const uint32_t i0 = nib & 3u, i1 = nib >> 2;
#pragma unroll
        for (int p = 0; p < 4; p++) {
          uint16_t v = 0;
          if (i0 == (uint32_t)p) v = (uint16_t)(vals[q] & 0xffffu);
          if (i1 == (uint32_t)p) v = (uint16_t)(vals[q] >> 16);
          vl[(4 * g + p) * kVStride + c] = v;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int q = tid + 256 * i, tok = q >> 4, c8 = q & 15;
    uint4 d = make_uint4(0, 0, 0, 0);
    if (mv != 0) {
      const uint2* s2 = reinterpret_cast<const uint2*>(vl + tok * kVStride + 8 * c8);
      const uint2 lo = s2[0], hi = s2[1];
      d = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
    *reinterpret_cast<uint4*>(vo + tok * HS_D + 8 * c8) = d;
  }
}

}  // namespace

hipError_t hs_launch_score(const uint16_t* K, const uint16_t* V, int64_t sb, int64_t sh, int64_t st_, int B, int Hkv,
                           int T, int rule, int dtype, int what, double* scores, hipStream_t st) {
  const dim3 grid(T, Hkv, B), block(256);
  // non-temporal reads once K and V together are larger than the 256 MB last-level cache
  const bool nt = 2.0 * B * Hkv * T * HS_BT * HS_D * 2.0 > 256e6;
#define HS_SCORE(F16_, WHAT_)                                                                                              \
  do {                                                                                                                     \
    if (nt) hipLaunchKernelGGL((score_kernel<F16_, WHAT_, true>), grid, block, 0, st, K, V, sb, sh, st_, Hkv, T, rule, scores); \
    else hipLaunchKernelGGL((score_kernel<F16_, WHAT_, false>), grid, block, 0, st, K, V, sb, sh, st_, Hkv, T, rule, scores);   \
  } while (0)
  if (dtype == HS_FP16) {
    if (what == 1) HS_SCORE(true, 1); else if (what == 2) HS_SCORE(true, 2); else HS_SCORE(true, 3);
  } else {
    if (what == 1) HS_SCORE(false, 1); else if (what == 2) HS_SCORE(false, 2); else HS_SCORE(false, 3);
  }
#undef HS_SCORE
  return hipGetLastError();
}

hipError_t hs_launch_select(const double* scores, int rows, int T, int n_skip, int n_sparse_k, int n_sparse_v,
                            int n_first, int n_last, int32_t* k_map, int32_t* v_map, hipStream_t st) {
#define HS_SELECT(CACHE_)                                                                                                  \
  hipLaunchKernelGGL(select_kernel<CACHE_>, dim3(rows), dim3(256), 0, st, scores, rows, T, n_skip, n_sparse_k, n_sparse_v, \
                     n_first, n_last, k_map, v_map)
  if (T <= 512) HS_SELECT(2);  // every pass over the keys costs by the slots a thread has for them
  else if (T <= 2048) HS_SELECT(8);
  else HS_SELECT(0);
#undef HS_SELECT
  return hipGetLastError();
}

hipError_t hs_launch_pack(const uint16_t* K, const uint16_t* V, int64_t sb, int64_t sh, int64_t st_, int B, int Hkv,
                          int T, hs_kv_dev kv, int uni_k, int uni_v, int n_first, int n_last, int rule, int v_f16, hipStream_t st) {
  if (2.0 * B * Hkv * T * HS_BT * HS_D * 2.0 > 256e6)  // K and V together beyond the 256 MB last-level cache
    hipLaunchKernelGGL((pack_kernel<true, false>), dim3(T, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, uni_k, uni_v, n_first, n_last,
                       rule, 0,
                       v_f16, (const int32_t*)nullptr, (int32_t*)nullptr, RankBy{});
  else
    hipLaunchKernelGGL((pack_kernel<false, false>), dim3(T, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, uni_k, uni_v, n_first, n_last,
                       rule, 0,
                       v_f16, (const int32_t*)nullptr, (int32_t*)nullptr, RankBy{});
  return hipGetLastError();
}

hipError_t hs_launch_rank_and_pack(const uint16_t* K, const uint16_t* V, int64_t sb, int64_t sh, int64_t st_, int B, int Hkv, int T,
                                   hs_kv_dev kv, const double* scores, int n_skip, int n_sparse_k, int n_sparse_v, int n_first, int n_last,
                                   int rule, int v_f16, hipStream_t st) {
  hipLaunchKernelGGL((pack_kernel<false, false, true>), dim3(T, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, 0, 0, n_first, n_last,
                     rule, 0, v_f16, (const int32_t*)nullptr, (int32_t*)nullptr, RankBy{scores, n_skip, n_sparse_k, n_sparse_v});
  return hipGetLastError();
}

hipError_t hs_launch_append(const uint16_t* K, const uint16_t* V, int64_t sb, int64_t sh, int64_t st_, int B, int Hkv,
                            int T, int tile, int n_tiles, const int32_t* tile_rows, int state_k, int state_v,
                            hs_kv_dev kv, int rule, int v_f16, int32_t* overflow, hipStream_t st) {
  // Few tiles: a workgroup of 8 waves each.  From 1024 on the chip is full and the smaller workgroups of pack_kernel are faster (us, 8 / 4
  // waves: 512 tiles 8.8 / 8.9, 1024 13.2 / 12.9, 8192 80.4 / 73.0).
  const bool one_launch = tile_rows != nullptr || (double)n_tiles * B * Hkv * T <= (double)(4 << 20);
  if (one_launch && (int64_t)n_tiles * B * Hkv <= 512) {
    hipLaunchKernelGGL(append_kernel, dim3(n_tiles, Hkv, B), dim3(512), 0, st, K, V, sb, sh, st_, T, kv, state_k, state_v, rule, tile, v_f16,
                       tile_rows, overflow);
    return hipGetLastError();
  }
  const bool nt = 2.0 * B * Hkv * n_tiles * HS_BT * HS_D * 2.0 > 256e6;
  // One launch while the map entries that all workgroups read to count are few (32 MB): 1 x 8 rows of 512 tiles, one tile
  // 8.1 -> 6.1 us, 64 tiles 10.7 -> 8.1 us; 1 x 8 rows of 2048, 256 tiles 26.6 -> 23.3 us, 1024 tiles 76.5 us either way;
  // 16 x 8 rows of 512, 128 tiles 137 -> 140 us.  Per-row places come one tile at a time and always take it.
  if (one_launch) {
    if (nt)
      hipLaunchKernelGGL((pack_kernel<true, true>), dim3(n_tiles, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, state_k,
                         state_v, 0, 0, rule, tile, v_f16, tile_rows, overflow, RankBy{});
    else
      hipLaunchKernelGGL((pack_kernel<false, true>), dim3(n_tiles, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, state_k,
                         state_v, 0, 0, rule, tile, v_f16, tile_rows, overflow, RankBy{});
    return hipGetLastError();
  }
  hipLaunchKernelGGL(append_slots_kernel, dim3(B * Hkv), dim3(256), 0, st, T, tile, n_tiles, state_k, state_v, kv, overflow);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nt)
    hipLaunchKernelGGL((pack_kernel<true, false>), dim3(n_tiles, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, 0, 0, 0, 0, rule, tile,
                       v_f16, (const int32_t*)nullptr, (int32_t*)nullptr, RankBy{});
  else
    hipLaunchKernelGGL((pack_kernel<false, false>), dim3(n_tiles, Hkv, B), dim3(256), 0, st, K, V, sb, sh, st_, Hkv, T, kv, 0, 0, 0, 0, rule, tile,
                       v_f16, (const int32_t*)nullptr, (int32_t*)nullptr, RankBy{});
  return hipGetLastError();
}

hipError_t hs_launch_states_to_maps(const int8_t* state_k, const int8_t* state_v, int rows, int T, hs_kv_dev kv,
                                    int32_t* flag, hipStream_t st) {
  hipLaunchKernelGGL(states_to_maps_kernel, dim3(rows), dim3(256), 0, st, state_k, state_v, T, kv.cap_dense_k,
                     kv.cap_sparse_k, kv.cap_dense_v, kv.cap_sparse_v, const_cast<int32_t*>(kv.k_map),
                     const_cast<int32_t*>(kv.v_map), flag);
  return hipGetLastError();
}

hipError_t hs_launch_recompress(int B, int Hkv, int T, hs_kv_dev src, const int8_t* tgt_k, const int8_t* tgt_v,
                                const int32_t* tgt_map_k, const int32_t* tgt_map_v, int frac_state_k, int frac_state_v,
                                int n_first, int n_last, hs_kv_dev dst, int rule, int v_f16, int32_t* overflow,
                                hipStream_t st) {
  const RestateTarget tg{tgt_k, tgt_v, tgt_map_k, tgt_map_v, frac_state_k, frac_state_v, n_first, n_last};
  // One launch while the entries that all workgroups read to count (rows x T x T) are few.  The line is where the worse of two
  // forms breaks even.  us, two launches / one, K and V dense -> 2:4 | keys dense -> 2:4, V 2:4 already: 8 rows of 512 tiles (at
  // the line) 44.2 / 44.4 | 33.6 / 31.2; 2 of 1024 (at the line) 28.9 / 25.4 | 21.3 / 18.8; 10 of 512 54.9 / 55.5 | 42.1 / 39.9;
  // 6 of 724 46.9 / 49.3 | 36.4 / 36.3; 16 of 512 81.5 / 84.1 | 63.9 / 61.6; 64 of 256 152.5 / 155.4 | 133.0 / 127.6.
  if ((double)B * Hkv * T * T <= (double)kCountEntries) {
    hipLaunchKernelGGL(repack_kernel<true>, dim3(T, Hkv, B), dim3(256), 0, st, Hkv, T, src, tg, dst, rule, v_f16, overflow);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(restate_kernel, dim3(B * Hkv), dim3(256), 0, st, T, src, tg, dst, overflow);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(repack_kernel<false>, dim3(T, Hkv, B), dim3(256), 0, st, Hkv, T, src, tg, dst, rule, v_f16, overflow);
  return hipGetLastError();
}

hipError_t hs_launch_unpack(int B, int Hkv, int T, hs_kv_dev kv, uint16_t* K_out, uint16_t* V_out, hipStream_t st) {
  hipLaunchKernelGGL(unpack_kernel, dim3(T, Hkv, B), dim3(256), 0, st, Hkv, T, kv, K_out, V_out);
  return hipGetLastError();
}
