// Prefill attention: number of tile ranges, choice of the kernel, and the kernels of tensors with one kind of tile.
#include "hs_prefill_kernel.h"

// Ranges to cut a workgroup's tiles into, from what was measured on 2:4 tensors (32/8 heads): a tile takes a workgroup
// 1.0 us alone on its compute unit and 1.2 us beside a second one, so 512 workgroups at a time are two on every unit;
// splitting costs 8 us for the merge launch and the caller's scratch (5 us on the GPU alone) and 0.028 us per workgroup
// for writing and reading its 66 KB of partials.
// The number of ranges that makes this sum smallest is taken.  Measured, one range / the chosen number: 64 queries on
// 32768 tokens 501 / 41.5 us (32 ranges), on 2048 tokens 37 / 18.8 us (8); 256 queries on 32768 tokens 504 / 101 us (8);
// 1024 queries on 32768 tokens 510 / 347 us (2); whole prompts of 256 to 2048 tokens are fastest unsplit (2048: 46 us, two
// ranges 56 us), and there the sum says one range too.  Beyond 512 workgroups one range is only
// worse where a last, nearly empty round of equally long workgroups follows: queries at the end of a long context (2304
// queries on 32768 tokens, 576 workgroups: 1116 / 828 us).  Skipped tiles cost nothing, so the tiles are counted by what
// the pools can hold.  Where that says nothing about how many are kept (hs_kept_by_pools) they count as a quarter: few enough
// that a call does not get slower where three quarters are skipped, and where none is the best number is not far.  us, one range /
// the chosen number / the number for all tiles, mixed tensors, none | half | three quarters | nine tenths skipped: 64 queries
// on 32768 tokens 526 / 52 (16 ranges) / 47 (32) | 276 / 41 / 39 | 142 / 32 / 33 | 73 / 25 / 30; 256 queries on 8192 tokens
// 137 / 51 (4) / 47 (8) | 79 / 38 / 38 | 45 / 30 / 33 | 29 / 24 / 29; 2 x 512 queries on 4096 tokens 74 / 74 (1) / 67 (2) |
// 48 / 48 / 48 | 34 / 34 / 37 | 22 / 22 / 32.
int hs_prefill_auto_splits(int B, int Hq, int Hkv, int T, int Lq, int q_start, int causal, const hs_kv_dev& kv) {
  const int64_t n_wg = (int64_t)(((Lq / 32) * (Hq / Hkv) + 3) / 4) * Hkv * B;
  const int64_t cap_tiles = (int64_t)kv.cap_dense_k + kv.cap_sparse_k;
  int n_tiles = causal ? (q_start + Lq + HS_BT - 1) / HS_BT : T;  // of the last query
  if (hs_kept_by_pools(kv, T) == HS_KEPT_UNKNOWN) n_tiles = (n_tiles + 3) / 4;
  else if (cap_tiles < n_tiles) n_tiles = (int)cap_tiles;
  if (n_wg > 2048 || (n_wg > 512 && causal && q_start < 3 * (int64_t)Lq)) return 1;
  int best = 1;
  double best_us = 0.0;
  for (int n = 1; n <= 128 && (n == 1 || (2 * n <= n_tiles && n_wg * n <= 4096)); n++) {
    const int64_t wgs = n_wg * n, full = wgs / 512, rest = wgs % 512;
    const int per = (n_tiles + n - 1) / n;
    const double us = per * (1.2 * full + (rest == 0 ? 0.0 : (rest <= 256 ? 1.0 : 1.2))) + (n > 1 ? 8.0 + 0.028 * wgs : 0.0);
    if (n == 1 || us < best_us) { best = n; best_us = us; }
  }
  return best;
}

hipError_t hs_launch_prefill(int B, int Hq, int Hkv, int T, int Tq, int q_start, float scale, int causal, const uint16_t* Q,
                             hs_kv_dev kv, uint16_t* O, float* LSE, hipStream_t st, int dtype, int n_splits, float* ws) {
  const bool f16 = dtype == HS_FP16;
  const float sl2 = scale * kLog2e;
  const int Lq = Tq * HS_BT;
  const int km = kv.cap_dense_k == 0 ? 0 : (kv.cap_sparse_k == 0 ? 1 : 2);
  const int vm = kv.cap_dense_v == 0 ? 0 : (kv.cap_sparse_v == 0 ? 1 : 2);
  const int64_t rows = (int64_t)B * Hq * Lq;
  float* ws_o = ws;
  float* ws_l = n_splits > 1 ? ws + rows * n_splits * HS_D : nullptr;
  hipError_t e = hipSuccess;
#define HS_GO(KM_, VM_)                                                                                                  \
  e = launch_prefill<KM_, VM_, 2>(B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l); \
  break
  switch (km * 3 + vm) {
    case 0: HS_GO(0, 0);
    case 1: HS_GO(0, 1);
    case 3: HS_GO(1, 0);
    case 4: HS_GO(1, 1);
    default: e = hs_launch_prefill_mixed(km, vm, B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l);
  }
#undef HS_GO
  if (e != hipSuccess || n_splits <= 1) return e;
  return hs_launch_merge(rows, n_splits, ws_o, ws_l, O, LSE, st, dtype);
}
