// Prefill attention: number of tile ranges, choice of the kernel, and the kernels of tensors with one kind of tile.
#include <math.h>

#include "hs_prefill_kernel.h"

static int tiles_to_expect(int T, int seen, const hs_kv_dev& kv) {  // of `seen` tiles, how many to reckon with: what the pools can hold (below)
  const int64_t cap_tiles = (int64_t)kv.cap_dense_k + kv.cap_sparse_k;
  if (hs_kept_by_pools(kv, T) == HS_KEPT_UNKNOWN) return (seen + 3) / 4;
  return cap_tiles < seen ? (int)cap_tiles : seen;
}

// Most ranges to cut a workgroup's tiles into, from what was measured on 2:4 tensors (32/8 heads): a tile takes a workgroup
// 1.0 us alone on its compute unit and 1.2 us beside a second one, so 512 workgroups at a time are two on every unit;
// splitting costs 8 us for the merge launch and the caller's scratch (5 us on the GPU alone) and 0.028 us per workgroup
// for writing and reading its 66 KB of partials.
// The number of ranges that makes this sum smallest is the most that hs_plan_prefill below chooses from.  It was fitted to slabs of
// 32 alone and its terms are rounded up where the other sum's are not: its part is to keep the scratch small.
// Measured with slabs of 32 queries, one range / the chosen number: 64 queries on
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
  const int n_tiles = tiles_to_expect(T, causal ? (q_start + Lq + HS_BT - 1) / HS_BT : T, kv);  // of the last query
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

// Slabs of 32 queries (NB = 2) or of 16 (NB = 1), those by one team of waves or by two, and in how many ranges (at most `fit`).  A tile takes a workgroup of NB = 1
// three quarters of the time for half of the work, so NB = 1 pays where NB = 2 has too few workgroups: one or none per compute
// unit, or a short second half of the work.  Measured, 32/8 heads, 2:4 tensors, us of NB = 2 / NB = 1 at the better number of
// ranges of each: whole prompts of 64 / 256 / 512 / 1024 / 1536 / 2048 / 4096 tokens 7.4 / 6.1, 10.3 / 8.0, 14.3 / 11.1, 22.4 /
// 19.1, 32.7 / 26.7, 41.5 / 39.1, 94.0 / 122; 64 queries on 1024 / 2048 / 8192 / 32768 tokens 14.4 / 12.1, 17.1 / 14.7, 25.4 /
// 23.3, 39.4 / 39.0; 512 queries on 2048 / 32768 tokens 31.8 (4 ranges) / 27.8 (1), 179 / 220; 4 prompts of 512 tokens 19.8 /
// 21.9, 13 of 192 21.2 / 21.4; both tensors dense, 1024 / 2048 tokens 26.1 / 20.7, 51.5 / 48.7; dense ends 30.1 / 22.5, 52.3 / 44.4.
// The sum below is fitted to 2:4 tensors.  It is up to 18 % low on these examples (4 prompts of 512 tokens 16.2 / 18.0, 13 of 192
// 17.5 / 19.9), and of 500 drawn calls of every kind 90 % lie between 0.93 and 1.1 of the time on 2:4 tensors, 0.75 and 1.05 on
// mixed and dense ones; what matters is the difference of the two slabs, where most of that cancels.  Of those 500, all of which it
// put in slabs of 16, the mean gain over slabs of 32 in all the ranges allowed is 1.20, and ten are 2 to 7.5 % slower (4 x 192 queries
// of 40/8 heads on 3584 tokens with dense ends, fp16, 57.2 / 61.5; 4 x 64 of 7/1 on 13760, values dense, 32.6 / 35.2).
// Its terms (us): a workgroup starts in `start`, a tile takes it `alone` with a compute unit
// to itself and `pair` beside a second one; at_once run at a time, the longest first, so the call ends with the longest, or when the
// whole is worked off, or with a pile of k + 1 where round k + 1 is just begun (queries at the end of a long context: all
// workgroups equally long); ranges add the merge launch and the partials.
// Two teams of waves per workgroup (one workgroup per compute unit, which takes two tiles in little more than the time one team takes
// for one) where slabs of 16 leave each compute unit one workgroup or none; one team / two, us: 64 workgroups of 16 tiles 15.7 / 13.3,
// 256 of up to 32 26.5 / 21.2, half of the keys dense 31.2 / 23.9, dense ends 31.2 / 23.6, 64 of up to 4 tiles 7.8 / 8.0.
// The more workgroups, the more a tile takes them (per_wg; 16 of 64 tiles 0.44 us a tile, 128 of 32 0.45, 256 of 32 0.47, and of 64, one to 64
// of them causal, 0.54 in bf16 and 0.44 in fp16: a prompt of 4096 tokens x 4 heads takes 36.9 and 35.4 in three ranges by one team, 40.8
// and 34.7 by two).  Not with more workgroups than compute units, which fill the chip by themselves (prompt of 1024 tokens
// 18.3 / 20.8, 352 workgroups of 40 tiles 35.5 / 43.8), and not in ranges: their tiles come from HBM, and both teams wait for the slower
// one's at every barrier (3 x 128 queries x 8 heads on 33088 tokens, half of them skipped, 45 / 58; 64 queries x 32 heads on 4096 17.1 / 17.0).
// The margins go by what the shape allows and not by `fit`, so a workspace of the size of the choice leads to the same choice.
hs_prefill_choice hs_plan_prefill(int B, int Hq, int Hkv, int T, int Lq, int q_start, int causal, const hs_kv_dev& kv, int fit) {
  static const struct { int nb, teams, at_once; double start, alone, pair, per_wg; } kWays[3] = {
      {2, 1, 512, 7.2, 0.905, 1.13, 0}, {1, 1, 512, 5.3, 0.70, 0.82, 0}, {1, 2, 256, 6.3, 0.43, 0.53, 0.0004}};
  const int most = hs_prefill_auto_splits(B, Hq, Hkv, T, Lq, q_start, causal, kv);
  const int seen = causal ? (q_start + Lq + HS_BT - 1) / HS_BT : T;  // tiles of the last query
  const double share = (double)tiles_to_expect(T, seen, kv) / seen;
  const double longest = seen * share, shortest = (causal ? seen - (Lq / HS_BT - 1) : seen) * share;
  hs_prefill_choice best = {2, 1, 1};
  double best_us = 0.0;
  for (const auto& w : kWays) {
    const double n_wg = (double)((int64_t)((Lq / (16 * w.nb) * (int64_t)(Hq / Hkv) + 3) / 4) * Hkv * B);
    for (int n = 1; n <= most && n <= fit; n++) {
      const double wgs = n_wg * n, rounds = ceil(wgs / w.at_once);
      if (w.teams == 2 && (n > 1 || rounds > 1)) break;
      double us = longest / n * (wgs <= 256 ? w.alone + w.per_wg * wgs : w.pair) + w.start;
      us = fmax(us, (longest + shortest) / 2 / n * w.pair * wgs / w.at_once + rounds * w.start);
      if (rounds > 1) {  // (k + 1) (first - k fall), k = 1 .. rounds - 1: largest beside its vertex, or at an end
        const double first = longest / n * w.pair + w.start, fall = (longest - shortest) * w.at_once / wgs / n * w.pair;
        const double k = fmin(fmax(fall > 0.0 ? floor((first / fall - 1) / 2) : rounds, 1.0), rounds - 1);
        us = fmax(us, fmax((k + 1) * (first - k * fall), k + 1 < rounds ? (k + 2) * (first - (k + 1) * fall) : 0.0));
      }
      if (n > 1) us += 3.0 + 0.014 * w.nb * wgs;
      // The wider slab in all the ranges allowed where things are even; ranges of the narrow one, two to a compute unit, are
      // where the sum is least sure (128 queries x 4 heads on 47104 tokens 25.8 / 28.0, 256 x 4 on 32768 29.6 / 27.0).
      if (w.nb == 1) us *= n > 1 && wgs > 256 ? 1.12 : (w.teams == 2 ? 1.08 : 1.03);
      else if (n != most) us *= 1.03;
      if (best_us == 0.0 || us < best_us) { best = {w.nb, n, w.teams}; best_us = us; }
    }
  }
  return best;
}

hipError_t hs_launch_prefill(int B, int Hq, int Hkv, int T, int Tq, int q_start, float scale, int causal, const uint16_t* Q,
                             hs_kv_dev kv, uint16_t* O, float* LSE, hipStream_t st, int dtype, hs_prefill_choice how, float* ws) {
  const bool f16 = dtype == HS_FP16;
  const float sl2 = scale * kLog2e;
  const int Lq = Tq * HS_BT;
  const int n_splits = how.n_splits;
  const int km = kv.cap_dense_k == 0 ? 0 : (kv.cap_sparse_k == 0 ? 1 : 2);
  const int vm = kv.cap_dense_v == 0 ? 0 : (kv.cap_sparse_v == 0 ? 1 : 2);
  const int64_t rows = (int64_t)B * Hq * Lq;
  float* ws_o = ws;
  float* ws_l = n_splits > 1 ? ws + rows * n_splits * HS_D : nullptr;
  hipError_t e = hipSuccess;
#define HS_GO(KM_, VM_)                                                                                                  \
  e = launch_prefill<KM_, VM_, 2>(B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l); \
  break
  if (how.nb == 1)
    e = hs_launch_prefill_narrow(how.teams, km, vm, B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l);
  else switch (km * 3 + vm) {
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
