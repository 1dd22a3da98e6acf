// Prefill attention with slabs of 16 queries, for calls with few query blocks (the rule is in hs_prefill.hip): tensors of one kind.
#include "hs_prefill_kernel.h"

hipError_t hs_launch_prefill_narrow(int teams, int km, int vm, int B, int Hq, int Hkv, int T, int Lq, int q_start, float sl2, int causal,
                                    const uint16_t* Q, const hs_kv_dev& kv, uint16_t* O, float* LSE, hipStream_t st, bool f16,
                                    int n_splits, float* ws_o, float* ws_l) {
#define HS_GO(KM_, VM_) \
  return launch_prefill_narrow<KM_, VM_>(teams, B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l)
  switch (km * 3 + vm) {
    case 0: HS_GO(0, 0);
    case 1: HS_GO(0, 1);
    case 3: HS_GO(1, 0);
    case 4: HS_GO(1, 1);
    default:
      return hs_launch_prefill_narrow_mixed(teams, km, vm, B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l);
  }
#undef HS_GO
}
