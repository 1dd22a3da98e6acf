// Prefill attention with slabs of 16 queries, tensors that mix dense and 2:4 tiles.  A translation unit of its own because these kernels
// want another scheduler (the flags are in build.py).
#include "hs_prefill_kernel.h"

hipError_t hs_launch_prefill_narrow_mixed(int teams, int km, int vm, int B, int Hq, int Hkv, int T, int Lq, int q_start, float sl2, int causal,
                                          const uint16_t* Q, const hs_kv_dev& kv, uint16_t* O, float* LSE, hipStream_t st, bool f16,
                                          int n_splits, float* ws_o, float* ws_l) {
#define HS_GO(KM_, VM_) \
  return launch_prefill_narrow<KM_, VM_>(teams, B, Hq, Hkv, T, Lq, q_start, sl2, causal, Q, kv, O, LSE, st, f16, n_splits, ws_o, ws_l)
  switch (km * 3 + vm) {
    case 2: HS_GO(0, 2);
    case 6: HS_GO(2, 0);
    case 7: HS_GO(2, 1);
    default: HS_GO(2, 2);  // dense K beside mixed V too, as in hs_prefill_mixed.hip
  }
#undef HS_GO
}
