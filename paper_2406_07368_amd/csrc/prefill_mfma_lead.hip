// The kernel of every bf16 prefill (prefill_mfma_ws.h) for short new sequences in one launch: LEAD.  A file of its own, so that the
// code of the other instantiations lies where it lay: it is 150 KB per kernel, and the order in the file alone moved a call of 5 groups on 256
// heads from 27.4 to 28.7 us.
#include "prefill_mfma_ws.h"

namespace linattn {

hipError_t launch_prefill_mfma_lead(const PrefillArgs& a, int d, bool grouped, hipStream_t st) {
  constexpr int C = 64;   // tokens per group
  if (d == 128) return grouped ? launch_ws_taps<128, C, true, true>(a, st) : launch_ws_taps<128, C, false, true>(a, st);
  return grouped ? launch_ws_taps<64, C, true, true>(a, st) : launch_ws_taps<64, C, false, true>(a, st);
}

}  // namespace linattn
