// The kernel of every bf16 prefill (prefill_mfma_ws.h): the first pass of the segmented form and the full pass.
#include "prefill_mfma_ws.h"

namespace linattn {

template <int D>
static hipError_t launch_ws_k(const PrefillArgs& a, bool state_only, bool grouped, hipStream_t st) {
  constexpr int C = 64;   // tokens per group
  if (state_only) return launch_ws<D, C, 3, true>(a, st);   // the conv taps play no part in the state
  return grouped ? launch_ws_taps<D, C, true, false>(a, st) : launch_ws_taps<D, C, false, false>(a, st);
}

// One pass of a prefill call over all its segments.  state_only: the first pass of the segmented
// form (segment increments into a.ws); otherwise the full pass (segment start states must be in a.ws).
// grouped: the three-branch form with 64-token groups (a.alpha weighs its linear branch).
hipError_t launch_prefill_mfma_ws(const PrefillArgs& a, int d, bool state_only, bool grouped, hipStream_t st) {
  return d == 128 ? launch_ws_k<128>(a, state_only, grouped, st) : launch_ws_k<64>(a, state_only, grouped, st);
}

}  // namespace linattn
