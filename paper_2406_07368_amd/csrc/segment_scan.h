// The prefix sum over the segments of a prefill call, for the kernel of prefill_mfma.hip and for the launch that has the long
// conv beside it (conv_mfma.hip).
#pragma once
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

namespace linattn {

// Prefix sum over the segments of one (b, h): slot 0 <- incoming state, slot g <- slot g-1 +
// increment of segment g-1 (or the increments of its 1 << fine parts, one after the other).  Also
// stages the incoming history so that the second pass never reads hist_in (which hist_out may
// alias).  One thread per state element walks the segments.
// Workgroup (bx, by) of dim3(ceil((D * D + D) / 256), B H m), 256 threads.
template <int D>
__device__ __forceinline__ void segment_scan_workgroup(const PrefillArgs& a, int bx, int by) {
  constexpr int SLOT = D * D + D;
  const HeadIndex hx = head_index(a, by, D);               // one (b, h, value block)
  const int bh = hx.bh;
  const int e = bx * 256 + threadIdx.x;
  float* ws_bh = a.ws + (size_t)hx.bhs * a.nseg * SLOT;
  if (e < SLOT) {
    float run = 0.f;
    if (a.S_in) run = e < D * D ? a.S_in[(size_t)bh * D * hx.dvt + (size_t)(e / D) * hx.dvt + hx.blk * D + e % D]
                                : a.z_in[(size_t)bh * D + (e - D * D)];
    ws_bh[e] = run;
    // sixteen increments at a time: all of them are requested before the first is added (read, add and
    // write back one by one, every segment would pay a trip to memory of its own: the compiler may not move a
    // load across the store before it)
    if (a.fine) {                                          // uniform: the parts' increments, in slots of their own
      const int n = ((a.nseg - 1) << a.fine) + 1, whole = (1 << a.fine) - 1;
      const float* from = a.ws_fine + (size_t)hx.bhs * n * SLOT;
      for (int g0 = 1; g0 < n; g0 += 16) {
        float inc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int g = g0 + i < n ? g0 + i : n - 1;       // past the end: the last one again, not used
          inc[i] = from[(size_t)g * SLOT + e];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          run += inc[i];
          if (g0 + i < n && ((g0 + i) & whole) == 0) ws_bh[(size_t)((g0 + i) >> a.fine) * SLOT + e] = run;
        }
      }
    } else {
      for (int g0 = 1; g0 < a.nseg; g0 += 16) {
        float inc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int g = g0 + i < a.nseg ? g0 + i : a.nseg - 1;
          inc[i] = ws_bh[(size_t)g * SLOT + e];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          run += inc[i];
          if (g0 + i < a.nseg) ws_bh[(size_t)(g0 + i) * SLOT + e] = run;
        }
      }
    }
  }
  if (a.hist_in && e < HALO * D) {
    float* staged = a.ws + (size_t)a.B * a.H * a.m * a.nseg * SLOT;
    const size_t se = (size_t)hx.bhs * HALO * D + e;
    const int r = e / D, cc = e % D;           // staged row r holds token r - HALO
    const int hr = (a.Kc - 1) - HALO + r;      // row of the incoming history
    const size_t he = hr >= 0 ? ((size_t)bh * (a.Kc - 1) + hr) * hx.dvt + hx.blk * D + cc : 0;
    if (a.f32) staged[se] = hr >= 0 ? static_cast<const float*>(a.hist_in)[he] : 0.f;
    else reinterpret_cast<uint16_t*>(staged)[se] = hr >= 0 ? static_cast<const uint16_t*>(a.hist_in)[he] : (uint16_t)0;
  }
}

}  // namespace linattn
