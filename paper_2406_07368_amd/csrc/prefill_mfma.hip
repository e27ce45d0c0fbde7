// Prefill of bf16 inputs (Sec. 4.1): the launch plan around the matrix-core kernel.
//
// The kernel itself (prefill_mfma_ws.h) walks one (b, h) -- or one segment of its
// sequence -- group by group with the state in registers.  When B*H alone cannot fill
// the chip the sequence axis is cut into segments: a first pass reduces each segment's
// K, V to its state increment, a prefix sum over the segments (here) turns the
// increments into segment start states, and the full pass starts every segment from its
// prefix (for a new sequence in few segments it adds the increments up itself).
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "segment_scan.h"

namespace linattn {

template <int D>
__global__ __launch_bounds__(256) void segment_scan_kernel(PrefillArgs a) {
  segment_scan_workgroup<D>(a, blockIdx.x, blockIdx.y);
}

// No tokens: S, z and the history as they came (zeros for a new sequence).  Plain copies, element by element, so that an
// output may be its input.
__global__ __launch_bounds__(256) void state_through_kernel(PrefillArgs a, size_t n_S, size_t n_z, size_t n_hist) {
  const size_t step = (size_t)gridDim.x * 256;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n_S || e < n_z || e < n_hist; e += step) {
    if (a.S_out && e < n_S) a.S_out[e] = a.S_in ? a.S_in[e] : 0.f;
    if (a.z_out && e < n_z) a.z_out[e] = a.z_in ? a.z_in[e] : 0.f;
    if (a.hist_out && e < n_hist) static_cast<uint16_t*>(a.hist_out)[e] = a.hist_in ? static_cast<const uint16_t*>(a.hist_in)[e] : (uint16_t)0;
  }
}

hipError_t launch_state_through(const PrefillArgs& a, int d, int elem_bytes, hipStream_t st) {
  const size_t BH = (size_t)a.B * a.H, n_S = BH * d * d * a.m, n_z = BH * d;
  const size_t n_hist = BH * (a.Kc - 1) * d * a.m * (elem_bytes / 2);      // in units of two bytes
  const size_t most = n_S > n_hist ? n_S : n_hist;
  const unsigned grid = (unsigned)((most + 255) / 256 < 2048 ? (most + 255) / 256 : 2048);
  hipLaunchKernelGGL(state_through_kernel, dim3(grid), dim3(256), 0, st, a, n_S, n_z, n_hist);
  return hipGetLastError();
}

// Segments per (b, h): as many as keep all workgroups of the second pass resident at once (at d = 128 one per compute
// unit: a workgroup takes most of a unit's LDS, so the 257th would wait for a whole segment; at d = 64 two), with at
// least 2 groups per segment, and no segments at all for sequences of fewer than 8 groups, where a second launch costs
// more than it saves.
int prefill_mfma_pick_segments(int BH, int L, int chunk, int d) {
  const int groups = (L + 63) / 64;            // the kernel walks groups of 64 tokens whatever `chunk` says
  const int chunks = (L + chunk - 1) / chunk;  // segments start on multiples of `chunk`
  int want = (d == 64 ? 512 : 256) / BH;
  int most = groups >= 8 ? groups / 2 : 1;
  if (most > chunks) most = chunks;
  if (want > most) want = most;
  if (want > 64) want = 64;
  return want < 1 ? 1 : want;
}

// A new sequence (no state and no history come in: nothing that an output could overwrite while another workgroup still
// reads it) needs no prefix sum as a launch of its own: every workgroup of the full pass adds up the increments of the
// segments before it while its first rows are on their way.  Returns the segments to use, 0: keep the prefix sum.
// What it costs is the last segment's reads, one slot (64 KB at d = 128) per segment through one compute unit, against
// a launch of 4 us and more.  Up to 6 segments it pays (us a call, prefix sum / this: 2 segments 100 / 93, 4 segments of
// 64 heads 69 / 65, 6 segments of 84 heads of 64 40.5 / 37, of 40 heads 78 / 75); at 8 it does not (d = 128, 32 heads:
// L = 1024 42 / 46, L = 8192 105 / 109).  Sequences of up to 16 groups are therefore cut into 6 at most, three groups each
// where the plan has two (L = 1024, us a call: d = 128, 32 heads 41 / 34, 16 heads 32 / 29.5, 12 heads 30 / 29; d = 64, 48 heads
// 29.7 / 26.6, 8 heads 25.7 / 23.0, and 23.5 / 23.8 as a graph, where launches cost less) -- at d = 128, where a group takes
// longer, not below 12 heads: 8 heads 27.1 / 27.2, as a graph 30.4 / 30.9, three-branch form 29.2 / 30.3; 4 heads 25.8 / 25.9, 27.7 /
// 29.3, 26.7 / 29.1.  Beyond 16 groups six segments have four groups and more: some gain (d = 128, 32 heads, L = 1300
// 42 / 40), others lose (three-branch form, 48 heads of 64, L = 1300 46 / 51; 12 heads of 128, L = 1200 31 / 32): the plan stays.
int prefill_mfma_fold_segments(int nseg, int L, int heads, int d) {
  if (nseg <= 1) return 0;
  if (nseg <= 6) return nseg;
  return L <= 16 * 64 && (d == 64 || heads >= 12) ? 6 : 0;
}

// A short new sequence in one launch, a workgroup per group of 64: the one of group g walks the g groups before its own for their
// state only, which takes half the time of a group with scores and outputs (1.6 us against 3.2 at d = 128), so the call is as long
// as its last group's walk instead of a walk that computes everything.  Costs g times the reads of the rows, from the last-level
// cache, and a compute unit per group.  (The front end fetches and maps Q of the groups before its own as well, which nobody
// reads.)  Returns the number of segments (= groups), 0: not that way.
// It pays while every group has a compute unit to itself, up to the length where the plan cuts the sequence (8 groups).  Measured,
// us a call, one workgroup per head / this:
//   d = 128: 16 heads: 2 groups 13.1 / 11.7, 3 16.1 / 13.2, 5 22.3 / 16.9, 6 25.4 / 18.8, 8 (in segments) 24.6 / 23.2, three-branch form
//   26.6 / 28.5; 32 heads of 6 26.0 / 20.1, 64 of 4 20.3 / 18.3, 128 of 2 14.5 / 14.5, 64 of 5 23.1 / 26.8, 96 of 3 17.3 / 21.4;
//   three-branch form 32 heads of 6 31.8 / 24.1, 64 of 4 24.6 / 21.6
//   d = 64: 16 heads of 6 22.1 / 16.4, 64 of 4 17.4 / 14.3, 128 of 2 12.1 / 11.0, 96 of 3 14.6 / 14.2, 96 of 4 17.6 / 19.1; three-branch
//   form 64 of 4 21.9 / 17.5, 96 of 3 17.7 / 21.0
int prefill_mfma_lead_segments(int L, int heads) {
  const int groups = (L + 63) / 64;
  return groups >= 2 && groups < 8 && (int64_t)groups * heads <= 256 ? groups : 0;
}

size_t prefill_mfma_workspace_bytes(int BH, int d, int nseg) {
  if (nseg <= 1) return 0;
  return (size_t)BH * nseg * ((size_t)d * d + d) * sizeof(float) + (size_t)BH * HALO * d * sizeof(uint16_t);
}

// Segments of the 256-token three-branch kernel: a workgroup takes all of a compute unit, so as many as fill the
// chip, down to one group per segment (the groups of a segment are walked one after the other).
int prefill_grouped256_pick_segments(int BH, int L) {
  const int groups = (L + 255) / 256;
  int want = 256 / BH;
  if (want > groups) want = groups;
  if (want > 64) want = 64;
  return want < 1 ? 1 : want;
}

// ... whose running state lives in its workspace slot: one slot per (b, h, segment) even without segments
size_t prefill_grouped256_workspace_bytes(int BH, int d, int nseg) {
  return (size_t)BH * nseg * ((size_t)d * d + d) * sizeof(float) + (size_t)BH * HALO * d * sizeof(uint16_t);
}

// The first pass over segments of one group, where they are few: 2 or 4 workgroups share a segment's 256 tokens, while each has
// a compute unit, and the prefix sum adds their increments up.  A workgroup's walk over four steps of 64 tokens was the longest
// part of such a call's first half (10.9 of 31 us at 8 heads of 1000 tokens).  What it costs are more slots written and read: a
// longer chain in the prefix sum where a head has many segments (at most 48 slots in four parts, 64 in two), and more of its
// traffic where the heads are many: sequences of two groups on more than 96 heads keep whole segments -- at d = 128 on more than 64,
// without a long conv beside the prefix sum --, but for long taps at d = 64, whose conv lasts longer than the prefix sum either way.
// us a call as a graph, whole segments / two parts / four:
//   63 taps, d = 128: 4 heads, 300 tokens 26.5 / - / 23.1; 8 heads, 1000 30.0 / - / 29.1, 2000 38.2 / 35.6 / 36.1, 3000 43.2 / 40.4; 4
//   heads, 3000 34.6 / 32.6 / 32.5; 1 head, 8000 37.6 / 36.0 / 39.0, 12000 35.2 / 33.4 / 37.5, 16000 37.5 / 37.8 / 44.1; two groups: 65 heads 55.7 / 53.0, 90
//   57.1 / 56.4, 110 65.5 / 66.8, 128 71.0 / 75.4; d = 64: 8 heads, 2000 23.1 / 21.4 / 21.3; 1 head, 4000 20.0 / 17.9 / 17.3, 16000 24.0 / 25.8 / 32.2;
//   128 heads, two groups 42.3 / 39.4
//   5 taps, d = 128: 8 heads, 2000 36.4 / 35.3 / 37.2; 1 head, 8000 36.3 / 36.0 / 39.5; 64 heads, three groups 53.9 / 53.3; two groups: 64 heads
//   47.2 / - / 46.9, 65 52.5 / 54.6, 128 61.0 / 63.6; d = 64: 1 head, 16000 22.1 / 23.9 / 30.8; two groups: 80 heads 28.8 / 28.6, 128 31.6 / 31.9
int prefill_grouped256_fine(int BH, int nseg, int seg_len, int d, int conv_k) {
  if (nseg <= 1 || seg_len != 256) return 0;
  const int64_t segs = (int64_t)BH * (nseg - 1);
  if (4 * segs <= 256 && 4 * (nseg - 1) <= 48) return 2;
  if (2 * segs > 256 || 2 * (nseg - 1) > 64) return 0;
  const bool long_conv = conv_k > 8;
  if (nseg == 2 && (d == 128 ? !long_conv || segs > 96 : !long_conv && segs > 96)) return 0;
  return 1;
}
size_t prefill_grouped256_fine_bytes(int BH, int d, int nseg, int fine) {
  return fine ? (size_t)BH * (((size_t)(nseg - 1) << fine) + 1) * ((size_t)d * d + d) * sizeof(float) : 0;
}

// The segments' increments into a.ws, or their parts' into a.ws_fine.
hipError_t launch_first_pass(const PrefillArgs& a, int d, hipStream_t st) {
  if (a.fine == 0) return launch_prefill_mfma_ws(a, d, true, false, st);
  PrefillArgs f = a;
  f.ws = a.ws_fine;
  f.nseg = ((a.nseg - 1) << a.fine) + 1;
  f.seg_len = a.seg_len >> a.fine;
  return launch_prefill_mfma_ws(f, d, true, false, st);
}

// The group size only blocks the computation; the result does not depend on it (the in-group
// part is the exact masked product).  A requested group of 128 tokens is walked as two steps of
// 64: two 128-token row buffers do not fit in LDS, and larger groups only add in-group MFMA work
// per token on this design.  Segment boundaries stay multiples of the requested size.
// grouped: the three-branch form, whose groups are exactly `chunk` tokens, 64 or 256 (segments start on
// group boundaries, so the first pass and the prefix sum are the same for both forms; groups of 256 have a
// kernel of their own for the full pass).
hipError_t launch_segment_scan(const PrefillArgs& a, int d, hipStream_t st) {
  const int BH = a.B * a.H * a.m;             // heads the kernels see: one per value block
  const int slot = d * d + d;
  const dim3 grid((unsigned)((slot + 255) / 256), (unsigned)BH);
  if (d == 128) hipLaunchKernelGGL((segment_scan_kernel<128>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((segment_scan_kernel<64>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_prefill_mfma(const PrefillArgs& a, int d, int chunk, bool grouped, hipStream_t st) {
  if (a.fold == 2) return launch_prefill_mfma_lead(a, d, grouped, st);
  hipError_t e;
  if (a.nseg > 1) {
    if ((e = launch_first_pass(a, d, st)) != hipSuccess) return e;
    if (!a.fold && (e = launch_segment_scan(a, d, st)) != hipSuccess) return e;
  }
  if (grouped && chunk == 256) return launch_prefill_grouped256(a, d, st);
  return launch_prefill_mfma_ws(a, d, false, grouped, st);
}

}  // namespace linattn
