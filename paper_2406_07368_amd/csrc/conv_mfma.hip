// Causal depthwise convolution of bf16 rows on the matrix cores (Sec. 4.1: the FLASH experiment runs the masked DWConv with
// kernel size 63), and the two gradients of a training step that are convolutions: the conv's share of dv and the gradient
// of the taps.
//
//   forward    out[t][c] (+)= sum_{j < Kc} w[c][j] Vext[t - j][c]        Vext = hist_in ++ V, zeros before that
//   backward   dv[s][c] = sum_j w[c][j] dO[s + j][c],    dw[c][j] = sum_t dO[t][c] v[t - j][c]
//
// A depthwise convolution contracts nothing across channels, but over tokens it is a Toeplitz product per channel.  With
// the tokens of a channel cut into blocks of 16 (t = 16a + i), U[i][a] = sum_k W[i][k] X[k][a], X[k][a] = v[16a - OFF + k]:
// 16 x 16 x 32 instructions with 16 blocks in the columns, so 256 tokens of one channel at a time; 63 taps are three
// contraction steps (96 token offsets, OFF = 80), up to 49 taps two, up to 17 one.  The taps enter as the sum of three
// bf16 terms, which is all 24 bits of a finite fp32 tap: products exact, sums fp32, like the fp32 multiply-adds they replace.
// The gradient of the taps is the same picture the other way round, D[i][r] = sum_a dO[16a + i] v[16(a - b) + r] (16 x 16 x
// 16, both factors bf16 as they are), summed along its diagonals: first over the four accumulator registers by shifts
// inside a row of 16 lanes, then over the four rows through LDS.
//
// One workgroup = 256 or 512 tokens of 32 channels (16 or 8 where few would run) of one (b, h[, value block]), four waves.
// The rows are turned around on their way into LDS ([channel][token], two tokens per dword: a thread takes 8 channels of
// two neighbouring tokens), so that an operand of eight consecutive tokens is one 16-byte read and one of every sixteenth
// token one transpose read; the results go back the same way.  The LDS rows are skewed per 8 channels so that those
// accesses hit 64 different banks.
// What bounds it: the LDS port, most of it the tap operands (nine KB per tile and channel), which is why a workgroup takes
// two tiles of 256 tokens where there are enough of them (104 -> 84 us below).  Measured on B8 H8 L8192 d128 with 63 taps:
// forward 84 us for 290 MB (158 us on the vector ALUs, a thread per channel: 63 multiply-adds per element); backward 185 us
// for both gradients beside the kernels of the other stream (158 + 355 us and more as two passes).
#include "common.h"
#include "conv_mfma.h"
#include "kernels.h"
#include "mfma_util.h"
#include "segment_scan.h"

namespace linattn {

namespace { constexpr int CM_NW = 4; }                     // waves per workgroup

template <int D, int KS, int MODE, int T, int CB>
__global__ __launch_bounds__(64 * CM_NW) void conv_mfma_kernel(ConvLongArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smu[];
  conv_mfma_workgroup<D, KS, MODE, T, CB, CM_NW>(a, blockIdx.x, blockIdx.y, smu);
}

// Tokens per workgroup: two tiles share the tap operands (104 -> 84 us at a chip-filling size, 0.81 of the time per tile);
// one where two would leave less than two workgroups per compute unit (B1 H8 L1000: 128 workgroups of one tile, 8 us), or
// where the second would be padding (256 heads of 128, 60 tokens: call of 43.7 us with two, 36.3 with one).
static int cm_tokens(int L, int heads, int d) {
  const int64_t two = (L + 2 * CM_SUB - 1) / (2 * CM_SUB), one = (L + CM_SUB - 1) / CM_SUB;
  return two * heads * (d / 32) >= 512 && 162 * two < 100 * one ? 2 * CM_SUB : CM_SUB;
}
int conv_mfma_blocks(int L, int heads, int d) {
  const int t = cm_tokens(L, heads, d);
  return (L + t - 1) / t;
}

template <int D, int KS, int MODE, int T, int CB>
static hipError_t launch_cm_one(const ConvLongArgs& a, hipStream_t st) {
  constexpr int bytes = ConvCfg<KS, MODE, T, CB, CM_NW>::TOTAL * 4;
  auto kern = conv_mfma_kernel<D, KS, MODE, T, CB>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.L + T - 1) / T * (D / CB)), (unsigned)(a.B * a.H * a.m)), dim3(64 * CM_NW), bytes, st, a);
  return hipGetLastError();
}

template <int D, int MODE, int T, int CB>
static hipError_t launch_cm_t(const ConvLongArgs& a, hipStream_t st) {
  return a.Kc <= 17 ? launch_cm_one<D, 1, MODE, T, CB>(a, st)
                    : a.Kc <= 49 ? launch_cm_one<D, 2, MODE, T, CB>(a, st) : launch_cm_one<D, 3, MODE, T, CB>(a, st);
}
// Channels per workgroup: a wave takes its channels one after another, so with few workgroups fewer channels each (and more
// workgroups) shorten the call: 32 / 16 / 8 channels, us a prefill call of 63 taps: 32 workgroups of 32 channels (B1 H4 L300 d128)
// 34.5 / 32.5 / 31.3, 64 (B1 H8 L1000 d64) 32.7 / 31.0 / 30.8, 96 32.7 / 32.1 / 32.3, 128 (B1 H4 L2000 d128) 37.8 / 35.7 / 36.4, 160 (B1 H32 L1000
// d64, two rounds of half a chip) 37.8 / 41.6 / 43.0.  More share the memory lines of a row.
template <int D, int MODE>
static hipError_t launch_cm(const ConvLongArgs& a, hipStream_t st) {
  const int heads = a.B * a.H * a.m;
  if (cm_tokens(a.L, heads, D) == 2 * CM_SUB) return launch_cm_t<D, MODE, 2 * CM_SUB, 32>(a, st);
  const int64_t wgs = (int64_t)((a.L + CM_SUB - 1) / CM_SUB) * heads * (D / 32);
  return wgs <= 64 ? launch_cm_t<D, MODE, CM_SUB, 8>(a, st)
                   : wgs <= 128 ? launch_cm_t<D, MODE, CM_SUB, 16>(a, st) : launch_cm_t<D, MODE, CM_SUB, 32>(a, st);
}

hipError_t launch_conv_mfma(const ConvLongArgs& a, int d, hipStream_t st) {
  if (a.bwd) return d == 128 ? launch_cm<128, CM_BWD>(a, st) : launch_cm<64, CM_BWD>(a, st);
  if (a.assign) return d == 128 ? launch_cm<128, CM_ASSIGN>(a, st) : launch_cm<64, CM_ASSIGN>(a, st);
  return d == 128 ? launch_cm<128, CM_ADD>(a, st) : launch_cm<64, CM_ADD>(a, st);
}

// The forward conv of a call in groups of 256 (out = conv, ahead of the kernel that adds the rest) in the launch of the prefix
// sum over its segments: neither needs anything from the other.  Both are short, a launch apart they were two gaps on the stream
// and two launches that leave most of the chip idle; the conv's workgroups are the longer ones and go first.  16 channels each
// (see launch_cm), the tap count chosen at run time, so the workgroups of the prefix sum hold the conv's LDS too: nothing to
// them, they use few registers and end early.
template <int D>
__global__ __launch_bounds__(64 * CM_NW) void segment_scan_conv_kernel(PrefillArgs p, ConvLongArgs c, int nconv) {
  extern __shared__ __attribute__((aligned(16))) uint32_t smu[];
  constexpr int CB = 16;
  static_assert(64 * CM_NW == 256, "the prefix sum's workgroups");
  if ((int)blockIdx.x < nconv) {                           // uniform; the longer ones first
    const int per = (c.L + CM_SUB - 1) / CM_SUB * (D / CB), bx = blockIdx.x % per, by = blockIdx.x / per;
    if (c.Kc <= 17) conv_mfma_workgroup<D, 1, CM_ASSIGN, CM_SUB, CB, CM_NW>(c, bx, by, smu);
    else if (c.Kc <= 49) conv_mfma_workgroup<D, 2, CM_ASSIGN, CM_SUB, CB, CM_NW>(c, bx, by, smu);
    else conv_mfma_workgroup<D, 3, CM_ASSIGN, CM_SUB, CB, CM_NW>(c, bx, by, smu);
    return;
  }
  constexpr int PER = (D * D + D + 255) / 256;
  const int e = blockIdx.x - nconv;
  segment_scan_workgroup<D>(p, e % PER, e / PER);
}

// Every conv of one tile a workgroup (with two tiles it lasts many times the prefix sum).  us a call, conv in a launch of its own /
// beside the prefix sum: d = 128, 63 taps: 8 heads, 1000 tokens 45.1 / 43.4; 8 heads, 2000 tokens 48.7 / 45.6; 32 heads, 700 tokens
// 54.6 / 50.2; 96 heads, 600 tokens (2304 workgroups) 90.4 / 85.1; d = 64: 8 heads, 1000 tokens 28.8 / 28.0; 4 heads, 8000 tokens
// 34.4 / 31.1.  A history written over the one that is read wants a kernel of its own after the conv (conv_long.hip).
bool conv_beside_scan(const ConvLongArgs& c, int d) {
  return c.L > 0 && cm_tokens(c.L, c.B * c.H * c.m, d) == CM_SUB && !(c.hist_out && c.hist_out == c.hist_in);
}

template <int D>
static hipError_t launch_scan_conv(const PrefillArgs& p, ConvLongArgs c, hipStream_t st) {
  constexpr int b3 = ConvCfg<3, CM_ASSIGN, CM_SUB, 16, CM_NW>::TOTAL, b1 = ConvCfg<1, CM_ASSIGN, CM_SUB, 16, CM_NW>::TOTAL;
  constexpr int bytes = 4 * (b3 > b1 ? b3 : b1);
  static_assert(ConvCfg<2, CM_ASSIGN, CM_SUB, 16, CM_NW>::TOTAL * 4 <= bytes, "LDS");
  auto kern = segment_scan_conv_kernel<D>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, bytes);
  if (e != hipSuccess) return e;
  c.hist_fused = c.hist_out != nullptr;
  const int heads = c.B * c.H * c.m, nconv = (c.L + CM_SUB - 1) / CM_SUB * (D / 16) * heads;
  hipLaunchKernelGGL(kern, dim3((unsigned)(nconv + (D * D + D + 255) / 256 * heads)), dim3(256), bytes, st, p, c, nconv);
  return hipGetLastError();
}
hipError_t launch_segment_scan_conv(const PrefillArgs& p, const ConvLongArgs& c, int d, hipStream_t st) {
  return d == 128 ? launch_scan_conv<128>(p, c, st) : launch_scan_conv<64>(p, c, st);
}

}  // namespace linattn
