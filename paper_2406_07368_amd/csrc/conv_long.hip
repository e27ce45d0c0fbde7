// Causal depthwise convolution on V with more than 8 taps (Sec. 4.1: the FLASH experiment runs the masked
// DWConv with kernel size 63), as a pass of its own behind the attention kernels:
//
//   out[t][c] += sum_{j < Kc} w[h][c][j] * Vext[t - j][c]        Vext = hist_in ++ V, zeros before that
//
// on the vector ALUs: fp32 rows (exact fp32 products), and bf16 rows with few taps or in short sequences (conv_vector_pays);
// the other bf16 rows run on the matrix cores (conv_mfma.hip).
// The attention kernels keep an 8-row halo of V in LDS and gather the taps per token; a 62-row halo does not
// fit next to their row buffers, and 63 taps per output are a vector-ALU workload of the size of the attention
// itself.  So long kernels are register-blocked here instead: a thread owns one channel, holds its taps in
// registers and slides over 8 outputs at a time, every value row read from LDS feeding that many multiply-adds.
// One workgroup = 64 (or 32) tokens of one (b, h); rows t0-62 .. t0+63 of V are staged in LDS as they lie in memory.
#include "common.h"
#include "kernels.h"

namespace linattn {

namespace {
constexpr int CL_TOK = 64;        // tokens per workgroup (32 when that still leaves compute units without one: a
                                  // workgroup's time is one thread's chain over its tokens, and half the chain is
                                  // worth more then than the halo rows it reads twice)
constexpr int CL_HALO = 62;       // rows before them that the longest kernel reaches
constexpr int CL_MAXK = 63;
constexpr int CL_BLK = 8;         // outputs a thread carries at once (fewer if it has fewer tokens)
}  // namespace

// KMAX: tap capacity of the instantiation (taps beyond Kc are zeros; the loops below are straight-line code for
// exactly KMAX taps: a branch per tap would put every LDS read into a basic block of its own, with a full wait
// behind it).
static __device__ __forceinline__ float elem_to_f32(float x) { return x; }
static __device__ __forceinline__ float elem_to_f32(uint16_t x) { return bf16_bits_to_f32(x); }

// bytes of the value rows, or of the taps before them
template <typename Elem, int D, int KMAX, int TOK>
static constexpr int conv_long_lds() {
  constexpr int rows = (CL_HALO + TOK) * D * (int)sizeof(Elem), taps = D * KMAX * (int)sizeof(float);
  return rows > taps ? rows : taps;
}

// Infinities and NaN among eight elements as they lie in memory: running maxima of the magnitudes' bits (bf16: two at a time).
typedef uint16_t cl_u16x2 __attribute__((ext_vector_type(2)));
static __device__ __forceinline__ uint32_t top_exponent(const u32x4& x, uint32_t top) {
  cl_u16x2 t = __builtin_bit_cast(cl_u16x2, top);
#pragma unroll
  for (int i = 0; i < 4; ++i) t = __builtin_elementwise_max(t, __builtin_bit_cast(cl_u16x2, x[i] & 0x7fff7fffu));
  return __builtin_bit_cast(uint32_t, t);
}
static __device__ __forceinline__ bool not_finite(uint32_t top, const u32x4&) { return (top >> 16) >= 0x7f80u || (top & 0xffffu) >= 0x7f80u; }
static __device__ __forceinline__ uint32_t top_exponent(const F32Raw8& x, uint32_t top) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a = __float_as_uint(x.lo[i]) & 0x7fffffffu, b = __float_as_uint(x.hi[i]) & 0x7fffffffu;
    top = a > top ? a : top;
    top = b > top ? b : top;
  }
  return top;
}
static __device__ __forceinline__ bool not_finite(uint32_t top, const F32Raw8&) { return top >= 0x7f800000u; }

template <typename Io, int D, int KMAX, int TOK>
__global__ __launch_bounds__(256) void conv_long_kernel(ConvLongArgs a) {
  // the value rows [CL_HALO + TOK][D] as they lie in memory (bf16 rows stay bf16: half the LDS of fp32 rows, so
  // twice the workgroups per compute unit); before them, for a moment, the taps as fp32
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_cl[];
  float* xs = reinterpret_cast<float*>(smem_cl);
  typename Io::elem* xe = reinterpret_cast<typename Io::elem*>(smem_cl);
  int* odd = reinterpret_cast<int*>(smem_cl + conv_long_lds<typename Io::elem, D, KMAX, TOK>());   // [waves]
  constexpr int NG = 256 / D;                 // token groups of threads
  constexpr int TPT = TOK / NG;            // tokens per thread
  // (a block also holds its own and the next block's elements of out)
  constexpr int BLK = TPT < CL_BLK ? TPT : CL_BLK;
  const int tid = threadIdx.x;
  // one (b, h, value block of D channels); d_v = D: one block per head
  const int bh = blockIdx.y / a.m, blk = blockIdx.y % a.m, b = bh / a.H, h = bh % a.H;
  const int DVT = a.m * D;
  // Neighbouring token blocks share 62 of their rows: block indices 8 apart land on the same chiplet, so they get
  // neighbouring token blocks, and the shared rows come from that chiplet's L2 (when the count is a multiple of 8).
  const int nblk = gridDim.x;
  const int tblk = nblk % 8 == 0 ? (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3) : (int)blockIdx.x;
  const int t0 = tblk * TOK;
  const int Kc = a.Kc, L = a.L;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh + (int64_t)blk * D;
  const int64_t hist_base = (int64_t)bh * (Kc - 1) * DVT + (int64_t)blk * D;
  const int c = tid % D, tg = tid / D;

  // this channel's taps; beyond Kc they are zero, so the unrolled loop below needs no tap count.  The D * Kc taps of
  // the block are contiguous in memory: they come in through LDS with whole-row requests (a thread reading its own
  // Kc consecutive floats would touch 64 cache lines per request), then each thread picks its own (stride Kc floats
  // between lanes; Kc odd or not, at most a 2-way bank conflict, once per workgroup).
  // Every request of the workgroup -- taps, value rows, the 32 elements of out that the thread adds to -- is issued
  // before the first wait: one trip to memory per workgroup instead of one per stage.
  constexpr int RIT = ((CL_HALO + TOK) * (D / 8) + 255) / 256;
  typename Io::raw8 raw[RIT];
  bool have[RIT];
  auto issue_rows = [&]() __attribute__((always_inline)) {
    // rows t0 - 62 .. t0 + 63: the sequence, before it the incoming history, before that (and past the end) zeros
#pragma unroll
    for (int i = 0; i < RIT; ++i) {
      const int e = tid + 256 * i;
      const int row = e / (D / 8), i0 = 8 * (e % (D / 8));
      const int tok = t0 - CL_HALO + row;
      // unconditional requests (a row that does not exist reads row 0 of the sequence instead and is dropped):
      // every branch around a request would end in a full wait
      const bool in_seq = tok >= 0 && tok < L;
      const bool in_hist = tok < 0 && a.hist_in != nullptr && Kc - 1 + tok >= 0;
      const void* src = in_hist ? a.hist_in : a.v;
      const int mt = in_seq ? tok : 0;     // where the token lies in memory
      const int64_t idx = in_hist ? hist_base + (int64_t)(Kc - 1 + tok) * DVT + i0 : base + (int64_t)mt * a.st + i0;
      raw[i] = Io::load_raw8(src, idx);
      have[i] = in_seq || in_hist;
    }
  };
  // what the attention kernels left in out, as it lies in memory (converted where it is added to), a block of tokens at a
  // time: the first block with the first requests, the next while the current ones are being computed (all 32
  // at once would cost the registers that let a second and third workgroup share the compute unit).  Past the end: the
  // first token's element, never stored.
  typename Io::elem prev[BLK];
  auto issue_prev = [&](int blk8, typename Io::elem (&dst)[BLK]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < BLK; ++e) {
      const int tok = t0 + tg * TPT + blk8 * BLK + e;
      const int mt = tok < L ? tok : 0;
      dst[e] = static_cast<const typename Io::elem*>(a.out)[base + (int64_t)mt * a.st + c];
    }
  };
  float wreg[KMAX];
  {
    // (16 bytes per request, every request of the thread issued before the first value is stored)
    const f32x4* wsrc = reinterpret_cast<const f32x4*>(a.conv_w + ((size_t)h * DVT + blk * D) * Kc);
    constexpr int WIT = (D * KMAX / 4 + 255) / 256;
    f32x4 wt[WIT];
#pragma unroll
    for (int i = 0; i < WIT; ++i) {
      const int e = tid + 256 * i;
      wt[i] = wsrc[e < D * Kc / 4 ? e : D * Kc / 4 - 1];   // unconditional: a branch would end in a full wait
    }
    issue_rows();                             // the value rows are on their way while the taps make their trip through LDS
#pragma unroll
    for (int i = 0; i < WIT; ++i) {
      const int e = tid + 256 * i;
      if (e < D * Kc / 4) *reinterpret_cast<f32x4*>(xs + 4 * e) = wt[i];
    }
    issue_prev(0, prev);                      // ... and the first of what is already in out
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KMAX; ++j) wreg[j] = j < Kc ? xs[c * Kc + j] : 0.f;
    __syncthreads();                          // the staging area is about to take the value rows
  }

  {
    uint32_t top = 0u;                        // largest exponent met, in the place where the type has it
#pragma unroll
    for (int i = 0; i < RIT; ++i) {
      const int e = tid + 256 * i;
      const int row = e / (D / 8), i0 = 8 * (e % (D / 8));
      if (e < (CL_HALO + TOK) * (D / 8)) {
        typename Io::raw8 y = raw[i];
        if (!have[i]) y = typename Io::raw8{};
        *reinterpret_cast<typename Io::raw8*>(xe + row * D + i0) = y;
        top = top_exponent(y, top);
      }
    }
    const int any = __any(not_finite(top, typename Io::raw8{}));
    if ((tid & 63) == 0) odd[tid >> 6] = any;
  }
  __syncthreads();
  // the zero taps beyond Kc would make a NaN of an infinity that lies beyond the window: such workgroups go tap by tap
  const bool by_tap = (odd[0] | odd[1] | odd[2] | odd[3]) != 0;

  // The history handed on (the last Kc - 1 rows of history ++ sequence), when the launcher asked for it here: every
  // workgroup writes the rows whose tokens it owns (t0 <= token < t0 + 64; the first one also the rows that stay
  // history rows), straight from its LDS copy.  Asked for only when no other workgroup can still have hist_in to read.
  if (a.hist_fused) {
    const int R = Kc - 1;
    for (int e = tid; e < R * (D / 8); e += 256) {
      const int r = e / (D / 8), i0 = 8 * (e % (D / 8));
      const int tok = L - R + r;                           // the token (negative: a row of the old history) that becomes row r
      const bool mine = tok < L && ((tok >= t0 && tok < t0 + TOK) || (tok < 0 && t0 == 0));
      const int row = tok - t0 + CL_HALO;                  // its row in the LDS copy
      if (mine && row >= 0)
        *reinterpret_cast<typename Io::raw8*>(static_cast<typename Io::elem*>(a.hist_out) + hist_base + (int64_t)r * DVT + i0) =
            *reinterpret_cast<const typename Io::raw8*>(xe + row * D + i0);
    }
  }

  // (one copy of the 500 multiply-adds in the instruction stream: the loop over the thread's blocks stays a loop)
#pragma unroll 1
  for (int blk8 = 0; blk8 < TPT / BLK; ++blk8) {
    const int tb0 = tg * TPT + blk8 * BLK;
    float acc[BLK];
    typename Io::elem next[BLK];
    issue_prev(blk8 + 1 < TPT / BLK ? blk8 + 1 : blk8, next);
#pragma unroll
    for (int e = 0; e < BLK; ++e) acc[e] = 0.f;
    // value rows from the newest output's own row backwards: row m feeds output e through tap e - 7 + m
    const typename Io::elem* newest = xe + (CL_HALO + tb0 + BLK - 1) * D + c;
    if (by_tap) {                               // uniform
      const float* wc = a.conv_w + ((size_t)h * DVT + blk * D + c) * Kc;
#pragma unroll 1
      for (int j = 0; j < Kc; ++j)
#pragma unroll
        for (int e = 0; e < BLK; ++e) acc[e] = fmaf(wc[j], elem_to_f32(newest[-(BLK - 1 - e + j) * D]), acc[e]);
    } else {
      // (fully unrolled, so that every tap index is a constant and the taps stay in registers)
#pragma unroll
      for (int m = 0; m < KMAX + BLK - 1; ++m) {
        const float x = elem_to_f32(newest[-m * D]);
#pragma unroll
        for (int e = 0; e < BLK; ++e) {
          constexpr int J0 = -(BLK - 1);
          const int j = e + J0 + m;
          if (j >= 0 && j < KMAX) acc[e] = fmaf(wreg[j], x, acc[e]);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < BLK; ++e) {
      const int tok = t0 + tb0 + e;
      if (tok < L)
        Io::store1(a.out, base + (int64_t)tok * a.st + c, elem_to_f32(prev[e]) + acc[e]);
    }
#pragma unroll
    for (int e = 0; e < BLK; ++e) prev[e] = next[e];
  }
}

// New history = the last Kc-1 rows of (incoming history ++ sequence), for the cases the conv kernel cannot do on the
// way (hist_out is hist_in on a sequence of several workgroups; no tokens).  Runs behind conv_long_kernel, which is the
// last reader of hist_in before this.  One workgroup per (b, h, value block): every element is read (all requests in
// flight at once) before, behind a barrier, any is written, so hist_out may be hist_in.
template <typename Io, int D>
__global__ __launch_bounds__(256) void conv_long_hist_kernel(ConvLongArgs a) {
  const int bh = blockIdx.x / a.m, blk = blockIdx.x % a.m, b = bh / a.H, h = bh % a.H;
  const int tid = threadIdx.x;
  const int R = a.Kc - 1, DVT = a.m * D;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh + (int64_t)blk * D;
  const int64_t hist_base = (int64_t)bh * R * DVT + (int64_t)blk * D;
  // whole vectors of 8 channels, as they lie in memory (history and value rows share their element type); every
  // request is unconditional -- a vector that does not exist reads the first one of hist_out instead and is
  // replaced by zeros -- so that all of them are in flight together
  using raw8 = typename Io::raw8;
  using elem = typename Io::elem;
  constexpr int VPR = D / 8;
  constexpr int EIT = (CL_HALO * VPR + 255) / 256;
  raw8 x[EIT];
  bool have[EIT];
#pragma unroll
  for (int i = 0; i < EIT; ++i) {
    const int el = tid + 256 * i;
    const int r = el / VPR, c = 8 * (el % VPR);
    const int e = a.L + r;                    // row of (history ++ sequence), the history being rows 0 .. R-1
    const bool from_v = r < R && e >= R;
    const bool from_h = r < R && e < R && a.hist_in != nullptr;
    const void* src = from_v ? a.v : from_h ? a.hist_in : a.hist_out;
    const int64_t idx = from_v ? base + (int64_t)(e - R) * a.st + c : from_h ? hist_base + (int64_t)e * DVT + c : hist_base;
    x[i] = Io::load_raw8(src, idx);
    have[i] = from_v || from_h;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < EIT; ++i) {
    const int el = tid + 256 * i;
    const int r = el / VPR, c = 8 * (el % VPR);
    if (r < R) {
      raw8 y = x[i];
      if (!have[i]) y = raw8{};
      *reinterpret_cast<raw8*>(static_cast<elem*>(a.hist_out) + hist_base + (int64_t)r * DVT + c) = y;
    }
  }
}

template <typename Io, int D, int KMAX, int TOK>
static hipError_t launch_cl_t(const ConvLongArgs& a, hipStream_t st) {
  constexpr int LDS = conv_long_lds<typename Io::elem, D, KMAX, TOK>() + 4 * (int)sizeof(int);
  auto kern = conv_long_kernel<Io, D, KMAX, TOK>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, LDS);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.L + TOK - 1) / TOK), (unsigned)(a.B * a.H * a.m)), dim3(256), LDS, st, a);
  return hipGetLastError();
}

template <typename Io, int D, int KMAX>
static hipError_t launch_cl_k(const ConvLongArgs& a, hipStream_t st) {
  // fewer 64-token workgroups than compute units: 32 tokens each
  const int64_t wgs = (int64_t)((a.L + CL_TOK - 1) / CL_TOK) * a.B * a.H * a.m;
  return wgs < 256 ? launch_cl_t<Io, D, KMAX, CL_TOK / 2>(a, st) : launch_cl_t<Io, D, KMAX, CL_TOK>(a, st);
}

// bf16 rows added to out: this kernel or the matrix cores?  The matrix-core kernel works on tiles of 256 tokens and takes
// about as long for 9 taps as for 17, for 18 as for 49; this one pays for the tokens and the taps there are (capacities of
// 16, 32 and 63; of those of 32 not 32 itself, whose taps come through LDS on one bank).  Measured, us a prefill call, this / matrix
// cores.  Up to 16 taps: d = 64: 1 head, 300 tokens 27.2 / 27.6, 32 heads, 1100 tokens 37.2 / 40.4, 256 heads, 300 tokens
// 37.3 / 44.7; d = 128: 16 heads, 300 tokens 32.0 / 33.1, 128 heads, 1100 tokens 97 / 107, 256 heads, 4096 tokens 442 / 438, but 1 head,
// 300 tokens 31.4 / 30.2.  Fewer than 32 taps, heads enough to fill the chip: d = 64: 32 heads, 300 tokens 29.1 / 31.1, 128 heads,
// 1100 tokens 64 / 72, 64 heads, 4000 tokens 95 / 91; d = 128: 64 heads, 300 tokens 39.0 / 40.5, 128 heads, 1100 tokens 103 / 107, 32
// heads, 500 tokens 41.3 / 39.2.  Any number of taps, sequences of half a tile: 63 taps, d = 64, 256 heads, 60 tokens 22.3 / 25.3, 120
// tokens 26.7 / 29.6, 200 tokens 38.8 / 40.6, 32 heads, 60 tokens 19.1 / 18.1; d = 128, 256 heads, 60 tokens 32 / 36, 200 tokens 56 / 52, 64
// heads, 60 tokens 23.4 / 22.9.
static bool conv_vector_pays(const ConvLongArgs& a, int d) {
  const int64_t heads = (int64_t)a.B * a.H * a.m, tiles = (int64_t)((a.L + 255) / 256) * heads * (d / 32);
  return (a.Kc <= 16 && (d == 64 || tiles >= 64)) || (a.Kc < 32 && a.L <= 2048 && 2 * heads >= d) || (a.L <= 128 && heads >= d);
}

template <typename Io, int D>
static hipError_t launch_cl(const ConvLongArgs& a_in, hipStream_t st) {
  constexpr bool BF16 = sizeof(typename Io::elem) == 2;
  hipError_t e = hipSuccess;
  // The history can be handed on by the conv kernel itself unless hist_out is hist_in and several workgroups share a
  // head: the first of them reads the old rows, the last would overwrite them, and nothing orders the two.  (The bf16
  // kernel writes it while its own waves may still be reading: never when hist_out is hist_in.)
  ConvLongArgs a = a_in;
  const bool vector = !BF16 || (!a.assign && conv_vector_pays(a, D));
  a.hist_fused = a.hist_out != nullptr && a.L > 0 && (a.hist_out != a.hist_in || (vector && a.L <= CL_TOK / 2));
  if (a.L > 0) {
    if (!vector) e = launch_conv_mfma(a, D, st);
    else e = a.Kc <= 16   ? launch_cl_k<Io, D, 16>(a, st)
             : a.Kc <= 32 ? launch_cl_k<Io, D, 32>(a, st)
                          : launch_cl_k<Io, D, CL_MAXK>(a, st);
    if (e != hipSuccess) return e;
  }
  if (a.hist_out && !a.hist_fused) {
    hipLaunchKernelGGL((conv_long_hist_kernel<Io, D>), dim3((unsigned)(a.B * a.H * a.m)), dim3(256), 0, st, a);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_conv_long(const ConvLongArgs& a, bool bf16, int d, hipStream_t st) {
  if (bf16) return d == 128 ? launch_cl<IoBf16, 128>(a, st) : launch_cl<IoBf16, 64>(a, st);
  return d == 128 ? launch_cl<IoF32, 128>(a, st) : launch_cl<IoF32, 64>(a, st);
}

}  // namespace linattn
