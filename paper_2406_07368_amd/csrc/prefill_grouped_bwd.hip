// Gradient of the three-branch form of Sec. 4.1 on the matrix cores (bf16 rows): the training direction of the
// paper's FLASH experiment (Sec. 5.3 times a training step, forward and backward, in groups of 256 tokens).
//
// With P_g = (S_g, z_g) the sums over everything before group g and D_g the gradient with respect to the sums after
// group g, for a token t of group g and the incoming gradient dO = d loss / d out:
//
//   grouped branch   N = S_g^T phi(q_t),  den = phi(q_t).z_g + eps,  f = alpha / den:
//                    W = S_g dO_t,  nd = phi(q_t).W,  dden = -f nd / den,
//                    dq_t += (f W + z_g dden) * phi'(q_t),   G_g += phi(q_t) (f dO_t)^T,   gz_g += phi(q_t) dden
//   local branch     p = softmax over the keys i <= t of the group of q_t.k_i / sqrt(d),  dp_i = dO_t.v_i,
//                    pbar = sum_i p_i dp_i,  ds_i = p_i (dp_i - pbar) / sqrt(d):
//                    dq_t += sum_i ds_i k_i,   dk_i += ds_i q_t,   dv_i += p_i dO_t
//   the sums         D_g = sum_{g' > g} (G_g', gz_g'):  dk_i += (D_g.S v_i + D_g.z) * phi'(k_i),  dv_i += D_g.S^T phi(k_i)
//   conv             dv_s += sum_j w[c][j] dO[s + j][c],   dw[c][j] = sum_t dO[t][c] v[t - j][c]   (conv_mfma.hip)
//
// Rows (dq, dk, dv): grouped_bwd_rows.hip.  Group-level sums, in this file one workgroup per (b, h, group):
//   grouped_bwd_gs_kernel     G_g = (f phi(Q))^T dO and gz_g, contraction over the group's tokens (32 x 32 x 16 bf16 MFMA).
//   grouped_bwd_suffix_kernel D_g = sum over the later groups, in place.
//                             (With heads enough, or few groups, one walk over the groups takes the place of these two and
//                             of the sums and their prefix sum: group_sums.hip.)
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

namespace linattn {

namespace {

template <int D, int GT>
struct BwdCfg {
  static constexpr int NW = GT / 32;         // waves: one 32-row tile each
  static constexpr int NT = NW * 64;
  static constexpr int CT = D / 32;          // 32-wide tiles of features / channels
  static constexpr int KS = D + 8;           // token rows: transposed reads
  static constexpr int OFF_A = 0;                  // Q (K) rows
  static constexpr int OFF_B = GT * KS * 2;        // dO (V) rows
  static constexpr int OFF_ST = 2 * GT * KS * 2;   // [2][GT] float: per-token scalars
  static constexpr int OFF_RED = OFF_ST + 2 * GT * 4;   // [NT] float: partial sums of the z passes
  static constexpr int TOTAL = OFF_RED + NT * 4;
  static constexpr int SLOT = D * D + D;
  static_assert(TOTAL <= 160 * 1024, "LDS");
  static_assert(NT >= D, "one thread per feature in the z passes");
};

// rows tok0 .. tok0 + GT - 1 of two tensors -> LDS (rows past the end are zero rows); every request before the first store
template <int D, int GT>
__device__ __forceinline__ void load_rows2(const uint16_t* ga, const uint16_t* gb, int64_t st, int tok0, int nt,
                                           uint16_t* La, uint16_t* Lb, int tid) {
  using G = BwdCfg<D, GT>;
  constexpr int NPC = GT * (D / 8) / G::NT;
  u32x4 ax[NPC], bx[NPC];
#pragma unroll
  for (int i = 0; i < NPC; ++i) {
    const int e = tid + G::NT * i;
    const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
    const int rr = r < nt ? r : nt - 1;        // unconditional requests; a row that does not exist is replaced by zeros
    ax[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ga + (int64_t)(tok0 + rr) * st + c0));
    bx[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gb + (int64_t)(tok0 + rr) * st + c0));
  }
#pragma unroll
  for (int i = 0; i < NPC; ++i) {
    const int e = tid + G::NT * i;
    const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
    const u32x4 zero = {0, 0, 0, 0};
    *reinterpret_cast<u32x4*>(La + r * G::KS + c0) = r < nt ? ax[i] : zero;
    *reinterpret_cast<u32x4*>(Lb + r * G::KS + c0) = r < nt ? bx[i] : zero;
  }
}

}  // namespace

// ---- what the queries of a group add to the gradient of the sums before it; and those sums themselves -----------------
// SUMS: the same contraction over a group's tokens with (K, V) in the place of (Q, dO) and weights of one: the group's
// own phi(K)^T V and sum of phi(K), written to the slot of the group after it (the prefix sum follows).  The forward's
// first pass is not used for this: it rounds phi(k) to one bf16, and with keys of the size 1/sqrt(d) most of what the
// keys say sits below that rounding, while the gradient of the grouped branch is a difference that lives on it.
template <int D, int GT, bool SUMS>
__global__ __launch_bounds__(GT * 2) void grouped_bwd_gs_kernel(GroupedBwdArgs a) {
  using G = BwdCfg<D, GT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* Ql = reinterpret_cast<uint16_t*>(smem + G::OFF_A);
  uint16_t* Dl = reinterpret_cast<uint16_t*>(smem + G::OFF_B);
  float* fs = reinterpret_cast<float*>(smem + G::OFF_ST);  // alpha / den per token
  float* dd = fs + GT;                                     // d den per token
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  // gradients: groups 1 .. ng-1 (group 0 has nothing before it); sums: groups 0 .. ng-2 (nothing follows the last)
  const int g = SUMS ? blockIdx.x : blockIdx.x + 1, bh = blockIdx.y;
  const int b = bh / a.H, h = bh % a.H;
  const int tok0 = g * GT;
  const int nt = (a.L - tok0) < GT ? (a.L - tok0) : GT;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const uint16_t* gq = static_cast<const uint16_t*>(SUMS ? a.k : a.q) + base;
  const uint16_t* gdo = static_cast<const uint16_t*>(SUMS ? a.v : a.dout) + base;
  float* slot = SUMS ? a.P + ((size_t)bh * a.ng + g + 1) * G::SLOT : a.Dg + ((size_t)bh * a.ng + g) * G::SLOT;
  const size_t n = (size_t)a.B * a.H * a.L, e0 = (size_t)bh * a.L + tok0;
  const float one = a.relu ? 0.f : 1.f;

  float f3 = 0.f, d4 = 0.f;
  if (tid < GT && tid < nt) {
    if (SUMS) f3 = d4 = 1.f;
    else { f3 = a.stats[3 * n + e0 + tid]; d4 = a.stats[4 * n + e0 + tid]; }
  }
  load_rows2<D, GT>(gq, gdo, a.st, tok0, nt, Ql, Dl, tid);
  if (tid < GT) { fs[tid] = f3; dd[tid] = d4; }
  __syncthreads();
  // gz[f] = sum_t phi(q_t[f]) dden_t: thread = (feature, one of NT / D runs of tokens), eight independent terms in
  // flight (one by one, every term would wait for its own LDS reads and exponential), the runs added up through LDS
  {
    constexpr int NP = G::NT / D, TPP = GT / NP;           // runs per feature, tokens per run
    float* zp = reinterpret_cast<float*>(smem + G::OFF_RED);   // [NP][D]
    const int f = tid % D, part = tid / D;
    float gz = 0.f;
#pragma unroll 8
    for (int i = 0; i < TPP; ++i) {
      const int t = part * TPP + i;                        // rows past the end are zero rows with weight 0
      gz = fmaf(phi_nb(bf16_bits_to_f32(Ql[t * G::KS + f]), one), dd[t], gz);
    }
    zp[part * D + f] = gz;
  }
  __syncthreads();
  if (tid < D) {
    const float* zp = reinterpret_cast<const float*>(smem + G::OFF_RED);
    float gz = 0.f;
#pragma unroll
    for (int p = 0; p < G::NT / D; ++p) gz += zp[p * D + tid];
    slot[D * D + tid] = gz;
  }
  // the tiles (feature block ib, channel block cb) over the waves; lanes = channels, registers = features.  The
  // operand (alpha / den_t) phi(q_t) is made from the raw rows as they are read (lane = feature, registers = tokens
  // 16ks + 8hi + 0..7) and enters as hi + lo: D.S v + D.z is again a difference of nearly equal parts.
  // A wave takes a feature block and CBG channel blocks at a time, so that the operand made above serves several tiles.
  constexpr int CBG = (G::CT * G::CT / G::NW) < 1 ? 1 : ((G::CT * G::CT / G::NW) > G::CT ? G::CT : (G::CT * G::CT / G::NW));
  constexpr int UPB = G::CT / CBG;                         // units per feature block
#pragma unroll 1
  for (int unit = w; unit < G::CT * UPB; unit += G::NW) {
    const int ib = unit / UPB, cb0 = (unit % UPB) * CBG;
    f32x16 sacc[CBG];
#pragma unroll
    for (int j = 0; j < CBG; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[j][r] = 0.f;
    for (int ks = 0; ks < GT / 16; ++ks) {
      const u32x4 raw = __builtin_bit_cast(u32x4, tr_operand(Ql, G::KS, 16 * ks, 32 * ib, lane));
      const float* fsp = fs + 16 * ks + 8 * hi;            // 0 for rows past the end
      u32x4 ah, al;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x0 = fsp[2 * i] * phi_nb(bf16_lo_to_f32(raw[i]), one);
        const float x1 = fsp[2 * i + 1] * phi_nb(bf16_hi_to_f32(raw[i]), one);
        ah[i] = pack_bf16x2(x0, x1);
        al[i] = pack_bf16x2(x0 - bf16_lo_to_f32(ah[i]), x1 - bf16_hi_to_f32(ah[i]));
      }
#pragma unroll
      for (int j = 0; j < CBG; ++j) {
        const bf16x8 dop = tr_operand(Dl, G::KS, 16 * ks, 32 * (cb0 + j), lane);
        sacc[j] = mfma(__builtin_bit_cast(bf16x8, ah), dop, sacc[j]);
        sacc[j] = mfma(__builtin_bit_cast(bf16x8, al), dop, sacc[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < CBG; ++j) {
      float* so = slot + (32 * ib + 4 * hi) * D + 32 * (cb0 + j) + l32;
#pragma unroll
      for (int r = 0; r < 16; ++r) so[(8 * (r >> 2) + (r & 3)) * D] = sacc[j][r];
    }
  }
}

// ---- D_g = sum over the later groups of what their queries added, in place (one thread per element) ----------------
__global__ __launch_bounds__(256) void grouped_bwd_suffix_kernel(GroupedBwdArgs a, int slot_elems) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= slot_elems) return;
  float* ws = a.Dg + (size_t)blockIdx.y * a.ng * slot_elems + e;
  float run = 0.f;
  // sixteen groups at a time, every request before the first store; slot 0 was never written and is not read
  for (int g1 = a.ng - 1; g1 >= 0; g1 -= 16) {
    float inc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int g = g1 - i;
      inc[i] = ws[(size_t)(g >= 1 ? g : 1) * slot_elems];     // (launched for two groups or more: slot 1 exists)
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int g = g1 - i;
      if (g >= 0) ws[(size_t)g * slot_elems] = run;
      if (g >= 1) run += inc[i];
    }
  }
}

// ---- dw: the partial sums of the token blocks (conv_mfma.hip) -------------------------------------------------------
// Sums over batch rows and token blocks in a fixed order, DW_RED partial sums at a time: in [H][n][per_head] ->
// out [H][ceil(n / DW_RED)][per_head]; the last stage writes dconv_w (n = 0: zeros).
namespace { constexpr int DW_RED = 32; }
__global__ __launch_bounds__(256) void grouped_bwd_dw_reduce_kernel(const float* in, float* out, int n, int per_head) {
  const int e = blockIdx.x * 256 + threadIdx.x, h = blockIdx.y, c = blockIdx.z;
  if (e >= per_head) return;
  const int nout = (n + DW_RED - 1) / DW_RED;
  const int i0 = c * DW_RED, i1 = (i0 + DW_RED) < n ? (i0 + DW_RED) : n;
  const float* p = in + ((size_t)h * n + i0) * per_head + e;
  float s = 0.f;
#pragma unroll 8
  for (int i = i0; i < i1; ++i, p += per_head) s += *p;
  out[((size_t)h * (nout > 0 ? nout : 1) + c) * per_head + e] = s;
}

template <int D, int GT>
static hipError_t launch_bwd_core(const GroupedBwdArgs& a, const ConvLongArgs* conv, hipStream_t st, hipEvent_t before_dkdv) {
  using G = BwdCfg<D, GT>;
  const int BH = a.B * a.H;
  hipError_t e;
  auto kg = grouped_bwd_gs_kernel<D, GT, false>;
  auto ks = grouped_bwd_gs_kernel<D, GT, true>;
  if ((e = LINATTN_MAX_LDS_ONCE(kg, G::TOTAL)) != hipSuccess) return e;
  if ((e = LINATTN_MAX_LDS_ONCE(ks, G::TOTAL)) != hipSuccess) return e;
  GroupSumsArgs s{};
  s.B = a.B; s.H = a.H; s.L = a.L; s.ng = a.ng; s.relu = a.relu; s.sb = a.sb; s.sh = a.sh; s.st = a.st;
  const bool walk = group_sums_pays(BH, a.ng, D, GT);
  if (walk) {
    s.a = a.k; s.b = a.v; s.slots = a.P;
    if ((e = launch_group_sums(s, D, GT, false, st)) != hipSuccess) return e;
  } else {
    // the sums before every group: every group's own sums, then the prefix sum (which also writes the zeros before group 0)
    hipLaunchKernelGGL(ks, dim3((unsigned)(a.ng - 1), (unsigned)BH), dim3(G::NT), G::TOTAL, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    PrefillArgs f{};
    f.ws = a.P; f.B = a.B; f.H = a.H; f.m = 1; f.nseg = a.ng;
    if ((e = launch_segment_scan(f, D, st)) != hipSuccess) return e;
  }
  if ((e = launch_grouped_bwd_rows(a, conv, D, false, st)) != hipSuccess) return e;
  if (walk && a.ng > 1) {
    const size_t n = (size_t)BH * a.L;
    s.a = a.q; s.b = a.dout; s.w = a.stats + 3 * n; s.wz = a.stats + 4 * n; s.slots = a.Dg;
    if ((e = launch_group_sums(s, D, GT, true, st)) != hipSuccess) return e;
  } else if (a.ng > 1) {
    hipLaunchKernelGGL(kg, dim3((unsigned)(a.ng - 1), (unsigned)BH), dim3(G::NT), G::TOTAL, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(grouped_bwd_suffix_kernel, dim3((unsigned)((G::SLOT + 255) / 256), (unsigned)BH), dim3(256), 0, st, a, (int)G::SLOT);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (conv && a.dconv_w && !dw_sums_ride(a) && (e = launch_grouped_bwd_dw(a, D, st)) != hipSuccess) return e;
  if (before_dkdv && (e = hipStreamWaitEvent(st, before_dkdv, 0)) != hipSuccess) return e;
  return launch_grouped_bwd_rows(a, conv, D, true, st);
}

// The conv-weight sums over batch rows and token blocks (no tokens: zeros).
hipError_t launch_grouped_bwd_dw(const GroupedBwdArgs& a, int d, hipStream_t st) {
  hipError_t e;
  const int per_head = d * a.Kc;
  // stages of 32: the partial sums ping-pong between the two halves of the buffer until one row per head is left
  const float* in = a.dw_part;
  float* other = a.dw_part + (size_t)a.B * a.H * (a.nwb > 0 ? a.nwb : 1) * per_head;
  int n = a.B * a.nwb;
  for (;;) {
    const int nout = (n + DW_RED - 1) / DW_RED;
    float* out = nout <= 1 ? a.dconv_w : other;
    hipLaunchKernelGGL(grouped_bwd_dw_reduce_kernel, dim3((unsigned)((per_head + 255) / 256), (unsigned)a.H, (unsigned)(nout > 0 ? nout : 1)),
                       dim3(256), 0, st, in, out, n, per_head);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (nout <= 1) break;
    other = const_cast<float*>(in);
    in = out;
    n = nout;
  }
  return hipSuccess;
}

// Everything but the conv's share and the conv-weight sums, in order; conv: those as well, on the way.
hipError_t launch_grouped_bwd_core(const GroupedBwdArgs& a, const ConvLongArgs* conv, int d, hipStream_t st, hipEvent_t before_dkdv) {
  if (a.L <= 0) return hipSuccess;
  if (d == 128) return a.group == 256 ? launch_bwd_core<128, 256>(a, conv, st, before_dkdv) : launch_bwd_core<128, 64>(a, conv, st, before_dkdv);
  return a.group == 256 ? launch_bwd_core<64, 256>(a, conv, st, before_dkdv) : launch_bwd_core<64, 64>(a, conv, st, before_dkdv);
}

}  // namespace linattn
