// Gradient of the three-branch form with respect to the rows of q, k and v (Sec. 4.1; the formulas stand in
// prefill_grouped_bwd.hip): the local branch inside a group and what the sums before / after the group add.
//
//   grouped_bwd_dq_kernel     queries of a run of RC tokens against the group's keys up to them; hands the per-token scalars on
//   grouped_bwd_dkdv_kernel   keys of a run of RC tokens against the group's queries from them on
//
// A workgroup owns RC = 128 tokens (a whole group of 64) and has four waves (two); the rows of the other side pass through
// LDS RC at a time.  A wave owns two tiles of 16 tokens, w and 2 NW - 1 - w: of the causal triangle inside the run every
// wave then has the same share.  Products are 16 x 16 x 32 bf16 MFMAs with fp32 accumulation, the wave's own rows being
// the operand with lane = token (lane % 16), so that softmax statistics and accumulators belong to a lane's token and the
// weights go from accumulators into the next product without passing through LDS.  An operand read from LDS serves both tiles.
// What bounds it: issue of vector and matrix instructions in turn, and the requests at the head of every run (about a
// quarter of the time in dq, less than half in dk/dv, whose accumulators leave room for half of a request).  With 76 KB of
// LDS two workgroups share a CU, one working while the other waits for its rows.  On B8 H8 L8192 d128 in groups of 256, each
// launch alone: dq 278 us, dk and dv 371 us.  One workgroup of eight waves per group, a 32-token tile each (1 to 8 units of
// work, all of a CU's LDS) and one launch half for dk, one for dv took 326 and 464 us: one wave per SIMD at work most of
// the time, and nothing behind its loads.
#include <type_traits>

#include "common.h"
#include "conv_mfma.h"
#include "kernels.h"
#include "mfma_util.h"

namespace linattn {

namespace {

template <int D, int GT>
struct RowsCfg {
  static constexpr int RC = GT < 128 ? GT : 128;   // tokens per workgroup, rows per pass through LDS
  static constexpr int NH = GT / RC;               // workgroups per group
  static constexpr int NW = RC / 32, NT = 64 * NW;
  static constexpr int KSD = D / 32;               // contraction steps over features / channels
  static constexpr int CT = D / 16;                // 16-wide tiles of features / channels
  static constexpr int KS = D + 16;                // LDS rows: row reads and transposed reads without bank conflicts
  static constexpr int OS = D + 4;                 // staged fp32 output rows
  // the d x d operand (two bf16 terms) and the staged outputs take the place of the token rows
  static constexpr int ROWS = 2 * RC * KS * 2, SREG = 2 * D * KS * 2, STG = RC * OS * 4;
  static constexpr int REGION = ((ROWS > SREG ? (ROWS > STG ? ROWS : STG) : (SREG > STG ? SREG : STG)) + 15) / 16 * 16;
  static constexpr int OFF_B = RC * KS * 2;        // the second tensor's rows
  static constexpr int OFF_Z = REGION;             // [D] float
  static constexpr int OFF_ST = OFF_Z + D * 4;     // [3][RC] float: per-token scalars
  static constexpr int TOTAL = OFF_ST + 3 * RC * 4;
  static constexpr int PPT = RC * (D / 8) / NT;    // 16-byte pieces of RC rows per thread
  static constexpr int SLOT = D * D + D;
  static_assert(TOTAL <= 80 * 1024, "two workgroups per CU");
};

template <int D> constexpr float kInvSqrt = D == 64 ? 0.125f : 0.08838834764831845f;
template <int D> constexpr float kToLog2 = 1.44269504088896340736f * kInvSqrt<D>;

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 16 x 32 operand: lane % 16 = row row0 + 0..15, registers = columns col0 + 8 (lane / 16) + 0..7
__device__ __forceinline__ bf16x8 rows16(const uint16_t* base, int stride, int row0, int col0, int lane) {
  return lds_row8(base + (row0 + (lane & 15)) * stride + col0 + 8 * (lane >> 4));
}
// transposed: lane % 16 = column col0 + 0..15, registers = rows row0 + 8 (lane / 16) + 0..7
__device__ __forceinline__ bf16x8 tr16(const uint16_t* base, int stride, int row0, int col0, int lane) {
  const uint16_t* p = base + (row0 + 8 * (lane >> 4) + ((lane & 15) >> 2)) * stride + col0 + 4 * (lane & 3);
  return cat4(lds_tr4(p), lds_tr4(p + 4 * stride));
}
// transposed, registers = the rows in the order in which two 16 x 16 accumulators hold them: row0 + 4 (lane / 16) + 0..3,
// then row0 + 16 + 4 (lane / 16) + 0..3
__device__ __forceinline__ bf16x8 tr16_acc_order(const uint16_t* base, int stride, int row0, int col0, int lane) {
  const uint16_t* p = base + (row0 + 4 * (lane >> 4) + ((lane & 15) >> 2)) * stride + col0 + 4 * (lane & 3);
  return cat4(lds_tr4(p), lds_tr4(p + 16 * stride));
}

// two 16 x 16 accumulators -> the operand of a contraction over their 32 rows, as hi + lo (two bf16 terms): with one term
// the rounding, met by cancelling products, would be the largest error of the gradient
__device__ __forceinline__ void split44(f32x4 x, f32x4 y, bf16x8& hi, bf16x8& lo) {
  u32x4 h, l;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    h[i] = pack_bf16x2(x[2 * i], x[2 * i + 1]);
    h[2 + i] = pack_bf16x2(y[2 * i], y[2 * i + 1]);
    l[i] = pack_bf16x2(x[2 * i] - bf16_lo_to_f32(h[i]), x[2 * i + 1] - bf16_hi_to_f32(h[i]));
    l[2 + i] = pack_bf16x2(y[2 * i] - bf16_lo_to_f32(h[2 + i]), y[2 * i + 1] - bf16_hi_to_f32(h[2 + i]));
  }
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}

// phi'(x) without a branch on the feature map: one = 1 for elu + 1 and 0 for max(x, 0)
__device__ __forceinline__ float dphi_nb(float x, float one) {
  return x > 0.f ? 1.f : one * __builtin_amdgcn_exp2f(x * 1.44269504088896340736f);
}

// four consecutive elements of a row as fp32
__device__ __forceinline__ f32x4 unpack4(u32x2 x) {
  return f32x4{bf16_lo_to_f32(x[0]), bf16_hi_to_f32(x[0]), bf16_lo_to_f32(x[1]), bf16_hi_to_f32(x[1])};
}

// Rows 0 .. RC - 1 of two tensors on their way into LDS, PARTS requests after one another (rows from nr on are zero rows).
// fetch and put are apart so that other requests and work can stand between them.
template <int D, int GT, int PARTS = 1>
struct RowLoad {
  using G = RowsCfg<D, GT>;
  static constexpr int N = G::RC * (D / 8) / G::NT / PARTS;
  u32x4 ax[N], bx[N];
  __device__ __forceinline__ void fetch(const uint16_t* ga, const uint16_t* gb, int64_t st, int nr, int tid, int part = 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e = tid + G::NT * (N * part + i);
      const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
      const int rr = r < nr ? r : nr - 1;      // unconditional requests; a row that does not exist is replaced by zeros
      ax[i] = *reinterpret_cast<const u32x4*>(ga + (int64_t)rr * st + c0);
      bx[i] = *reinterpret_cast<const u32x4*>(gb + (int64_t)rr * st + c0);
    }
  }
  __device__ __forceinline__ void put(uint16_t* La, uint16_t* Lb, int nr, int tid, int part = 0) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e = tid + G::NT * (N * part + i);
      const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
      const u32x4 zero = {0, 0, 0, 0};
      *reinterpret_cast<u32x4*>(La + r * G::KS + c0) = r < nr ? ax[i] : zero;
      *reinterpret_cast<u32x4*>(Lb + r * G::KS + c0) = r < nr ? bx[i] : zero;
    }
  }
};

// A slot's d x d part -> LDS as two bf16 arrays [feature][channel], hi = bf16(x) at Sl and lo = bf16(x - hi) behind it; its
// d-vector -> LDS as fp32.  Two terms because what is computed from these sums is a difference of two nearly equal parts
// (the derivative of a ratio: numerator part minus denominator part), which the rounding of one bf16 term (2^-9 of the
// common part) would swamp.
template <int D, int GT, int PARTS = 1>
struct SlotLoad {
  using G = RowsCfg<D, GT>;
  static constexpr int N = D * D / 4 / G::NT / PARTS;
  f32x4 sx[N];
  __device__ __forceinline__ void fetch(const float* slot, int tid, int part = 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) sx[i] = reinterpret_cast<const f32x4*>(slot)[tid + G::NT * (N * part + i)];
  }
  __device__ __forceinline__ void put(uint16_t* Sl, int tid, int part = 0) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e = 4 * (tid + G::NT * (N * part + i));
      const u32x2 h = {pack_bf16x2(sx[i][0], sx[i][1]), pack_bf16x2(sx[i][2], sx[i][3])};
      const u32x2 l = {pack_bf16x2(sx[i][0] - bf16_lo_to_f32(h[0]), sx[i][1] - bf16_hi_to_f32(h[0])),
                       pack_bf16x2(sx[i][2] - bf16_lo_to_f32(h[1]), sx[i][3] - bf16_hi_to_f32(h[1]))};
      *reinterpret_cast<u32x2*>(Sl + (e / D) * G::KS + e % D) = h;
      *reinterpret_cast<u32x2*>(Sl + D * G::KS + (e / D) * G::KS + e % D) = l;
    }
  }
};

// acc[n][ct][r] = X[token 16 tile[n] + lane % 16][column 16ct + 4 (lane / 16) + r] -> global bf16 rows, staged through LDS in
// fp32.  held: rows that are added (one rounding).  Starts with a barrier: every wave is past its use of LDS.
template <int D, int GT>
struct HeldRows { u32x4 x[RowsCfg<D, GT>::PPT]; };
template <int D, int GT>
__device__ __forceinline__ void hold_rows(HeldRows<D, GT>& held, const uint16_t* gout, int64_t st, int nr, int tid) {
  using G = RowsCfg<D, GT>;
#pragma unroll
  for (int i = 0; i < RowsCfg<D, GT>::PPT; ++i) {
    const int e = tid + G::NT * i, r = e / (D / 8), c0 = 8 * (e % (D / 8));
    held.x[i] = *reinterpret_cast<const u32x4*>(gout + (int64_t)(r < nr ? r : nr - 1) * st + c0);
  }
}
template <int D, int GT, bool ADD>
__device__ __forceinline__ void store_rows(const f32x4 (&acc)[2][D / 16], const HeldRows<D, GT>& held, float* Ol,
                                           uint16_t* gout, int64_t st, int nr, int tid, const int (&tile)[2], int lane) {
  using G = RowsCfg<D, GT>;
  constexpr int PPT = G::PPT;
  static_assert(PPT * G::NT == G::RC * (D / 8), "whole pieces per thread");
  __syncthreads();
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    float* orow = Ol + (16 * tile[n] + (lane & 15)) * G::OS + 4 * (lane >> 4);
#pragma unroll
    for (int ct = 0; ct < G::CT; ++ct) *reinterpret_cast<f32x4*>(orow + 16 * ct) = acc[n][ct];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int e = tid + G::NT * i, r = e / (D / 8), c0 = 8 * (e % (D / 8));
    if (r < nr) {
      const float* src = Ol + r * G::OS + c0;
      f32x4 y0 = *reinterpret_cast<const f32x4*>(src), y1 = *reinterpret_cast<const f32x4*>(src + 4);
      if constexpr (ADD) {
        y0 += unpack4(u32x2{held.x[i][0], held.x[i][1]});
        y1 += unpack4(u32x2{held.x[i][2], held.x[i][3]});
      }
      *reinterpret_cast<u32x4*>(gout + (int64_t)r * st + c0) =
          u32x4{pack_bf16x2(y0[0], y0[1]), pack_bf16x2(y0[2], y0[3]), pack_bf16x2(y1[0], y1[1]), pack_bf16x2(y1[2], y1[3])};
    }
  }
}

// The workgroups of a group read the same rows: with two of them they get block indices 8 apart, which the dispatcher
// places on the same chiplet, so that the second finds the rows in that chiplet's L2 (blocks 0..7 = groups 0..7 with
// half `first`, 8..15 = the same groups with the other half, and so on; a remainder of fewer than 8 groups alternates).
template <int NH>
__device__ __forceinline__ void group_and_half(int bx, int ng, int first, int& g, int& half) {
  if constexpr (NH == 1) {
    g = bx;
    half = 0;
  } else {
    const int full = (ng >> 3) << 3;
    half = first ^ (bx < 2 * full ? (bx >> 3) & 1 : (bx - 2 * full) & 1);
    g = bx < 2 * full ? ((bx >> 4) << 3) | (bx & 7) : full + ((bx - 2 * full) >> 1);
  }
}

}  // namespace

// ---- dq and the per-token scalars ---------------------------------------------------------------------------------
// Pass 1 over the key rows up to the queries: scores, running maximum and sum, and the running sum of e_i dp_i (so pbar
// needs no pass of its own).  Pass 2, from the last rows (still in LDS) back: scores and dp again, dQ^T += K^T ds^T.  Then
// the grouped branch with S_g in LDS.
//
// CONV: the workgroups behind the first `ndq` are the conv's (its share of dv and the partial sums of the tap gradient).  A
// small gradient call does not fill the chip, and as launches of their own on a side stream these cost more host time (events
// to fork and join, 6 to 7 us each) than the whole call's work; see conv_rides.
template <int D, int GT> struct RidingConv {
  static constexpr int NW = RowsCfg<D, GT>::NW, CB = 4 * NW;   // four channels per wave
  template <int KS> using Cfg = ConvCfg<KS, CM_BWD, CM_SUB, CB, NW>;
};
template <int D, int GT, bool CONV>
__global__ __launch_bounds__((RowsCfg<D, GT>::NT), 2) void grouped_bwd_dq_kernel(GroupedBwdArgs a, ConvLongArgs c, int ndq) {
  using G = RowsCfg<D, GT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if constexpr (CONV) {
    if ((int)blockIdx.x >= ndq) {                          // uniform
      using R = RidingConv<D, GT>;
      const int per = (c.L + CM_SUB - 1) / CM_SUB * (D / R::CB), e = blockIdx.x - ndq, bx = e % per, by = e / per;
      uint32_t* smu = reinterpret_cast<uint32_t*>(smem);
      if (c.Kc <= 17) conv_mfma_workgroup<D, 1, CM_BWD, CM_SUB, R::CB, R::NW>(c, bx, by, smu);
      else if (c.Kc <= 49) conv_mfma_workgroup<D, 2, CM_BWD, CM_SUB, R::CB, R::NW>(c, bx, by, smu);
      else conv_mfma_workgroup<D, 3, CM_BWD, CM_SUB, R::CB, R::NW>(c, bx, by, smu);
      return;
    }
  }
  uint16_t* Kl = reinterpret_cast<uint16_t*>(smem);
  uint16_t* Vl = reinterpret_cast<uint16_t*>(smem + G::OFF_B);
  float* zl = reinterpret_cast<float*>(smem + G::OFF_Z);
  uint16_t* Sl = Kl;                                       // S_g, once the key rows are done with
  float* Ol = reinterpret_cast<float*>(smem);

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  int g, half;
  const int per_head = G::NH * a.ng;
  group_and_half<G::NH>(blockIdx.x % per_head, a.ng, G::NH - 1, g, half);   // the longer one (later queries, more keys) first
  const int bh = blockIdx.x / per_head, b = bh / a.H, h = bh % a.H;
  const int tok0 = g * GT, q0 = half * G::RC;
  const int nt = (a.L - tok0) < GT ? (a.L - tok0) : GT;
  if (q0 >= nt) return;                                    // uniform: no queries in this run
  const int nq = nt - q0 < G::RC ? nt - q0 : G::RC;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh + (int64_t)tok0 * a.st;
  const uint16_t* gq = static_cast<const uint16_t*>(a.q) + base + (int64_t)q0 * a.st;
  const uint16_t* gdo = static_cast<const uint16_t*>(a.dout) + base + (int64_t)q0 * a.st;
  const uint16_t* gk = static_cast<const uint16_t*>(a.k) + base;
  const uint16_t* gv = static_cast<const uint16_t*>(a.v) + base;
  uint16_t* gdq = static_cast<uint16_t*>(a.dq) + base + (int64_t)q0 * a.st;
  const float* slot = a.P + ((size_t)bh * a.ng + g) * G::SLOT;
  constexpr float to_log2 = kToLog2<D>;
  const float one = a.relu ? 0.f : 1.f;

  // this wave's queries and their incoming gradients as MFMA operands: lane % 16 = query, registers = features /
  // channels 32ks + 8 (lane / 16) + 0..7.  A query past the end reads the last row; it is never stored.
  const int tile[2] = {w, 2 * G::NW - 1 - w};
  RowLoad<D, GT> rows;
  rows.fetch(gk, gv, a.st, nt < G::RC ? nt : G::RC, tid);
  const uint16_t* qrow[2];
  u32x4 qop[2][G::KSD], dop[2][G::KSD];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int q = 16 * tile[n] + l16;
    const int64_t off = (int64_t)(q < nq ? q : nq - 1) * a.st;
    qrow[n] = gq + off;
#pragma unroll
    for (int ks = 0; ks < G::KSD; ++ks) {
      qop[n][ks] = *reinterpret_cast<const u32x4*>(qrow[n] + 32 * ks + 8 * g4);
      dop[n][ks] = *reinterpret_cast<const u32x4*>(gdo + off + 32 * ks + 8 * g4);
    }
  }

  // sc, dp [n][s][r]: key 32kt + 16s + 4 (lane / 16) + r, query 16 tile[n] + lane % 16; tiles N0 .. 1
  auto scores = [&](auto n0, int kt, f32x4 (&sc)[2][2], f32x4 (&dp)[2][2]) __attribute__((always_inline)) {
    constexpr int N0 = decltype(n0)::value;
#pragma unroll
    for (int n = N0; n < 2; ++n) sc[n][0] = sc[n][1] = dp[n][0] = dp[n][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ks = 0; ks < G::KSD; ++ks) {
        const bf16x8 ka = rows16(Kl, G::KS, 32 * kt + 16 * s, 32 * ks, lane);
        const bf16x8 va = rows16(Vl, G::KS, 32 * kt + 16 * s, 32 * ks, lane);
#pragma unroll
        for (int n = N0; n < 2; ++n) {
          sc[n][s] = mfma16(ka, __builtin_bit_cast(bf16x8, qop[n][ks]), sc[n][s]);
          dp[n][s] = mfma16(va, __builtin_bit_cast(bf16x8, dop[n][ks]), dp[n][s]);
        }
      }
  };
  using Both = std::integral_constant<int, 0>;
  using Second = std::integral_constant<int, 1>;
  // which tile has its own queries among the 32 keys of a unit (keys later than the query do not exist for it).  Groups of 64 are
  // two units, each some tile's own: the select in both tiles and one body for either unit is the faster way (us a gradient call, B4 H4 L15958
  // d128 787 / 777, B16 H8 L1000 356 / 351).
  using Whole = std::integral_constant<int, -1>;
  using First = std::integral_constant<int, 0>;
  using Each = std::integral_constant<int, 2>;

  // ---- pass 1: largest logit, sum of the weights and sum of e_i dp_i per query, of the keys that this lane holds (the four
  // lanes of a query are merged behind the loop).  The maximum starts from the lowest finite number: a lane may have met
  // only keys that do not exist for its query.
  float mtop[2] = {-3.402823466e38f, -3.402823466e38f}, mass[2] = {0.f, 0.f}, racc[2] = {0.f, 0.f};
  auto stats_unit = [&](auto n0, int kt, auto diag) __attribute__((always_inline)) {
    constexpr int N0 = decltype(n0)::value, DIAG = decltype(diag)::value;
    f32x4 sc[2][2], dp[2][2];
    scores(n0, kt, sc, dp);
#pragma unroll
    for (int n = N0; n < 2; ++n) {
      const int qi = 16 * tile[n] + l16;
      float mnew = mtop[n];
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (DIAG == 2 || n == DIAG) sc[n][s][r] = 32 * kt + 16 * s + 4 * g4 + r <= qi ? sc[n][s][r] : -INFINITY;
          mnew = fmaxf(mnew, sc[n][s][r]);
        }
      const float corr = __builtin_amdgcn_exp2f((mtop[n] - mnew) * to_log2);
      const float shift = -mnew * to_log2;
      float rs = 0.f, rd = 0.f;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float e = __builtin_amdgcn_exp2f(fmaf(sc[n][s][r], to_log2, shift));
          rs += e;
          rd = fmaf(e, dp[n][s][r], rd);
        }
      mass[n] = fmaf(mass[n], corr, rs);
      racc[n] = fmaf(racc[n], corr, rd);
      mtop[n] = mnew;
    }
  };
  // the units of one run of key rows: both tiles, then (on the diagonal) the later tile alone; every tile's last one is its own
  auto walk = [&](auto&& unit, bool diag) __attribute__((always_inline)) {
    int kt = 0;
    if constexpr (G::NH == 1) {                            // (the one run of a group is its own)
#pragma unroll 1
      for (; kt <= tile[0] / 2; ++kt) unit(Both{}, kt, Each{});
#pragma unroll 1
      for (; kt <= tile[1] / 2; ++kt) unit(Second{}, kt, Each{});
      return;
    }
    const int d0 = diag ? tile[0] / 2 : G::NW, d1 = tile[1] / 2;   // d0 < d1
#pragma unroll 1
    for (; kt < d0; ++kt) unit(Both{}, kt, Whole{});
    if (!diag) return;                                     // uniform
    unit(Both{}, kt++, First{});
#pragma unroll 1
    for (; kt < d1; ++kt) unit(Second{}, kt, Whole{});
    unit(Second{}, kt, Second{});
  };
  rows.put(Kl, Vl, nt < G::RC ? nt : G::RC, tid);
  __syncthreads();
  if (G::NH > 1 && half) {                                 // the next rows are under way while these are worked on
    rows.fetch(gk + (int64_t)G::RC * a.st, gv + (int64_t)G::RC * a.st, a.st, nq, tid);
    walk(stats_unit, false);
    __syncthreads();                                       // every wave is done with the rows before
    rows.put(Kl, Vl, nq, tid);
    __syncthreads();
  }
  walk(stats_unit, true);
  // p = exp2(x - mlog2) * inv_mass.  (The sum's logarithm as part of mlog2 saved a multiplication and a scalar and cost bits: mlog2
  // is the size of the logits, and what its rounding takes off has to be what it took off in the sum, where it cancels.  Logits of
  // 60 to 330: weights of 1 off by up to 5e-5, now 1e-7; a training step of B8 H8 L8192 d128 takes 0.2 % longer.)
  float mlog2[2], inv_mass[2], pbar[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    float top = fmaxf(mtop[n], __shfl_xor(mtop[n], 16));
    top = fmaxf(top, __shfl_xor(top, 32));
    const float corr = __builtin_amdgcn_exp2f((mtop[n] - top) * to_log2);
    float ms = mass[n] * corr, rc = racc[n] * corr;
    ms += __shfl_xor(ms, 16);
    rc += __shfl_xor(rc, 16);
    ms += __shfl_xor(ms, 32);
    rc += __shfl_xor(rc, 32);
    inv_mass[n] = 1.f / ms;                                // the token itself is always seen: the sum is at least 1
    pbar[n] = rc * inv_mass[n];
    mlog2[n] = top * to_log2;
  }

  // ---- pass 2: ds = p (dp - pbar), dQ^T += K^T ds^T (the 1 / sqrt(d) once, behind the loop) ----------------------
  // dqa[n][ft][r] = dQ[query 16 tile[n] + lane % 16][feature 16ft + 4 (lane / 16) + r]
  f32x4 dqa[2][G::CT];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int ft = 0; ft < G::CT; ++ft) dqa[n][ft] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto dq_unit = [&](auto n0, int kt, auto diag) __attribute__((always_inline)) {
    constexpr int N0 = decltype(n0)::value, DIAG = decltype(diag)::value;
    f32x4 sc[2][2], dp[2][2];
    scores(n0, kt, sc, dp);
    bf16x8 dh[2], dl[2];
#pragma unroll
    for (int n = N0; n < 2; ++n) {
      const int qi = 16 * tile[n] + l16;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // (the mask as a select on the exponent, exp2(-inf) = 0: a branch per element would cut the loop into pieces)
          float arg = fmaf(sc[n][s][r], to_log2, -mlog2[n]);
          if (DIAG == 2 || n == DIAG) arg = 32 * kt + 16 * s + 4 * g4 + r <= qi ? arg : -INFINITY;
          sc[n][s][r] = __builtin_amdgcn_exp2f(arg) * inv_mass[n] * (dp[n][s][r] - pbar[n]);
        }
      split44(sc[n][0], sc[n][1], dh[n], dl[n]);
    }
#pragma unroll
    for (int ft = 0; ft < G::CT; ++ft) {
      const bf16x8 ko = tr16_acc_order(Kl, G::KS, 32 * kt, 16 * ft, lane);
#pragma unroll
      for (int n = N0; n < 2; ++n) {
        dqa[n][ft] = mfma16(ko, dh[n], dqa[n][ft]);
        dqa[n][ft] = mfma16(ko, dl[n], dqa[n][ft]);
      }
    }
  };
  walk(dq_unit, true);
  if (G::NH > 1 && half) {                                 // (the first run's rows: all there, and in L2)
    rows.fetch(gk, gv, a.st, G::RC, tid);
    __syncthreads();
    rows.put(Kl, Vl, G::RC, tid);
    __syncthreads();
    walk(dq_unit, false);
  }

  // ---- the grouped branch: S_g -> LDS as bf16 [feature][channel], z_g -> LDS ------------------------------------
  constexpr int PARTS = D * D / 4 / G::NT > 16 ? D * D / 4 / G::NT / 16 : 1;
  SlotLoad<D, GT, PARTS> sums;
  sums.fetch(slot, tid);
  constexpr int ZN = (D + G::NT - 1) / G::NT;
  float zx[ZN];
#pragma unroll
  for (int i = 0; i < ZN; ++i) zx[i] = slot[D * D + (tid + G::NT * i) % D];
  u32x2 qx[2][G::CT];                                      // the query in the accumulator's order of features
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int ft = 0; ft < G::CT; ++ft) qx[n][ft] = *reinterpret_cast<const u32x2*>(qrow[n] + 16 * ft + 4 * g4);
  __syncthreads();                                         // every wave is done with the key and value rows
  sums.put(Sl, tid);
#pragma unroll
  for (int p = 1; p < PARTS; ++p) {
    sums.fetch(slot, tid, p);
    sums.put(Sl, tid, p);
  }
#pragma unroll
  for (int i = 0; i < ZN; ++i)
    if (tid + G::NT * i < D) zl[tid + G::NT * i] = zx[i];
  __syncthreads();
  // W[f][t] = sum_c S_g[f][c] dO[t][c]; den = phi(q).z + eps and nd = phi(q).W, both with phi(q) in fp32: f W and z dden
  // nearly cancel, so neither may carry the rounding of a bf16 phi(q)
  f32x4 wt[2][G::CT];
  float nd[2] = {0.f, 0.f}, dz[2] = {0.f, 0.f};
#pragma unroll
  for (int ft = 0; ft < G::CT; ++ft) {
    wt[0][ft] = wt[1][ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < G::KSD; ++ks) {
      const bf16x8 sh = rows16(Sl, G::KS, 16 * ft, 32 * ks, lane);
      const bf16x8 sl = rows16(Sl + D * G::KS, G::KS, 16 * ft, 32 * ks, lane);
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        wt[n][ft] = mfma16(sh, __builtin_bit_cast(bf16x8, dop[n][ks]), wt[n][ft]);
        wt[n][ft] = mfma16(sl, __builtin_bit_cast(bf16x8, dop[n][ks]), wt[n][ft]);
      }
    }
    const f32x4 zf = *reinterpret_cast<const f32x4*>(zl + 16 * ft + 4 * g4);
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const f32x4 qv = unpack4(qx[n][ft]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float f = phi_nb(qv[r], one);
        nd[n] = fmaf(f, wt[n][ft][r], nd[n]);
        dz[n] = fmaf(f, zf[r], dz[n]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);                     // (reads of later tiles moved up here would cost spills)
  }
  const size_t ntok = (size_t)a.B * a.H * a.L;
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    nd[n] += __shfl_xor(nd[n], 16);
    dz[n] += __shfl_xor(dz[n], 16);
    nd[n] += __shfl_xor(nd[n], 32);
    dz[n] += __shfl_xor(dz[n], 32);
    const float gden = dz[n] + a.eps;
    const float fscale = gden != 0.f ? a.alpha / gden : 0.f;   // nothing before the group: no branch
    const float dden = gden != 0.f ? -fscale * nd[n] / gden : 0.f;
#pragma unroll
    for (int ft = 0; ft < G::CT; ++ft) {
      // (opaque, so that the exponentials above are made again here: kept, they would be spilled)
      asm volatile("" : "+v"(qx[n][ft]));
      const f32x4 qv = unpack4(qx[n][ft]);
      const f32x4 zf = *reinterpret_cast<const f32x4*>(zl + 16 * ft + 4 * g4);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        dqa[n][ft][r] = fmaf(fmaf(fscale, wt[n][ft][r], zf[r] * dden), dphi_nb(qv[r], one), dqa[n][ft][r] * kInvSqrt<D>);
    }
    // the per-token scalars for the kernels that follow
    const int q = 16 * tile[n] + l16;
    if (g4 == 0 && q < nq) {
      const size_t e = (size_t)bh * a.L + tok0 + q0 + q;
      a.stats[e] = mlog2[n];
      a.stats[ntok + e] = inv_mass[n];
      a.stats[2 * ntok + e] = pbar[n];
      a.stats[3 * ntok + e] = fscale;
      a.stats[4 * ntok + e] = dden;
    }
  }
  const HeldRows<D, GT> none{};
  store_rows<D, GT, false>(dqa, none, Ol, gdq, a.st, nq, tid, tile, lane);
}

// ---- dk, dv ---------------------------------------------------------------------------------------------------------
// Elements NT block .. NT block + NT - 1 of the tap gradient: the partial sums of the token blocks, 32 at a time and those
// sums in turn, the order of the stages of grouped_bwd_dw_reduce_kernel (two of them: dw_sums_ride).
template <int NT>
__device__ __forceinline__ void dw_sums(const GroupedBwdArgs& a, int d, int block) {
  const int e = block * NT + threadIdx.x, per_head = d * a.Kc, n = a.B * a.nwb;
  if (e >= a.H * per_head) return;
  const float* p = a.dw_part + (size_t)(e / per_head) * n * per_head + e % per_head;
  float sum = 0.f;
  for (int i0 = 0; i0 < n; i0 += 32) {
    float x[32], s = 0.f;                                  // every request before the first sum; past the end the last one again, not used
#pragma unroll
    for (int i = 0; i < 32; ++i) x[i] = p[(size_t)(i0 + i < n ? i0 + i : n - 1) * per_head];
#pragma unroll
    for (int i = 0; i < 32; ++i) s = i0 + i < n ? s + x[i] : s;
    sum += s;
  }
  a.dconv_w[e] = sum;
}

// SPLIT: dk and dv in workgroups of their own (see split_pays); otherwise both from one pass over the scores.
template <int D, int GT, bool SPLIT>
__global__ __launch_bounds__((RowsCfg<D, GT>::NT), 2) void grouped_bwd_dkdv_kernel(GroupedBwdArgs a) {
  using G = RowsCfg<D, GT>;
  if ((int)blockIdx.y >= a.B * a.H) {                      // uniform: the sums of the tap gradient ride along
    dw_sums<G::NT>(a, D, ((blockIdx.y - a.B * a.H) * gridDim.z + blockIdx.z) * gridDim.x + blockIdx.x);
    return;
  }
  const bool with_dv = !SPLIT || blockIdx.z != 0, with_dk = !SPLIT || blockIdx.z == 0;   // uniform
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* Ql = reinterpret_cast<uint16_t*>(smem);
  uint16_t* Dl = reinterpret_cast<uint16_t*>(smem + G::OFF_B);
  float* zl = reinterpret_cast<float*>(smem + G::OFF_Z);
  float* ml = reinterpret_cast<float*>(smem + G::OFF_ST);  // largest logit (log2 units), 1 / sum, pbar per query
  float* il = ml + G::RC;
  float* pl = il + G::RC;
  uint16_t* Sl = Ql;                                       // D_g, once the token rows are done with
  float* Ol = reinterpret_cast<float*>(smem);

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  int g, half;
  group_and_half<G::NH>(blockIdx.x, a.ng, 0, g, half);     // the longer one (earlier keys, more queries) first
  const int bh = blockIdx.y, b = bh / a.H, h = bh % a.H;
  const int tok0 = g * GT, k0 = half * G::RC;
  const int nt = (a.L - tok0) < GT ? (a.L - tok0) : GT;
  if (k0 >= nt) return;                                    // uniform: no keys in this run
  const int nk = nt - k0 < G::RC ? nt - k0 : G::RC;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh + (int64_t)tok0 * a.st;
  const uint16_t* gq = static_cast<const uint16_t*>(a.q) + base;
  const uint16_t* gdo = static_cast<const uint16_t*>(a.dout) + base;
  const uint16_t* gk = static_cast<const uint16_t*>(a.k) + base + (int64_t)k0 * a.st;
  const uint16_t* gv = static_cast<const uint16_t*>(a.v) + base + (int64_t)k0 * a.st;
  uint16_t* gdk = static_cast<uint16_t*>(a.dk) + base + (int64_t)k0 * a.st;
  uint16_t* gdv = static_cast<uint16_t*>(a.dv) + base + (int64_t)k0 * a.st;
  const float* slot = a.Dg + ((size_t)bh * a.ng + g) * G::SLOT;
  const size_t ntok = (size_t)a.B * a.H * a.L, e0 = (size_t)bh * a.L + tok0;
  constexpr float to_log2 = kToLog2<D>;
  const float one = a.relu ? 0.f : 1.f;

  // this wave's keys and their values as MFMA operands: lane % 16 = key, registers = features 32ks + 8 (lane / 16) + 0..7
  const int tile[2] = {w, 2 * G::NW - 1 - w};
  RowLoad<D, GT> rows;
  rows.fetch(gq + (int64_t)k0 * a.st, gdo + (int64_t)k0 * a.st, a.st, nk, tid);
  // the scalars of queries r0 .. r0 + RC - 1 (queries past the end weigh nothing)
  static_assert(G::RC <= G::NT, "one thread per query");
  float s0 = 0.f, s1 = 0.f, s2 = 0.f;
  auto fetch_scalars = [&](int r0, int nr) __attribute__((always_inline)) {
    const size_t e = e0 + r0 + (tid < nr ? tid : nr - 1);
    s0 = a.stats[e];
    s1 = a.stats[ntok + e];
    s2 = a.stats[2 * ntok + e];
  };
  auto put_scalars = [&](int nr) __attribute__((always_inline)) {
    if (tid < G::RC) {
      ml[tid] = tid < nr ? s0 : 0.f;
      il[tid] = tid < nr ? s1 : 0.f;
      pl[tid] = tid < nr ? s2 : 0.f;
    }
  };
  fetch_scalars(k0, nk);
  int64_t koff[2];
  u32x4 kop[2][G::KSD], vop[2][G::KSD];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int t = 16 * tile[n] + l16;
    koff[n] = (int64_t)(t < nk ? t : nk - 1) * a.st;
#pragma unroll
    for (int ks = 0; ks < G::KSD; ++ks) {
      kop[n][ks] = *reinterpret_cast<const u32x4*>(gk + koff[n] + 32 * ks + 8 * g4);
      vop[n][ks] = *reinterpret_cast<const u32x4*>(gv + koff[n] + 32 * ks + 8 * g4);
    }
  }
  // dka, dva [n][ct][r] = dK, dV [key 16 tile[n] + lane % 16][column 16ct + 4 (lane / 16) + r]
  f32x4 dkb[2][G::CT], dva[2][G::CT];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int ct = 0; ct < G::CT; ++ct) dkb[n][ct] = dva[n][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 (&dka)[2][G::CT] = SPLIT ? dva : dkb;              // (a workgroup with one of them has one set of accumulators)

  // 32 queries against tiles 0 .. N1 - 1; DIAG: the tile that has its own tokens among them (queries earlier than the key do
  // not see it)
  auto unit = [&](auto n1, int qt, auto diag) __attribute__((always_inline)) {
    constexpr int N1 = decltype(n1)::value, DIAG = decltype(diag)::value;
    f32x4 sc[2][2], dp[2][2];                              // [n][s][r]: query 32qt + 16s + 4 (lane / 16) + r, key lane % 16
    auto product = [&](const uint16_t* rl, const u32x4 (&op)[2][G::KSD], f32x4 (&x)[2][2]) __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < N1; ++n) x[n][0] = x[n][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int ks = 0; ks < G::KSD; ++ks) {
          const bf16x8 ra = rows16(rl, G::KS, 32 * qt + 16 * s, 32 * ks, lane);
#pragma unroll
          for (int n = 0; n < N1; ++n) x[n][s] = mfma16(ra, __builtin_bit_cast(bf16x8, op[n][ks]), x[n][s]);
        }
    };
    // X^T += rows^T p, p as hi + lo
    auto gather = [&](const uint16_t* rl, const f32x4 (&p)[2][2], f32x4 (&x)[2][G::CT]) __attribute__((always_inline)) {
      bf16x8 ph[2], pw[2];
#pragma unroll
      for (int n = 0; n < N1; ++n) split44(p[n][0], p[n][1], ph[n], pw[n]);
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct) {
        const bf16x8 rt = tr16_acc_order(rl, G::KS, 32 * qt, 16 * ct, lane);
#pragma unroll
        for (int n = 0; n < N1; ++n) x[n][ct] = mfma16(rt, ph[n], x[n][ct]);
#pragma unroll
        for (int n = 0; n < N1; ++n) x[n][ct] = mfma16(rt, pw[n], x[n][ct]);
      }
    };
    product(Ql, kop, sc);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int t0 = 32 * qt + 16 * s + 4 * g4;
      const f32x4 mt = *reinterpret_cast<const f32x4*>(ml + t0), it = *reinterpret_cast<const f32x4*>(il + t0);
#pragma unroll
      for (int n = 0; n < N1; ++n) {
        const int ki = 16 * tile[n] + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float x = fmaf(sc[n][s][r], to_log2, -mt[r]);
          sc[n][s][r] = __builtin_amdgcn_exp2f((DIAG != 2 && n != DIAG) || t0 + r >= ki ? x : -INFINITY) * it[r];
        }
      }
    }
    if (with_dv) gather(Dl, sc, dva);                      // dV^T += dO^T P
    if (with_dk) {
      product(Dl, vop, dp);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const f32x4 pb = *reinterpret_cast<const f32x4*>(pl + 32 * qt + 16 * s + 4 * g4);
#pragma unroll
        for (int n = 0; n < N1; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) dp[n][s][r] = sc[n][s][r] * (dp[n][s][r] - pb[r]);
      }
      gather(Ql, dp, dka);                                 // dK^T += Q^T ds (the 1 / sqrt(d) once, behind the loop)
    }
  };
  using One = std::integral_constant<int, 1>;
  using Both = std::integral_constant<int, 2>;
  using Whole = std::integral_constant<int, -1>;
  using First = std::integral_constant<int, 0>;
  using Second = std::integral_constant<int, 1>;
  using Each = std::integral_constant<int, 2>;             // (groups of 64: as in the dq kernel)
  auto walk = [&](int nr, bool diag) __attribute__((always_inline)) {
    const int nqt = (nr + 31) / 32, d0 = tile[0] / 2, d1 = tile[1] / 2;   // d0 < d1
    int qt = 0;
    if constexpr (G::NH == 1) {
#pragma unroll 1
      for (qt = d0; qt < (d1 < nqt ? d1 : nqt); ++qt) unit(One{}, qt, Each{});
#pragma unroll 1
      for (; qt < nqt; ++qt) unit(Both{}, qt, Each{});
      return;
    }
    if (diag) {                                            // uniform
      qt = d0;
      if (qt < nqt) unit(One{}, qt++, First{});
#pragma unroll 1
      for (; qt < (d1 < nqt ? d1 : nqt); ++qt) unit(One{}, qt, Whole{});
      if (d1 < nqt) unit(Both{}, qt++, Second{});
    }
#pragma unroll 1
    for (; qt < nqt; ++qt) unit(Both{}, qt, Whole{});
  };
  put_scalars(nk);
  rows.put(Ql, Dl, nk, tid);
  __syncthreads();
  walk(nk, true);
  if (G::NH > 1 && half == 0 && nt > G::RC) {              // uniform: the later queries
    constexpr int PARTS = SPLIT ? 1 : 2;                   // what fits beside the accumulators (almost: with both sets of them
                                                           // 34 registers spill at D = 128, 30 in groups of 64)
    RowLoad<D, GT, PARTS> more;
    const int nr = nt - G::RC;
    const uint16_t *gq1 = gq + (int64_t)G::RC * a.st, *gdo1 = gdo + (int64_t)G::RC * a.st;
    more.fetch(gq1, gdo1, a.st, nr, tid, 0);
    fetch_scalars(G::RC, nr);
    __syncthreads();                                       // every wave is done with the rows before
    put_scalars(nr);
    more.put(Ql, Dl, nr, tid, 0);
#pragma unroll
    for (int p = 1; p < PARTS; ++p) {
      more.fetch(gq1, gdo1, a.st, nr, tid, p);
      more.put(Ql, Dl, nr, tid, p);
    }
    __syncthreads();
    walk(nr, false);
  }
  if (with_dk)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct) dka[n][ct] *= kInvSqrt<D>;

  // ---- the group's keys and values entered the sums every later group read ---------------------------------------
  if (g + 1 < a.ng) {                                      // uniform; after the last group nothing reads the sums
    constexpr int PARTS = D * D / 4 / G::NT > 8 ? D * D / 4 / G::NT / 8 : 1;   // what fits beside the accumulators
    SlotLoad<D, GT, PARTS> sums;
    sums.fetch(slot, tid, 0);
    __syncthreads();                                       // every wave is done with the query and gradient rows
    sums.put(Sl, tid, 0);
#pragma unroll
    for (int p = 1; p < PARTS; ++p) {
      sums.fetch(slot, tid, p);
      sums.put(Sl, tid, p);
    }
    for (int f = tid; f < D; f += G::NT) zl[f] = slot[D * D + f];
    u32x2 kx[2][G::CT];                                    // the key in the accumulator's order of features
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int ft = 0; ft < G::CT; ++ft) kx[n][ft] = *reinterpret_cast<const u32x2*>(gk + koff[n] + 16 * ft + 4 * g4);
    __syncthreads();
    if (with_dv) {
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int ks = 0; ks < G::KSD; ++ks) kop[n][ks] = phi_pack8_nb(kop[n][ks], one);
#pragma unroll
      for (int ct = 0; ct < G::CT; ++ct) {                   // dV^T += D.S^T phi(K)^T
#pragma unroll
        for (int ks = 0; ks < G::KSD; ++ks) {
          const bf16x8 sh = tr16(Sl, G::KS, 32 * ks, 16 * ct, lane);
          const bf16x8 sl = tr16(Sl + D * G::KS, G::KS, 32 * ks, 16 * ct, lane);
#pragma unroll
          for (int n = 0; n < 2; ++n) dva[n][ct] = mfma16(sh, __builtin_bit_cast(bf16x8, kop[n][ks]), dva[n][ct]);
#pragma unroll
          for (int n = 0; n < 2; ++n) dva[n][ct] = mfma16(sl, __builtin_bit_cast(bf16x8, kop[n][ks]), dva[n][ct]);
        }
        if (ct % 2) __builtin_amdgcn_sched_barrier(0);       // (reads of later tiles moved up here would cost spills)
      }
    }
    if (with_dk) {
#pragma unroll
      for (int ft = 0; ft < G::CT; ++ft) {                   // dK += (D.S V^T + D.z) * phi'(K)
        f32x4 lin[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < G::KSD; ++ks) {
          const bf16x8 sh = rows16(Sl, G::KS, 16 * ft, 32 * ks, lane);
          const bf16x8 sl = rows16(Sl + D * G::KS, G::KS, 16 * ft, 32 * ks, lane);
#pragma unroll
          for (int n = 0; n < 2; ++n) {
            lin[n] = mfma16(sh, __builtin_bit_cast(bf16x8, vop[n][ks]), lin[n]);
            lin[n] = mfma16(sl, __builtin_bit_cast(bf16x8, vop[n][ks]), lin[n]);
          }
        }
        const f32x4 zf = *reinterpret_cast<const f32x4*>(zl + 16 * ft + 4 * g4);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const f32x4 kv = unpack4(kx[n][ft]);
#pragma unroll
          for (int r = 0; r < 4; ++r) dka[n][ft][r] = fmaf(lin[n][r] + zf[r], dphi_nb(kv[r], one), dka[n][ft][r]);
        }
        if (ft % 2) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // dk is written; dv is added to what the conv's share left there (written ahead of this kernel)
  HeldRows<D, GT> held;
  if (with_dv) hold_rows<D, GT>(held, gdv, a.st, nk, tid);
  if (with_dk) store_rows<D, GT, false>(dka, held, Ol, gdk, a.st, nk, tid, tile, lane);
  if (with_dv) store_rows<D, GT, true>(dva, held, Ol, gdv, a.st, nk, tid, tile, lane);
}

namespace {
// dk and dv in workgroups of their own: twice the workgroups, each with half of the products and none of the other half's
// accumulators, but the scores computed twice.  Pays while all of them fit the chip at once (two to a CU) and the extra ones
// take CUs that would stand idle.  Measured, us a gradient call as a graph, together / apart, by workgroups: D = 128, groups of 64: 64
// 61.5 / 53.1, 128 65.9 / 57.6, 256 83.6 / 79.2, 320 102.0 / 100.3 and 77.4 / 76.1, 400 95.8 / 96.6; groups of 256: 64 79.0 / 66.2, 128 94.0 /
// 86.3, 256 109 / 101, 320 80.5 / 79.3, 384 64.7 / 63.4, 512 76.5 / 78.5.  D = 64, where a workgroup is short: groups of 64: 64 29.6 /
// 28.3, 128 35.7 / 35.8, 256 40.2 / 40.2; groups of 256: 32 36.4 / 34.6, 64 47.3 / 45.6, 96 52.5 / 53.2, 128 51.2 / 52.2, 256 25.2 / 25.7: up to 64
// it pays, from there to the line neither way is ahead by more than 2 %.
template <int D>
bool split_pays(int64_t wgs) { return wgs <= (D == 128 ? 256 : 128); }

template <int D, int GT>
int riding_blocks(const GroupedBwdArgs& a) {
  return (a.L + CM_SUB - 1) / CM_SUB * (D / RidingConv<D, GT>::CB) * a.B * a.H;
}

template <int D, int GT>
hipError_t launch_rows(const GroupedBwdArgs& a, const ConvLongArgs* conv, bool keys, hipStream_t st) {
  using G = RowsCfg<D, GT>;
  using R = RidingConv<D, GT>;
  hipError_t e;
  const int runs = G::NH * a.ng * a.B * a.H;
  if (!keys && !conv) {
    auto kq = grouped_bwd_dq_kernel<D, GT, false>;
    if ((e = LINATTN_MAX_LDS_ONCE(kq, G::TOTAL)) != hipSuccess) return e;
    hipLaunchKernelGGL(kq, dim3((unsigned)runs), dim3(G::NT), G::TOTAL, st, a, ConvLongArgs{}, runs);
  } else if (!keys) {
    constexpr int conv_bytes = 4 * (R::template Cfg<3>::TOTAL > R::template Cfg<2>::TOTAL ? R::template Cfg<3>::TOTAL : R::template Cfg<2>::TOTAL);
    static_assert(conv_bytes <= G::TOTAL && R::template Cfg<1>::TOTAL * 4 <= G::TOTAL, "the conv's workgroups in the rows' LDS");
    auto kq = grouped_bwd_dq_kernel<D, GT, true>;
    if ((e = LINATTN_MAX_LDS_ONCE(kq, G::TOTAL)) != hipSuccess) return e;
    hipLaunchKernelGGL(kq, dim3((unsigned)(runs + riding_blocks<D, GT>(a))), dim3(G::NT), G::TOTAL, st, a, *conv, runs);
  } else {
    const bool split = split_pays<D>(runs);
    auto kk = grouped_bwd_dkdv_kernel<D, GT, false>;
    auto k2 = grouped_bwd_dkdv_kernel<D, GT, true>;
    if ((e = split ? LINATTN_MAX_LDS_ONCE(k2, G::TOTAL) : LINATTN_MAX_LDS_ONCE(kk, G::TOTAL)) != hipSuccess) return e;
    dim3 grid((unsigned)(G::NH * a.ng), (unsigned)(a.B * a.H), split ? 2 : 1);
    if (conv && a.dconv_w && dw_sums_ride(a)) {
      const unsigned blocks = (unsigned)((a.H * D * a.Kc + G::NT - 1) / G::NT);
      grid.y += (blocks + grid.x * grid.z - 1) / (grid.x * grid.z);
    }
    hipLaunchKernelGGL(split ? k2 : kk, grid, dim3(G::NT), G::TOTAL, st, a);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_grouped_bwd_rows(const GroupedBwdArgs& a, const ConvLongArgs* conv, int d, bool keys, hipStream_t st) {
  if (d == 128) return a.group == 256 ? launch_rows<128, 256>(a, conv, keys, st) : launch_rows<128, 64>(a, conv, keys, st);
  return a.group == 256 ? launch_rows<64, 256>(a, conv, keys, st) : launch_rows<64, 64>(a, conv, keys, st);
}

// The conv's workgroups in the dq launch and the sums of the tap gradient in the dk / dv launch, instead of launches of their
// own on a side stream.  Calls that do not fill the chip gain: the events that fork and join the stream cost the host 40 us, more
// than such a call's work, and in the dq launch the conv costs the GPU next to nothing.  Where the rows' workgroups fill the chip by
// themselves, the conv in its own shape (four waves, more channels: memory lines shared) is the better one, more so against the two
// waves of groups of 64.  us a gradient call as a graph (in brackets: as plain calls, where the host's share differs), side stream /
// riding, by runs of queries:
//   groups of 256, d = 128: 64 57.8 / 45.4 (68 / 46), 512 138 / 136, 768 223 / 216 and 196 / 197, 1000 303 / 301, 1024 235 / 242
//   and 274 / 270; d = 64: 64 30.1 / 20.9 (76 / 23), 1024 119 / 110, 2048 205 / 198, 2560 254 / 254 and 301 / 286
//   groups of 64, d = 128: 128 68 / 61 (82 / 62), 256 63 / 60, 314 114 / 106, 320 81 / 81 and 85 / 88, 384 86 / 89, 448 95 / 104,
//   512 98 / 106 and 118 / 124; d = 64: 256 49 / 40 (80 / 40), 768 60.7 / 56.0 and 71.9 / 72.1 (91 / 72), 896 77 / 80 and 65 / 63
//   (89 / 80 and 90 / 63), 1000 102 / 106 (101 / 106), 1024 81 / 86 (92 / 87)
// A workgroup of the conv takes a tile of 256 tokens, whatever the sequence has of them: in groups of 64 at d = 128, where 16 of them
// (two waves, eight channels each) go to a head's tile, many short sequences are the conv's call, not the rows': 64 tokens, 128
// heads 47.3 / 43.1, 160 49.5 / 50.1, 240 58 / 68, 320 72 / 88.
bool conv_rides(const GroupedBwdArgs& a, int d) {
  if (conv_mfma_blocks(a.L, a.B * a.H, d) != (a.L + CM_SUB - 1) / CM_SUB) return false;   // (two tiles per workgroup: calls that fill the chip)
  const int run = a.group < 128 ? a.group : 128;
  const int64_t heads = (int64_t)a.B * a.H, runs = (a.L + run - 1) / run * heads;
  if (a.group == 64 && d == 128 && (a.L + CM_SUB - 1) / CM_SUB * heads > 160) return false;
  return runs <= (a.group == 256 ? (d == 128 ? 768 : 2560) : (d == 128 ? 320 : 896));
}

// The sums over the partial sums are one chain per thread, 32 of them a step: beyond 384 it outlasts the rows, and launches that
// deal the partial sums out over workgroups are the faster way.  us a gradient call as a graph, launches / riding, by partial sums
// (batch rows times token blocks): d = 64: groups of 256: 256 43 / 39, 512 67 / 71, 1024 107 / 123, 2560 257 / 321; groups of 64:
// 384 61.7 / 58.4, 512 39.2 / 43.2; d = 128, groups of 256: 400 157 / 151, 512 141 / 141, 800 199 / 200.  (Eight at a time, and
// riding at any number: 2560 403.)
bool dw_sums_ride(const GroupedBwdArgs& a) { return (int64_t)a.B * a.nwb <= 384; }

}  // namespace linattn
