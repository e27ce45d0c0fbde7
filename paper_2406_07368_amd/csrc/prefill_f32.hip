// Prefill of fp32 rows on the fp32 matrix instructions (v_mfma_f32_32x32x2: exact fp32 products, fp32 sums), both forms
// of Sec. 4.1: the token-level form and the three-branch form in groups of 64 tokens.
//
// One workgroup per (b, h, value block[, segment]), D / 32 waves, 32 tokens per step.  Wave w owns the value channels
// 32w .. 32w+31: its column block of S stays in accumulator registers for the whole walk (lane = channel, registers =
// features) and is the right operand of phi(Q) S as it is -- an accumulator register holds features
// 8(r/4) + 4(lane/32) + r%4, which is a legal pair of contraction indices for one 32x32x2 step, and the left operand is
// read from LDS in the same order.  The same order serves P V: the scores are computed with keys in the rows of the
// accumulator, so they are the left operand of P V without passing through LDS again.
//   scores     the contraction over features is dealt out over the waves (32 features each); the partial tiles meet in
//              LDS, together with the partial sums of phi(q).z
//   outputs    O = phi(Q) S + P V in one accumulator (lane = channel, registers = tokens), normalised and with the conv
//              taps added from the V rows in LDS, stored as whole 128-byte row pieces
//   state      S += phi(K)^T V, z += column sums of phi(K)
//
// What bounds it: the fp32 matrix rate (160 instructions of 64 cycles per wave, step and SIMD at D = 128), and for short
// sequences the latency of a step, about 3 us.  Sequences are cut into segments when the heads alone do not fill the
// chip: three launches (state-only pass, prefix sum, full pass).  Short sequences on few heads take the quadratic kernel
// below instead, which has no serial chain.  Measured (us a call, launches queued; before: one workgroup per head on the
// vector ALUs): B1 H4 L1024 D64 26 (1160 before), B2 H32 L1024 D128 118 (4190); the three-branch form 36 (2830) and 148 (6490).
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

#include <type_traits>

namespace linattn {

namespace {
constexpr int FT = 32;                       // tokens per step
constexpr int FGROUP = 64;                   // tokens per group of the three-branch form: two steps

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
// phi for fp32 rows: the map of the fp32 generation step (under elu + 1 a NaN stays one), without a branch on the feature
// map: one = 1 for elu + 1 and 0 for max(x, 0), whose lower branch is 0 whatever x is.
__device__ __forceinline__ float phi_f32(float x, float one) {
  const uint32_t keep = one != 0.f ? 0xffffffffu : 0u;
  const float e = __uint_as_float(__float_as_uint(__expf(x)) & keep);
  return x > 0.f ? x + one : e;
}
// row of accumulator register r in a lane of half hi
__device__ __forceinline__ constexpr int acc_row(int r, int hi) { return 8 * (r >> 2) + 4 * hi + (r & 3); }

// Values that are not finite.  In the tile that holds the queries themselves a key later than the query has weight 0, but 0
// times an infinity or a NaN is a NaN in an earlier token's output.  The products therefore take the largest finite numbers
// in the place of such values, and what the values themselves give the queries that see them is added behind a tile, key by
// key; weights are not negative, so what the replacement has added of itself has the infinity's sign (or meets a NaN).
// (A branch behind the products: ahead of them it would keep the requests of a tile from being spread over the products
// before, and cost spills.)  t becomes a NaN with the first such value.
__device__ __forceinline__ float finite_part(float v, float& t) {
  t = fmaf(v, 0.f, t);
  return __builtin_amdgcn_fmed3f(v, -3.402823466e38f, 3.402823466e38f);
}
// w: the key's weights by query; v: the key's value in this lane's channel; o[r]: query acc_row(r) of the tile, `seen` of
// them on see the key.
__device__ __forceinline__ void add_non_finite(const float* w, float v, int seen, f32x16& o, int hi) {
  const bool is = !__builtin_isfinite(v);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 w4 = *reinterpret_cast<const f32x4*>(w + 8 * g + 4 * hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[4 * g + e] = is && 8 * g + 4 * hi + e >= seen ? fmaf(w4[e], v, o[4 * g + e]) : o[4 * g + e];
  }
}

template <int D, bool GROUPED>
struct F32Cfg {
  static constexpr int NW = D / 32, NT = 64 * NW;
  static constexpr int ST = D + 8;                         // row stride in floats: 16-byte row reads of 8 rows, and 4-byte
                                                           // reads of two rows 4 apart, hit different banks
  static constexpr int KROWS = GROUPED ? FGROUP : FT;      // the rows of the step, or of the group
  static constexpr int TILES = GROUPED ? 2 : 1;            // key tiles a query tile meets
  static constexpr int Q = 0;                              // [FT][ST]
  static constexpr int K = Q + FT * ST;                    // [KROWS][ST]
  static constexpr int V = K + KROWS * ST;                 // [HALO + KROWS][ST]
  static constexpr int P = V + (HALO + KROWS) * ST;        // [TILES][NW][1024] partial score tiles, accumulator order
  static constexpr int PZ = P + TILES * NW * 1024;         // [NW][32] partial phi(q).z
  static constexpr int ZZ = PZ + NW * 32;                  // [D]; features 32w.. belong to wave w
  static constexpr int SC = ZZ + D;                        // [NW][2][32] per-token factors, one copy per wave
  static constexpr int TOTAL = SC + NW * 64;
  static constexpr int SLOT = D * D + D;
};
}  // namespace

template <int D, int KCM, bool STATE_ONLY, bool GROUPED>
__global__ __launch_bounds__(2 * D, GROUPED ? 1 : 2) void prefill_f32_kernel(PrefillArgs a) {
  using G = F32Cfg<D, GROUPED>;
  constexpr int NW = G::NW, NT = G::NT, ST = G::ST, IB = D / 32;
  extern __shared__ __attribute__((aligned(16))) float smf[];
  float* Ql = smf + G::Q;
  float* Kl = smf + G::K;
  float* Vl = smf + G::V;
  float* Pp = smf + G::P;
  float* Pz = smf + G::PZ;
  float* zl = smf + G::ZZ;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const int seg = blockIdx.y;                              // (heads along x: there may be more of them than y can count)
  const HeadIndex hx = head_index(a, blockIdx.x, D);       // one (b, h, value block)
  const int L = a.L, Kc = a.Kc;
  const int t_beg = seg * a.seg_len;
  const int t_end = (L - t_beg) < a.seg_len ? L : t_beg + a.seg_len;
  const float one = a.relu ? 0.f : 1.f;
  const float* gq = static_cast<const float*>(a.q) + (int64_t)hx.b * a.sb + (int64_t)hx.h * a.sh;
  const float* gk = static_cast<const float*>(a.k) + (int64_t)hx.b * a.sb + (int64_t)hx.h * a.sh;
  const int64_t base_v = (int64_t)hx.b * a.sb_v + (int64_t)hx.h * a.sh_v + (int64_t)hx.blk * D;
  const float* gv = static_cast<const float*>(a.v) + base_v;
  float* go = static_cast<float*>(a.out) + base_v;
  const int64_t S_base = (int64_t)hx.bh * D * hx.dvt + (int64_t)hx.blk * D;
  const int64_t hist_base = (int64_t)hx.bh * (Kc - 1) * hx.dvt + (int64_t)hx.blk * D;
  const bool slots = a.nseg > 1;                           // start states come from the workspace
  float* slot = slots ? a.ws + ((size_t)hx.bhs * a.nseg + seg) * G::SLOT : nullptr;
  const int ch = 32 * w + l32;                             // this lane's value channel

  // ---- start state: S[f][ch] of the wave's channels, z of its features ---------------------------------------
  f32x16 Sa[IB];
  float zr = 0.f;                                          // z[32w + l32], in both halves of the wave
  if (STATE_ONLY || (!slots && !a.S_in)) {
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) Sa[ib][r] = 0.f;
  } else {
    const float* src = slots ? slot : a.S_in + S_base;
    const int row = slots ? D : hx.dvt;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) Sa[ib][r] = src[(size_t)(32 * ib + acc_row(r, hi)) * row + ch];
    zr = slots ? slot[D * D + ch] : a.z_in[(size_t)hx.bh * D + ch];
  }
  if (hi == 0) zl[ch] = zr;

  const int taps = a.no_conv ? 0 : Kc;
  float wreg[KCM];
#pragma unroll
  for (int j = 0; j < KCM; ++j) wreg[j] = 0.f;
  if (!STATE_ONLY && !a.no_conv) {
    const float* wp = a.conv_w + ((size_t)hx.h * hx.dvt + hx.blk * D + ch) * Kc;
#pragma unroll
    for (int j = 0; j < KCM; ++j) {
      const float x = wp[j < Kc ? j : 0];
      wreg[j] = j < Kc ? x : 0.f;
    }
  }

  // a thread's pieces of 32 rows: 16 bytes of rows tid / (D/4) + 8i
  constexpr int RPI = NT / (D / 4);                        // rows per pass: 8
  static_assert(RPI == 8 && HALO == 8, "pieces per thread");
  const int pr = tid / (D / 4), pc = 4 * (tid % (D / 4));
  f32x4 xq[4], xk[4], xv[4];
  auto request = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tok = t0 + pr + RPI * i;
      const int64_t t = tok < L ? tok : L - 1;             // unconditional; what does not exist is replaced by zeros
      xk[i] = *reinterpret_cast<const f32x4*>(gk + t * a.st + pc);
      xv[i] = *reinterpret_cast<const f32x4*>(gv + t * a.st_v + pc);
      if constexpr (!STATE_ONLY) xq[i] = *reinterpret_cast<const f32x4*>(gq + t * a.st + pc);
    }
  };

  // The eight value rows before the first token go where the loop looks for the tail of the previous rows.
  {
    const int tok = t_beg - HALO + pr;                    // t_beg = 0 or a multiple of 32
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
    if (tok >= 0 && t_beg < L) y = *reinterpret_cast<const f32x4*>(gv + (int64_t)tok * a.st_v + pc);
    else if (tok < 0 && a.hist_in && Kc - 1 + tok >= 0)
      y = slots ? *reinterpret_cast<const f32x4*>(a.ws + (size_t)a.B * a.H * a.m * a.nseg * G::SLOT + ((size_t)hx.bhs * HALO + pr) * D + pc)
                : *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.hist_in) + hist_base + (int64_t)(Kc - 1 + tok) * hx.dvt + pc);
    *reinterpret_cast<f32x4*>(Vl + (G::KROWS + pr) * ST + pc) = y;
  }
  if (t_beg < t_end) request(t_beg);
  __syncthreads();

  float vr[16];                                            // V[acc_row(r)][ch] of the rows at hand
  auto value_regs = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) vr[r] = Vl[(HALO + 32 * p + acc_row(r, hi)) * ST + ch];
  };
  // S += phi(K)^T V and z += sum of phi(K) over the 32 rows of half p (n of them exist)
  auto add_keys = [&](int p, int n) __attribute__((always_inline)) {
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      float zs = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float x = Kl[(32 * p + acc_row(r, hi)) * ST + 32 * ib + l32];
        if constexpr (GROUPED) {                           // raw rows
          x = phi_f32(x, one);
          x = acc_row(r, hi) < n ? x : 0.f;
        }
        Sa[ib] = mfma32(x, vr[r], Sa[ib]);
        zs += x;
      }
      if (ib == w) zr += zs + __shfl_xor(zs, 32);          // uniform
    }
  };

  static_assert(D == 64 || D == 128, "1 / sqrt(d) below");
  constexpr float to_log2 = 1.44269504088896340736f * (D == 64 ? 0.125f : 0.08838834764831845f);
  int n_last = 0;                                          // rows in V behind the halo that exist
  for (int t0 = t_beg; t0 < t_end; t0 += FT) {
    const int p = GROUPED ? (t0 / FT) & 1 : 0;
    const int nt = (L - t0) < FT ? (L - t0) : FT;
    n_last = 32 * p + nt;
    // ---- rows to LDS; the tail of the previous rows becomes the halo ------------------------------------------
    f32x4 tail;
    if (p == 0) tail = *reinterpret_cast<const f32x4*>(Vl + (G::KROWS + pr) * ST + pc);
    __syncthreads();
    if (p == 0) *reinterpret_cast<f32x4*>(Vl + pr * ST + pc) = tail;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = pr + RPI * i;
      const bool is = r < nt;
      f32x4 q4, k4, v4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        k4[e] = is ? (GROUPED ? xk[i][e] : phi_f32(xk[i][e], one)) : 0.f;
        v4[e] = is ? xv[i][e] : 0.f;
        if constexpr (!STATE_ONLY) q4[e] = GROUPED ? xq[i][e] : phi_f32(xq[i][e], one);
      }
      *reinterpret_cast<f32x4*>(Kl + (32 * p + r) * ST + pc) = k4;
      *reinterpret_cast<f32x4*>(Vl + (HALO + 32 * p + r) * ST + pc) = v4;
      if constexpr (!STATE_ONLY) *reinterpret_cast<f32x4*>(Ql + r * ST + pc) = q4;
    }
    if (t0 + FT < t_end) request(t0 + FT);
    __syncthreads();
    if constexpr (STATE_ONLY) {
      value_regs(0);
      add_keys(0, nt);
    } else {
      // ---- partial scores over the wave's 32 features, partial phi(q).z ---------------------------------------
      f32x4 qf[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) qf[j] = *reinterpret_cast<const f32x4*>(Ql + l32 * ST + 32 * w + 8 * j + 4 * hi);
#pragma unroll
      for (int kt = 0; kt < G::TILES; ++kt) {
        if (kt > p) break;                                 // uniform
        f32x16 sc;
        constexpr int CH = !GROUPED ? 1 : D == 64 ? 4 : 2; // logits: chains of D / 8 features (see the quadratic kernel)
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          f32x16 part;
#pragma unroll
          for (int r = 0; r < 16; ++r) part[r] = 0.f;
#pragma unroll
          for (int j = 4 / CH * c; j < 4 / CH * (c + 1); ++j) {
            const f32x4 kf = *reinterpret_cast<const f32x4*>(Kl + (32 * kt + l32) * ST + 32 * w + 8 * j + 4 * hi);
#pragma unroll
            for (int e = 0; e < 4; ++e) part = mfma32(kf[e], qf[j][e], part);
          }
          sc = c == 0 ? part : sc + part;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(Pp + ((kt * NW + w) * 4 + g) * 256 + 4 * lane) = f32x4{sc[4 * g], sc[4 * g + 1], sc[4 * g + 2], sc[4 * g + 3]};
      }
      float qz = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 z4 = *reinterpret_cast<const f32x4*>(zl + 32 * w + 8 * j + 4 * hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) qz = fmaf(GROUPED ? phi_f32(qf[j][e], one) : qf[j][e], z4[e], qz);
      }
      qz += __shfl_xor(qz, 32);
      if (hi == 0) Pz[32 * w + l32] = qz;
      // ---- O = phi(Q) S: needs nothing from the other waves ---------------------------------------------------
      f32x16 o;
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = 0.f;
#pragma unroll
      for (int ib = 0; ib < IB; ++ib)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 qa = *reinterpret_cast<const f32x4*>(Ql + l32 * ST + 32 * ib + 8 * j + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) o = mfma32(GROUPED ? phi_f32(qa[e], one) : qa[e], Sa[ib][4 * j + e], o);
        }
      __syncthreads();
      // ---- the scores of the step: pr_[kt][r] = key 32kt + acc_row(r), query l32 --------------------------------
      float pt[G::TILES][16];
#pragma unroll
      for (int kt = 0; kt < G::TILES; ++kt) {
        if (kt > p) break;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 s = *reinterpret_cast<const f32x4*>(Pp + (kt * NW * 4 + g) * 256 + 4 * lane);
#pragma unroll
          for (int v = 1; v < NW; ++v) s += *reinterpret_cast<const f32x4*>(Pp + ((kt * NW + v) * 4 + g) * 256 + 4 * lane);
#pragma unroll
          for (int e = 0; e < 4; ++e) pt[kt][4 * g + e] = s[e];
        }
      }
      float den = a.eps;
#pragma unroll
      for (int v = 0; v < NW; ++v) den += Pz[32 * v + l32];
      float* sc0 = smf + G::SC + 64 * w;
      if constexpr (!GROUPED) {
        float rs = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          pt[0][r] = acc_row(r, hi) <= l32 ? pt[0][r] : 0.f;
          rs += pt[0][r];
        }
        den += rs + __shfl_xor(rs, 32);
        if (hi == 0) sc0[l32] = 1.f / den;
      } else {
        // causal softmax over the group's keys so far: the first tile of a second half is seen whole
        float top = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          if (kt > p) break;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            pt[kt][r] = (kt < p || acc_row(r, hi) <= l32) ? pt[kt][r] : -INFINITY;
            top = fmaxf(top, pt[kt][r]);
          }
        }
        top = fmaxf(top, __shfl_xor(top, 32));
        float sum[4] = {};
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          if (kt > p) break;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            pt[kt][r] = __builtin_amdgcn_exp2f((pt[kt][r] - top) * to_log2);
            sum[r % 4] += pt[kt][r];
          }
        }
        float mass = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        mass += __shfl_xor(mass, 32);                      // the token itself is always seen: mass >= 1
        const float f = den != 0.f ? a.alpha / den : 0.f;  // nothing before the group: no branch
        if (hi == 0) { sc0[l32] = 1.f / mass; sc0[32 + l32] = f * mass; }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 fm = *reinterpret_cast<const f32x4*>(sc0 + 32 + 8 * g + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[4 * g + e] *= fm[e];
        }
      }
#pragma unroll
      for (int kt = 0; kt < G::TILES; ++kt) {
        if (kt > p) break;
        value_regs(kt);
        float odd = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) o = mfma32(pt[kt][r], finite_part(vr[r], odd), o);
        if (__any(odd != odd)) {                                  // uniform; two keys at a time through the wave's own 32 floats
#pragma unroll 1
          for (int s = 0; s < 16; ++s) {
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
              const int key = acc_row(s, h2);
              asm volatile("" ::: "memory");
              if (hi == h2) sc0[32 + l32] = pt[kt][0];
              asm volatile("" ::: "memory");
              add_non_finite(sc0 + 32, Vl[(HALO + 32 * kt + key) * ST + ch], kt == p ? key : 0, o, hi);
            }
#pragma unroll
            for (int i = 0; i < 15; ++i) pt[kt][i] = pt[kt][i + 1];
          }
        }
      }
      // ---- outputs: o[r] = token t0 + acc_row(r), channel ch ----------------------------------------------------
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 iv = *reinterpret_cast<const f32x4*>(sc0 + 8 * g + 4 * hi);
        float back[KCM - 1 + 1];                           // value rows before the four tokens, newest first
        const float* vb = Vl + (HALO + 32 * p + 8 * g + 4 * hi) * ST + ch;
#pragma unroll
        for (int j = 1; j < KCM; ++j) back[j] = vb[-j * ST];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float u = o[4 * g + e] * iv[e];
#pragma unroll
          for (int j = 0; j < KCM; ++j) {                  // (a tap that does not exist is left out: 0 times an infinity is none)
            const float x = e - j >= 0 ? vr[4 * g + e - j < 0 ? 0 : 4 * g + e - j] : back[j - e > 0 ? j - e : 1];
            u = j < taps ? fmaf(wreg[j], x, u) : u;
          }
          const int row = 8 * g + 4 * hi + e;
          if (row < nt) go[(int64_t)(t0 + row) * a.st_v + ch] = u;
        }
      }
      // ---- the keys enter the sums: at once, or at the end of their group ----------------------------------------
      if constexpr (!GROUPED) {
        add_keys(0, nt);
        if (hi == 0) zl[ch] = zr;
      } else if (p == 1 || t0 + FT >= t_end) {
        add_keys(p, nt);
        if (p == 1) {
          value_regs(0);
          add_keys(0, FT);
        }
        if (hi == 0) zl[ch] = zr;
      }
    }
  }

  if constexpr (STATE_ONLY) {
    float* so = a.ws + ((size_t)hx.bhs * a.nseg + seg + 1) * G::SLOT;   // the segment's increment, for the segment after it
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) so[(32 * ib + acc_row(r, hi)) * D + ch] = Sa[ib][r];
    if (hi == 0) so[D * D + ch] = zr;
  } else if (seg == a.nseg - 1) {
    if (a.S_out) {
#pragma unroll
      for (int ib = 0; ib < IB; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) a.S_out[S_base + (int64_t)(32 * ib + acc_row(r, hi)) * hx.dvt + ch] = Sa[ib][r];
    }
    if (a.z_out && hx.blk == 0 && hi == 0) a.z_out[(size_t)hx.bh * D + ch] = zr;   // the same in every value block
    if (a.hist_out) {
      // the last Kc - 1 value rows; with no tokens at all the rows that were to become the halo
      __syncthreads();
      const int end = t_beg < t_end ? HALO + n_last : G::KROWS + HALO;
      for (int e = tid; e < (Kc - 1) * (D / 4); e += NT) {
        const int r = e / (D / 4), c4 = 4 * (e % (D / 4));
        *reinterpret_cast<f32x4*>(static_cast<float*>(a.hist_out) + hist_base + (int64_t)r * hx.dvt + c4) =
            *reinterpret_cast<const f32x4*>(Vl + (end - (Kc - 1) + r) * ST + c4);
      }
    }
  }
}

// Short sequences on few heads: every 32-query tile by a workgroup of its own, straight from the masked quadratic form
// -- no running state, no chain from one group to the next, one launch.  The key tiles are dealt out over the eight
// waves; a wave takes its K, Q and V operands from memory into registers (all requests before the first product), forms
// its tile of scores with keys in the rows of the accumulator (the left operand of P V as it is), and the partial outputs
// meet in LDS.  An incoming state is one more tile: phi(Q) S_in.  Workgroups behind the query tiles form what is handed
// on: 32 features of S and z each, the tokens dealt out over the waves in the same way.  In the three-branch form the
// tiles of earlier groups go into a linear sum of their own and one wave takes the group's own (at most two) tiles with
// the softmax.
// What bounds it: one trip to memory, then the fp32 matrix rate of one compute unit (0.43 us per pair of tiles at D = 64,
// 0.85 us at D = 128), quadratic in the length -- hence for short sequences only.  Measured: B1 H4 L256 D64 18 us a call
// (294 us before, 26 us as the three launches of the walk).
namespace {
constexpr int DW = 8;                                      // waves
template <int D>
struct DirectCfg {
  static constexpr int IB = D / 32;
  static constexpr int O = 0;                              // [DW][IB][4][64][4] partial outputs, accumulator order
  static constexpr int RS = O + DW * 32 * D;               // [DW][32] partial normalisers
  static constexpr int SC = RS + DW * 32;                  // [32] sum of the local weights
  static constexpr int TOTAL = SC + 32;
};
}  // namespace

template <int D, bool GROUPED>
__global__ __launch_bounds__(64 * DW, 2) void prefill_f32_direct_kernel(PrefillArgs a) {
  using G = DirectCfg<D>;
  constexpr int IB = G::IB, NT = 64 * DW;
  extern __shared__ __attribute__((aligned(16))) float smf[];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const HeadIndex hx = head_index(a, blockIdx.x, D);
  const int L = a.L, Kc = a.Kc, nq = (L + FT - 1) / FT;
  const float one = a.relu ? 0.f : 1.f;
  const float* gq = static_cast<const float*>(a.q) + (int64_t)hx.b * a.sb + (int64_t)hx.h * a.sh;
  const float* gk = static_cast<const float*>(a.k) + (int64_t)hx.b * a.sb + (int64_t)hx.h * a.sh;
  const int64_t base_v = (int64_t)hx.b * a.sb_v + (int64_t)hx.h * a.sh_v + (int64_t)hx.blk * D;
  const float* gv = static_cast<const float*>(a.v) + base_v;
  float* go = static_cast<float*>(a.out) + base_v;
  const int64_t S_base = (int64_t)hx.bh * D * hx.dvt + (int64_t)hx.blk * D;
  const int64_t hist_base = (int64_t)hx.bh * (Kc - 1) * hx.dvt + (int64_t)hx.blk * D;
  const float* gh = static_cast<const float*>(a.hist_in);
  // value row t, which may lie in the history
  auto value_at = [&](int t, int c) __attribute__((always_inline)) -> float {
    const bool old = t < 0, none = old && (!gh || Kc - 1 + t < 0);
    const float* p = none ? gv : old ? gh + hist_base + (int64_t)(Kc - 1 + t) * hx.dvt : gv + (int64_t)t * a.st_v;
    const float x = p[c];
    return none ? 0.f : x;
  };
  f32x16 acc[IB];
#pragma unroll
  for (int cb = 0; cb < IB; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
  auto spill = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int cb = 0; cb < IB; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(smf + G::O + ((slot * IB + cb) * 4 + g) * 256 + 4 * lane) =
            f32x4{acc[cb][4 * g], acc[cb][4 * g + 1], acc[cb][4 * g + 2], acc[cb][4 * g + 3]};
  };

  if ((int)blockIdx.y >= nq) {
    // ---- what is handed on: features 32ib .. of S (all the block's channels) and z, and the history --------------
    const int ib = blockIdx.y - nq;
    float zs = 0.f;
    for (int kt = w; kt < nq; kt += DW) {
      float kx[16], vx[IB][16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int tok = FT * kt + acc_row(r, hi);
        const int64_t t = tok < L ? tok : L - 1;
        kx[r] = gk[t * a.st + 32 * ib + l32];
#pragma unroll
        for (int cb = 0; cb < IB; ++cb) vx[cb][r] = gv[t * a.st_v + 32 * cb + l32];
      }
      if (kt == nq - 1) {                                  // uniform: rows past the end are zero rows
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int cb = 0; cb < IB; ++cb) vx[cb][r] = FT * kt + acc_row(r, hi) < L ? vx[cb][r] : 0.f;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x = FT * kt + acc_row(r, hi) < L ? phi_f32(kx[r], one) : 0.f;
        zs += x;
#pragma unroll
        for (int cb = 0; cb < IB; ++cb) acc[cb] = mfma32(x, vx[cb][r], acc[cb]);
      }
    }
    zs += __shfl_xor(zs, 32);
    spill(w);
    if (hi == 0) smf[G::RS + 32 * w + l32] = zs;
    __syncthreads();
    for (int e = tid; e < 32 * D; e += NT) {
      const int f = e / D, c = e % D, cb = c / 32;
      const int at = (cb * 4 + (f >> 3)) * 256 + 4 * (((f >> 2) & 1) * 32 + (c & 31)) + (f & 3);
      float s = a.S_in ? a.S_in[S_base + (int64_t)(32 * ib + f) * hx.dvt + c] : 0.f;
#pragma unroll
      for (int v = 0; v < DW; ++v) s += smf[G::O + v * 32 * D + at];
      if (a.S_out) a.S_out[S_base + (int64_t)(32 * ib + f) * hx.dvt + c] = s;
    }
    if (a.z_out && hx.blk == 0 && tid < 32) {
      float s = a.z_in ? a.z_in[(size_t)hx.bh * D + 32 * ib + tid] : 0.f;
#pragma unroll
      for (int v = 0; v < DW; ++v) s += smf[G::RS + 32 * v + tid];
      a.z_out[(size_t)hx.bh * D + 32 * ib + tid] = s;
    }
    if (a.hist_out && ib == 0)
      for (int e = tid; e < (Kc - 1) * D; e += NT)
        static_cast<float*>(a.hist_out)[hist_base + (int64_t)(e / D) * hx.dvt + e % D] = value_at(L - (Kc - 1) + e / D, e % D);
    return;
  }

  // ---- one query tile (the longest first) ------------------------------------------------------------------------
  const int qt = nq - 1 - blockIdx.y;
  const int kt0 = GROUPED ? qt & ~1 : qt + 1;              // tiles from here on belong to the query's own group
  f32x4 qf[IB][4];                                         // query l32, features 32ib + 8j + 4hi + e
  {
    const int tok = FT * qt + l32;
    const float* p = gq + (int64_t)(tok < L ? tok : L - 1) * a.st + 4 * hi;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int j = 0; j < 4; ++j) qf[ib][j] = *reinterpret_cast<const f32x4*>(p + 32 * ib + 8 * j);
  }
  if (!GROUPED || w != 0) {                                // only the softmax of the query's own group takes the raw rows
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) qf[ib][j][e] = phi_f32(qf[ib][j][e], one);
  }
  static_assert(D == 64 || D == 128, "1 / sqrt(d) below");
  constexpr float to_log2 = 1.44269504088896340736f * (D == 64 ? 0.125f : 0.08838834764831845f);
  // value rows of key tile kt
  auto values = [&](int kt, float (&vx)[IB][16]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int tv = FT * kt + acc_row(r, hi);
#pragma unroll
      for (int cb = 0; cb < IB; ++cb) vx[cb][r] = gv[(int64_t)(tv < L ? tv : L - 1) * a.st_v + 32 * cb + l32];
    }
  };
  // scores of key tile kt: sc[r] = key acc_row(r), query l32; raw: the rows as they are, else under the feature map.
  // In the three-branch form all sums are cut into short chains, so that the outputs are no further from the exact ones
  // than those of the vector ALUs that did this before (logits in four chains per row, weights times values in four): raw
  // scores eight chains of D / 8 features (a logit may be a small difference of large products), mapped ones four (two
  // at d = 128, where four spill: 30 us -> 28 at B1 H4 L256 with two), the own group's weights times values chains of 8 keys,
  // the earlier groups' of 16 at d = 64.  2-norm error, rows of d^-1/2 / unit normals, against 4.8e-8 / 6.0e-8 (d = 64) and
  // 4.9e-8 / 6.6e-8 (d = 128): one chain each 5.2 / 8.2 and 5.3 / 9.9; as it is 4.8 / 5.9 and 4.9 / 6.2, for 0 to 3 % of the time
  // (B1 H4 L256 d64 18 us either way, B2 H8 L289 d128 28 -> 28.5).  The token form is closer than the vector ALUs with one chain.
  auto scores = [&](int kt, bool raw, f32x16& sc) __attribute__((always_inline)) {
    f32x4 kf[IB][4];
    const int tok = FT * kt + l32;
    const float* p = gk + (int64_t)(tok < L ? tok : L - 1) * a.st + 4 * hi;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib)
#pragma unroll
      for (int j = 0; j < 4; ++j) kf[ib][j] = *reinterpret_cast<const f32x4*>(p + 32 * ib + 8 * j);
    const int chains = raw ? 8 : !GROUPED ? 1 : D == 64 ? 4 : 2;
#pragma unroll
    for (int c = 0; c < chains; ++c) {
      f32x16 part;
#pragma unroll
      for (int r = 0; r < 16; ++r) part[r] = 0.f;
#pragma unroll
      for (int j = 0; j < 4 * IB / chains; ++j) {
        const int ib = (4 * IB / chains * c + j) / 4, jj = (4 * IB / chains * c + j) % 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) part = mfma32(raw ? kf[ib][jj][e] : phi_f32(kf[ib][jj][e], one), qf[ib][jj][e], part);
      }
      sc = c == 0 ? part : sc + part;
    }
  };
  // acc += weights times value(cb, r), in chains of 32 / n keys, a channel block at a time
  auto add_in_chains = [&](auto n, const f32x16& sc, auto value) __attribute__((always_inline)) {
    constexpr int PER = 16 / decltype(n)::value;
#pragma unroll
    for (int cb = 0; cb < IB; ++cb)
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += PER) {
        f32x16 part;
#pragma unroll
        for (int r = 0; r < 16; ++r) part[r] = 0.f;
#pragma unroll
        for (int r = r0; r < r0 + PER; ++r) part = mfma32(sc[r], value(cb, r), part);
        acc[cb] += part;
      }
  };
  auto weigh = [&](const f32x16& sc, const float (&vx)[IB][16]) __attribute__((always_inline)) {
    if constexpr (D == 64) {
      add_in_chains(std::integral_constant<int, 2>(), sc, [&](int cb, int r) { return vx[cb][r]; });
    } else {                                               // (no registers left for a second sum)
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int cb = 0; cb < IB; ++cb) acc[cb] = mfma32(sc[r], vx[cb][r], acc[cb]);
    }
  };
  // the same with values that may not be finite, and what those add
  auto weigh_finite = [&](const f32x16& sc, const float (&vx)[IB][16]) __attribute__((always_inline)) {
    float odd = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int cb = 0; cb < IB; ++cb) acc[cb] = mfma32(sc[r], finite_part(vx[cb][r], odd), acc[cb]);
    return odd;
  };
  auto weigh_rest = [&](float odd, int kt, const f32x16& sc) __attribute__((always_inline)) {
    if (!__any(odd != odd)) return;                        // uniform
    float* own = smf + G::O + w * 32 * D;                  // the wave's part of the outputs, free until they go there
#pragma unroll
    for (int r = 0; r < 16; ++r) own[32 * acc_row(r, hi) + l32] = sc[r];
    asm volatile("" ::: "memory");
#pragma unroll 1
    for (int key = 0; key < FT; ++key) {
      const float* vp = gv + (int64_t)(FT * kt + key < L ? FT * kt + key : L - 1) * a.st_v + l32;
#pragma unroll
      for (int cb = 0; cb < IB; ++cb) add_non_finite(own + 32 * key, vp[32 * cb], kt == qt ? key : 0, acc[cb], hi);
    }
    asm volatile("" ::: "memory");
  };
  float rs = 0.f;                                          // what the wave's tiles add to the normaliser of query l32
  const int first = GROUPED ? w - 1 : w;                   // three-branch form: wave 0 has the query's own group
  const int step = GROUPED ? DW - 1 : DW;
  if (GROUPED && w == 0) {
    // causal softmax over the group's own tiles; unnormalised weights, their sum to LDS
    f32x16 s0, s1;
    float v0[IB][16], v1[IB][16];
    const bool two = qt > kt0;                             // uniform
    if (D == 64) {
      values(qt, v1);
      values(kt0, v0);
    }
    scores(qt, true, s1);
    scores(kt0, true, s0);
    if (D == 128) {                                        // (all requests at once would not fit)
      __builtin_amdgcn_sched_barrier(0);
      values(qt, v1);
      values(kt0, v0);
    }
    float top = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s1[r] = acc_row(r, hi) <= l32 ? s1[r] : -INFINITY;
      if (!two) s0[r] = -INFINITY;
      top = fmaxf(top, fmaxf(s0[r], s1[r]));
    }
    top = fmaxf(top, __shfl_xor(top, 32));
    float sum[4] = {};
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s0[r] = __builtin_amdgcn_exp2f((s0[r] - top) * to_log2);
      s1[r] = __builtin_amdgcn_exp2f((s1[r] - top) * to_log2);
      sum[r % 4] += s0[r] + s1[r];
    }
    float mass = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    mass += __shfl_xor(mass, 32);                          // the token itself is always seen: mass >= 1
    if (hi == 0) smf[G::SC + l32] = mass;
    float odd = 0.f;
    const std::integral_constant<int, 4> four;
    add_in_chains(four, s1, [&](int cb, int r) { return finite_part(v1[cb][r], odd); });
    if (two) add_in_chains(four, s0, [&](int cb, int r) { return v0[cb][r]; });
    weigh_rest(odd, qt, s1);
  } else {
    for (int kt = first; kt < kt0; kt += step) {
      f32x16 sc;
      float vx[IB][16];
      if (!GROUPED || D == 64) values(kt, vx);             // (ahead of the scores where there are registers)
      scores(kt, false, sc);
      if (GROUPED && D == 128) values(kt, vx);
      float sum[4] = {};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (!GROUPED) sc[r] = (kt < qt || acc_row(r, hi) <= l32) ? sc[r] : 0.f;
        sum[r % 4] += sc[r];
      }
      rs += (sum[0] + sum[1]) + (sum[2] + sum[3]);
      if constexpr (GROUPED) weigh(sc, vx);                // whole tiles of earlier groups
      else weigh_rest(weigh_finite(sc, vx), kt, sc);
    }
    if (w == DW - 1 && a.S_in) {                           // the incoming state
#pragma unroll
      for (int ib = 0; ib < IB; ++ib)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 z4 = *reinterpret_cast<const f32x4*>(a.z_in + (size_t)hx.bh * D + 32 * ib + 8 * j + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = qf[ib][j][e];
            rs = fmaf(x, z4[e], rs);
            const float* sp = a.S_in + S_base + (int64_t)(32 * ib + 8 * j + 4 * hi + e) * hx.dvt + l32;
#pragma unroll
            for (int cb = 0; cb < IB; ++cb) acc[cb] = mfma32(x, sp[32 * cb], acc[cb]);
          }
        }
    }
  }
  rs += __shfl_xor(rs, 32);
  spill(w);
  if (hi == 0) smf[G::RS + 32 * w + l32] = rs;
  // the conv of this thread's outputs (one channel, every NT / D-th token), four taps at a time: their requests leave
  // together (tap by tap, every one would pay its own trip to memory)
  constexpr int NO = 32 * D / NT;
  static_assert(NT % D == 0, "one channel per thread");
  float u[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) u[i] = 0.f;
  if (!a.no_conv) {
    const int c = tid % D;
    const float* wp = a.conv_w + ((size_t)hx.h * hx.dvt + hx.blk * D + c) * Kc;
    for (int jb = 0; jb < Kc; jb += 4) {
      float wt[4], x[NO][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        wt[j] = wp[jb + j < Kc ? jb + j : Kc - 1];
#pragma unroll
        for (int i = 0; i < NO; ++i) {
          const int tok = FT * qt + (tid + NT * i) / D;
          x[i][j] = value_at((tok < L ? tok : L - 1) - jb - j, c);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < NO; ++i) u[i] = jb + j < Kc ? fmaf(wt[j], x[i][j], u[i]) : u[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int t = (tid + NT * i) / D, c = (tid + NT * i) % D, tok = FT * qt + t, cb = c / 32;
    const int at = (cb * 4 + (t >> 3)) * 256 + 4 * (((t >> 2) & 1) * 32 + (c & 31)) + (t & 3);
    float den = a.eps, y = 0.f;
#pragma unroll
    for (int v = GROUPED ? 1 : 0; v < DW; ++v) {
      den += smf[G::RS + 32 * v + t];
      y += smf[G::O + v * 32 * D + at];
    }
    if (GROUPED) y = (den != 0.f ? a.alpha / den : 0.f) * y + smf[G::O + at] / smf[G::SC + t];
    else y /= den;
    if (tok < L) go[(int64_t)tok * a.st_v + c] = y + u[i];
  }
}

// The quadratic kernel or the walk?  The quadratic kernel's time grows with the longest query tile's chain and with the
// sum of all tile pairs over the chip, the walk's is three launches and hardly moves at these sizes.  Measured, us per call
// quadratic / walk: D = 64: 12 heads of 16 tiles (1632 pairs) 21 / 26, 48 of 8 (1728) 24 / 28, 4 of 24 26 / 25, 4 of 32 32 / 26; D = 128: 4 of
// 8 (144) 24 / 33, 28 of 8 (1008) 30 / 39, 7 of 16 (952) 36 / 35, 8 of 16 (1088) 36 / 36, 64 of 8 (2304) 51 / 44.  Three-branch form (two
// kinds of steps in the walk): D = 64: 4 of 32 (2112) 33 / 49, 32 of 16 (4352) 40 / 51, 12 of 32 (6336) 47 / 50; D = 128: 8 of 16 (1088)
// 36 / 70, 4 of 32 (2112) 59 / 70, 64 of 8 (2304) 59 / 75.
static bool prefill_f32_direct_pays(int heads, int tiles, int d, bool grouped) {
  const int64_t pairs = (int64_t)heads * tiles * (tiles + 1) / 2;
  if (grouped) return tiles <= 48 && pairs <= (d == 64 ? 4400 : 2200);
  return tiles <= 16 && pairs <= (d == 64 ? 1700 : 1000);
}

// Segments per (b, h, value block), or the quadratic kernel.  Steps of 32 tokens (groups of 64 in the three-branch form)
// are the unit.
F32Plan prefill_f32_plan(int heads, int L, int d, bool grouped, int per_cu) {
  F32Plan p{1, L > 0 ? L : 1, false};
  const int tiles = (L + FT - 1) / FT;
  if (prefill_f32_direct_pays(heads, tiles, d, grouped)) {
    p.direct = true;
    return p;
  }
  const int unit = grouped ? FGROUP : FT;
  const int units = (L + unit - 1) / unit;
  // As many workgroups as keep the chip busy.  Token form at d = 64: four per compute unit (two waves each and 38 KB of LDS; with
  // two, half of the matrix units' time went by: us a call, 512 / 1024 workgroups: 12 heads L = 9164 96 / 79, 24 heads L = 4180
  // 95 / 69, 128 heads L = 300 49 / 40, 320 heads L = 700 194 / 125, 16 heads L = 16000 200 / 126), but not for sequences of fewer
  // than 8 steps on 256 heads or more (512 heads, 130 tokens: 49 / 59; 256 heads, 200 tokens 52 / 53).  d = 128: one (two: 32 heads
  // L = 1400 86 / 83, 64 heads L = 500 64 / 66, 160 heads L = 300, which 256 leaves whole, 87 / 101).  Three-branch form: the
  // registers and LDS of two and one.
  int want = (d == 64 ? (grouped || per_cu <= 2 ? 512 : 1024) : 256) / heads;
  if (d == 64 && !grouped && heads >= 256 && units < 8) want = 512 / heads;
  const int most = units / 2 < 64 ? units / 2 : 64;
  if (want > most) want = most;
  if (want < 2) return p;
  const int per = (units + want - 1) / want;
  p.seg_len = per * unit;
  p.nseg = (units + per - 1) / per;
  return p;
}

size_t prefill_f32_workspace_bytes(int heads, int d, const F32Plan& p) {
  if (p.nseg <= 1) return 0;
  return (size_t)heads * p.nseg * ((size_t)d * d + d) * sizeof(float) + (size_t)heads * HALO * d * sizeof(float);
}

template <int D, int KCM, bool STATE_ONLY, bool GROUPED>
static hipError_t launch_f32_one(const PrefillArgs& a, hipStream_t st) {
  using G = F32Cfg<D, GROUPED>;
  constexpr int bytes = G::TOTAL * (int)sizeof(float);
  static_assert(bytes <= 160 * 1024, "LDS");
  auto kern = prefill_f32_kernel<D, KCM, STATE_ONLY, GROUPED>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * a.H * a.m), (unsigned)(STATE_ONLY ? a.nseg - 1 : a.nseg)), dim3(G::NT), bytes, st, a);
  return hipGetLastError();
}

template <int D, bool GROUPED>
static hipError_t launch_f32_direct(const PrefillArgs& a, hipStream_t st) {
  constexpr int bytes = DirectCfg<D>::TOTAL * (int)sizeof(float);
  static_assert(bytes <= 160 * 1024, "LDS");
  auto kern = prefill_f32_direct_kernel<D, GROUPED>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, bytes);
  if (e != hipSuccess) return e;
  const bool hand_on = a.S_out || a.z_out || a.hist_out;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * a.H * a.m), (unsigned)((a.L + FT - 1) / FT + (hand_on ? D / 32 : 0))), dim3(64 * DW), bytes, st, a);
  return hipGetLastError();
}

template <int D, bool GROUPED>
static hipError_t launch_f32_d(const PrefillArgs& a, hipStream_t st) {
  if (a.direct) return launch_f32_direct<D, GROUPED>(a, st);
  if (a.nseg > 1) {
    hipError_t e = launch_f32_one<D, 3, true, false>(a, st);
    if (e != hipSuccess) return e;
    if ((e = launch_segment_scan(a, D, st)) != hipSuccess) return e;
  }
  return a.Kc <= 3 ? launch_f32_one<D, 3, false, GROUPED>(a, st) : a.Kc <= 5 ? launch_f32_one<D, 5, false, GROUPED>(a, st)
                                                                             : launch_f32_one<D, 8, false, GROUPED>(a, st);
}

hipError_t launch_prefill_f32(const PrefillArgs& a, int d, bool grouped, hipStream_t st) {
  if (d == 128) return grouped ? launch_f32_d<128, true>(a, st) : launch_f32_d<128, false>(a, st);
  return grouped ? launch_f32_d<64, true>(a, st) : launch_f32_d<64, false>(a, st);
}

}  // namespace linattn
