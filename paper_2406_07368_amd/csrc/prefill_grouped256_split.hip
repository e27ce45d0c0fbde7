// The three-branch form in groups of 256 tokens (see prefill_grouped256.hip for the arithmetic) when the groups are few: P = 2, 4
// or 8 workgroups share a group, each with 256 / P of its queries, and P of a workgroup's eight waves share a 32-query tile, each
// with every P-th key tile.
//
// With one workgroup per group, 8 heads of 1000 tokens are 32 workgroups on 256 compute units, and the call waits for one wave's
// walk over eight key tiles, the state update behind it and 256 rows of output.  Here that walk is 8 / P tiles, the outputs are
// shared, and the state after the last token is the work of a workgroup of its own.
//
//   local branch   online softmax over the wave's key tiles (products, order and rounding of a tile as in the other kernel); the
//                  waves of a query tile then exchange their largest logits and sums through LDS and scale what they have
//   linear branch  O_lin^T = S^T phi(Q)^T one 32-channel tile at a time, the tiles dealt out over the waves that share the
//                  queries; the state's operand comes straight from memory into registers, requested ahead of the rows
//   outputs        the waves' partial sums meet in LDS in fp32 (the key rows' memory), 64 channels at a time; one rounding
//
// Measured: see prefill_grouped256_parts.
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

namespace linattn {

namespace {

template <int D>
struct G256SCfg {
  static constexpr int GT = 256, NW = 8, NT = 64 * NW;
  static constexpr int KSD = D / 16, CT = D / 32;
  static constexpr int KS = D + 8;           // key rows: 16-byte row reads, transpose reads
  static constexpr int VS = D + 4;           // value rows: transpose reads, 8-byte row reads
  static constexpr int OS = 64 + 4;          // partial outputs: 64 channels of 32 queries per wave, fp32
  static constexpr int SZK = GT * KS * 2, SZO = NW * 32 * OS * 4;
  static constexpr int OFF_K = 0;
  static constexpr int OFF_V = SZK > SZO ? SZK : SZO;                 // row r = token r - HALO
  static constexpr int OFF_Z = (OFF_V + (HALO + GT) * VS * 2 + 15) / 16 * 16;   // [D] float: z before the group
  static constexpr int OFF_R = OFF_Z + D * 4;                         // [NW][D] float: per-wave tops and sums
  static constexpr int OFF_W = OFF_R + NW * D * 4;                    // [8][D] float conv taps, tap-major
  static constexpr int TOTAL = OFF_W + 8 * D * 4;
  static_assert(TOTAL <= 160 * 1024, "LDS");
};

}  // namespace

template <int D, int KCM, int P>
__global__ __launch_bounds__(512) void prefill_grouped256_split_kernel(PrefillArgs a) {
  using G = G256SCfg<D>;
  constexpr int GT = G::GT, NQ = GT / P, CT = G::CT, KSD = G::KSD;
  constexpr int SLOT = D * D + D;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* Kl = reinterpret_cast<uint16_t*>(smem + G::OFF_K);
  uint16_t* Vl = reinterpret_cast<uint16_t*>(smem + G::OFF_V);
  float* zl = reinterpret_cast<float*>(smem + G::OFF_Z);
  float* redl = reinterpret_cast<float*>(smem + G::OFF_R);
  float* wl = reinterpret_cast<float*>(smem + G::OFF_W);
  float* Ol = reinterpret_cast<float*>(smem + G::OFF_K);

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  // Workgroups: the last (longest) part of every group first, then the ones before it; behind them one per head for the
  // state after the last token and the history.
  const int ngh = a.B * a.H * a.nseg;
  const bool hand_on = (int)blockIdx.x >= P * ngh;         // uniform
  const int gh = hand_on ? (blockIdx.x - P * ngh) * a.nseg + a.nseg - 1 : blockIdx.x % ngh;
  const int part = hand_on ? P - 1 : P - 1 - blockIdx.x / ngh;
  const int bh = gh / a.nseg, seg = gh % a.nseg;
  const int b = bh / a.H, h = bh % a.H;
  const int tok0 = seg * GT;
  const int nt = (a.L - tok0) < GT ? (a.L - tok0) : GT;
  if (!hand_on && NQ * part >= nt) return;                 // uniform: no queries there
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const uint16_t* gq = static_cast<const uint16_t*>(a.q) + base;
  const uint16_t* gk = static_cast<const uint16_t*>(a.k) + base;
  const uint16_t* gv = static_cast<const uint16_t*>(a.v) + base;
  uint16_t* gout = static_cast<uint16_t*>(a.out) + base;
  // the state before the group: a slot of the workspace, or (one group) what came in
  const bool slots = a.nseg > 1, have_state = slots || a.S_in != nullptr;
  const float* S0 = slots ? a.ws + (size_t)gh * SLOT : a.S_in ? a.S_in + (size_t)bh * D * D : a.conv_w;
  const float* z0 = slots ? S0 + D * D : a.S_in ? a.z_in + (size_t)bh * D : nullptr;
  const uint16_t* staged_hist = reinterpret_cast<const uint16_t*>(a.ws + (size_t)a.B * a.H * a.nseg * SLOT) + (size_t)bh * HALO * D;
  const uint16_t* hin = static_cast<const uint16_t*>(a.hist_in);
  static_assert(D == 64 || D == 128, "1 / sqrt(d) below");
  constexpr float to_log2 = 1.44269504088896340736f * (D == 64 ? 0.125f : 0.08838834764831845f);

  // The rows up to the last query's, in one go; rows past that re-read the last one (nobody looks at them), rows past the end
  // of the sequence are zero rows.
  constexpr int NPC = GT * (D / 8) / G::NT;
  u32x4 kx[NPC], vx[NPC];
  const int rows = NQ * (part + 1) < nt ? NQ * (part + 1) : nt;
  auto request_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NPC; ++i) {
      const int e = tid + G::NT * i;
      const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
      const int64_t off = (int64_t)(tok0 + (r < rows ? r : rows - 1)) * a.st + c0;
      kx[i] = *reinterpret_cast<const u32x4*>(gk + off);
      vx[i] = *reinterpret_cast<const u32x4*>(gv + off);
    }
  };

  if (hand_on) {
    // ======================= S, z and the history after the last token ===========================================
    if (a.S_out || a.z_out) {
      request_rows();
      float zp[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NPC; ++i) {
        const int e = tid + G::NT * i;
        const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
        u32x4 f = phi_pack8_nb(kx[i], a.relu ? 0.f : 1.f);
        if (r >= nt) f = vx[i] = u32x4{0, 0, 0, 0};
        *reinterpret_cast<u32x4*>(Kl + r * G::KS + c0) = f;
        u32x2* vrow = reinterpret_cast<u32x2*>(Vl + (HALO + r) * G::VS + c0);
        vrow[0] = u32x2{vx[i][0], vx[i][1]};
        vrow[1] = u32x2{vx[i][2], vx[i][3]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          zp[2 * j] += bf16_lo_to_f32(f[j]);
          zp[2 * j + 1] += bf16_hi_to_f32(f[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
#pragma unroll
        for (int m = D / 8; m < 64; m *= 2) zp[j] += __shfl_xor(zp[j], m);
      }
      if (lane < D / 8) {
        *reinterpret_cast<f32x4*>(redl + w * D + 8 * lane) = f32x4{zp[0], zp[1], zp[2], zp[3]};
        *reinterpret_cast<f32x4*>(redl + w * D + 8 * lane + 4) = f32x4{zp[4], zp[5], zp[6], zp[7]};
      }
      __syncthreads();
      // one 32 x 32 tile of S at a time and wave
      if (a.S_out) {
        for (int tile = w; tile < CT * CT; tile += G::NW) {
          const int64_t so = (int64_t)(32 * (tile / CT) + 4 * hi) * D + 32 * (tile % CT) + l32;
          f32x16 s;
#pragma unroll
          for (int r = 0; r < 16; ++r) s[r] = have_state ? S0[so + (8 * (r >> 2) + (r & 3)) * D] : 0.f;
#pragma unroll 8
          for (int ks = 0; ks < GT / 16; ++ks)
            s = mfma(tr_operand(Kl, G::KS, 16 * ks, 32 * (tile / CT), lane), tr_operand(Vl + HALO * G::VS, G::VS, 16 * ks, 32 * (tile % CT), lane), s);
#pragma unroll
          for (int r = 0; r < 16; ++r) a.S_out[(size_t)bh * D * D + so + (8 * (r >> 2) + (r & 3)) * D] = s[r];
        }
      }
      if (a.z_out && tid < D) {
        float zs = have_state ? z0[tid] : 0.f;
#pragma unroll
        for (int i = 0; i < G::NW; ++i) zs += redl[i * D + tid];
        a.z_out[(size_t)bh * D + tid] = zs;
      }
    }
    if (a.hist_out && tid < D) {
      uint16_t* hout = static_cast<uint16_t*>(a.hist_out) + (size_t)bh * (a.Kc - 1) * D;
      for (int r = 0; r < a.Kc - 1; ++r) {
        const int tok = a.L - (a.Kc - 1) + r;
        uint16_t x = 0;
        if (tok >= 0) x = gv[(int64_t)tok * a.st + tid];
        else if (hin) x = slots ? staged_hist[(size_t)(HALO + tok) * D + tid] : hin[((size_t)bh * (a.Kc - 1) + (a.Kc - 1 + tok)) * D + tid];
        hout[(size_t)r * D + tid] = x;
      }
    }
    return;
  }

  // ---- 1. requests: this wave's queries, its channels' columns of the state, the rows, z ------------------------------
  const int ql = w / P, j = w % P;                         // query tile of this workgroup; the wave's turn among the key tiles
  const int qtile = NQ / 32 * part + ql;
  const int qt = 32 * qtile + l32;
  u32x4 qraw[KSD];
  {
    const uint16_t* qp = gq + (int64_t)(tok0 + (qt < nt ? qt : nt - 1)) * a.st + 8 * hi;
#pragma unroll
    for (int ks = 0; ks < KSD; ++ks) qraw[ks] = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
  }
  constexpr int LT = (CT + P - 1) / P;                     // channel tiles of the linear branch per wave
  float sx[LT][KSD][8];
#pragma unroll
  for (int t = 0; t < LT; ++t) {
    const int ct = j + P * t < CT ? j + P * t : CT - 1;
#pragma unroll
    for (int ks = 0; ks < KSD; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) sx[t][ks][e] = have_state ? S0[(16 * ks + 8 * hi + e) * D + 32 * ct + l32] : 0.f;
  }
  const float zx = have_state ? z0[tid < D ? tid : 0] : 0.f;
  request_rows();
  uint16_t hx[KCM > 0 ? HALO * D / G::NT : 1];
  float wx[KCM > 0 ? 8 * D / G::NT : 1];
  if constexpr (KCM > 0) {
#pragma unroll
    for (int i = 0; i < 8 * D / G::NT; ++i) {
      const int e = tid + G::NT * i;
      wx[i] = a.conv_w[((size_t)h * D + e % D) * a.Kc + (e / D < a.Kc ? e / D : 0)];
    }
#pragma unroll
    for (int i = 0; i < HALO * D / G::NT; ++i) {
      const int e = tid + G::NT * i;
      const int r = e / D, cc = e % D;
      const int tok = tok0 - HALO + r;
      const bool staged = tok < 0 && hin != nullptr && slots;
      const bool given = tok < 0 && hin != nullptr && !slots && a.Kc - 1 + tok >= 0;
      const uint16_t* src = staged ? staged_hist + (int64_t)(HALO + tok) * D + cc
                          : given ? hin + ((int64_t)bh * (a.Kc - 1) + (a.Kc - 1 + tok)) * D + cc
                                  : gv + (int64_t)(tok >= 0 ? tok : 0) * a.st + cc;
      const uint16_t x = *src;
      hx[i] = tok >= 0 || staged || given ? x : (uint16_t)0;
    }
  }
  // ---- 2. into LDS, the state's columns into operands ----------------------------------------------------------------
  bf16x8 sop[LT][KSD];                                     // lanes = channels, registers = features 16ks + 8hi + 0..7
#pragma unroll
  for (int t = 0; t < LT; ++t)
#pragma unroll
    for (int ks = 0; ks < KSD; ++ks)
      sop[t][ks] = __builtin_bit_cast(bf16x8, u32x4{pack_bf16x2(sx[t][ks][0], sx[t][ks][1]), pack_bf16x2(sx[t][ks][2], sx[t][ks][3]),
                                                    pack_bf16x2(sx[t][ks][4], sx[t][ks][5]), pack_bf16x2(sx[t][ks][6], sx[t][ks][7])});
  if (tid < D) zl[tid] = zx;
#pragma unroll
  for (int i = 0; i < NPC; ++i) {
    const int e = tid + G::NT * i;
    const int r = e / (D / 8), c0 = 8 * (e % (D / 8));
    if (r >= nt) kx[i] = vx[i] = u32x4{0, 0, 0, 0};
    *reinterpret_cast<u32x4*>(Kl + r * G::KS + c0) = kx[i];
    u32x2* vrow = reinterpret_cast<u32x2*>(Vl + (HALO + r) * G::VS + c0);
    vrow[0] = u32x2{vx[i][0], vx[i][1]};
    vrow[1] = u32x2{vx[i][2], vx[i][3]};
  }
  if constexpr (KCM > 0) {
#pragma unroll
    for (int i = 0; i < 8 * D / G::NT; ++i) {
      const int e = tid + G::NT * i;
      wl[e] = e / D < a.Kc ? wx[i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < HALO * D / G::NT; ++i) {
      const int e = tid + G::NT * i;
      Vl[(e / D) * G::VS + e % D] = hx[i];
    }
  }
  __syncthreads();                                         // A: the rows are in LDS

  // ---- 3. local branch over key tiles j, j + P, .. <= qtile -----------------------------------------------------------
  f32x16 o[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ct][r] = 0.f;
  float mtop = -INFINITY, mass = 0.f;
  for (int kt = j; kt <= qtile; kt += P) {                 // uniform per wave
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const uint16_t* ka = Kl + (32 * kt + l32) * G::KS + 8 * hi;
#pragma unroll
    for (int ks = 0; ks < KSD; ++ks) acc = mfma(lds_row8(ka + 16 * ks), __builtin_bit_cast(bf16x8, qraw[ks]), acc);
    // acc[r]: key 32kt + 8(r/4) + 4hi + r%4, query 32 qtile + l32; later keys are -inf, their weight an exact zero
    float top = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int kl = 8 * (r >> 2) + 4 * hi + (r & 3);
      acc[r] = (kt < qtile || kl <= l32) ? acc[r] : -INFINITY;
      top = fmaxf(top, acc[r]);
    }
    top = fmaxf(top, __shfl_xor(top, 32));
    // (a wave may have met only logits of -inf, another one the tile with the finite ones: weights of zero, not NaN)
    const float mnew = fmaxf(mtop, top), from = mnew == -INFINITY ? 0.f : mnew;
    const float corr = __builtin_amdgcn_exp2f((mtop - from) * to_log2);
    const float shift = -from * to_log2;
    float rs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[r] = __builtin_amdgcn_exp2f(fmaf(acc[r], to_log2, shift));
      rs += acc[r];
    }
    mass = fmaf(mass, corr, rs);
    mtop = mnew;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[ct][r] *= corr;
    const bf16x8 p0 = pack8(acc, 0), p1 = pack8(acc, 8);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      o[ct] = mfma(tr_operand_acc_order(Vl + HALO * G::VS, G::VS, 32 * kt, 32 * ct, lane), p0, o[ct]);
      o[ct] = mfma(tr_operand_acc_order(Vl + HALO * G::VS, G::VS, 32 * kt + 16, 32 * ct, lane), p1, o[ct]);
    }
  }
  mass += __shfl_xor(mass, 32);
  if (lane < 32) {
    redl[64 * w + l32] = mtop;
    redl[64 * w + 32 + l32] = mass;
  }
  // ---- 4. phi(Q), phi(q).z, the wave's channels of the linear branch ----------------------------------------------------
  float dz = 0.f;
  bf16x8 fq[KSD];
#pragma unroll
  for (int ks = 0; ks < KSD; ++ks) {
    const u32x4 f = phi_pack8_nb(qraw[ks], a.relu ? 0.f : 1.f);
    fq[ks] = __builtin_bit_cast(bf16x8, f);
    const float* zp = zl + 16 * ks + 8 * hi;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      dz = fmaf(bf16_lo_to_f32(f[i]), zp[2 * i], dz);
      dz = fmaf(bf16_hi_to_f32(f[i]), zp[2 * i + 1], dz);
    }
  }
  dz += __shfl_xor(dz, 32);
  const float gden = dz + a.eps;
  const float fscale = gden != 0.f ? a.alpha * __builtin_amdgcn_rcpf(gden) : 0.f;   // nothing before the group: no branch
  f32x16 lin[LT];
#pragma unroll
  for (int t = 0; t < LT; ++t) {
#pragma unroll
    for (int r = 0; r < 16; ++r) lin[t][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KSD; ++ks) lin[t] = mfma(sop[t][ks], fq[ks], lin[t]);
  }
  // what this thread adds its outputs to (long conv: the pass that ran first left it there)
  constexpr int ROUNDS = D / 64, PPT = (NQ * 8 + G::NT - 1) / G::NT;
  u32x4 held[KCM == 0 ? ROUNDS * PPT : 1];
  if constexpr (KCM == 0) {
#pragma unroll
    for (int i = 0; i < ROUNDS * PPT; ++i) {
      const int e = tid + G::NT * (i % PPT);
      const int r = NQ * part + e / 8, c0 = 64 * (i / PPT) + 8 * (e % 8);
      held[i] = *reinterpret_cast<const u32x4*>(gout + (int64_t)(tok0 + (r < rows ? r : rows - 1)) * a.st + c0);
    }
  }
  __syncthreads();                                         // B: every wave's top and sum; the key rows are done with
  float all = -INFINITY, total = 0.f;
#pragma unroll
  for (int v = 0; v < P; ++v) all = fmaxf(all, redl[64 * (ql * P + v) + l32]);
#pragma unroll
  for (int v = 0; v < P; ++v)
    total = fmaf(redl[64 * (ql * P + v) + 32 + l32], __builtin_amdgcn_exp2f((redl[64 * (ql * P + v) + l32] - all) * to_log2), total);
  // the query itself is always seen: total >= 1; a wave without a key tile has zeros
  const float scale = __builtin_amdgcn_exp2f((mtop - all) * to_log2) * __builtin_amdgcn_rcpf(total);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ct][r] *= scale;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
    if (ct % P == j) {                                     // uniform per wave
#pragma unroll
      for (int r = 0; r < 16; ++r) o[ct][r] = fmaf(lin[ct / P][r], fscale, o[ct][r]);
    }

  // ---- 5. outputs, 64 channels at a time ----------------------------------------------------------------------------------
#pragma unroll
  for (int half = 0; half < ROUNDS; ++half) {
    if (half > 0) __syncthreads();                         // the partial sums of the round before are read
    float* orow = Ol + (32 * w + l32) * G::OS + 4 * hi;
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16& x = o[2 * half + c2];
        *reinterpret_cast<f32x4*>(orow + 32 * c2 + 8 * g) = f32x4{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int e = tid + G::NT * i;
      const int q = e / 8, cl = 8 * (e % 8), c0 = 64 * half + cl;
      const int r = NQ * part + q;
      if (q < NQ && r < nt) {
        float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < P; ++v) {
          const float* src = Ol + (32 * ((q / 32) * P + v) + q % 32) * G::OS + cl;
          const f32x4 y0 = *reinterpret_cast<const f32x4*>(src), y1 = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
          for (int c = 0; c < 4; ++c) { y[c] += y0[c]; y[4 + c] += y1[c]; }
        }
        if constexpr (KCM == 0) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            y[2 * c] += bf16_lo_to_f32(held[half * PPT + i][c]);
            y[2 * c + 1] += bf16_hi_to_f32(held[half * PPT + i][c]);
          }
        } else {
#pragma unroll
          for (int tap = 0; tap < KCM; ++tap) {
            const u32x2* vp = reinterpret_cast<const u32x2*>(Vl + (HALO + r - tap) * G::VS + c0);
            const u32x2 x[2] = {vp[0], vp[1]};
            const f32x4 wt[2] = {*reinterpret_cast<const f32x4*>(wl + tap * D + c0), *reinterpret_cast<const f32x4*>(wl + tap * D + c0 + 4)};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              y[c] = fmaf(wt[c / 4][c % 4], c % 2 ? bf16_hi_to_f32(x[c / 4][(c % 4) / 2]) : bf16_lo_to_f32(x[c / 4][(c % 4) / 2]), y[c]);
            }
          }
        }
        *reinterpret_cast<u32x4*>(gout + (int64_t)(tok0 + r) * a.st + c0) =
            u32x4{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]), pack_bf16x2(y[6], y[7])};
      }
    }
  }
}

// Workgroups per group.  As many as get a compute unit each (a workgroup takes most of one's LDS), with those that hand on the
// state; two also where the last few have to wait.  Only where the plan has one group per segment: from 128 workgroups on the chip is
// half full anyway.  Measured, us a call of 63 taps, 1 / 2 / 4 / 8 parts: d = 128: 4 heads, 200 tokens 31.7 / 17.8 / 16.1 / 15.6, 4 heads, 1500
// 41.4 / 34.4 / 30.5 / 29.9; 8 heads: 1000 tokens (8 parts: 264 workgroups) 43.1 / 35.6 / 31.6 / 38.7, 1300 43.1 / 38.3 / 34.3 / 43.3, 2000
// 45.2 / 38.6 / 41.2 / 51.9, 4000 53.5 / 51.2 / 59.6 / 79.6; 24 heads, 1200 tokens 51.9 / 49.8 / 51.7 / 70.8; 40 heads, 100 tokens
// 34.9 / 19.7 / 19.1 / 19.2; d = 64: 4 heads, 400 tokens 26.6 / 22.8 / 21.4 / 20.9, 8 heads, 1000 27.9 / 23.5 / 22.2 / 25.3, 2000 27.9 / 24.0 /
// 26.0 / 31.5, 4000 31.8 / 30.5 / 36.2 / 46.4.
int prefill_grouped256_parts(const PrefillArgs& a) {
  const int64_t heads = (int64_t)a.B * a.H, groups = (a.L + 255) / 256;
  if (a.L <= 0 || a.nseg != groups) return 1;
  // without segments the incoming state and history are read where they are: not while another workgroup writes over them
  if (a.nseg == 1 && ((a.S_in && a.S_in == a.S_out) || (a.z_in && a.z_in == a.z_out) || (a.hist_in && a.hist_in == a.hist_out))) return 1;
  for (int p = 8; p > 2; p /= 2)
    if (heads * ((a.L + 256 / p - 1) / (256 / p) + (a.S_out || a.z_out || a.hist_out)) <= 256) return p;
  return heads * groups <= 128 ? 2 : 1;
}

template <int D, int KCM, int P>
static hipError_t launch_split(const PrefillArgs& a, hipStream_t st) {
  using G = G256SCfg<D>;
  auto kern = prefill_grouped256_split_kernel<D, KCM, P>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, G::TOTAL);
  if (e != hipSuccess) return e;
  const int heads = a.B * a.H;
  hipLaunchKernelGGL(kern, dim3((unsigned)(P * heads * a.nseg + (a.S_out || a.z_out || a.hist_out ? heads : 0))), dim3(G::NT), G::TOTAL, st, a);
  return hipGetLastError();
}
template <int D, int KCM>
static hipError_t launch_split_p(const PrefillArgs& a, int parts, hipStream_t st) {
  return parts == 8 ? launch_split<D, KCM, 8>(a, st) : parts == 4 ? launch_split<D, KCM, 4>(a, st) : launch_split<D, KCM, 2>(a, st);
}
template <int D>
static hipError_t launch_split_d(const PrefillArgs& a, int parts, hipStream_t st) {
  if (a.no_conv) return launch_split_p<D, 0>(a, parts, st);
  // (as many tap counts as prefill_grouped256.hip: a tap that does not exist weighs its row with 0, and 0 times an infinity is a NaN)
  return a.Kc <= 3 ? launch_split_p<D, 3>(a, parts, st) : a.Kc <= 5 ? launch_split_p<D, 5>(a, parts, st) : launch_split_p<D, 8>(a, parts, st);
}
hipError_t launch_prefill_grouped256_split(const PrefillArgs& a, int d, int parts, hipStream_t st) {
  return d == 128 ? launch_split_d<128>(a, parts, st) : launch_split_d<64>(a, parts, st);
}

}  // namespace linattn
