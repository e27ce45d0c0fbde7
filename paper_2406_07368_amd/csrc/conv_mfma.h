// The work of one workgroup of the convolution on the matrix cores (conv_mfma.hip says what it computes and how), for the
// kernels of that file and for the gradient's dq kernel, which takes such workgroups along where few run.
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

namespace linattn {

namespace {
constexpr int CM_SUB = 256;                                // tokens of one 16 x 16 tile; a workgroup takes one or two
constexpr int CM_SKEW = 16;                                // dwords per 8 channels
typedef uint32_t __attribute__((may_alias)) u32_any;      // dwords of an array that is written in 16-bit pieces
typedef uint16_t __attribute__((may_alias)) u16_any;      // and the other way round
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
enum { CM_ASSIGN = 0, CM_ADD = 1, CM_BWD = 2 };

template <int KS, int MODE, int T, int CB, int NW>   // NW: waves; channels are dealt out over them
struct ConvCfg {
  static constexpr int OFF = 32 * KS - 16;                 // tokens beyond the block that the taps reach; taps <= OFF + 1
  static constexpr int NB = KS == 1 ? 2 : KS == 2 ? 4 : 5; // 16-token lags of the tap gradient
  static constexpr int VOFF = 16 * (NB - 1);
  static constexpr int XN = 32 * KS + 16;                  // Toeplitz line of the taps: entry x, contraction index k, row i: x = k - i + 15
  static constexpr int XD = (T + OFF) / 2;            // dwords per channel
  static constexpr int VD = MODE == CM_BWD ? (T + VOFF) / 2 : MODE == CM_ADD ? T / 2 : 0;
  static_assert(XD % 8 == 0 && VD % 8 == 0, "bank skew");
  static constexpr int X = 0;
  static constexpr int V = X + CB * XD + CM_SKEW * (CB / 8);            // value rows (backward), low halves of the results (add)
  static constexpr int W = V + (VD ? CB * VD + CM_SKEW * (CB / 8) : 0); // per wave: [2 copies][3 terms][XN] u16
  static constexpr int ED = MODE == CM_BWD ? 4 * 80 : 0;                      // backward: the tap sums' rows, [4][80] float, in the same place
  static constexpr int WB = ((3 * XN / 2 + 31) / 64) * 64 + 32;              // the copy shifted by one entry: other banks than the first
  static constexpr int WLEN = WB + 3 * XN / 2;
  static constexpr int WD = WLEN > ED ? WLEN : ED;
  static constexpr int ODD = W + NW * WD;                // [waves]: rows that are not finite
  static constexpr int TOTAL = ODD + NW;                // dwords
};

__device__ __forceinline__ int cm_row(int c, int dwords) { return c * dwords + (c >> 3) * CM_SKEW; }
// two tokens of two channels: (a = token 0, b = token 1; two channels each) -> channel 0's pair, channel 1's pair; and back
__device__ __forceinline__ uint32_t low_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t high_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// lane s of a row of 16 reads lane s + N (SHL) or s - N (SHR); 0 from outside the row
template <int N>
__device__ __forceinline__ float row_shl(float x) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x100 + N, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ float row_shr(float x) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), 0x110 + N, 0xf, 0xf, true));
}

// Rows tok0 .. tok0 + 2 NP - 1 of CB channels on their way to LDS: requested, then turned around and stored.
template <int NP, int CB, int NT>
struct RowPairs {
  static constexpr int NG = CB / 8, PPI = NT / NG, IT = (NP + PPI - 1) / PPI;
  u32x4 x[IT][2];
  // row(tok, &ok): the memory row of a token and whether it exists (a row that does not is requested all the same)
  template <typename Row>
  __device__ __forceinline__ void request(int tok0, int tid, Row row) {
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int p = tid / NG + PPI * i;
        bool ok;
        const uint16_t* r = row(tok0 + 2 * (p < NP ? p : NP - 1) + u, ok);
        const u32x4 y = *reinterpret_cast<const u32x4*>(r + 8 * (tid % NG));
        x[i][u] = y;
      }
  }
  // returns whether one of the thread's elements is an infinity or a NaN
  template <typename Row>
  __device__ __forceinline__ bool store(uint32_t* lds, int dwords, int tok0, int tid, Row row) {
    const int g = tid % NG;
    u16x2 top = {0, 0};
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int p = tid / NG + PPI * i;
      bool ok0, ok1;
      row(tok0 + 2 * p, ok0);
      row(tok0 + 2 * p + 1, ok1);
      if (p < NP) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t a = ok0 ? x[i][0][e] : 0u, b = ok1 ? x[i][1][e] : 0u;
          lds[cm_row(8 * g + 2 * e, dwords) + p] = low_halves(a, b);
          lds[cm_row(8 * g + 2 * e + 1, dwords) + p] = high_halves(a, b);
          top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, a & 0x7fff7fffu));
          top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, b & 0x7fff7fffu));
        }
      }
    }
    return top[0] >= 0x7f80 || top[1] >= 0x7f80;
  }
};
}  // namespace

// workgroup (bx, by) of dim3(token blocks x channel blocks, B H m)
template <int D, int KS, int MODE, int T, int CB, int NW>
__device__ __forceinline__ void conv_mfma_workgroup(const ConvLongArgs& a, int bx, int by, uint32_t* smu) {
  using G = ConvCfg<KS, MODE, T, CB, NW>;
  constexpr int NT = 64 * NW;
  constexpr int CPW = CB / NW;                          // channels per wave
  constexpr bool BWD = MODE == CM_BWD;
  uint32_t* Xl = smu + G::X;
  uint32_t* Vl = smu + G::V;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, col = lane & 15, q = lane >> 4;
  uint16_t* wl = reinterpret_cast<uint16_t*>(smu + G::W + w * G::WD);
  float* el = reinterpret_cast<float*>(wl);

  // CB channels of one (b, h, value block)
  const int bh = by / a.m, b = bh / a.H, h = bh % a.H;
  // Block indices 8 apart land on the same chiplet.  The channel blocks of a token block share its memory lines and
  // neighbouring token blocks share rows, so both are kept on one chiplet, close together in time (when the number of
  // token blocks is a multiple of 8; otherwise the channel blocks of a token block lie side by side).
  constexpr int CBLK = D / CB;
  const int nblk = (a.L + T - 1) / T;
  const int seq = nblk % 8 == 0 ? bx >> 3 : bx;
  const int tblk = seq / CBLK + (nblk % 8 == 0 ? (bx & 7) * (nblk >> 3) : 0);
  const int DVT = a.m * D, cblk = seq % CBLK * CB, ch0 = (by % a.m) * D + cblk;
  const int t0 = tblk * T;
  const int L = a.L, Kc = a.Kc, R = Kc - 1;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh + ch0;
  const int64_t hist_base = (int64_t)bh * R * DVT + ch0;
  const uint16_t* gx = static_cast<const uint16_t*>(a.v) + base;             // backward: the gradient rows
  uint16_t* go = static_cast<uint16_t*>(a.out) + base;

  // ---- every request of the workgroup: rows, taps ------------------------------------------------------------------
  auto x_row = [&](int tok, bool& ok) __attribute__((always_inline)) {
    const bool in_hist = !BWD && tok < 0 && a.hist_in != nullptr && R + tok >= 0;
    ok = (tok >= 0 && tok < L) || in_hist;
    return in_hist ? static_cast<const uint16_t*>(a.hist_in) + hist_base + (int64_t)(R + tok) * DVT
                   : gx + (int64_t)((tok >= 0 && tok < L) ? tok : 0) * a.st;
  };
  const uint16_t* gv = BWD ? static_cast<const uint16_t*>(a.dw_v) + base : nullptr;
  auto v_row = [&](int tok, bool& ok) __attribute__((always_inline)) {
    ok = tok >= 0 && tok < L;
    return gv + (int64_t)(ok ? tok : 0) * a.st;
  };
  const int x0 = BWD ? t0 : t0 - G::OFF;                   // first token of the rows at hand
  RowPairs<G::XD, CB, NT> xr;
  xr.request(x0, tid, x_row);
  [[maybe_unused]] RowPairs<BWD ? G::VD : 1, CB, NT> vr;
  if constexpr (BWD) vr.request(t0 - G::VOFF, tid, v_row);
  const float* wsrc = a.conv_w + ((size_t)h * DVT + ch0 + w * CPW) * Kc + (lane < Kc ? lane : 0);
  float tap = wsrc[0];
  for (int i = lane; i < G::WD; i += 64) reinterpret_cast<u32_any*>(wl)[i] = 0u;

  const int odd_rows = __any(xr.store(Xl, G::XD, x0, tid, x_row));
  if (lane == 0) smu[G::ODD + w] = odd_rows;
  if constexpr (BWD) vr.store(Vl, G::VD, t0 - G::VOFF, tid, v_row);
  // the history handed on, by the workgroups that own its rows (the launcher sees to it that nobody still reads it)
  if (!BWD && a.hist_fused) {
#pragma unroll
    for (int i = 0; i < xr.IT; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int p = tid / xr.NG + xr.PPI * i, tok = x0 + 2 * p + u, r = tok - (L - R);
        bool ok;
        x_row(tok, ok);
        if (p < G::XD && tok < L && r >= 0 && (tok >= t0 || t0 == 0))
          *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(a.hist_out) + hist_base + (int64_t)r * DVT + 8 * (tid % xr.NG)) =
              ok ? xr.x[i][u] : u32x4{0, 0, 0, 0};
      }
  }
  __syncthreads();

  // A row of the Toeplitz operand also holds the zeros of the tokens that an output does not see, and 0 times an infinity or a
  // NaN is a NaN: a workgroup that has met such an element sums its outputs tap by tap on the vector ALUs (rare).
  uint32_t odd = 0;
#pragma unroll
  for (int v = 0; v < NW; ++v) odd |= smu[G::ODD + v];
  const bool by_tap = odd != 0;

  // Toeplitz operand: lane (i = col, q) takes entries x = 8q + 32ks - i + 15 + 0..7 of the tap line; odd starts read the
  // copy that is shifted by one entry, so that every read is whole dwords
  const int xs = 8 * q - col + 15;
  const u32_any* wop = reinterpret_cast<const u32_any*>(wl) + (xs & 1 ? G::WB : 0) + (xs >> 1);
  const int at = BWD ? lane + 15 : G::OFF + 15 - lane;     // where this lane's tap sits in the line
  auto channels = [&](auto taps_alone) __attribute__((always_inline)) {
#pragma unroll 1
    for (int cc = 0; cc < CPW; ++cc) {
      const int c = w * CPW + cc;
      uint32_t* xrow = Xl + cm_row(c, G::XD);
      if constexpr (BWD) {
        if (a.dw_part) {                                     // uniform
          // D_b[i][r] = sum over the blocks a of dO[16a + i] v[16(a + b) - VOFF + r]: lag 16(NB-1-b) + i - r
          const uint16_t* grow = reinterpret_cast<const uint16_t*>(xrow) + 4 * lane;
          const uint16_t* vrow = reinterpret_cast<const uint16_t*>(Vl + cm_row(c, G::VD)) + 4 * lane;
          f32x4 dacc[G::NB];
#pragma unroll
          for (int bb = 0; bb < G::NB; ++bb) dacc[bb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int sub = 0; sub < T / CM_SUB; ++sub) {
            const s16x4 ga = __builtin_bit_cast(s16x4, lds_tr4(grow + CM_SUB * sub));
#pragma unroll
            for (int bb = 0; bb < G::NB; ++bb)
              dacc[bb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ga, __builtin_bit_cast(s16x4, lds_tr4(vrow + CM_SUB * sub + 16 * bb)), dacc[bb], 0, 0, 0);
          }
          // register e of row q: i = 4q + e.  Shifted by e lanes, every register has lag 16(NB-1-b) + 4q - s in lane s; what
          // leaves the row belongs to the block of the next larger lag (beyond the last tap for block 0)
#pragma unroll
          for (int bb = 0; bb < G::NB; ++bb) {
            float y = dacc[bb][0] + row_shl<1>(dacc[bb][1]) + row_shl<2>(dacc[bb][2]) + row_shl<3>(dacc[bb][3]);
            if (bb + 1 < G::NB) y += row_shr<15>(dacc[bb + 1 < G::NB ? bb + 1 : bb][1]) + row_shr<14>(dacc[bb + 1 < G::NB ? bb + 1 : bb][2]) +
                                     row_shr<13>(dacc[bb + 1 < G::NB ? bb + 1 : bb][3]);
            el[80 * q + 16 * (G::NB - 1 - bb) - col + 15] = y;
          }
          if (lane < Kc) {
            float y = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) y += el[80 * r + lane - 4 * r + 15];
            a.dw_part[((((size_t)h * a.B + b) * nblk + tblk) * D + ch0 + c) * Kc + lane] = y;
          }
          // the tap line takes its place back (its entries around the taps are zeros)
          asm volatile("" ::: "memory");
          for (int i = lane; i < G::WLEN; i += 64) reinterpret_cast<u32_any*>(wl)[i] = 0u;
          asm volatile("" ::: "memory");
        }
      }
      if (lane < Kc) {
        // (cut, not rounded: a tap at the end of the range stays finite; an infinity has no rest)
        const uint16_t w1 = (uint16_t)(__float_as_uint(tap) >> 16);
        const float r1 = __builtin_isinf(tap) ? 0.f : tap - bf16_bits_to_f32(w1);
        const uint16_t w2 = (uint16_t)(__float_as_uint(r1) >> 16);
        const uint16_t w3 = (uint16_t)(__float_as_uint(r1 - bf16_bits_to_f32(w2)) >> 16);
        const uint16_t t3[3] = {w1, w2, w3};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          wl[G::XN * t + at] = t3[t];
          wl[2 * G::WB + G::XN * t + at - 1] = t3[t];        // at >= 15
        }
      }
      tap = wsrc[(cc + 1 < CPW ? cc + 1 : cc) * Kc];
      bf16x8 wf[3][KS];
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const u32_any* p = wop + G::XN / 2 * t + 16 * ks;
          wf[t][ks] = __builtin_bit_cast(bf16x8, u32x4{p[0], p[1], p[2], p[3]});
        }
#pragma unroll
      for (int sub = 0; sub < T / CM_SUB; ++sub) {
        uint32_t* xs_row = xrow + CM_SUB / 2 * sub;
        f32x4 u1 = {0.f, 0.f, 0.f, 0.f}, u2 = u1, u3 = u1;
        if constexpr (decltype(taps_alone)::value) {
          const u16_any* xe = reinterpret_cast<const u16_any*>(xs_row) + 16 * col + 4 * q + (BWD ? 0 : G::OFF);
          const float* wc = a.conv_w + ((size_t)h * DVT + ch0 + c) * Kc;
#pragma unroll 1
          for (int j = 0; j < Kc; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) u1[i] = fmaf(wc[j], bf16_bits_to_f32(xe[BWD ? i + j : i - j]), u1[i]);
        } else {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 xb = *reinterpret_cast<const bf16x8*>(xs_row + 8 * col + 4 * q + 16 * ks);
            u1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[0][ks], xb, u1, 0, 0, 0);
            u2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[1][ks], xb, u2, 0, 0, 0);
            u3 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[2][ks], xb, u3, 0, 0, 0);
          }
          u1 += u2 + u3;
        }
        // tokens 16col + 4q + 0..3 of the tile: over the row they came from (nobody else reads it, and this wave is done
        // with this part of it)
        u32x2 hv;
        if constexpr (MODE == CM_ADD) {                      // the fp32 sum in two halves: it is rounded when out is added
          u32x2 lv;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const uint32_t x = __float_as_uint(u1[2 * i]), y = __float_as_uint(u1[2 * i + 1]);
            hv[i] = high_halves(x, y);
            lv[i] = low_halves(x, y);
          }
          *reinterpret_cast<u32x2*>(Vl + cm_row(c, G::VD) + CM_SUB / 2 * sub + 8 * col + 2 * q) = lv;
        } else {
          hv = u32x2{pack_bf16x2(u1[0], u1[1]), pack_bf16x2(u1[2], u1[3])};
        }
        *reinterpret_cast<u32x2*>(xs_row + 8 * col + 2 * q) = hv;
      }
    }
  };
  if (by_tap) channels(std::true_type{});                  // uniform
  else channels(std::false_type{});

  // ---- whole rows out ------------------------------------------------------------------------------------------------
  constexpr int NG = CB / 8, PPI = NT / NG, OIT = (T / 2 + PPI - 1) / PPI;
  const int g = tid % NG;
  [[maybe_unused]] u32x4 held[OIT][2];
  if constexpr (MODE == CM_ADD) {
#pragma unroll
    for (int i = 0; i < OIT; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int tok = t0 + 2 * (tid / NG + PPI * i) + u;
        held[i][u] = *reinterpret_cast<const u32x4*>(go + (int64_t)(tok < L ? tok : L - 1) * a.st + 8 * g);
      }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < OIT; ++i) {
    const int p = tid / NG + PPI * i;
    if (T / 2 % PPI != 0 && p >= T / 2) break;
    uint32_t d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = Xl[cm_row(8 * g + e, G::XD) + p];
    u32x4 o[2];
    if constexpr (MODE == CM_ADD) {
      float y[2][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t lo = Vl[cm_row(8 * g + e, G::VD) + p];
        y[0][e] = __uint_as_float(low_halves(lo, d[e]));
        y[1][e] = __uint_as_float(high_halves(lo, d[e]));
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[u][e] = pack_bf16x2(y[u][2 * e] + bf16_lo_to_f32(held[i][u][e]), y[u][2 * e + 1] + bf16_hi_to_f32(held[i][u][e]));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[0][e] = low_halves(d[2 * e], d[2 * e + 1]);
        o[1][e] = high_halves(d[2 * e], d[2 * e + 1]);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int tok = t0 + 2 * p + u;
      if (tok < L) *reinterpret_cast<u32x4*>(go + (int64_t)tok * a.st + 8 * g) = o[u];
    }
  }
}

}  // namespace linattn
