// The three-branch form of Sec. 4.1 for fp32 rows in groups of 256 tokens, with fp32 arithmetic on the vector ALUs.  (fp32
// rows in groups of 64, and the token-level form, run on the fp32 matrix instructions: prefill_f32.hip.)
#include "common.h"
#include "kernels.h"

namespace linattn {

namespace {
constexpr int HMAX = 7;            // history rows kept in LDS: enough for the largest conv kernel (8 taps)
constexpr int D = 64, GCT = 256;   // rows and groups (rows of 128 in groups of 256 would need 266 KB of LDS: no kernel)
typedef IoF32 Io;
}  // namespace

// The three-branch form (grouped linear attention over the groups before a token's own, weight alpha + causal
// softmax attention inside its group + masked conv) with fp32 arithmetic.
// One workgroup walks one (b, h) group by group and, inside a group, token by token; S and z are only advanced
// at the end of a group, which is exactly what the linear branch is defined on.  The state sits in registers
// (thread (c, tg) holds S[i][c] for i = tg, tg + NG, ...), the group's raw key rows and value rows in LDS in
// the i/o dtype.  Exact to fp32 rounding; not built for speed.
namespace {
struct GroupedSimtLayout {
  typedef Io::elem elem;
  static constexpr int KSTR = D + 4 / (int)sizeof(elem);                  // key row stride: one 4-byte word of padding
  static constexpr int KR = 0;                                             // [GCT][KSTR] raw key rows of the group (elem)
  static constexpr int VV = KR + GCT * KSTR * (int)sizeof(elem);           // [HMAX+GCT][D]: history rows, then the group's value rows (elem)
  static constexpr int F0 = (VV + (HMAX + GCT) * D * (int)sizeof(elem) + 15) / 16 * 16;   // floats from here
  static constexpr int QR = 0;                        // [D] raw q_t
  static constexpr int FQ = QR + D;                   // [D] phi(q_t)
  static constexpr int LG = FQ + D;                   // [GCT] logits, then weights
  static constexpr int PART = LG + GCT;               // [256 / D][D] partial outputs
  static constexpr int ZZ = PART + 256;               // [D]
  static constexpr int SCAL = ZZ + D;                 // [16]: alpha / denominator; per-wave maxima and sums
  static constexpr int NFLOAT = SCAL + 16;
  static constexpr int TOTAL = F0 + NFLOAT * (int)sizeof(float);
};
}  // namespace

__global__ __launch_bounds__(256) void prefill_grouped_simt_kernel(PrefillArgs a) {
  using Lay = GroupedSimtLayout;
  typedef Io::elem elem;
  constexpr int NG = 256 / D;
  constexpr int NS = D / NG;                           // state rows per thread
  constexpr int KSTR = Lay::KSTR;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  elem* kr = reinterpret_cast<elem*>(smem + Lay::KR);
  elem* vv = reinterpret_cast<elem*>(smem + Lay::VV);
  float* fl = reinterpret_cast<float*>(smem + Lay::F0);
  float* qr = fl + Lay::QR;
  float* fq = fl + Lay::FQ;
  float* lg = fl + Lay::LG;
  float* part = fl + Lay::PART;
  float* zz = fl + Lay::ZZ;
  float* scal = fl + Lay::SCAL;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bh = blockIdx.x, b = bh / a.H, h = bh % a.H;
  const int Kc = a.Kc, L = a.L;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const int c = tid % D, tg = tid / D;
  static_assert(D == 64 || D == 128, "1 / sqrt(d) below");
  constexpr float inv_sqrt_d = D == 64 ? 0.125f : 0.08838834764831845f;

  float wreg[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) wreg[j] = (j < Kc && !a.no_conv) ? a.conv_w[((size_t)h * D + c) * Kc + j] : 0.f;
  float Sreg[NS];                                      // S[tg + NG m][c]
#pragma unroll
  for (int m = 0; m < NS; ++m) Sreg[m] = a.S_in ? a.S_in[(size_t)bh * D * D + (size_t)(tg + NG * m) * D + c] : 0.f;
  if (tid < D) zz[tid] = a.z_in ? a.z_in[(size_t)bh * D + tid] : 0.f;
  for (int e = tid; e < HMAX * D; e += 256) {
    const int row = e / D, cc = e % D;
    const int r = row - (HMAX - (Kc - 1));   // row of the incoming history, oldest first
    if (r >= 0 && a.hist_in) vv[e] = static_cast<const elem*>(a.hist_in)[((int64_t)bh * (Kc - 1) + r) * D + cc];
    else vv[e] = (elem)0;
  }
  __syncthreads();

  for (int t0 = 0; t0 < L; t0 += GCT) {
    const int nt = (L - t0) < GCT ? (L - t0) : GCT;
    // a. the group's raw key and value rows, as they are
    for (int e = tid; e < nt * D; e += 256) {
      const int t = e / D, i = e % D;
      const int64_t off = base + (int64_t)(t0 + t) * a.st + i;
      kr[t * KSTR + i] = static_cast<const elem*>(a.k)[off];
      vv[(HMAX + t) * D + i] = static_cast<const elem*>(a.v)[off];
    }
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      // b. the token's query, raw and under the feature map
      if (tid < D) {
        const float x = Io::load1(a.q, base + (int64_t)(t0 + t) * a.st + tid);
        qr[tid] = x;
        fq[tid] = phi_any(x, a.relu);
      }
      __syncthreads();
      // c. logits against the group's rows up to the token (four lanes per row); the linear normaliser
      for (int i0 = 0; i0 <= t; i0 += 64) {
        const int i = i0 + tid / 4, sub = tid % 4;
        float acc = 0.f;
        if (i <= t) {
          const elem* y = kr + i * KSTR + sub * (D / 4);
          const float* x = qr + sub * (D / 4);
#pragma unroll 8
          for (int f = 0; f < D / 4; ++f) acc = fmaf(x[f], y[f], acc);
        }
        acc += __shfl_xor(acc, 1);
        acc += __shfl_xor(acc, 2);
        if (sub == 0 && i < GCT) lg[i] = acc * inv_sqrt_d;
      }
      if (wave == 3) {                          // the last wave: phi(q_t).z
        float dz = 0.f;
        for (int f = lane; f < D; f += 64) dz = fmaf(fq[f], zz[f], dz);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) dz += __shfl_xor(dz, off);
        if (lane == 0) {
          const float gden = dz + a.eps;
          scal[0] = gden != 0.f ? a.alpha / gden : 0.f;
        }
      }
      __syncthreads();
      // d. softmax over rows 0..t, one row per thread: largest logit and mass over the workgroup
      {
        const bool seen = tid < GCT && tid <= t;
        const float x = seen ? lg[tid] : -INFINITY;
        float top = x;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
        if (lane == 0) scal[4 + wave] = top;
        __syncthreads();
        top = fmaxf(fmaxf(scal[4], scal[5]), fmaxf(scal[6], scal[7]));   // row 0 is always seen: finite
        const float p = seen ? __expf(x - top) : 0.f;
        float mass = p;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mass += __shfl_xor(mass, off);
        if (lane == 0) scal[8 + wave] = mass;
        __syncthreads();
        mass = (scal[8] + scal[9]) + (scal[10] + scal[11]);
        if (tid < GCT) lg[tid] = p / mass;
      }
      __syncthreads();
      // e. both branches for channel c, the features / rows dealt out over the NG thread groups
      {
        float lin = 0.f, loc = 0.f;
#pragma unroll
        for (int m = 0; m < NS; ++m) lin = fmaf(fq[tg + NG * m], Sreg[m], lin);
        for (int s2 = tg; s2 <= t; s2 += NG) loc = fmaf(lg[s2], vv[(HMAX + s2) * D + c], loc);
        part[tg * D + c] = fmaf(scal[0], lin, loc);
      }
      __syncthreads();
      if (tid < D) {
        float y = 0.f;
#pragma unroll
        for (int g = 0; g < NG; ++g) y += part[g * D + tid];
        float u = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (j < Kc) u = fmaf(wreg[j], vv[(HMAX + t - j) * D + tid], u);
        Io::store1(a.out, base + (int64_t)(t0 + t) * a.st + tid, y + u);
      }
      // the next token's step b writes qr, fq (read in c, e: both behind barriers by then); lg, part and scal are
      // written by the next token's c, d, e after barriers of their own
    }
    __syncthreads();
    // f. the group enters the sums: S += phi(K)^T V, z += colsum phi(K); the history slides forward by nt rows
    for (int s2 = 0; s2 < nt; ++s2) {
      const float x = vv[(HMAX + s2) * D + c];
#pragma unroll
      for (int m = 0; m < NS; ++m) Sreg[m] = fmaf(phi_any(kr[s2 * KSTR + tg + NG * m], a.relu), x, Sreg[m]);
    }
    if (tid < D) {
      float zs = zz[tid];
      for (int s2 = 0; s2 < nt; ++s2) zs += phi_any(kr[s2 * KSTR + tid], a.relu);
      zz[tid] = zs;
      for (int r = 0; r < HMAX; ++r) vv[r * D + tid] = vv[(r + nt) * D + tid];
    }
    __syncthreads();
  }

  if (a.S_out) {
#pragma unroll
    for (int m = 0; m < NS; ++m) a.S_out[(size_t)bh * D * D + (size_t)(tg + NG * m) * D + c] = Sreg[m];
  }
  if (a.z_out && tid < D) a.z_out[(size_t)bh * D + tid] = zz[tid];
  if (a.hist_out)
    for (int e = tid; e < (Kc - 1) * D; e += 256) {
      const int r = e / D, cc = e % D;
      static_cast<elem*>(a.hist_out)[((int64_t)bh * (Kc - 1) + r) * D + cc] = vv[(HMAX - (Kc - 1) + r) * D + cc];
    }
}

hipError_t launch_prefill_grouped_simt(const PrefillArgs& a, int d, hipStream_t st) {
  if (d != D || a.group != GCT) return hipErrorInvalidValue;
  constexpr int bytes = GroupedSimtLayout::TOTAL;
  static_assert(bytes <= 160 * 1024, "LDS");
  hipError_t e = LINATTN_MAX_LDS_ONCE(prefill_grouped_simt_kernel, bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(prefill_grouped_simt_kernel, dim3((unsigned)(a.B * a.H)), dim3(256), bytes, st, a);
  return hipGetLastError();
}

}  // namespace linattn
