// The group-level sums of the three-branch form (Sec. 4.1), walked in one launch:
//
//   forward    slot[g] = sums over everything before group g of phi(k) v^T and phi(k)          (S_g, z_g)
//   backward   slot[g] = sums over everything after group g of f phi(q) dO^T and dden phi(q)   (their gradients)
//
// One workgroup walks one (b, h) for 32 features (D = 64: all 64) in four 32 x 32 tiles of the sums (lane = channel,
// registers = features), a wave each (groups of 256: two, see below), in accumulator registers from the first group to the
// last; at the start of every group they go to the group's slot as they are.  Rows come 128 tokens at a time (64 in groups of
// 64), requested two steps ahead into registers; on their way into one of two LDS buffers the left rows get the feature map and their weight and are
// split into two bf16 terms (hi = bf16(x), lo = bf16(x - hi)): once per element, where making the operand as it is read
// would repeat it in every wave.  Both operands are then transpose reads; the vector part is summed in fp32 by the
// threads that map the rows.
// What bounds it: the traffic, every row once from memory (the four workgroups of a head are neighbours on one chiplet and
// share the right rows through its L2: FETCH_SIZE counts them once) and one slot per group written and never read back by a
// prefix sum.  On B8 H8 L8192 d128 in groups of 256 either direction takes 117 us for 403 MB (one workgroup per group and
// the prefix sum: 165 us).  Two waves share a tile in groups of 256: with one wave per SIMD nothing covered the mapping of the
// rows and the LDS reads (145 us; 167 us with the rows requested one step ahead instead of two).
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

namespace linattn {

namespace {
template <int D, int GT>
struct SumsCfg {
  static constexpr int FW = D == 128 ? 32 : 64;            // features per workgroup
  static constexpr int CT = GT < 128 ? GT : 128;           // tokens per step
  static constexpr int CPG = GT / CT;                      // steps per group
  static constexpr int AP = FW / 8, BP = D / 8;            // 16-byte pieces per row
  static constexpr int KH = GT == 256 ? 2 : 1;             // waves per tile: the steps' tokens dealt out between them
  static constexpr int NT = 256 * KH;
  static constexpr int AI = CT * AP / NT, BI = CT * BP / NT;     // pieces per thread
  static constexpr int AS = FW == 32 ? 48 : 72, BS = D + 16;     // row strides: four rows of a transpose read on different banks
  static constexpr int A = 0;                              // [2 buffers][hi, lo][CT][AS]
  static constexpr int B = A + 4 * CT * AS * 2;            // [2][CT][BS]
  static constexpr int ZR = B + 2 * CT * BS * 2;           // [2][waves][FW] float
  static constexpr int CO = ZR + 2 * 4 * KH * FW * 4;      // [4 tiles][16][64] float: what the second wave of a tile summed up
  static constexpr int TOTAL = CO + (KH - 1) * 4 * 16 * 64 * 4;
  static constexpr int SLOT = D * D + D;
  static_assert(TOTAL <= 160 * 1024 && AI >= 1 && BI >= 1, "LDS, pieces");
};
}  // namespace

template <int D, int GT, bool BACK>
__global__ __launch_bounds__(GT == 256 ? 512 : 256) void group_sums_kernel(GroupSumsArgs a) {
  using G = SumsCfg<D, GT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* Al = reinterpret_cast<uint16_t*>(smem + G::A);
  uint16_t* Bl = reinterpret_cast<uint16_t*>(smem + G::B);
  float* zred = reinterpret_cast<float*>(smem + G::ZR);
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  // The D / FW workgroups of a head get block indices 8 apart (the same chiplet) while there are whole eights of heads.
  constexpr int NF = D / G::FW;
  const int full = a.B * a.H / 8 * 8, bx = blockIdx.x;
  const int bh = bx < full * NF ? (bx & 7) + bx / (8 * NF) * 8 : full + (bx - full * NF) / NF;
  const int fb = bx < full * NF ? (bx >> 3) % NF : (bx - full * NF) % NF;
  const int b = bh / a.H, h = bh % a.H;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const uint16_t* ga = static_cast<const uint16_t*>(a.a) + base + fb * G::FW;
  const uint16_t* gb = static_cast<const uint16_t*>(a.b) + base;
  const float* gw = BACK ? a.w + (size_t)bh * a.L : nullptr;
  const float* gwz = BACK ? a.wz + (size_t)bh * a.L : nullptr;
  float* slots = a.slots + (size_t)bh * a.ng * G::SLOT;
  const float one = a.relu ? 0.f : 1.f;
  // this wave's tile: features f0 .. f0 + 31, channels c0 .. c0 + 31
  const int wt4 = w & 3, kh = w >> 2;                      // tile, and which part of a step's tokens
  const int fl = D == 128 ? 0 : 32 * (wt4 >> 1);           // within the workgroup's features
  const int f0 = fb * G::FW + fl, c0 = 32 * (D == 128 ? wt4 : wt4 & 1);

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int zf = fb * G::FW + tid;                         // threads below FW: the feature whose vector part they carry
  float zrun = 0.f;

  // group of step s, first token of step s
  auto group_of = [&](int s) __attribute__((always_inline)) { return BACK ? a.ng - 1 - s / G::CPG : s / G::CPG; };
  auto token_of = [&](int s) __attribute__((always_inline)) { return group_of(s) * GT + s % G::CPG * G::CT; };
  struct Rows { u32x4 a[G::AI], b[G::BI]; float w[G::AI], wz[G::AI]; };
  auto request = [&](int s, Rows& x) __attribute__((always_inline)) {
    const int t0 = token_of(s);
#pragma unroll
    for (int i = 0; i < G::AI; ++i) {
      const int e = tid + G::NT * i, tok = t0 + e / G::AP;
      const int64_t t = tok < a.L ? tok : a.L - 1;         // unconditional; a row that does not exist gets weight zero
      x.a[i] = *reinterpret_cast<const u32x4*>(ga + t * a.st + 8 * (e % G::AP));
      if constexpr (BACK) { x.w[i] = gw[t]; x.wz[i] = gwz[t]; }
    }
#pragma unroll
    for (int i = 0; i < G::BI; ++i) {
      const int e = tid + G::NT * i, tok = t0 + e / G::BP;
      x.b[i] = *reinterpret_cast<const u32x4*>(gb + (int64_t)(tok < a.L ? tok : a.L - 1) * a.st + 8 * (e % G::BP));
    }
  };
  float zacc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) zacc[e] = 0.f;
  // the rows of step s, mapped, weighed and split, to their buffer; at the end of a group its vector part to zred
  auto place = [&](int s, const Rows& x) __attribute__((always_inline)) {
    const int buf = s & 1, t0 = token_of(s);
    uint16_t* Ah = Al + buf * 2 * G::CT * G::AS;
    uint16_t* Bh = Bl + buf * G::CT * G::BS;
#pragma unroll
    for (int i = 0; i < G::AI; ++i) {
      const int e = tid + G::NT * i, row = e / G::AP;
      const bool is = t0 + row < a.L;
      const float wt = is ? (BACK ? x.w[i] : 1.f) : 0.f, wzt = is ? (BACK ? x.wz[i] : 1.f) : 0.f;
      u32x4 xh, xl;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float p0 = phi_nb(bf16_lo_to_f32(x.a[i][j]), one), p1 = phi_nb(bf16_hi_to_f32(x.a[i][j]), one);
        zacc[2 * j] = fmaf(p0, wzt, zacc[2 * j]);
        zacc[2 * j + 1] = fmaf(p1, wzt, zacc[2 * j + 1]);
        const float y0 = p0 * wt, y1 = p1 * wt;
        xh[j] = pack_bf16x2(y0, y1);
        xl[j] = pack_bf16x2(y0 - bf16_lo_to_f32(xh[j]), y1 - bf16_hi_to_f32(xh[j]));
      }
      uint16_t* p = Ah + row * G::AS + 8 * (e % G::AP);
      *reinterpret_cast<u32x4*>(p) = xh;
      *reinterpret_cast<u32x4*>(p + G::CT * G::AS) = xl;
    }
#pragma unroll
    for (int i = 0; i < G::BI; ++i) {
      const int e = tid + G::NT * i, row = e / G::BP;
      *reinterpret_cast<u32x4*>(Bh + row * G::BS + 8 * (e % G::BP)) = t0 + row < a.L ? x.b[i] : u32x4{0, 0, 0, 0};
    }
    if ((s + 1) % G::CPG == 0) {                           // uniform: over the lanes that map the same features, then the waves
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float y = add_xor8(zacc[e]);
        if (G::AP == 4) y = dpp_add<0x124>(y);             // rotation by 4 inside a row of 16
        y = add_xor32(add_xor16(y));
        if (lane < G::AP) zred[(buf * 4 * G::KH + w) * G::FW + 8 * lane + e] = y;
        zacc[e] = 0.f;
      }
    }
  };
  auto write_slot = [&](int g) __attribute__((always_inline)) {
    float* so = slots + (size_t)g * G::SLOT;
    if (kh == 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) so[(f0 + 8 * (r >> 2) + 4 * hi + (r & 3)) * D + c0 + l32] = acc[r];
    if (tid < G::FW) so[D * D + zf] = zrun;
  };

  // the second wave's part of the sums joins the first's: left in LDS behind a group's products, taken behind the barrier
  float* co = reinterpret_cast<float*>(smem + G::CO) + wt4 * 1024 + lane;
  auto leave = [&]() __attribute__((always_inline)) {
    if (G::KH > 1 && kh == 1)
#pragma unroll
      for (int r = 0; r < 16; ++r) { co[64 * r] = acc[r]; acc[r] = 0.f; }
  };
  auto take = [&]() __attribute__((always_inline)) {
    if (G::KH > 1 && kh == 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += co[64 * r];
  };
  // Step s: its products, and between them the rows of step s + 1 on their way to the other buffer and the requests of
  // step s + 3 (two steps of rows are in registers: with one wave per SIMD nothing else hides a trip to memory).
  auto step = [&](int s, int steps, Rows& x) __attribute__((always_inline)) {
    const int buf = s & 1;
    const uint16_t* Ah = Al + buf * 2 * G::CT * G::AS;
    const uint16_t* Bh = Bl + buf * G::CT * G::BS;
    if (s % G::CPG == 0) {
      if (s > 0) take();
      write_slot(group_of(s));
    }
    if ((s + 1) % G::CPG == 0 && tid < G::FW) {
#pragma unroll
      for (int v = 0; v < 4 * G::KH; ++v) zrun += zred[(buf * 4 * G::KH + v) * G::FW + tid];
    }
#pragma unroll
    for (int k1 = 0; k1 < G::CT / 16 / G::KH; ++k1) {
      const int ks = kh * (G::CT / 16 / G::KH) + k1;
      const bf16x8 bop = tr_operand(Bh, G::BS, 16 * ks, c0, lane);
      acc = mfma(tr_operand(Ah, G::AS, 16 * ks, fl, lane), bop, acc);
      acc = mfma(tr_operand(Ah + G::CT * G::AS, G::AS, 16 * ks, fl, lane), bop, acc);
    }
    if ((s + 1) % G::CPG == 0) leave();
    if (s + 1 < steps) place(s + 1, x);
    if (s + 3 < steps) request(s + 3, x);
    __syncthreads();
  };
  const int steps = (a.ng - 1) * G::CPG;                   // nothing follows the last group of the walk
  if (steps > 0) {
    Rows x0, x1;
    request(0, x1);
    if (steps > 1) request(1, x0);
    place(0, x1);
    if (steps > 2) request(2, x1);
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {
      step(s, steps, x0);
      if (s + 1 < steps) step(s + 1, steps, x1);
    }
  }
  if (steps > 0) take();
  write_slot(group_of(steps));
}

template <int D, int GT, bool BACK>
static hipError_t launch_sums_one(const GroupSumsArgs& a, hipStream_t st) {
  using G = SumsCfg<D, GT>;
  auto kern = group_sums_kernel<D, GT, BACK>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, G::TOTAL);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * a.H * (D / G::FW))), dim3(G::NT), G::TOTAL, st, a);
  return hipGetLastError();
}
template <int D, int GT>
static hipError_t launch_sums_dir(const GroupSumsArgs& a, bool back, hipStream_t st) {
  return back ? launch_sums_one<D, GT, true>(a, st) : launch_sums_one<D, GT, false>(a, st);
}

// Against one workgroup per group and a prefix sum over the slots, which has no chain over the groups but moves every slot
// three times: the walk pays with workgroups for half the chip (groups of 64: three quarters), or few groups.  Measured, us
// per gradient call, per-group kernels / walk.  Few heads, by the number of groups: groups of 64, 8 heads: D = 64: 4 62 / 60, 5
// 73 / 68, 6 61 / 66; D = 128: 4 81 / 72, 5 81 / 74, 6 82 / 78, 8 84 / 83, 12 85 / 96; groups of 256: D = 64: 3 79 / 75, 4 80 / 81, 5 81 / 87;
// D = 128: 4 110 / 99, 5 111 / 106, 6 111 / 111, 8 112 / 123.  Many groups, by the number of heads: groups of 256, D = 128, 32
// groups: 8 heads 179 / 295, 32 heads 645 / 615; D = 64, 16 groups of 48 heads (48 workgroups) 248 / 279; groups of 64, D = 128, 64
// groups: 32 heads 426 / 456, 64 heads 851 / 712.
bool group_sums_pays(int heads, int ng, int d, int group) {
  return ng <= (d == 64 && group == 256 ? 4 : 5) || heads * (d == 128 ? 4 : 1) >= (group == 256 ? 128 : 192);
}

hipError_t launch_group_sums(const GroupSumsArgs& a, int d, int group, bool back, hipStream_t st) {
  if (d == 128) return group == 256 ? launch_sums_dir<128, 256>(a, back, st) : launch_sums_dir<128, 64>(a, back, st);
  return group == 256 ? launch_sums_dir<64, 256>(a, back, st) : launch_sums_dir<64, 64>(a, back, st);
}

}  // namespace linattn
