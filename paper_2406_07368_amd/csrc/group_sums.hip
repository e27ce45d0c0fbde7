// The group-level sums of the three-branch form (Sec. 4.1), walked in one launch:
//
//   forward    slot[g] = sums over everything before group g of phi(k) v^T and phi(k)          (S_g, z_g)
//   backward   slot[g] = sums over everything after group g of f phi(q) dO^T and dden phi(q)   (their gradients)
//
// One workgroup walks one (b, h) for 32 features (D = 64: all 64) in four 32 x 32 tiles of the sums (lane = channel,
// registers = features), a wave each (groups of 256: two, see below), in accumulator registers from the first group to the
// last; at the start of every group they go to the group's slot as they are.  Where the heads are few, a workgroup has one tile
// and all its waves share a step's tokens (one_tile).  Rows come 128 tokens at a time (64 in groups of 64), requested two steps
// ahead into registers; on their way into one of two LDS buffers the left rows get the feature map and their weight and are split
// into two bf16 terms (hi = bf16(x), lo = bf16(x - hi)): once per element, where making the operand as it is read would repeat it
// in every wave.  Both operands are then transpose reads; the vector part is summed in fp32 by the
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
template <int D, int GT, int TILES>
struct SumsCfg {
  static constexpr int FW = D == 128 || TILES == 1 ? 32 : 64;    // features per workgroup
  static constexpr int CW = TILES == 1 ? 32 : D;           // channels per workgroup
  static constexpr int CT = GT < 128 ? GT : 128;           // tokens per step
  static constexpr int CPG = GT / CT;                      // steps per group
  static constexpr int AP = FW / 8, BP = CW / 8;           // 16-byte pieces per row
  static constexpr int KH = (GT == 256 ? 8 : 4) / TILES;   // waves per tile: the steps' tokens dealt out between them
  static constexpr int NWV = TILES * KH, NT = 64 * NWV;
  static constexpr int AI = CT * AP / NT, BI = CT * BP / NT;     // pieces per thread
  static constexpr int AS = FW == 32 ? 48 : 72, BS = CW + 16;    // row strides: four rows of a transpose read on different banks
  static constexpr int A = 0;                              // [2 buffers][hi, lo][CT][AS]
  static constexpr int B = A + 4 * CT * AS * 2;            // [2][CT][BS]
  static constexpr int ZR = B + 2 * CT * BS * 2;           // [2][waves][FW] float
  static constexpr int CO = ZR + 2 * NWV * FW * 4;         // [KH - 1][TILES][16][64] float: what the other waves of a tile summed up
  static constexpr int SZC = (KH - 1) * TILES * 16 * 64 * 4;
  static constexpr int TOTAL = CO + (CPG == 1 ? 2 : 1) * SZC;    // groups of one step: left and taken in the same step, two buffers
  static constexpr int SLOT = D * D + D;
  static_assert(TOTAL <= 160 * 1024 && AI >= 1 && BI >= 1, "LDS, pieces");
};
}  // namespace

template <int D, int GT, bool BACK, int TILES>
__global__ __launch_bounds__(GT == 256 ? 512 : 256) void group_sums_kernel(GroupSumsArgs a) {
  using G = SumsCfg<D, GT, TILES>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* Al = reinterpret_cast<uint16_t*>(smem + G::A);
  uint16_t* Bl = reinterpret_cast<uint16_t*>(smem + G::B);
  float* zred = reinterpret_cast<float*>(smem + G::ZR);
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  // The NB workgroups of a head get block indices 8 apart (the same chiplet) while there are whole eights of heads.
  constexpr int NF = D / G::FW, NB = NF * (D / G::CW);
  const int full = a.B * a.H / 8 * 8, bx = blockIdx.x;
  const int bh = bx < full * NB ? (bx & 7) + bx / (8 * NB) * 8 : full + (bx - full * NB) / NB;
  const int blk = bx < full * NB ? (bx >> 3) % NB : (bx - full * NB) % NB;
  const int fb = blk % NF, cblk = blk / NF;
  const int b = bh / a.H, h = bh % a.H;
  const int64_t base = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const uint16_t* ga = static_cast<const uint16_t*>(a.a) + base + fb * G::FW;
  const uint16_t* gb = static_cast<const uint16_t*>(a.b) + base + cblk * G::CW;
  const float* gw = BACK ? a.w + (size_t)bh * a.L : nullptr;
  const float* gwz = BACK ? a.wz + (size_t)bh * a.L : nullptr;
  float* slots = a.slots + (size_t)bh * a.ng * G::SLOT;
  const float one = a.relu ? 0.f : 1.f;
  // this wave's tile: features f0 .. f0 + 31, channels c0 .. c0 + 31
  const int wt4 = w % TILES, kh = w / TILES;               // tile, and which part of a step's tokens
  const int fl = G::FW == 32 ? 0 : 32 * (wt4 >> 1);        // within the workgroup's features, channels
  const int cl = TILES == 1 ? 0 : 32 * (D == 128 ? wt4 : wt4 & 1);
  const int f0 = fb * G::FW + fl, c0 = cblk * G::CW + cl;

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
        if (lane < G::AP) zred[(buf * G::NWV + w) * G::FW + 8 * lane + e] = y;
        zacc[e] = 0.f;
      }
    }
  };
  auto write_slot = [&](int g) __attribute__((always_inline)) {
    float* so = slots + (size_t)g * G::SLOT;
    if (kh == 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) so[(f0 + 8 * (r >> 2) + 4 * hi + (r & 3)) * D + c0 + l32] = acc[r];
    if (tid < G::FW && cblk == 0) so[D * D + zf] = zrun;
  };

  // the other waves' parts of the sums join the first's: left in LDS behind a group's products, taken behind the barrier
  float* co = reinterpret_cast<float*>(smem + G::CO) + wt4 * 1024 + lane;
  auto leave = [&](int s) __attribute__((always_inline)) {
    if (G::KH > 1 && kh > 0) {
      float* p = co + (G::CPG == 1 ? s & 1 : 0) * (G::SZC / 4) + (kh - 1) * TILES * 1024;
#pragma unroll
      for (int r = 0; r < 16; ++r) { p[64 * r] = acc[r]; acc[r] = 0.f; }
    }
  };
  auto take = [&](int s) __attribute__((always_inline)) {  // what step s left
    if (G::KH > 1 && kh == 0) {
      const float* p = co + (G::CPG == 1 ? s & 1 : 0) * (G::SZC / 4);
#pragma unroll
      for (int v = 0; v < G::KH - 1; ++v)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += p[v * TILES * 1024 + 64 * r];
    }
  };
  // Step s: its products, and between them the rows of step s + 1 on their way to the other buffer and the requests of
  // step s + 3 (two steps of rows are in registers: with one wave per SIMD nothing else hides a trip to memory).
  auto step = [&](int s, int steps, Rows& x) __attribute__((always_inline)) {
    const int buf = s & 1;
    const uint16_t* Ah = Al + buf * 2 * G::CT * G::AS;
    const uint16_t* Bh = Bl + buf * G::CT * G::BS;
    if (s % G::CPG == 0) {
      if (s > 0) take(s - 1);
      write_slot(group_of(s));
    }
    if ((s + 1) % G::CPG == 0 && tid < G::FW) {
#pragma unroll
      for (int v = 0; v < G::NWV; ++v) zrun += zred[(buf * G::NWV + v) * G::FW + tid];
    }
#pragma unroll
    for (int k1 = 0; k1 < G::CT / 16 / G::KH; ++k1) {
      const int ks = kh * (G::CT / 16 / G::KH) + k1;
      const bf16x8 bop = tr_operand(Bh, G::BS, 16 * ks, cl, lane);
      acc = mfma(tr_operand(Ah, G::AS, 16 * ks, fl, lane), bop, acc);
      acc = mfma(tr_operand(Ah + G::CT * G::AS, G::AS, 16 * ks, fl, lane), bop, acc);
    }
    if ((s + 1) % G::CPG == 0) leave(s);
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
  if (steps > 0) take(steps - 1);
  write_slot(group_of(steps));
}

template <int D, int GT, bool BACK, int TILES>
static hipError_t launch_sums_one(const GroupSumsArgs& a, hipStream_t st) {
  using G = SumsCfg<D, GT, TILES>;
  auto kern = group_sums_kernel<D, GT, BACK, TILES>;
  hipError_t e = LINATTN_MAX_LDS_ONCE(kern, G::TOTAL);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.B * a.H * (D / G::FW) * (D / G::CW))), dim3(G::NT), G::TOTAL, st, a);
  return hipGetLastError();
}
// One tile per workgroup, or four?  A workgroup takes most of a compute unit's LDS: one tile while every workgroup has a unit to itself
// (16 heads at D = 128, 64 at D = 64).  Measured, us per gradient call, four / one: groups of 256, 4 groups: D = 128: 8 heads 68.9 / 66.6,
// 16 heads 77.3 / 75.3, 24 heads 81.5 / 95.9; D = 64: 8 heads 50.3 / 46.4, 64 heads 82.4 / 79.4, 80 heads 98.0 / 111; groups of 64: D = 128:
// 16 heads 45.2 / 44.4, 32 heads 51.2 / 52.4; D = 64: 48 heads 38.1 / 37.5.
static bool one_tile(int heads, int d) { return (int64_t)heads * (d / 32) * (d / 32) <= 256; }
template <int D, int GT>
static hipError_t launch_sums_dir(const GroupSumsArgs& a, bool back, hipStream_t st) {
  if (one_tile(a.B * a.H, D)) return back ? launch_sums_one<D, GT, true, 1>(a, st) : launch_sums_one<D, GT, false, 1>(a, st);
  return back ? launch_sums_one<D, GT, true, 4>(a, st) : launch_sums_one<D, GT, false, 4>(a, st);
}

// Against one workgroup per group and a prefix sum over the slots, which has no chain over the groups but moves every slot
// three times: the walk pays with workgroups for half the chip (groups of 64: three quarters), or few groups.  Measured, us
// per gradient call, per-group kernels / walk.  Few heads, by the number of groups: groups of 64, 8 heads: D = 64: 4 62 / 60, 5
// 73 / 68, 6 61 / 66; D = 128: 4 81 / 72, 5 81 / 74, 6 82 / 78, 8 84 / 83, 12 85 / 96; groups of 256: D = 64: 3 79 / 75, 4 80 / 81, 5 81 / 87;
// D = 128: 4 110 / 99, 5 111 / 106, 6 111 / 111, 8 112 / 123.  Many groups, by the number of heads: groups of 256, D = 128, 32
// groups: 8 heads 179 / 295, 32 heads 645 / 615; D = 64, 16 groups of 48 heads (48 workgroups) 248 / 279; groups of 64, D = 128, 64
// groups: 32 heads 426 / 456, 64 heads 851 / 712.
// With one tile per workgroup, D = 128, few groups go further: groups of 256: 6 groups of 4, 8, 16 heads 76.0 / 74.3, 84.0 / 82.6, 94.0 / 91.7,
// 7 groups 77.3 / 80.8, 85.2 / 88.5, 101.6 / 103.3; groups of 64: 6 groups 47.7 / 44.7, 52.2 / 47.8, 55.0 / 50.7, 7 groups 49.2 / 47.9, 52.6 / 50.4,
// 55.5 / 53.3, 8 groups 48.5 / 49.9, 53.6 / 52.9, 60.5 / 59.5.  D = 64: 5 groups of 256 48.7 / 52.3, 6 of 64 30.4 / 34.3.
bool group_sums_pays(int heads, int ng, int d, int group) {
  const int few = d == 64 ? (group == 256 ? 4 : 5) : one_tile(heads, d) ? (group == 256 ? 6 : 7) : 5;
  return ng <= few || heads * (d == 128 ? 4 : 1) >= (group == 256 ? 128 : 192);
}

hipError_t launch_group_sums(const GroupSumsArgs& a, int d, int group, bool back, hipStream_t st) {
  if (d == 128) return group == 256 ? launch_sums_dir<128, 256>(a, back, st) : launch_sums_dir<128, 64>(a, back, st);
  return group == 256 ? launch_sums_dir<64, 256>(a, back, st) : launch_sums_dir<64, 64>(a, back, st);
}

}  // namespace linattn
