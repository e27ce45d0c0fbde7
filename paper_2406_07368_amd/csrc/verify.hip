// Speculative verification / decode step (Sec. 4.2; decode = one draft that is
// always kept).  Memory-bound: every head's fp32 state S (d x d) is read once
// and, if any draft is accepted, written once; everything else is tiny.
//
// One workgroup of NT threads owns one (b, h) (value rows wider than 128: the column
// slice S[:, c0 : c0+CW] of it).  The state streams through registers in row passes
// with 16-byte loads (rows are contiguous, so a wave reads whole 256..512 B row
// segments; nontemporal: the state is touched once per step), a few
// passes in flight at a time: each row adds its term to the kk read-outs
// phi(q_j)^T S, receives the accepted rank-1 updates and is written straight back.
// The read-outs are then reduced across the threads that share a column group,
// completed with the causal in-block term, normalised, and joined with the
// convolution over (history ++ drafts <= j).
//
// What bounds it: with few heads the one launch and its chain of request, products,
// reduction (5.2 us as a graph for one draft, as long as a plain call's host part); with many the state's
// traffic.  Few heads get more threads each (pick_threads), so that the whole state
// is requested at once.  Splitting a head's columns over four workgroups instead put as
// many requests under way, but then all of them read the old z and a second launch had
// to advance it, and every slice repeated the drafts' feature maps and scores.  us a call
// as a graph, slices / whole heads: B1 H32 d128 one draft 8.1 / 5.5, eight 12.6 / 10.9; B8 H32 d128 eight 18.2 /
// 14.6; 200 heads of 64, sixteen 26.4 / 10.9.
#include "common.h"
#include "kernels.h"

namespace linattn {

template <int D, int CW, int KP, int NT>
struct VerifySmem {
  float fq[D][KP];          // phi(q_j)[i], feature-major so one thread reads all drafts of its row
  float fk[D][KP];          // phi(k_j)[i]
  float vv[KP][CW];         // v_j[c0 + c]
  float red[NT / kWave][KP][CW];   // per-wave partial read-outs
  float amat[KP][KP];       // phi(q_j).phi(k_j') for j' <= j, else 0
  float den[KP];            // phi(q_j).z + sum_j' amat + eps
  float zz[D];
  float wt[8][CW];          // conv taps of the slice's channels, tap-major (taps >= Kc are 0)
  float hh[8][CW];          // hh[t]: the value row t+1 positions before the first draft (t < Kc-1)
};

template <int KP>
__device__ __forceinline__ void load_row(const float* row, float (&f)[KP]) {
  if constexpr (KP >= 4) {
#pragma unroll
    for (int g = 0; g < KP / 4; ++g) {
      f32x4 t = *reinterpret_cast<const f32x4*>(row + 4 * g);
      f[4 * g] = t[0]; f[4 * g + 1] = t[1]; f[4 * g + 2] = t[2]; f[4 * g + 3] = t[3];
    }
  } else {
#pragma unroll
    for (int j = 0; j < KP; ++j) f[j] = row[j];
  }
}

// At most 128 registers per thread for up to 8 drafts: 16 waves fit on a compute unit, so that B*H = 1024 heads of
// 256 threads are all resident at once (a partial second round would run at a fraction of the bandwidth).
template <typename Io, int D, int CW, int KP, int NT>
__global__ __launch_bounds__(NT, (KP <= 8 ? 4 : 2)) void verify_kernel(VerifyArgs a) {
  constexpr int CG = CW / 4;          // float4 column groups per row slice
  constexpr int RPP = NT / CG;        // rows covered per pass
  constexpr int NPASS = D / RPP;
  static_assert(NPASS >= 1 && RPP * NPASS == D, "tile shape");
  __shared__ VerifySmem<D, CW, KP, NT> sm;

  const int tid = threadIdx.x;
  // value rows of DV = a.dv elements (a multiple of D; DV == D: d_v = d_k): DV / CW column slices per head, and
  // DV is the row length of v, out, hist, conv_w and S
  const int DV = a.dv, nslice = DV / CW;
  const int bh = blockIdx.x / nslice;
  const int c0 = (blockIdx.x % nslice) * CW;
  const int b = bh / a.H, h = bh % a.H;
  const int kk = a.kk, Kc = a.Kc;
  const int cg = tid % CG, r0 = tid / CG;

  // ---- 0. every request of the step is issued before anything waits, the small inputs FIRST: every workgroup of
  //         the launch is about to ask for its state at the same moment, and anything requested after that waits
  //         behind it.  All requests unconditional -- indices past the end are clamped, what they bring is dropped --:
  //         under conditions on the thread index every one of them sat in a block of its own with a full wait at its
  //         end, a dozen trips to memory in a row before the state was asked for. ------------------------------------
  const int64_t tok0 = (int64_t)bh * kk * D;              // q, k
  const int64_t vtok0 = (int64_t)bh * kk * DV;            // v, out
  const int64_t hist0 = (int64_t)bh * (Kc - 1) * DV;
  constexpr int QK_IT = (KP * (D / 8) + NT - 1) / NT;   // 8-element pieces of q and k per thread
  constexpr int V_IT = (KP * (CW / 8) + NT - 1) / NT;
  typename Io::raw8 rq[QK_IT], rk[QK_IT], rv[V_IT];
#pragma unroll
  for (int m = 0; m < QK_IT; ++m) {
    const int c8 = tid + NT * m;
    const int j = c8 / (D / 8), i0 = (c8 % (D / 8)) * 8;
    const int64_t off = tok0 + (int64_t)(j < kk ? j : kk - 1) * D + i0;
    rq[m] = Io::load_raw8(a.q, off);
    rk[m] = Io::load_raw8(a.k, off);
  }
#pragma unroll
  for (int m = 0; m < V_IT; ++m) {
    const int c8 = tid + NT * m;
    const int j = c8 / (CW / 8), cc = (c8 % (CW / 8)) * 8;
    rv[m] = Io::load_raw8(a.v, vtok0 + (int64_t)(j < kk ? j : kk - 1) * DV + c0 + cc);
  }
  const float zreg = a.z[(size_t)bh * D + tid % D];
  // taps and history rows of the slice's channels: element e = tid + NT m of the [8][CW] arrays in LDS
  constexpr int TAP_IT = (8 * CW + NT - 1) / NT;
  float tap_reg[TAP_IT], hist_reg[TAP_IT];
  // (one tap: no history; the request then reads a draft's value row, which is dropped)
  const void* hsrc = Kc > 1 ? a.hist : a.v;
  const int64_t hbase = (Kc > 1 ? hist0 : vtok0) + c0;
#pragma unroll
  for (int m = 0; m < TAP_IT; ++m) {
    const int e = (tid + NT * m) % (8 * CW);
    const int t = e / CW, cc = e % CW;
    tap_reg[m] = a.conv_w[((size_t)h * DV + c0 + cc) * Kc + (t < Kc ? t : 0)];
    hist_reg[m] = Io::load1(hsrc, hbase + (int64_t)(t < Kc - 1 ? Kc - 2 - t : 0) * DV + cc);
  }
  int n = kk;
  if (a.n_commit) { n = a.n_commit[b]; n = n < 0 ? 0 : (n > kk ? kk : n); }

  // ---- 0. the state slice streams through a window of PD row passes: the first PD loads are
  //         in flight before anything else, each later one is issued when its slot frees up ----
  constexpr int PDW = KP == 8 ? 2 : 4;        // fewer passes in flight when the read-outs need the registers
  constexpr int PD = NPASS < PDW ? NPASS : PDW;
  float* Sg = a.S + (size_t)bh * D * DV + c0 + 4 * cg;
  f32x4 s[PD];
#pragma unroll
  for (int p = 0; p < PD; ++p) s[p] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Sg + (size_t)(p * RPP + r0) * DV));
  // (values that only some threads use: kept ahead of the state's requests, or the compiler moves their requests down
  // to the uses, behind the state's)
#pragma unroll
  for (int m = 0; m < QK_IT; ++m) { Io::needed_here(rq[m]); Io::needed_here(rk[m]); }
#pragma unroll
  for (int m = 0; m < V_IT; ++m) Io::needed_here(rv[m]);

  // ---- 1. drafts -> LDS (phi applied), normaliser, taps and history -> LDS -----------------------
#pragma unroll
  for (int m = 0; m < QK_IT; ++m) {
    const int c8 = tid + NT * m;
    const int j = c8 / (D / 8), i0 = (c8 % (D / 8)) * 8;
    if (c8 < KP * (D / 8)) {
      float xq[8], xk[8];
      Io::unpack8(rq[m], xq);
      Io::unpack8(rk[m], xk);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sm.fq[i0 + e][j] = j < kk ? phi_any(xq[e], a.relu) : 0.f;
        sm.fk[i0 + e][j] = j < kk ? phi_any(xk[e], a.relu) : 0.f;
      }
    }
  }
#pragma unroll
  for (int m = 0; m < V_IT; ++m) {
    const int c8 = tid + NT * m;
    const int j = c8 / (CW / 8), cc = (c8 % (CW / 8)) * 8;
    if (c8 < KP * (CW / 8)) {
      float xv[8];
      Io::unpack8(rv[m], xv);
#pragma unroll
      for (int e = 0; e < 8; ++e) sm.vv[j][cc + e] = j < kk ? xv[e] : 0.f;
    }
  }
  if (tid < D) sm.zz[tid] = zreg;
#pragma unroll
  for (int m = 0; m < TAP_IT; ++m) {
    const int e = tid + NT * m;
    if (e < 8 * CW) {
      const int t = e / CW, cc = e % CW;
      sm.wt[t][cc] = t < Kc ? tap_reg[m] : 0.f;
      sm.hh[t][cc] = t < Kc - 1 ? hist_reg[m] : 0.f;
    }
  }
  __syncthreads();

  // ---- 2. in-block scores and denominators ----------------------------------------
  if constexpr (KP == 16) {
    // 16 drafts: phi(Q) phi(K)^T on wave 0, phi(Q) z on wave 1, fp32 products on 16 x 16 x 4 matrix instructions (lane =
    // draft lane % 16 and feature lane / 16 of a step) in four chains over the features.  A thread per pair of drafts
    // had 64 steps of LDS reads in a row (us a call, d = 128: 4 heads 17.5, now 14.3; 256 heads 22.4, now 17.2).
    const int wv = tid / kWave, lane = tid % kWave, l16 = lane % 16, g4 = lane / 16;
    if (wv < 2) {                                          // uniform per wave
      f32x4 part[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) part[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int i = 0; i < D; i += 16)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int f = i + 4 * c + g4;
          part[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(sm.fq[f][l16], wv == 0 ? sm.fk[f][l16] : sm.zz[f], part[c], 0, 0, 0);
        }
      const f32x4 x = (part[0] + part[1]) + (part[2] + part[3]);   // row (draft of q) 4 g4 + e, column (draft of k) l16
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * g4 + e;
        if (wv == 0) sm.amat[j][l16] = (l16 <= j && j < kk) ? x[e] : 0.f;
        else if (l16 == 0) sm.den[j] = x[e];               // completed below
      }
    }
  } else {
    constexpr int NPAIR = KP * KP;
    constexpr int TPP = (NT / NPAIR) > 64 ? 64 : (NT / NPAIR);   // threads per (j, j') pair
    if (tid < NPAIR * TPP) {
      const int pair = tid / TPP, sub = tid % TPP;
      const int j = pair / KP, jp = pair % KP;
      float acc = 0.f, dz = 0.f;
      for (int i = sub; i < D; i += TPP) {
        const float fqv = sm.fq[i][j];
        acc += fqv * sm.fk[i][jp];
        dz += fqv * sm.zz[i];
      }
#pragma unroll
      for (int off = TPP / 2; off >= 1; off >>= 1) {
        acc += __shfl_xor(acc, off);
        dz += __shfl_xor(dz, off);
      }
      if (sub == 0) {
        sm.amat[j][jp] = (jp <= j && j < kk) ? acc : 0.f;
        if (jp == 0) sm.den[j] = dz;     // completed below
      }
    }
  }

  // ---- 3. read-outs phi(q_j)^T S from registers; accepted drafts folded in and the row
  //         streamed back as soon as it has been used (reads of later rows are still in flight)
  float acc[KP][4];
#pragma unroll
  for (int j = 0; j < KP; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[j][e] = 0.f;
  float vr[KP][4];
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    f32x4 t = *reinterpret_cast<const f32x4*>(&sm.vv[j][4 * cg]);
    const bool keep = j < n;
    vr[j][0] = keep ? t[0] : 0.f; vr[j][1] = keep ? t[1] : 0.f;
    vr[j][2] = keep ? t[2] : 0.f; vr[j][3] = keep ? t[3] : 0.f;
  }
#pragma unroll 1
  for (int pb = 0; pb < NPASS; pb += PD) {
#pragma unroll
    for (int q = 0; q < PD; ++q) {
      const int p = pb + q;
      const int i = p * RPP + r0;
      float f[KP], g[KP];
      f32x4 cur = s[q];
      load_row<KP>(&sm.fq[i][0], f);
#pragma unroll
      for (int j = 0; j < KP; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(f[j], cur[e], acc[j][e]);
      if (n > 0) {   // uniform per workgroup; n == 0 leaves the state untouched
        load_row<KP>(&sm.fk[i][0], g);
#pragma unroll
        for (int j = 0; j < KP; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) cur[e] = fmaf(g[j], vr[j][e], cur[e]);
        __builtin_nontemporal_store(cur, reinterpret_cast<f32x4*>(Sg + (size_t)i * DV));
      }
      if (p + PD < NPASS) s[q] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Sg + (size_t)((p + PD) * RPP + r0) * DV));
    }
  }
  // threads that share a column group sit CG lanes apart inside a wave
#pragma unroll
  for (int off = CG; off < kWave; off <<= 1)
#pragma unroll
    for (int j = 0; j < KP; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][e] += __shfl_xor(acc[j][e], off);
  if ((tid % kWave) < CG) {
    const int wv = tid / kWave;
#pragma unroll
    for (int j = 0; j < KP; ++j)
      *reinterpret_cast<f32x4*>(&sm.red[wv][j][4 * cg]) = f32x4{acc[j][0], acc[j][1], acc[j][2], acc[j][3]};
  }
  __syncthreads();
  if (tid < kk) {
    float dsum = sm.den[tid] + a.eps;
    for (int jp = 0; jp <= tid; ++jp) dsum += sm.amat[tid][jp];
    sm.den[tid] = dsum;
  }
  __syncthreads();

  // ---- 4. outputs: normalise, add the causal convolution -------------------------------
  for (int idx = tid; idx < kk * CW; idx += NT) {
    const int j = idx / CW, c = idx % CW;
    float num = 0.f;
#pragma unroll
    for (int v = 0; v < NT / kWave; ++v) num += sm.red[v][j][c];
    for (int jp = 0; jp <= j; ++jp) num = fmaf(sm.amat[j][jp], sm.vv[jp][c], num);
    float u = 0.f;
    for (int t = 0; t < Kc; ++t) {
      // tap t looks t rows back from draft j: another draft if t <= j, else history row (t - j) back
      const float x = t <= j ? sm.vv[j - t][c] : sm.hh[t - j - 1][c];
      u = fmaf(sm.wt[t][c], x, u);
    }
    Io::store1(a.out, vtok0 + (int64_t)j * DV + c0 + c, num / sm.den[j] + u);
  }

  // ---- 5. the rest of the state: normaliser and history ----------------------------------
  if (n == 0) return;   // uniform per workgroup: nothing accepted, state untouched
  if (nslice == 1 && tid < D) {   // with several slices per head a separate launch updates z
    float zs = sm.zz[tid];
    for (int j = 0; j < n; ++j) zs += sm.fk[tid][j];
    a.z[(size_t)bh * D + tid] = zs;
  }
  if (Kc > 1) {
    __syncthreads();   // every conv read of the old history is done
    for (int c = tid; c < CW; c += NT) {
      for (int r = 0; r < Kc - 1; ++r) {
        const int sidx = n - (Kc - 1) + r;   // position in (history ++ accepted drafts)
        const int64_t dst = hist0 + (int64_t)r * DV + c0 + c;
        if (sidx >= 0) Io::store1(a.hist, dst, sm.vv[sidx][c]);
        else Io::store1(a.hist, dst, sm.hh[-sidx - 1][c]);   // an old history row, -sidx positions back
      }
    }
  }
}

// z += sum of the accepted phi(k_j); used when several workgroups have a head's value columns
// (they all read the old z, so it cannot be updated by one of them).
template <typename Io, int D>
__global__ __launch_bounds__(256) void verify_z_kernel(VerifyArgs a) {
  const int gid = blockIdx.x * 256 + threadIdx.x;
  if (gid >= a.B * a.H * D) return;
  const int bh = gid / D, i = gid % D;
  const int b = bh / a.H;
  // every draft's element requested at once, whatever the count says (a loop up to the count was one trip to memory
  // per draft, one after the other); kept or dropped by select
  constexpr int KMAX = 16;   // drafts per call at most (the entry point refuses more)
  float x[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) x[j] = Io::load1(a.k, ((int64_t)bh * a.kk + (j < a.kk ? j : a.kk - 1)) * D + i);
  float zs = a.z[gid];
  int n = a.kk;
  if (a.n_commit) { n = a.n_commit[b]; n = n < 0 ? 0 : (n > a.kk ? a.kk : n); }
  if (n == 0) return;
#pragma unroll
  for (int j = 0; j < KMAX; ++j) zs += j < n ? phi_any(x[j], a.relu) : 0.f;
  a.z[gid] = zs;
}

// z += sum of the accepted phi(k_j) for every head, as a launch of its own (fp32 sums of fp32 feature maps).
hipError_t launch_verify_z(const VerifyArgs& a, bool bf16, int d, hipStream_t st) {
  const int total = a.B * a.H * d;
  const dim3 grid((unsigned)((total + 255) / 256)), block(256);
  if (bf16) {
    if (d == 128) hipLaunchKernelGGL((verify_z_kernel<IoBf16, 128>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((verify_z_kernel<IoBf16, 64>), grid, block, 0, st, a);
  } else {
    if (d == 128) hipLaunchKernelGGL((verify_z_kernel<IoF32, 128>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((verify_z_kernel<IoF32, 64>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}

template <typename Io, int D, int CW, int KP, int NT>
static hipError_t launch_nt(const VerifyArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((verify_kernel<Io, D, CW, KP, NT>), dim3((unsigned)(a.B * a.H * (a.dv / CW))), dim3(NT), 0, st, a);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || a.dv == CW ? e : launch_verify_z(a, sizeof(typename Io::elem) == 2, D, st);
}

// Threads per workgroup.  More threads ask for more of the state at once and shorten the chain of row passes, which
// is all that counts while every workgroup has a compute unit of its own; beyond that, fewer threads let more workgroups
// share one (and 8 drafts, 120 registers, fill it with 1024 threads).  Measured, us a call as a graph (a plain call takes the
// host about 5), 256 / 512 / 1024 threads, 128 x 128 state:
//   1 draft    4 heads 7.3 / 5.9 / 5.2, 256 13.0 / 9.8 / 7.6, 512 17.5 / 13.5 / 12.9, 576 19.2 / 16.2 / 15.4, 640 19.5 / 16.7 / 17.8,
//              767 20.6 / 18.6 / 20.4; fp32 rows 832 22.4 / 22.5, 900 23.9 / 24.7, 1000 25.7 / 27.7, 1024 26.1 / 28.2
//   2 drafts   4 heads 8.2 / 6.5 / 5.7, 256 15.1 / 10.7 / 8.2, 512 18.5 / 14.1 / 13.7, 576 20.3 / 16.5 / 16.9, 640 20.8 / 17.1 / 19.5;
//              fp32 rows 832 23.9 / 23.8, 900 24.5 / 25.1, 1000 27.0 / 27.6, 1024 27.2 / 28.0
//   4 drafts   4 heads 9.3 / 7.5 / 7.8, 64 9.9 / 8.1 / 8.5, 128 13.1 / 9.8 / 9.2, 256 15.9 / 11.7 / 9.9, 320 18.4 / 14.1 / 16.5,
//              512 19.9 / 15.6 / 17.2, 576 21.8 / 21.1 / 23.6, 640 22.2 / 22.9 / 23.8
//   8 drafts   4 heads 14.6 / 10.6 / 11.2, 64 15.9 / 11.8 / 12.0, 128 15.4 / 11.7 / 12.1, 192 16.7 / 13.1 / 12.9, 256 21.4 / 15.9 / 14.6,
//              320 22.7 / 18.3 / 23.2, 512 26.5 / 21.5 / 27.2, 576 28.9 / 30.4 / 36.3
//   16 drafts  one kernel, of 512 threads (1024 have too few registers): 4 heads 14.2, 256 17.3, 767 46; fp32 rows 1024 61
// 64 x 128 state, 256 / 512 threads: 1 draft 32 heads 6.0 / 5.2, 384 7.6 / 7.1; 8 drafts 32 11.2 / 8.9, 256 11.9 / 9.8, 384 12.9 / 12.8,
// 767 19.4 / 22.3; 16 drafts 256 15.6 / 12.7, 288 17.2 / 22.6, 1024 37.8 / 45.2.  Slices of 128 x 64 (launch_d) likewise.
// 64 x 64: 256 threads have a row each in four passes.
static int pick_threads(int state, int kp, int blocks) {
  if (state == 64 * 64) return 256;
  if (state == 64 * 128) return blocks <= (kp == 16 ? 256 : 384) ? 512 : 256;
  if (kp == 16) return 512;
  if (kp <= 2) return blocks <= 576 ? 1024 : blocks < 832 ? 512 : 256;
  if (blocks <= (kp == 8 ? 128 : 64)) return 512;
  return blocks <= 256 ? 1024 : blocks <= 512 ? 512 : 256;
}

template <typename Io, int D, int CW, int KP>
static hipError_t launch_kp(const VerifyArgs& a, hipStream_t st) {
  const int blocks = a.B * a.H * (a.dv / CW);
  const int nt = pick_threads(D * CW, KP, blocks);
  if constexpr (D * CW == 128 * 128 && KP < 16)
    if (nt >= 1024) return launch_nt<Io, D, CW, KP, 1024>(a, st);
  if constexpr (D * CW >= 64 * 128)
    if (nt >= 512) return launch_nt<Io, D, CW, KP, 512>(a, st);
  // (768 blocks of bf16 rows and more are verify_mfma.hip's: one and two drafts of them never come here)
  if constexpr (D * CW < 128 * 128 || (KP < 16 && (KP > 2 || sizeof(typename Io::elem) == 4))) return launch_nt<Io, D, CW, KP, 256>(a, st);
  return hipErrorInvalidValue;                             // (not reached)
}

template <typename Io, int D, int CW>
static hipError_t launch_cw(const VerifyArgs& a, hipStream_t st) {
  if (a.kk <= 1) return launch_kp<Io, D, CW, 1>(a, st);
  if (a.kk <= 2) return launch_kp<Io, D, CW, 2>(a, st);
  if (a.kk <= 4) return launch_kp<Io, D, CW, 4>(a, st);
  if (a.kk <= 8) return launch_kp<Io, D, CW, 8>(a, st);
  return launch_kp<Io, D, CW, 16>(a, st);
}

// Whole heads where the value rows have up to 128 elements, slices otherwise, z in a launch of its own: of D columns, but at D =
// 128 of 64 while the chip has room for all of them (up to 384, of 512 threads), and of 64 or 32 where blocks of 128 would leave a
// second round to a few workgroups.  Measured, us a call as a graph, d_v = 256 and 1024, by blocks of 128 columns, slices of 32 /
// 64 / 128:
//   1 draft    64 blocks 8.0 / 7.8 / 8.1, 192 9.2 / 9.1 / 9.1, 256 9.8 / 10.2 / 9.9, 288 11.7 / 12.4 / 13.0, 384 14.4 / 14.3 / 13.0
//   2 drafts   64 8.7 / 8.4 / 8.7, 192 10.1 / 9.9 / 9.9, 288 12.0 / 13.0 / 13.6, 384 15.2 / 15.2 / 15.2
//   4 drafts   64 9.2 / 9.4 / 10.9, 128 10.4 / 10.1 / 11.6, 192 11.3 / 11.7 / 11.6, 256 12.9 / 11.5 / 12.1, 320 14.3 / 13.7 / 16.1
//   8 drafts   64 12.5 / 12.2 / 13.7, 128 14.3 / 12.9 / 15.0, 192 15.8 / 15.2 / 15.5, 256 18.3 / 15.6 / 16.3, 320 24.0 / 18.6 / 19.5
//   16 drafts  64 14.2 / 14.4 / 17.2, 128 17.6 / 14.9 / 17.6, 192 25.2 / 19.6 / 17.8, 320 36 / 30 / 31
// d = 64 (d_v = 256 on): slices of 64 columns as before the whole heads: 64 blocks, 1, 8 and 16 drafts 7.3, 11.3, 13.3.
template <typename Io, int D>
static hipError_t launch_d(const VerifyArgs& a, hipStream_t st) {
  if constexpr (D == 64)
    if (a.dv == 128) return launch_cw<Io, D, 2 * D>(a, st);
  if constexpr (D == 128)
    if (a.dv > D) {
      const int blocks = a.B * a.H * (a.dv / D);
      const bool odd_round = blocks > 256 && blocks < 384;
      if (odd_round && a.kk <= 2) return a.kk == 1 ? launch_nt<Io, D, D / 4, 1, 256>(a, st) : launch_nt<Io, D, D / 4, 2, 256>(a, st);
      if (odd_round || blocks <= (a.kk > 8 ? 128 : 192)) return launch_cw<Io, D, D / 2>(a, st);
    }
  return launch_cw<Io, D, D>(a, st);
}

hipError_t launch_verify(const VerifyArgs& a, bool bf16, int d, hipStream_t st) {
  if (bf16) return d == 128 ? launch_d<IoBf16, 128>(a, st) : launch_d<IoBf16, 64>(a, st);
  return d == 128 ? launch_d<IoF32, 128>(a, st) : launch_d<IoF32, 64>(a, st);
}

}  // namespace linattn
