// Value-tiled DeltaLog decode step (Sec. 3.3, the kernel ownership path): the state of
// one (slot, head) is split along the value dimension into NV tiles of dk x dv/NV, one
// workgroup per (token row, head, tile):
//
//   replay_prep_kernel  (split replay only) once per (row, head): the key-side replay
//                       coefficients g_i(k), g_i(q) of every live entry, into an fp32
//                       scratch buffer [n, H, 2, C] owned by the caller, and the commit of
//                       the live length (append: L + 1; merge: 0);
//   tile_step_kernel    per value tile: stream the dense-base tile, replay the live log
//                       on the tile's columns (coefficients from the scratch buffer, or
//                       recomputed by every tile in the fused variant), write the
//                       output slice, then either append the tile's U_log[L] shard --
//                       tile 0 being the designated writer of the shared K_log[L] and
//                       Lam_log[L] -- or merge the tile's columns of the base;
//   finalize_kernel     (fused replay only) commit L after every tile has read it.
//
// With split replay the length is committed ahead of the tiles: append maps L to L + 1 in
// 1 .. C and merge maps C to 0, so every committed length has one L it came from and the
// tiles read that (GDN 32x32 heads 128x128, M = 8, 4 tiles: the launch it saves is about
// 4 us of the 23.5 us a step took with it).  Where the tile launch is refused the commit is
// taken back by a launch of its own, the same map the other way.
//
// The arithmetic per element is that of dl_kernel.hpp; the coefficient routine is shared
// by the prepare kernel and the fused tile kernel, so the split and fused variants give
// bit-identical results.  Only fp32 dense state is supported on this path.
#pragma once

#include "dl_kernel.hpp"

namespace dl {

constexpr int tile_threads(int dk, int dv, int nv) {
  return dk * (dv / nv) / 16 > 256 ? 256 : dk * (dv / nv) / 16;   // 4 rows x 4 columns per thread
}

template <int DK, int DV, int NV>
struct TileCfg {
  static constexpr int DVT = DV / NV;              // value columns per tile
  static constexpr int NCG = DVT / 4;              // float4 column groups
  static constexpr int NT = tile_threads(DK, DV, NV);
  static constexpr int NRG = NT / NCG;             // row groups
  static constexpr int RPT = DK / NRG;             // rows per thread
  static constexpr int NW = NT / 64;               // waves
  static constexpr int WK = DK / 64;               // waves of the per-row work
  static constexpr int CH = 16;                    // log entries staged per merge chunk
  static constexpr int KTS = CH + 4;               // LDS row stride of a staged K~ chunk
  static constexpr int LPE = 16, EPP = NT / LPE, RPL = DK / LPE;   // coefficient pass
  static constexpr int UQ = 32 / NRG < 1 ? 1 : 32 / NRG;           // log values loaded ahead
  static_assert(DV % NV == 0 && DVT % 4 == 0 && DVT <= NT, "value tiles of whole column quads");
  static_assert(NT % 64 == 0 && NT >= DK, "whole waves; one thread per key row in the prologue");
  static_assert(64 % NCG == 0 && NT == NCG * NRG && DK == NRG * RPT && RPT % 4 == 0, "thread layout");
};

// Sum over the lanes of a wave that share a column group (NCG apart).
template <int NCG>
__device__ __forceinline__ float column_sum(float v) {
  static_assert(NCG == 4 || NCG == 8 || NCG == 16 || NCG == 32, "column groups");
  if constexpr (NCG <= 4) v += dpp_move<0x124>(v);   // row_ror:4
  if constexpr (NCG <= 8) v += dpp_move<0x128>(v);   // row_ror:8
  if constexpr (NCG <= 16) v = xor16_sum(v);
  return xor32_sum(v);
}
template <int NCG>
__device__ __forceinline__ float4 column_sum(float4 v) {
  return make_float4(column_sum<NCG>(v.x), column_sum<NCG>(v.y), column_sum<NCG>(v.z),
                     column_sum<NCG>(v.w));
}

// Replay coefficients of the live entries for the readout vectors k and q (LDS s_kf,
// s_qf) at readout log-decay s_lr:  g_i(x) = sum_r e^(s_lr[r] - Lam_i,r) x_r K_i,r.
// The LDS vectors hold row c * RPL + x at x * 16 + c (lane c's run, element x).
// Every entry is reduced by 16 lanes of dk/16 rows each, whatever the workgroup size, so
// every caller produces the same bits.  Results go to gk[i], gq[i] (i < L).
template <int OP, int DK, int NT, typename TIN, typename Sink>
__device__ __forceinline__ void replay_coefficients(const TIN* Kb, const float* Lb, size_t LS,
                                                    int L, const float* s_kf, const float* s_qf,
                                                    const float* s_lr, Sink sink) {
  using TR = OpTraits<OP>;
  constexpr int DL = TR::PER_KEY ? DK : 1;
  constexpr int LPE = 16, EPP = NT / LPE, RPL = DK / LPE;
  const int tid = threadIdx.x;
  const int e_ = tid / LPE, c_ = tid % LPE;
  for (int i0 = 0; i0 < L; i0 += EPP) {           // uniform trip count
    const int i = i0 + e_, ic = min(i, L - 1);    // lanes past the log re-read its last entry
    RawRun<TIN, RPL> kr;
    RawRun<float, DL == 1 ? 4 : RPL> lr;
    float l0 = 0.f;
    kr.load(Kb + size_t(ic) * DK + c_ * RPL);
    if constexpr (TR::DECAY) {
      if constexpr (DL == 1) l0 = Lb[size_t(ic) * LS];
      else lr.load(Lb + size_t(ic) * LS + c_ * RPL);
    }
    float ak = 0.f, aq = 0.f;
#pragma unroll
    for (int x = 0; x < RPL; ++x) {
      const int pr = x * LPE + c_;
      float kx = kr.at(x);
      if constexpr (TR::DECAY && DL != 1) kx *= dl_exp(s_lr[pr] - lr.at(x));
      if constexpr (TR::DELTA) ak = fmaf(kx, s_kf[pr], ak);
      aq = fmaf(kx, s_qf[pr], aq);
    }
    if constexpr (TR::DECAY && DL == 1) {
      const float w = dl_exp(s_lr[0] - l0);
      ak *= w;
      aq *= w;
    }
    if constexpr (TR::DELTA) ak = group_sum<LPE>(ak);
    aq = group_sum<LPE>(aq);
    if (c_ == 0 && i < L) sink(i, ak, aq);
  }
}

// LDS position of key row r in the coefficient pass's vectors.
template <int DK>
__device__ __forceinline__ int tile_pos(int r) { return (r % (DK / 16)) * 16 + r / (DK / 16); }

// Cumulative log-decay of a (slot, head) at live length L, element x: the newest
// snapshot, 0 with an empty log (it is not stored; see the step kernel).
template <int DL>
__device__ __forceinline__ float cumulative_decay(const float* Lb, size_t LS, int L, int x) {
  if constexpr (DL == 1) return L > 0 ? scalar_ld(Lb + size_t(L - 1) * LS) : 0.f;
  else return L > 0 ? Lb[size_t(L - 1) * LS + x] : 0.f;
}

// ------------------------------------------------------------------ ReplayPrep
template <int OP, int DK, typename TIN>
__global__ __launch_bounds__(256) void replay_prep_kernel(const int32_t* slots, int32_t* len,
                                                          const void* k_, const void* q_,
                                                          float* coef, int H, uint32_t h_magic,
                                                          int C, KParams p) {
  using TR = OpTraits<OP>;
  constexpr int DL = TR::PER_KEY ? DK : 1;
  __shared__ float s_kf[DK], s_qf[DK], s_lr[DL];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int row, h;
  split_row(blockIdx.x, H, h_magic, row, h);
  int slot = row;
  if (slots) {
    slot = slots[row];
    if (slot < 0 || slot >= p.B) return;           // reported by the tiles
  }
  const size_t sh = size_t(slot) * H + h, th = size_t(row) * H + h;
  const int L_raw = len[sh];
  const int rl = min(tid, DK - 1);
  const TIN k_raw = (static_cast<const TIN*>(k_) + th * DK)[rl];
  const TIN q_raw = (static_cast<const TIN*>(q_) + th * DK)[rl];
  float lam = 0.f;
  if constexpr (TR::DECAY && !TR::BONUS) {
    if constexpr (DL == 1) lam = scalar_ld(p.lam + th);
    else lam = p.lam[th * DL + rl];
  }
  const float* Lb = nullptr;
  const size_t LS = DL == 1 ? size_t(H) : size_t(DL);
  if constexpr (TR::DECAY)
    Lb = p.lam_log + (DL == 1 ? size_t(slot) * size_t(C) * H + h : sh * size_t(C) * DL);
  const int L = __builtin_amdgcn_readfirstlane(L_raw);
  if (L < 0 || L > C) return;                      // reported by the tiles
  if (L > 0) {                                     // uniform per workgroup
    if (w < DK / 64) {
      const int pr = tile_pos<DK>(tid);
      s_kf[pr] = to_f32(k_raw);
      s_qf[pr] = to_f32(q_raw);
      float lr = 0.f;
      // readout decay, as in the step
      if constexpr (TR::DECAY) lr = cumulative_decay<DL>(Lb, LS, L, DL == 1 ? 0 : tid) + lam;
      if (tid < DL) s_lr[pr] = lr;
    }
    __syncthreads();                               // (also: every wave has read the length)
    float* out = coef + th * 2 * size_t(C);
    replay_coefficients<OP, DK, 256>(static_cast<const TIN*>(p.k_log) + sh * size_t(C) * DK, Lb,
                                     LS, L, s_kf, s_qf, s_lr, [&](int i, float gk, float gq) {
                                       if constexpr (TR::DELTA) out[i] = gk;
                                       out[C + i] = gq;
                                     });
  }
  if (L == 0) __syncthreads();                     // every wave has read the length
  if (tid == 0) len[sh] = L < C ? L + 1 : 0;
}

// ------------------------------------------------------------------ tile step
template <int OP, int DK, int DV, int NV, bool SPLIT, typename TIN>
__global__ __launch_bounds__(tile_threads(DK, DV, NV))
void tile_step_kernel(const int32_t* slots, const int32_t* len, void* S_, const void* k_,
                      const void* q_, int H, uint32_t h_magic, int n, int C, KParams p,
                      const float* __restrict__ coef) {
  using TC = TileCfg<DK, DV, NV>;
  using TR = OpTraits<OP>;
  using TU = typename UType<OP, TIN>::type;
  constexpr int NT = TC::NT, NCG = TC::NCG, NRG = TC::NRG, RPT = TC::RPT, DVT = TC::DVT;
  constexpr int CH = TC::CH, KTS = TC::KTS, WK = TC::WK, LPE = TC::LPE, RPL = TC::RPL;
  constexpr int EPP = TC::EPP, UQ = TC::UQ, GW = 64 / NCG;
  constexpr int DL = TR::PER_KEY ? DK : 1;
  constexpr bool NEEDS_C = TR::DELTA;

  __shared__ float s_kf[DK], s_qf[DK];             // coefficient-pass order
  __shared__ float2 s_x[DK];
  __shared__ float s_em[DK];
  __shared__ float s_lr[DL], s_lm[DL];             // coefficient-pass order
  constexpr int NG = SPLIT ? 1 : DL_MAX_MERGE_INTERVAL;
  __shared__ float s_gk[NG], s_gq[NG];             // replay coefficients (fused)
  __shared__ __align__(16) float s_red[TC::NW * 2 * DVT];
  __shared__ float s_dotw[WK];
  __shared__ __align__(16) float s_bv[DVT];
  __shared__ __align__(16) float s_kt[DK * KTS];   // K~ chunk [DK][KTS] (merge)
  __shared__ float4 s_u[CH * NCG];                 // U chunk  [CH][NCG] (merge)

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Chunks of consecutive (row, head, tile) triples are dealt to the XCDs in turn (as in
  // the untiled kernel); a head's tiles sit in one chunk and share one L2.
  const uint32_t lin = xcd_chunked(blockIdx.x, uint32_t(n) * uint32_t(H) * NV);
  const int j = int(lin % NV);                     // value tile
  int row, h;
  split_row(lin / NV, H, h_magic, row, h);
  int slot = row;
  if (slots) {
    slot = slots[row];
    if (slot < 0 || slot >= p.B) {
      if (tid == 0 && p.err) atomicOr(p.err, 1);
      return;
    }
  }
  const size_t sh = size_t(slot) * H + h;
  const size_t th = size_t(row) * H + h;

  // ---- loads: length, token rows, the tile slice, then the log (as in the step kernel) --
  const int L_raw = len[sh];
  const int rl = min(tid, DK - 1), cl = min(tid, DVT - 1);
  const TIN k_raw = (static_cast<const TIN*>(k_) + th * DK)[rl];
  const TIN q_raw = (static_cast<const TIN*>(q_) + th * DK)[rl];
  float lam = 0.f, uf = 0.f, beta = 0.f;
  if constexpr (TR::DECAY && DL != 1) lam = p.lam[th * DL + rl];
  sched_fence();
  const int cg = tid % NCG, rg = tid / NCG;
  const int c0 = j * DVT + 4 * cg;                 // this thread's first value column
  // rows rg + NRG * i, columns c0 .. c0 + 3
  float* const Sh = static_cast<float*>(S_) + sh * size_t(DK) * DV;
  const auto srs = state_rsrc(Sh, DK * DV * sizeof(float));
  const uint32_t toff = uint32_t(rg * DV + c0) * sizeof(float);
  constexpr uint32_t kRowBlock = NRG * DV * sizeof(float);
  StateQuad<float> t[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) t[i].load(srs, toff, i * kRowBlock);
  if constexpr (TR::DECAY && DL == 1) lam = scalar_ld(p.lam + th);
  if constexpr (TR::BONUS) uf = p.u[size_t(h) * DK + rl];
  const TIN v_raw = (static_cast<const TIN*>(p.v) + th * DV + j * DVT)[cl];
  if constexpr (TR::DELTA) beta = scalar_ld(p.beta + th);
  const TIN* Kb = static_cast<const TIN*>(p.k_log) + sh * size_t(C) * DK;
  const TU* Ub = static_cast<const TU*>(p.u_log) + sh * size_t(C) * DV;
  float* Lb = nullptr;
  const size_t LS = DL == 1 ? size_t(H) : size_t(DL);
  if constexpr (TR::DECAY)
    Lb = p.lam_log + (DL == 1 ? size_t(slot) * size_t(C) * H + h : sh * size_t(C) * DL);
  asm volatile("" ::"s"(Kb), "s"(Ub), "s"(Lb), "s"(coef));
  sched_fence();

  int L = __builtin_amdgcn_readfirstlane(L_raw);
  if (L < 0 || L > C) {
    if (tid == 0 && p.err) atomicOr(p.err, 2);
    return;
  }
  // Split replay: the length is already committed (C == 0 has no prepare launch and
  // nothing to commit).
  if constexpr (SPLIT) L = L == 0 ? C : L - 1;
  // The log values of this row group and, with split replay, their prepared coefficients.
  Raw4<TU> u_raw[UQ];
  float gk[UQ] = {}, gq[UQ] = {};
  const float* const cp = SPLIT ? coef + th * 2 * size_t(C) : nullptr;
#pragma unroll
  for (int a = 0; a < UQ; ++a) {
    if (a * NRG + w * GW < L) {                    // uniform per wave
      const int ic = min(a * NRG + rg, L - 1);
      u_raw[a].load(Ub + size_t(ic) * DV + c0);
      if constexpr (SPLIT) {
        if constexpr (NEEDS_C) gk[a] = cp[ic];
        gq[a] = cp[C + ic];
      }
    }
  }

  // ---- prologue: per-row decay factors, token vectors, the token dot product --------
  if (w < WK) {
    float ell = 0.f;
    if constexpr (TR::DECAY) ell = cumulative_decay<DL>(Lb, LS, L, DL == 1 ? 0 : tid);
    const float kf = to_f32(k_raw), qf = to_f32(q_raw);
    const float lm = ell + lam;
    const float lr = TR::BONUS ? ell : lm;
    const float er = dl_exp(lr);
    const int pr = tile_pos<DK>(tid);
    s_kf[pr] = kf;
    s_qf[pr] = qf;
    s_x[tid] = make_float2(er * kf, er * qf);
    s_em[tid] = dl_exp(lm);
    if (tid < DL) {
      s_lr[pr] = lr;
      s_lm[pr] = lm;
    }
    float d = TR::BONUS ? qf * uf * kf : qf * kf;
    d = xor32_sum(xor16_sum(group_sum<16>(d)));
    if ((tid & 63) == 0) s_dotw[w] = d;
  }
  __syncthreads();

  // ---- base readout of the tile's columns, replay coefficients, log replay -----------
  float4 cv = f4(0.f), ov = f4(0.f);
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const float2 x = s_x[rg + NRG * i];
    const float4 sj = t[i].get();
    if constexpr (NEEDS_C) cv = fma4(x.x, sj, cv);
    ov = fma4(x.y, sj, ov);
  }
  if constexpr (!SPLIT) {
    replay_coefficients<OP, DK, NT>(Kb, Lb, LS, L, s_kf, s_qf, s_lr, [&](int i, float gk, float gq) {
      if constexpr (NEEDS_C) s_gk[i] = gk;
      s_gq[i] = gq;
    });
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < UQ; ++a) {
    if (a * NRG + w * GW < L) {                    // uniform per wave
      const int i = a * NRG + rg, ic = min(i, L - 1);
      const float4 u = u_raw[a].get();
      if constexpr (!SPLIT) {
        if constexpr (NEEDS_C) gk[a] = s_gk[ic];
        gq[a] = s_gq[ic];
      }
      if (i < L) {                                 // as in the step kernel
        if constexpr (NEEDS_C) cv = fma4(gk[a], u, cv);
        ov = fma4(gq[a], u, ov);
      }
    }
  }
  for (int i = UQ * NRG + rg; i < L; i += NRG) {   // entries past those loaded ahead
    const float4 u = ld4(Ub + size_t(i) * DV + c0);
    if constexpr (NEEDS_C) cv = fma4(SPLIT ? cp[i] : s_gk[i], u, cv);
    ov = fma4(SPLIT ? cp[C + i] : s_gq[i], u, ov);
  }
  if constexpr (NEEDS_C) cv = column_sum<NCG>(cv);
  ov = column_sum<NCG>(ov);
  if ((tid & 63) < NCG) {
    if constexpr (NEEDS_C) st4(&s_red[w * 2 * DVT + 4 * cg], cv);
    st4(&s_red[(w * 2 + 1) * DVT + 4 * cg], ov);
  }
  __syncthreads();

  // ---- update factors, the output slice and the append (Eq. 5), one thread per column ---
  if (tid < DVT) {
    float c = 0.f, o = 0.f, dot = 0.f;
#pragma unroll
    for (int x = 0; x < TC::NW; ++x) {
      if constexpr (NEEDS_C) c += s_red[x * 2 * DVT + tid];
      o += s_red[(x * 2 + 1) * DVT + tid];
    }
#pragma unroll
    for (int x = 0; x < WK; ++x) dot += s_dotw[x];
    const float v = to_f32(v_raw);
    const float b = TR::DELTA ? beta * (v - c) : v;
    p.o[th * DV + j * DVT + tid] = fmaf(dot, b, o);
    if (L < C) {
      TU* Ud = static_cast<TU*>(p.u_log) + (sh * size_t(C) + L) * DV + j * DVT;
      if constexpr (TR::DELTA) reinterpret_cast<float*>(Ud)[tid] = b;
      else Ud[tid] = v_raw;
    }
    s_bv[tid] = b;
  }
  if (L < C) {                                     // tile 0 writes the shared entries
    if (j == 0 && w < WK) {
      static_cast<TIN*>(p.k_log)[(sh * size_t(C) + L) * DK + tid] = k_raw;
      if constexpr (TR::DECAY) {
        if (tid < DL) Lb[size_t(L) * LS + tid] = s_lm[tile_pos<DK>(tid)];
      }
    }
    return;
  }

  // ---- merge (Eq. 6) of the tile's columns, on MFMA as in the step kernel --------------
  __syncthreads();
  const float4 bv = *reinterpret_cast<const float4*>(&s_bv[4 * cg]);
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  constexpr int NRB = RPT / 4;
  f32x4 acc[NRB][4];
  int a_off[NRB];
  constexpr int EB = NCG / 4;                      // entries per read of the A operand
  constexpr int CB = EB == 4 ? 2 : EB == 2 ? 1 : 0;
  static_assert(EB == 1 || EB == 2 || EB == 4, "blocks of a row group");
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    a_off[rb] = tile_pos<DK>(rg + NRG * (4 * rb + (cg & 3))) * KTS + (cg >> 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = rg + NRG * (4 * rb + i);
      const float4 m = fma4(s_kf[tile_pos<DK>(r)], bv, s_em[r] * t[4 * rb + i].get());
      acc[rb][0][i] = m.x; acc[rb][1][i] = m.y; acc[rb][2][i] = m.z; acc[rb][3][i] = m.w;
    }
  }
  const int e_ = tid / LPE, c_ = tid % LPE;
  for (int i0 = 0; i0 < L; i0 += CH) {              // uniform trip count
    const int nn = min(CH, L - i0);
    if (i0 > 0) __syncthreads();                    // the previous chunk is consumed
#pragma unroll
    for (int e0 = 0; e0 < CH; e0 += EPP) {          // K~_i[r] = e^(l'_r - Lam_i,r) K_i[r]
      const int e = e0 + e_, i = i0 + e, ic = min(i, L - 1);
      if (e < CH) {
        RawRun<TIN, RPL> kg;
        RawRun<float, DL == 1 ? 4 : RPL> lg;
        float wt = 1.f;
        kg.load(Kb + size_t(ic) * DK + c_ * RPL);
        if constexpr (DL != 1) lg.load(Lb + size_t(ic) * LS + c_ * RPL);
        else if constexpr (TR::DECAY) wt = dl_exp(s_lm[0] - Lb[size_t(ic) * LS]);
#pragma unroll
        for (int x = 0; x < RPL; ++x) {
          const int pr = x * LPE + c_;
          if constexpr (DL != 1) wt = dl_exp(s_lm[pr] - lg.at(x));
          s_kt[pr * KTS + e] = i < L ? wt * kg.at(x) : 0.f;
        }
      }
    }
    for (int x = tid; x < CH * NCG; x += NT) {
      const int ii = x / NCG, c4 = x % NCG;
      s_u[x] = ii < nn ? ld4(Ub + size_t(i0 + ii) * DV + j * DVT + 4 * c4) : f4(0.f);
    }
    __syncthreads();
    for (int ii = 0; ii < nn; ii += 4) {            // zero-padded to a multiple of 4
#pragma unroll
      for (int e4 = 0; e4 < 4; e4 += EB) {
        float a[NRB];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) a[rb] = s_kt[a_off[rb] + ii + e4];
#define DL_MERGE_ENTRY(e)                                                                   \
  if constexpr (e < EB) {                                                                   \
    const float4 b = s_u[(ii + e4 + e) * NCG + cg];                                         \
    _Pragma("unroll") for (int rb = 0; rb < NRB; ++rb) {                                    \
      acc[rb][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.x, acc[rb][0], CB, e % EB, 0); \
      acc[rb][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.y, acc[rb][1], CB, e % EB, 0); \
      acc[rb][2] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.z, acc[rb][2], CB, e % EB, 0); \
      acc[rb][3] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.w, acc[rb][3], CB, e % EB, 0); \
    }                                                                                       \
  }
        DL_MERGE_ENTRY(0) DL_MERGE_ENTRY(1) DL_MERGE_ENTRY(2) DL_MERGE_ENTRY(3)
#undef DL_MERGE_ENTRY
      }
    }
  }
  // Rows gathered into registers of their own and held until the last store has issued
  // (see the step kernel).
  u32x4 x[RPT];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    asm volatile("s_nop 7\n\ts_nop 7"
                 : "+v"(acc[rb][0]), "+v"(acc[rb][1]), "+v"(acc[rb][2]), "+v"(acc[rb][3]));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[4 * rb + i] = u32x4{__float_as_uint(acc[rb][0][i]), __float_as_uint(acc[rb][1][i]),
                            __float_as_uint(acc[rb][2][i]), __float_as_uint(acc[rb][3][i])};
      asm volatile("" : "+v"(x[4 * rb + i]));
    }
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i)
    __builtin_amdgcn_raw_buffer_store_b128(x[i], srs, toff, i * kRowBlock, kStateStorePolicy);
#pragma unroll
  for (int i = 0; i < RPT; ++i) asm volatile("" ::"v"(x[i]));
}

// ------------------------------------------------------------------ Finalize
// One thread per (row, head): append -> L + 1; merge -> L = 0.  The cumulative log-decay
// follows from Lam_log[L] (written by tile 0) and L, so L is all there is to commit.
// BACK: the length before such a commit (the prepare kernel's, whose tiles did not run).
template <int OP, bool BACK>
__global__ __launch_bounds__(256) void finalize_kernel(const int32_t* slots, int32_t* len,
                                                       int n, int H, uint32_t h_magic,
                                                       int B, int C) {
  const uint32_t lin = blockIdx.x * 256u + threadIdx.x;
  if (lin >= uint32_t(n) * uint32_t(H)) return;
  int row, h;
  split_row(lin, H, h_magic, row, h);
  const int slot = slots ? slots[row] : row;
  if (slot < 0 || slot >= B) return;                // invalid: reported by the tiles
  const size_t sh = size_t(slot) * H + h;
  const int L = len[sh];
  if (L < 0 || L > C) return;                       // invalid: reported by the tiles
  if constexpr (BACK) len[sh] = L > 0 ? L - 1 : C;
  else len[sh] = L < C ? L + 1 : 0;
}

// ------------------------------------------------------------------ dispatch
template <int OP, int DK, int DV, int NV, bool SPLIT, typename TIN>
hipError_t launch_tiled_one(const KParams& p, const float* coef, hipStream_t s) {
  using TC = TileCfg<DK, DV, NV>;
  const int32_t* slots = p.slots;
  const int32_t* len = p.len;
  void* S = p.S;
  const void *k = p.k, *q = p.q;
  int H = p.H, n = p.n, C = p.C;
  uint32_t h_magic = 0xffffffffu / uint32_t(p.H);
  KParams rest = p;
  const float* carg = coef;
  void* args[] = {&slots, &len, &S, &k, &q, &H, &h_magic, &n, &C, &rest, &carg};
  return hipLaunchKernel(reinterpret_cast<const void*>(&tile_step_kernel<OP, DK, DV, NV, SPLIT, TIN>),
                         dim3(unsigned(p.n) * unsigned(p.H) * NV), dim3(TC::NT), args, 0, s);
}

template <int OP, int DK, typename TIN>
hipError_t launch_prep(const KParams& p, float* coef, hipStream_t s) {
  const int32_t* slots = p.slots;
  int32_t* len = p.len;
  const void *k = p.k, *q = p.q;
  float* carg = coef;
  int H = p.H, C = p.C;
  uint32_t h_magic = 0xffffffffu / uint32_t(p.H);
  KParams rest = p;
  void* args[] = {&slots, &len, &k, &q, &carg, &H, &h_magic, &C, &rest};
  return hipLaunchKernel(reinterpret_cast<const void*>(&replay_prep_kernel<OP, DK, TIN>),
                         dim3(unsigned(p.n) * unsigned(p.H)), dim3(256), args, 0, s);
}

template <int OP, bool BACK>
hipError_t launch_finalize(const KParams& p, hipStream_t s) {
  const int32_t* slots = p.slots;
  int32_t* len = p.len;
  int n = p.n, H = p.H, B = p.B, C = p.C;
  uint32_t h_magic = 0xffffffffu / uint32_t(p.H);
  void* args[] = {&slots, &len, &n, &H, &h_magic, &B, &C};
  const unsigned total = unsigned(p.n) * unsigned(p.H);
  return hipLaunchKernel(reinterpret_cast<const void*>(&finalize_kernel<OP, BACK>),
                         dim3((total + 255) / 256), dim3(256), args, 0, s);
}

// Split replay with a log: [ReplayPrep and commit] -> tiles.  Otherwise: tiles ->
// Finalize (with no log there is nothing to prepare, and the length stays 0).
template <int OP, int DK, int DV, typename TIN>
hipError_t launch_tiled_shape(int nv, bool split, const KParams& p, float* coef, hipStream_t s) {
  hipError_t e = hipSuccess;
  split = split && p.C > 0;
  if (split) e = launch_prep<OP, DK, TIN>(p, coef, s);
  if (e != hipSuccess) return e;
  if (nv == 2) e = split ? launch_tiled_one<OP, DK, DV, 2, true, TIN>(p, coef, s)
                         : launch_tiled_one<OP, DK, DV, 2, false, TIN>(p, coef, s);
  else if (nv == 4) e = split ? launch_tiled_one<OP, DK, DV, 4, true, TIN>(p, coef, s)
                              : launch_tiled_one<OP, DK, DV, 4, false, TIN>(p, coef, s);
  else e = hipErrorInvalidValue;
  if (split) {
    if (e != hipSuccess) (void)launch_finalize<OP, true>(p, s);   // e is what the caller hears
    return e;
  }
  if (e != hipSuccess || p.C == 0) return e;
  return launch_finalize<OP, false>(p, s);
}

template <int OP, typename TIN>
hipError_t launch_tiled_in(int dk, int dv, int nv, bool split, const KParams& p, float* coef,
                           hipStream_t s) {
  if (dk == 128 && dv == 128) return launch_tiled_shape<OP, 128, 128, TIN>(nv, split, p, coef, s);
  if (dk == 64 && dv == 64) return launch_tiled_shape<OP, 64, 64, TIN>(nv, split, p, coef, s);
  if (dk == 64 && dv == 128) return launch_tiled_shape<OP, 64, 128, TIN>(nv, split, p, coef, s);
  if (dk == 128 && dv == 64) return launch_tiled_shape<OP, 128, 64, TIN>(nv, split, p, coef, s);
  return hipErrorInvalidValue;
}

template <int OP>
hipError_t launch_tiled_op(int dk, int dv, bool bf16, int nv, bool split, const KParams& p,
                           float* coef, hipStream_t s) {
  return bf16 ? launch_tiled_in<OP, uint16_t>(dk, dv, nv, split, p, coef, s)
              : launch_tiled_in<OP, float>(dk, dv, nv, split, p, coef, s);
}

}  // namespace dl
