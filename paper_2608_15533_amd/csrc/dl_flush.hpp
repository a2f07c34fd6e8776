// The flush (dl_merge without a token): Eq. 7 materialised into the base, the log emptied.
//
// There is no readout and so no partial sums to agree on with the step kernel, and the
// layout is chosen for the merge alone: 256 threads for every head, the log in chunks of 16
// entries for any interval (in registers of its own the whole log would cost the tile's
// bytes in flight), each chunk loaded while the one before is contracted.  A wave holds 16
// column quads of 4 row groups, so that the output fragment of v_mfma_f32_16x16x4f32 is the
// tile itself: lane l holds output column l % 16, component c of its quad in accumulator c,
// and rows 4 (l / 16) + i, which are rows 4 mb + i of its own row group.  Its A operand is
// the decayed key of entry l / 16 at output row l % 16, its B operand the log value of that
// entry at its own quad.
//
// us per flush of 1536 heads in a captured graph (with a fill of the lengths, about 2 us),
// as a mode of the step kernel (whole log in two LDS chunks of 32, 4x4x1 MFMA) and so:
//   KDA 64x64, bf16 state, M = 64, L = 40   16.7 / 13.9
//   KDA 128x64, M = 64, L = 40              34.1 / 28.8
//   KDA 128x128, M = 64, L = 63             57.8 / 53.9
//   GLA 128x128, bf16 state, M = 64, L = 63 47.6 / 42.0
//   GDN 128x128, M = 16, L = 15             38.2 / 38.9
//   KDA 64x128, all fp32, M = 16, L = 15    20.9 / 22.5 (the largest loss)
// 0.926 over 672 combinations of operator, shape, types, interval and length (geometric
// mean).
#pragma once

#include "dl_kernel.hpp"

namespace dl {

template <int DK, int DV>
struct FlushCfg {
  static constexpr int NT = 256;
  static constexpr int NCG = DV / 4;             // float4 column groups
  static constexpr int NRG = NT / NCG;           // row groups
  static constexpr int RPT = DK / NRG;           // state rows per thread
  static constexpr int WH = NCG / 16;            // waves side by side
  static constexpr int NMB = RPT / 4;            // blocks of 16 output rows per wave
  static constexpr int CH = 16;                  // log entries per chunk
  static constexpr int LPE = NT / CH;            // lanes per log entry (staging)
  static constexpr int RPL = DK / LPE;           // key rows per lane (staging)
  static constexpr int UQ = CH / NRG;            // log-value quads per thread and chunk
  // LDS stride of an entry's decayed keys: the four entries of a read hit other banks.
  static constexpr int KTS = DK + 20;
  // Waves per SIMD by registers: what the tile leaves.
  static constexpr int WAVES = RPT == 16 ? 4 : RPT == 8 ? 5 : 7;
  static_assert(RPT % 4 == 0 && NRG % 4 == 0 && CH % NRG == 0 && NT >= DK, "layout");
  // Position of state row r among an entry's decayed keys: output rows in lane order, so
  // that a wave's read of a block is consecutive words.
  static __device__ __forceinline__ int pos(int r) {
    const int rg = r % NRG, j = r / NRG;
    return ((rg / 4) * NMB + j / 4) * 16 + 4 * (rg % 4) + j % 4;
  }
};

template <int OP, int DK, int DV, typename TIN, typename TS>
__global__ __launch_bounds__((FlushCfg<DK, DV>::NT)) __attribute__((amdgpu_waves_per_eu((FlushCfg<DK, DV>::WAVES))))
void flush_kernel(const int32_t* slots, int32_t* len, void* S_, const void* k_log,
                  const void* u_log, int H, uint32_t h_magic, int n, int C, KParams p) {
  using FC = FlushCfg<DK, DV>;
  using TR = OpTraits<OP>;
  using TU = typename UType<OP, TIN>::type;
  constexpr int NCG = FC::NCG, NRG = FC::NRG, RPT = FC::RPT, CH = FC::CH, KTS = FC::KTS;
  constexpr int LPE = FC::LPE, RPL = FC::RPL, UQ = FC::UQ, NMB = FC::NMB;
  constexpr int EW = 64 / LPE;                    // log entries per wave (keys)
  constexpr int DL = TR::PER_KEY ? DK : 1;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

  __shared__ float s_l[DL], s_e[DL];              // ell, e^ell (per-key decay)
  __shared__ float s_kt[CH * KTS];                // decayed keys of a chunk
  __shared__ float4 s_u[CH * NCG];                // ... and its log values

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int row, h;                                     // row of the slot list and head
  split_row(xcd_chunked(blockIdx.x, uint32_t(n) * uint32_t(H)), H, h_magic, row, h);
  int slot = row;
  if (slots) {
    slot = slots[row];
    if (slot < 0 || slot >= p.B) {                // uniform per workgroup
      if (tid == 0 && p.err) atomicOr(p.err, 1);
      return;
    }
  }
  const size_t sh = size_t(slot) * H + h;
  const int L_raw = len[sh];
  sched_fence();
  const int wr = w / FC::WH;                      // the wave's row groups 4 wr .. 4 wr + 3
  const int cg = 16 * (w % FC::WH) + (lane & 15), rg = 4 * wr + (lane >> 4);
  TS* const Sh = static_cast<TS*>(S_) + sh * size_t(DK) * DV;
  const auto srs = state_rsrc(Sh, DK * DV * sizeof(TS));
  const uint32_t toff = uint32_t(rg * DV + 4 * cg) * sizeof(TS);
  constexpr uint32_t kRowBlock = NRG * DV * sizeof(TS);
  StateQuad<TS> t[RPT];
#pragma unroll
  for (int j = 0; j < RPT; ++j) t[j].load(srs, toff, j * kRowBlock);
  const size_t LS = DL == 1 ? size_t(H) : size_t(DL);
  const TIN* Kb = static_cast<const TIN*>(k_log) + sh * size_t(C) * DK;
  const TU* Ub = static_cast<const TU*>(u_log) + sh * size_t(C) * DV;
  const float* Lb = nullptr;
  if constexpr (TR::DECAY)
    Lb = p.lam_log + (DL == 1 ? size_t(slot) * size_t(C) * H + h : sh * size_t(C) * DL);
  asm volatile("" ::"s"(Kb), "s"(Ub), "s"(Lb));
  sched_fence();
  const int L = __builtin_amdgcn_readfirstlane(L_raw);
  if (L < 0 || L > C) {                           // every address below is in bounds
    if (tid == 0 && p.err) atomicOr(p.err, 2);
    return;
  }

  // Chunk c0 of the log: lanes past the live length re-read entry L-1 (staged as zeros).
  const int e_ = tid / LPE, c_ = tid % LPE, ew = w * EW;
  RawRun<TIN, RPL> k_raw{};
  RawRun<float, DL == 1 ? 4 : RPL> l_raw{};
  float l0 = 0.f;
  const int ue = tid / NCG, uc = tid % NCG;       // log value: entry, quad
  const int uw = w * 64 / NCG;                    // ... the wave's first entry
  Raw4<TU> u_raw[UQ] = {};
  auto load_chunk = [&](int c0) {
    if (c0 + ew < L) {                            // uniform per wave
      const int i = min(c0 + e_, L - 1);
      k_raw.load(Kb + size_t(i) * DK + c_ * RPL);
      if constexpr (DL != 1) l_raw.load(Lb + size_t(i) * DK + c_ * RPL);
      else if constexpr (TR::DECAY) l0 = Lb[size_t(i) * LS];
    }
#pragma unroll
    for (int a = 0; a < UQ; ++a)
      if (c0 + a * NRG + uw < L)                  // uniform per wave
        u_raw[a].load(Ub + size_t(min(c0 + a * NRG + ue, L - 1)) * DV + 4 * uc);
  };
  float ell = 0.f;                                // the newest snapshot (see the step kernel)
  if constexpr (DL != 1) {
    if (w < DK / 64) {
      if (L > 0) ell = Lb[size_t(L - 1) * DK + tid];
      s_l[tid] = ell;
      s_e[tid] = dl_exp(ell);
    }
    __syncthreads();
  } else if constexpr (TR::DECAY) {
    if (L > 0) ell = scalar_ld(Lb + size_t(L - 1) * LS);
  }

  // The decayed base, as the MFMA's accumulators: component c of the thread's row 4 mb + i
  // is acc[mb][c][i].
  f32x4 acc[NMB][4];
  float e1 = dl_exp(ell);                         // one decay per head
  pin(e1);                                        // 1 without decay: the products copy the tile
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const float4 m = (DL == 1 ? e1 : s_e[DL == 1 ? 0 : rg + NRG * j]) * t[j].get();
    acc[j / 4][0][j % 4] = m.x;
    acc[j / 4][1][j % 4] = m.y;
    acc[j / 4][2][j % 4] = m.z;
    acc[j / 4][3][j % 4] = m.w;
  }
  load_chunk(0);                                  // issued earlier it costs small heads 5%
  for (int c0 = 0; c0 < L; c0 += CH) {            // uniform
    if (c0 > 0) __syncthreads();                  // the chunk before is consumed
    const int nn = min(CH, (L - c0 + 3) / 4 * 4);   // entries read, four at a time
    if (ew < nn) {                                // uniform per wave
      float wt = 1.f;
      if constexpr (DL == 1 && TR::DECAY) wt = dl_exp(ell - l0);
      const bool live = c0 + e_ < L;
#pragma unroll
      for (int x = 0; x < RPL; ++x) {
        const int r = c_ * RPL + x;
        if constexpr (DL != 1) wt = dl_exp(s_l[r] - l_raw.at(x));
        s_kt[e_ * KTS + FC::pos(r)] = live ? wt * k_raw.at(x) : 0.f;
      }
    }
#pragma unroll
    for (int a = 0; a < UQ; ++a) {
      const int e = a * NRG + ue;
      s_u[e * NCG + uc] = c0 + e < L ? u_raw[a].get() : f4(0.f);
    }
    __syncthreads();
    load_chunk(c0 + CH);
    for (int i = 0; i < nn; i += 4) {
      const int e = i + (lane >> 4);
      const float4 b = s_u[e * NCG + cg];
#pragma unroll
      for (int mb = 0; mb < NMB; ++mb) {
        const float a = s_kt[e * KTS + (wr * NMB + mb) * 16 + (lane & 15)];
        acc[mb][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b.x, acc[mb][0], 0, 0, 0);
        acc[mb][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b.y, acc[mb][1], 0, 0, 0);
        acc[mb][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b.z, acc[mb][2], 0, 0, 0);
        acc[mb][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b.w, acc[mb][3], 0, 0, 0);
      }
    }
  }
  if (tid == 0) len[sh] = 0;                      // every wave has read it: a barrier where L > 0
#pragma unroll
  for (int mb = 0; mb < NMB; ++mb)                // wait states, as in the step kernel
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7"
                 : "+v"(acc[mb][0]), "+v"(acc[mb][1]), "+v"(acc[mb][2]), "+v"(acc[mb][3]));
  if constexpr (sizeof(TS) == 4) {
    // Rows in registers of their own until the last store has issued (see the step kernel).
    u32x4 x[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      x[j] = u32x4{__float_as_uint(acc[j / 4][0][j % 4]), __float_as_uint(acc[j / 4][1][j % 4]),
                   __float_as_uint(acc[j / 4][2][j % 4]), __float_as_uint(acc[j / 4][3][j % 4])};
      asm volatile("" : "+v"(x[j]));
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(x[j], srs, toff, j * kRowBlock, kStateStorePolicy);
#pragma unroll
    for (int j = 0; j < RPT; ++j) asm volatile("" ::"v"(x[j]));
  } else {
#pragma unroll
    for (int j = 0; j < RPT; ++j)
      StateQuad<TS>::store(srs, toff, j * kRowBlock,
                           make_float4(acc[j / 4][0][j % 4], acc[j / 4][1][j % 4],
                                       acc[j / 4][2][j % 4], acc[j / 4][3][j % 4]));
  }
}

}  // namespace dl
