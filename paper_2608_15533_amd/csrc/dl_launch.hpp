// Template dispatch from runtime (mode, dk, dv, dtype) to a kernel instantiation.
#pragma once

#include "dl_flush.hpp"
#include "dl_kernel.hpp"

namespace dl {

template <int OP, int DK, int DV, int MODE, typename TIN, typename TS, int CE>
hipError_t launch_build(const KParams& p, hipStream_t s) {
  const dim3 grid(unsigned(p.n) * unsigned(p.H));
  const dim3 block(threads_per_head(DK, DV, CE));
  const int32_t* slots = p.slots;
  int32_t* len = p.len;
  void* S = p.S;
  const void *k = p.k, *q = p.q;
  int H = p.H, n = p.n, C = p.C;
  uint32_t h_magic = 0xffffffffu / uint32_t(p.H);
  KParams rest = p;
  void* args[] = {&slots, &len, &S, &k, &q, &H, &h_magic, &n, &C, &rest};
  return hipLaunchKernel(
      reinterpret_cast<const void*>(&deltalog_kernel<OP, DK, DV, MODE, TIN, TS, CE>), grid,
      block, args, 0, s);
}

template <int OP, int DK, int DV, typename TIN, typename TS>
hipError_t launch_flush(const KParams& p, hipStream_t s) {
  const int32_t* slots = p.slots;
  int32_t* len = p.len;
  void* S = p.S;
  const void *k_log = p.k_log, *u_log = p.u_log;
  int H = p.H, n = p.n, C = p.C;
  uint32_t h_magic = 0xffffffffu / uint32_t(p.H);
  KParams rest = p;
  void* args[] = {&slots, &len, &S, &k_log, &u_log, &H, &h_magic, &n, &C, &rest};
  return hipLaunchKernel(reinterpret_cast<const void*>(&flush_kernel<OP, DK, DV, TIN, TS>),
                         dim3(unsigned(p.n) * unsigned(p.H)), dim3(FlushCfg<DK, DV>::NT), args, 0, s);
}

// The build for the descriptor's log capacity (the eager kernel has no log).  The readout
// keeps all three as well: with the 64-entry build alone it takes 4.3% longer over operators,
// head shapes and types at 40 and 1536 heads (M = 16: 5.0%, M = 32: 3.4%; 0.95 to 1.24 of the
// time), the most at short lengths.
template <int OP, int DK, int DV, int MODE, typename TIN, typename TS>
hipError_t launch_one(const KParams& p, hipStream_t s) {
  if constexpr (MODE != M_EAGER) {
    if (log_build(p.C) == 64) return launch_build<OP, DK, DV, MODE, TIN, TS, 64>(p, s);
    if (log_build(p.C) == 32) return launch_build<OP, DK, DV, MODE, TIN, TS, 32>(p, s);
  }
  return launch_build<OP, DK, DV, MODE, TIN, TS, 16>(p, s);
}

template <int OP, int DK, int DV, typename TIN, typename TS>
hipError_t launch_mode(int mode, const KParams& p, hipStream_t s) {
  switch (mode) {
    case M_EAGER: return launch_one<OP, DK, DV, M_EAGER, TIN, TS>(p, s);
    case M_STEP: return launch_one<OP, DK, DV, M_STEP, TIN, TS>(p, s);
    case M_MERGE: return launch_one<OP, DK, DV, M_MERGE, TIN, TS>(p, s);
    case M_FLUSH: return launch_flush<OP, DK, DV, TIN, TS>(p, s);
    case M_READOUT: return launch_one<OP, DK, DV, M_READOUT, TIN, TS>(p, s);
  }
  return hipErrorInvalidValue;
}

template <int OP, typename TIN, typename TS>
hipError_t launch_shape(int mode, int dk, int dv, const KParams& p, hipStream_t s) {
  if (dk == 128 && dv == 128) return launch_mode<OP, 128, 128, TIN, TS>(mode, p, s);
  if (dk == 64 && dv == 64) return launch_mode<OP, 64, 64, TIN, TS>(mode, p, s);
  if (dk == 64 && dv == 128) return launch_mode<OP, 64, 128, TIN, TS>(mode, p, s);
  if (dk == 128 && dv == 64) return launch_mode<OP, 128, 64, TIN, TS>(mode, p, s);
  return hipErrorInvalidValue;
}

template <int OP, typename TS>
hipError_t launch_in(int mode, int dk, int dv, bool bf16, const KParams& p, hipStream_t s) {
  return bf16 ? launch_shape<OP, uint16_t, TS>(mode, dk, dv, p, s)
              : launch_shape<OP, float, TS>(mode, dk, dv, p, s);
}

template <int OP>
hipError_t launch_op(int mode, int dk, int dv, bool bf16, bool state_bf16, const KParams& p,
                     hipStream_t s) {
  return state_bf16 ? launch_in<OP, uint16_t>(mode, dk, dv, bf16, p, s)
                    : launch_in<OP, float>(mode, dk, dv, bf16, p, s);
}

}  // namespace dl
