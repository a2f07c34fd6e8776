// DeltaLog decode kernels for gfx950 (CDNA4, wave64).
//
// One workgroup owns one (slot, head) state: a dk x dv matrix (64 KiB at 128x128 fp32).
// Thread layout: NCG = dv/4 column groups (one float4 column slice each) times NRG row
// groups; every thread keeps RPT = dk/NRG rows x 4 columns of the state in registers (rows
// rg, rg+NRG, ..., so one wave-wide float4 load covers whole consecutive rows, 1 KiB
// contiguous).  The state is read from HBM exactly once per step and, when the step
// materialises (merge / eager / flush), written back exactly once from the same registers
// -- the read, the key-dimension reductions and the write never leave the workgroup.
// Because one workgroup owns all of a head's value columns, the replay coefficients are
// computed once per (slot, head) and the shared log metadata (K_log[L], Lam_log[L], L) has
// a single writer without any cross-workgroup finalisation (the ownership problem of
// Sec. 3.3).  The cumulative log-decay ell is not stored: it equals the newest snapshot
// Lam_log[L-1], or 0 with an empty log.
//
// The kernel is bound by HBM at large launches and by the chain launch -> live length and
// tile -> log entries -> sums -> store at small ones.  The layout depends on the head shape
// and the log capacity only, not on the number of rows: a slot's results do not depend on
// what else is in the batch.  256 threads up to 16 log entries; 128 x 128 heads with
// longer logs take 512 threads (twice the entries per coefficient pass, half the log
// values per thread).  us per step in a captured graph, 256 against 512 threads:
//   GDN 64x32 heads   M = 16: 25.9 / 26.8      KDA 128x32 heads  M = 16: 53.2 / 53.6
//   KDA 128x32 heads  M = 32: 67.9 / 59.7      KDA 64x32 heads   M = 64: 39.6 / 39.1
//   RetNet 8x16 heads M = 64: 4.99 / 4.57      GLA 100x32, bf16 state, M = 64: 43.5 / 41.7
//
// Modes (one template per mode; the per-slot append/merge branch of Alg. 1 is taken on the
// device from that slot's live length; the flush has a kernel of its own, dl_flush.hpp):
//   EAGER   Eq. 3 on a dense state (no log).
//   STEP    Alg. 1: readout + replay, then append (Eq. 5) if L < C, else merge (Eq. 6).
//   MERGE   the merge branch at the current L (a forced merge, any 0 <= L <= C).
//   READOUT o = x^T (Eq. 7 state), no writes to the state.
//
// Per (slot, head) and step the arithmetic is (l' = ell + lambda):
//   replay coefficient of entry i for a vector x:  g_i(x) = sum_r e^(l_r - Lam_i,r) x_r K_i,r
//   base readout:   sum_r e^(l_r) x_r S_r,:      (l = ell for RWKV6, l' otherwise)
//   correction c = base(k) + sum_i g_i(k) U_i ;  b = beta (v - c)             (GDN/KDA)
//              b = v                             (RWKV6, linear attention, RetNet, GLA)
//   output     o = base(q) + sum_i g_i(q) U_i + (q.k) b    (post-update: all but RWKV6)
//              o = base(r) + sum_i g_i(r) U_i + (r.(u*k)) v                   (RWKV6)
//   merge      S <- diag(e^l') S + sum_i diag(e^(l'-Lam_i)) K_i U_i^T + k b^T  (Eq. 6)
// Linear attention has no decay: every e^(.) above is 1 and ell, Lam_log and lambda are
// never touched.
// Every decay factor is evaluated as exp of a log-decay *difference* (<= 0 in normal
// use), never as a product of exp(l') and exp(-Lam_i).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dl_internal.h"

namespace dl {

// ------------------------------------------------------------------ loads/stores
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 ld4(const uint16_t* p) {
  const uint2 w = *reinterpret_cast<const uint2*>(p);
  return make_float4(bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y));
}

__device__ __forceinline__ void st4(float* d, float4 v) { *reinterpret_cast<float4*>(d) = v; }

__device__ __forceinline__ float4 f4(float a) { return make_float4(a, a, a, a); }
__device__ __forceinline__ float4 operator+(float4 a, float4 b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float4 operator-(float4 a, float4 b) {
  return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
}
__device__ __forceinline__ float4 operator*(float s, float4 a) {
  return make_float4(s * a.x, s * a.y, s * a.z, s * a.w);
}
// a + s * b, written as separate fused multiply-adds per lane element.
__device__ __forceinline__ float4 fma4(float s, float4 b, float4 a) {
  return make_float4(fmaf(s, b.x, a.x), fmaf(s, b.y, a.y), fmaf(s, b.z, a.z), fmaf(s, b.w, a.w));
}

// Sum over aligned groups of N lanes (N = 4, 8 or 16), every lane of a group ending with
// the group's sum.  The lane exchanges are DPP moves inside a 16-lane row (mirror over 16
// lanes, mirror over 8, then swaps of lane pairs of pairs and of lane pairs), and the
// exchanges across rows below are the gfx950 row-swap instructions: none needs an LDS
// round trip.  Callers reduce only where every lane of the wave is active.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(N == 4 || N == 8 || N == 16, "DPP rows hold 16 lanes");
  if constexpr (N == 16) v += dpp_move<0x140>(v);   // row_mirror: lane i <- 15 - i
  if constexpr (N >= 8) v += dpp_move<0x141>(v);    // row_half_mirror: lane i <- 7 - i
  v += dpp_move<0x4E>(v);                           // quad_perm [2,3,0,1]
  v += dpp_move<0xB1>(v);                           // quad_perm [1,0,3,2]
  return v;
}
// Sums over lane pairs that leave each lane one of the two sums: a(l) + a(l ^ 32) in lanes
// 0-31 and b(l) + b(l ^ 32) in lanes 32-63 (v_permlane32_swap trades a's upper half for
// b's lower half), and likewise a in the even 16-lane rows and b in the odd ones.  One swap
// and one addition do what two all-lane sums take two of each and two copies for.
__device__ __forceinline__ float swap32_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// v(lane) + v(lane ^ 16) and v(lane) + v(lane ^ 32) in every lane.
__device__ __forceinline__ float xor16_sum(float v) { return swap16_sum(v, v); }
__device__ __forceinline__ float xor32_sum(float v) { return swap32_sum(v, v); }

// f(x0) + ... + f(x0 + N - 1) in pairs: the last and largest partial sums take log2(N)
// roundings instead of N - 1.  Mean error of the outputs against 64 bits, in turn and in
// pairs, at the same time: linear attention 64 x 128, M = 13, 6.43e-8 and 6.24e-8; RetNet
// 128 x 128, M = 64, 1.58e-7 and 1.55e-7.
template <int N, typename F>
__device__ __forceinline__ auto pair_sum(F f, int x0 = 0) {
  if constexpr (N == 1) return f(x0);
  else return pair_sum<N / 2>(f, x0) + pair_sum<N / 2>(f, x0 + N / 2);
}

// Decay factors exp(x) for log-decay differences x <= 0: the hardware base-2
// exponential of x * log2(e) (two instructions instead of the 13 of a correctly
// rounded expf).  Its relative error is about 2^-24 * |x| * log2(e) plus one ulp
// (below 2e-6 for |x| <= 40); exp(0) is exactly 1.
__device__ __forceinline__ float dl_exp(float x) { return __expf(x); }

// State-tile traffic.  The base is streamed once per step and not reused by this
// workgroup, so by default its loads and stores carry the non-temporal hint.
#ifndef DL_NT_STATE
#define DL_NT_STATE 1
#endif
// Cache policy of the state-tile stores alone (the merged base): -1 = as the loads;
// by default non-temporal with device scope (nt sc1), so that the base is written
// through the XCD's L2 rather than held there as dirty lines while the other
// workgroups of the launch stream their tiles in.
#ifndef DL_STATE_STORE_POLICY
#define DL_STATE_STORE_POLICY (DL_NT_STATE ? 18 : -1)
#endif
// The state tile of one (slot, head) is addressed through a buffer resource: the
// head's base address lives in scalar registers, each lane keeps one 32-bit offset and
// the row blocks differ by a scalar offset, so no per-row 64-bit addresses occupy
// vector registers between the load and the store.  The resource covers exactly the
// head's dk x dv state elements; the hardware drops accesses outside it.
constexpr int kStateCachePolicy = DL_NT_STATE ? 2 : 0;   // 2 = non-temporal (nt)
constexpr int kStateStorePolicy =            // 18 = nt (2) + device scope (sc1, 16)
    DL_STATE_STORE_POLICY >= 0 ? DL_STATE_STORE_POLICY : kStateCachePolicy;
constexpr int kRawBufferFlags = 0x00020000;                // 32-bit data format, raw access

__device__ __forceinline__ __amdgpu_buffer_rsrc_t state_rsrc(void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, int(bytes), kRawBufferFlags);
}

// Round fp32 to bf16, nearest even (finite values).
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// Four consecutive state elements of one row, as held by one lane between the load and
// the store.  fp32 state: one 16-byte access (stored by the kernels themselves, see the
// merge); bf16 state: one 8-byte access, widened to fp32 on use and rounded (nearest even)
// on store.
template <typename TS> struct StateQuad;
template <> struct StateQuad<float> {
  float4 w;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kStateCachePolicy);
    w = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]),
                    __uint_as_float(v[3]));
  }
  __device__ __forceinline__ float4 get() const { return w; }
  __device__ __forceinline__ void opaque() {}
};
template <> struct StateQuad<uint16_t> {
  uint2 w;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, kStateCachePolicy);
    w = make_uint2(v[0], v[1]);
  }
  // The compiler takes the words as changed here: it widens them again for a later use
  // instead of keeping the widened row (twice the registers) live until then.
  __device__ __forceinline__ void opaque() { asm volatile("" : "+v"(w.x), "+v"(w.y)); }
  __device__ __forceinline__ float4 get() const {
    return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
                       __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
  }
  static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t voff,
                                               uint32_t soff, float4 v) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 x = {bf16_rne(v.x) | (bf16_rne(v.y) << 16), bf16_rne(v.z) | (bf16_rne(v.w) << 16)};
    __builtin_amdgcn_raw_buffer_store_b64(x, r, voff, soff, kStateStorePolicy);
  }
};

constexpr uint32_t kXcds = 8;   // accelerator complex dies of an MI355X
// (row, head) pairs per XCD chunk: 32 heads' 4-byte metadata is one 128-byte line.
// 0 gives each XCD a single contiguous range instead.
#ifndef DL_XCD_CHUNK
#define DL_XCD_CHUNK 32
#endif
constexpr uint32_t kXcdChunk = DL_XCD_CHUNK;

// Raw register images of loads whose conversion to fp32 is deferred: converting right
// after a load makes the wave wait for it, and (loads completing in issue order) for
// every load issued before it -- the state tile included.
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(uint16_t x) { return __uint_as_float(uint32_t(x) << 16); }

template <typename T> struct Raw4;                 // four consecutive elements
template <> struct Raw4<float> {
  float4 w;
  __device__ __forceinline__ void load(const float* p) { w = *reinterpret_cast<const float4*>(p); }
  __device__ __forceinline__ float4 get() const { return w; }
};
template <> struct Raw4<uint16_t> {
  uint2 w;
  __device__ __forceinline__ void load(const uint16_t* p) { w = *reinterpret_cast<const uint2*>(p); }
  __device__ __forceinline__ float4 get() const {
    return make_float4(bf_lo(w.x), bf_hi(w.x), bf_lo(w.y), bf_hi(w.y));
  }
};

template <typename T, int N> struct RawRun;         // N consecutive elements, N % 4 == 0
template <int N> struct RawRun<float, N> {
  float4 w[N / 4];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) w[i] = reinterpret_cast<const float4*>(p)[i];
  }
  __device__ __forceinline__ float at(int x) const {   // x a compile-time constant
    const float4 v = w[x / 4];
    return x % 4 == 0 ? v.x : x % 4 == 1 ? v.y : x % 4 == 2 ? v.z : v.w;
  }
};
template <int N> struct RawRun<uint16_t, N> {
  static_assert(N % 4 == 0, "run length");
  static constexpr bool W16 = N % 8 == 0;           // 16-byte words, else 8-byte words
  using Word = std::conditional_t<W16, uint4, uint2>;
  Word w[W16 ? N / 8 : N / 4];
  __device__ __forceinline__ void load(const uint16_t* p) {
#pragma unroll
    for (int i = 0; i < (W16 ? N / 8 : N / 4); ++i) w[i] = reinterpret_cast<const Word*>(p)[i];
  }
  __device__ __forceinline__ float at(int x) const {   // x a compile-time constant
    uint32_t d;
    if constexpr (W16) {
      const uint4 v = w[x / 8];
      const int y = x % 8 / 2;
      d = y == 0 ? v.x : y == 1 ? v.y : y == 2 ? v.z : v.w;
    } else {
      const uint2 v = w[x / 4];
      d = x % 4 / 2 == 0 ? v.x : v.y;
    }
    return x % 2 ? bf_hi(d) : bf_lo(d);
  }
};

// Read one float at a workgroup-uniform address through the scalar path (the constant
// address space): the read waits on its own counter instead of queueing behind the
// vector loads in flight.  Only for data that no workgroup of the launch writes (the
// scalar cache is invalidated at every kernel launch).
__device__ __forceinline__ float scalar_ld(const float* ptr) {
  typedef const float __attribute__((address_space(4))) const_float;
  return *(const_float*)ptr;
}

// Nothing may be scheduled across this point (loads keep their issue order).
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// The value is recomputed or re-read from here on, not kept: an empty asm block that
// claims to change it.  Bounds how far the compiler moves the sums it feeds.
__device__ __forceinline__ void pin(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(float4& v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

// ------------------------------------------------------------------ configuration
// What distinguishes the operators of Table 1 inside the kernel.
template <int OP>
struct OpTraits {
  static constexpr bool DELTA = OP == OP_GDN || OP == OP_KDA;   // b = beta (v - correction)
  static constexpr bool PER_KEY = OP == OP_KDA || OP == OP_RWKV6 || OP == OP_GLA;
  static constexpr bool DECAY = OP != OP_LINATTN;               // linear attention: none
  static constexpr bool BONUS = OP == OP_RWKV6;   // pre-update readout plus r^T diag(u) k v^T
};

// U_log holds the delta rule's corrected values in fp32, and exact copies of v (in the
// activation dtype) for every other operator.
template <int OP, typename TIN>
struct UType { using type = std::conditional_t<OpTraits<OP>::DELTA, float, TIN>; };

// Log capacities the kernel is built for (CE entries; the host takes the smallest that
// holds C = M - 1).  The log entries of a build are replayed from registers, loaded in one
// go, so a longer log takes more registers and its own build.
constexpr int log_build(int capacity) { return capacity <= 16 ? 16 : capacity <= 32 ? 32 : 64; }

// Threads per workgroup: 256, and 512 for 128 x 128 heads with more than 16 log entries
// (see the top).
constexpr int threads_per_head(int dk, int dv, int ce) {
  return dk == 128 && dv == 128 && ce > 16 ? 512 : 256;
}

template <int OP, int DK, int DV, int MODE, int CE_>
struct Cfg {
  static constexpr int CE = CE_;                 // log entries of the build (C <= CE)
  static constexpr int NT = threads_per_head(DK, DV, CE);
  static constexpr int NCG = DV / 4;             // float4 column groups
  static constexpr int NRG = NT / NCG;           // row groups
  static constexpr int RPT = DK / NRG;           // state rows per thread
  static constexpr int NW = NT / 64;             // waves
  static constexpr int DL = OpTraits<OP>::PER_KEY ? DK : 1;   // log-decay width
  static constexpr int LPE = DK == DV ? 16 : 8;  // lanes per log entry (coefficient pass)
  static constexpr int RPL = DK / LPE;           // key rows per lane (coefficient pass)
  // Log entries staged per merge chunk: the 64-entry build stages two chunks of 32 in
  // turn (all 64 at once take LDS that leaves 64 x 64 heads four workgroups per CU: GLA
  // 250x32 heads, bf16 state, M = 40: 34.2 us a step, in chunks 29.7).
  static constexpr int CH = CE < 32 ? CE : 32;
  static constexpr int EPP = NT / LPE < CH ? NT / LPE : CH;   // log entries per pass
  static constexpr int NP = CE / EPP;            // coefficient passes
  static constexpr int UQ = (CE + NRG - 1) / NRG;             // log-value quads per thread
  static constexpr int KTS = CH + 4;             // LDS row stride of the decayed log keys
  static constexpr bool DELTA = OpTraits<OP>::DELTA;
  static constexpr bool DECAY = OpTraits<OP>::DECAY;
  static constexpr bool BONUS = OpTraits<OP>::BONUS;
  static constexpr bool HAS_LOG = MODE != M_EAGER;
  static constexpr bool HAS_TOKEN = MODE == M_EAGER || MODE == M_STEP || MODE == M_MERGE;
  static constexpr bool NEEDS_C = DELTA && HAS_TOKEN;
  static constexpr bool CAN_MERGE = MODE != M_READOUT;
  static constexpr bool MERGES_LOG = CAN_MERGE && HAS_LOG;
  // Waves of the per-row and the per-column work.
  static constexpr int WK = DK / 64, WV = DV / 64;
  // LDS floats of the cross-wave partial sums, and of the staged log values, which take
  // the same place once the sums are read.
  static constexpr int LRED = NW * 2 * DV;
  static constexpr int LU = MERGES_LOG ? CH * DV : 0;
  static constexpr int LSCR = LRED > LU ? LRED : LU;
  // Registers over latency: the readout and coefficient loops are kept from running
  // ahead of themselves (see pin).  It fits 128 x 128 heads with long logs in three
  // workgroups of 512 threads per CU, and 64 entries in the registers of 256 (KDA 64x32
  // heads 128x64, M = 63: 35.6 us with spills, 25.9 without).
  static constexpr bool LEAN = NT == 512 || CE == 64;
  static_assert(NT % 64 == 0 && NT >= DK && NT >= DV, "a thread per key row and value column");
  static_assert(DK % NRG == 0 && RPT % 4 == 0, "whole blocks of four rows per thread");
  static_assert(64 % NCG == 0 && (NCG == 16 || NCG == 32), "a wave holds whole rows");
  static_assert(NT % LPE == 0 && (RPL == 4 || RPL == 8 || RPL == 16), "coefficient runs");
  static_assert(CE % EPP == 0 && EPP % (64 / LPE) == 0, "whole passes of whole waves");
  static_assert(CE % CH == 0 && CH % EPP == 0, "a chunk is whole passes");
  static_assert(!(BONUS && DL == 1), "the bonus readout is only defined with per-key decay");
  // LDS position of key row r in the vectors the coefficient pass reads and in the
  // decayed log keys: the pass reads element x of every lane's run of RPL rows at once, so
  // row r = c * RPL + x is kept at x * LPE + c (consecutive words for an entry's lanes).
  static __device__ __forceinline__ int pos(int r) { return (r % RPL) * LPE + r / RPL; }
};

// Waves per SIMD the register allocator aims at: 4 (128 registers; a kernel that needs fewer
// takes fewer).
//
// The 512 threads of 17 to 32 log entries: 6 (80), or 8 (64) with a bf16 state and bf16
// activations, which keeps two KDA merges from 81 and 65 registers; every other kernel of
// them measures the same at 4, 6 and 8, but for spills: with fp32 state and activations at 6
// (KDA 64x32 heads, M = 32, us a step: 47.0, 34.4 at 4), with bf16 activations and an fp32
// state at 8 (KDA 48x32 heads, M = 18 to 33: 36.1, 21.4 at 6 and at 4).
//
// 64 entries in 256 threads of a rectangular head do not fit 128 registers where the
// snapshots are per key and everything is fp32 in 128 x 64 heads (16 rows of a log entry a
// lane), and in some merges with the token: 3 (168).  us a call, 1536 heads 128 x 64, all
// fp32, steps of M = 33 to 64 (geometric mean): KDA 20.0 at 4 with spills, 18.6 with 512
// threads, 17.7 at 3; GLA 18.3, 18.2, 17.3; RWKV6 19.8, 17.7, 16.9; at 40 heads KDA 4.9,
// 4.4, 4.5.  dl_merge of KDA 64 x 128 heads, all fp32, M = 64: 34.7 at 4 with spills, 32.5
// at 3.  Steps of 64 x 128 heads fit at 4 and are better there (KDA 15.5, at 3 15.8).
template <int OP>
constexpr int waves_target(int dk, int dv, int mode, int ce, int in_bytes, int state_bytes) {
  const bool fp32 = in_bytes == 4 && state_bytes == 4, bf16 = in_bytes == 2 && state_bytes == 2;
  if (threads_per_head(dk, dv, ce) == 512) return ce > 32 || fp32 ? 4 : bf16 ? 8 : 6;
  if (ce == 64 && dk != dv &&
      (mode == M_MERGE || (dk == 128 && fp32 && OpTraits<OP>::PER_KEY)))
    return 3;
  return 4;
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).  Map
// them so that each XCD owns whole chunks of DL_XCD_CHUNK consecutive (row, head)
// pairs: the 4-byte per-head metadata (L and the head-wise log-decay snapshots) and token
// scalars of a chunk then fill whole 128-byte lines in one L2 instead of being
// written back partially by eight different caches.  Chunks are dealt to the XCDs
// in turn, so a run of consecutive slots that merge in the same step (slots admitted
// together) is spread over all eight XCDs instead of loading one of them.  Rows past
// the last whole round of chunks keep the hardware order.
__device__ __forceinline__ uint32_t xcd_chunked(uint32_t lin, uint32_t nblk) {
  if constexpr (kXcdChunk > 0) {
    const uint32_t full = nblk - nblk % (kXcds * kXcdChunk);
    if (lin < full) {
      const uint32_t x = lin % kXcds, j = lin / kXcds;
      lin = ((j / kXcdChunk) * kXcds + x) * kXcdChunk + j % kXcdChunk;
    }
  } else if (nblk % kXcds == 0) {
    lin = (lin % kXcds) * (nblk / kXcds) + lin / kXcds;   // one contiguous range per XCD
  }
  return lin;
}

// Token row lin / H and head lin % H.  h_magic = floor((2^32 - 1) / H) gives the
// quotient or one less for any lin < 2^32.
__device__ __forceinline__ void split_row(uint32_t lin, int H, uint32_t h_magic, int& row, int& h) {
  row = int(__umulhi(lin, h_magic));
  h = int(lin) - row * H;
  if (h >= H) {
    h -= H;
    ++row;
  }
}

// ------------------------------------------------------------------ the kernel
// One workgroup per (token row, head).
//
// The leading arguments are scalars, not a struct, so that they arrive in scalar registers
// with the wave (the build asks for 14 preloaded argument words): the first loads then
// wait for no argument load.  The order of the loads is by what waits for them: the live
// length, the token's key and query (the prologue), the tile, and, once the length is
// back, the log entries; the pointers of the latter are read meanwhile.  Measured against
// a struct argument with the token rows under a branch (GDN 128 x 128, M = 16, us per
// step in a captured graph): 64 heads 4.97 -> 4.03, 256 heads 6.31 -> 5.26, 2048 heads
// 27.6 -> 25.9; RWKV6 64 x 64 with a bf16 state, 5120 heads: 15.4 -> 13.3.
template <int OP, int DK, int DV, int MODE, typename TIN, typename TS, int CE>
__global__
__launch_bounds__(threads_per_head(DK, DV, CE))
__attribute__((amdgpu_waves_per_eu(
    waves_target<OP>(DK, DV, MODE, CE, int(sizeof(TIN)), int(sizeof(TS))))))
void deltalog_kernel(const int32_t* slots, int32_t* len, void* S_, const void* k_,
                     const void* q_, int H, uint32_t h_magic, int n, int C, KParams p) {
  using CF = Cfg<OP, DK, DV, MODE, CE>;
  using TU = typename UType<OP, TIN>::type;
  constexpr int NT = CF::NT, NCG = CF::NCG, NRG = CF::NRG, RPT = CF::RPT, DL = CF::DL;
  constexpr int RPL = CF::RPL, LPE = CF::LPE, EPP = CF::EPP, NP = CF::NP, UQ = CF::UQ;
  constexpr int KTS = CF::KTS, NW = CF::NW, WK = CF::WK, WV = CF::WV;
  constexpr int EW = 64 / LPE;                    // log entries per wave and pass
  constexpr int GW = 64 / NCG;                    // row groups per wave

  __shared__ float s_kf[DK], s_qf[DK];            // k, q (coefficient-pass order)
  __shared__ float2 s_x[DK];                      // (k_r, q_r), times e^(l_r) per key
  __shared__ float s_em[DL == 1 ? 1 : DK];        // e^(l'_r)              (per-key decay)
  __shared__ float s_lr[DL], s_lm[DL];            // l, l' (coefficient-pass order; per key)
  __shared__ float s_gk[CE], s_gq[CE];            // replay coefficients
  __shared__ float s_dotw[WK];
  __shared__ __align__(16) float s_bv[DV];
  __shared__ __align__(16) float s_scr[CF::LSCR];
  __shared__ __align__(16) float s_kt[CF::MERGES_LOG ? DK * KTS : 1];   // decayed log keys
  float* const s_red = s_scr;                     // [NW][2][DV] partial sums
  float4* const s_u = reinterpret_cast<float4*>(s_scr);   // [CH][NCG] log values

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int row, h;                                     // token row and head
  split_row(xcd_chunked(blockIdx.x, uint32_t(n) * uint32_t(H)), H, h_magic, row, h);
  int slot = row;                                 // no list: the host has checked n <= B
  if (slots) {
    slot = slots[row];
    if (slot < 0 || slot >= p.B) {                // uniform per workgroup
      if (tid == 0 && p.err) atomicOr(p.err, 1);
      return;
    }
  }
  const size_t sh = size_t(slot) * H + h;         // state (slot, head) index
  const size_t th = size_t(row) * H + h;          // token (row, head) index

  // ---- 1. loads ------------------------------------------------------------------------
  int L_raw = 0;
  if constexpr (CF::HAS_LOG) L_raw = len[sh];
  // Every thread loads token elements (threads past the row repeat its last element): a
  // load under a branch is waited for at the branch's end.
  const int rl = min(tid, DK - 1), cl = min(tid, DV - 1);
  TIN k_raw = TIN(0), q_raw = TIN(0), v_raw = TIN(0);
  Raw4<TIN> v4_raw{};
  float lam = 0.f, ell = 0.f, uf = 0.f, beta = 0.f;
  if constexpr (CF::HAS_TOKEN) k_raw = (static_cast<const TIN*>(k_) + th * DK)[rl];
  q_raw = (static_cast<const TIN*>(q_) + th * DK)[rl];
  if constexpr (CF::HAS_TOKEN && CF::DECAY && DL != 1) lam = p.lam[th * DL + rl];
  // An eager step has nothing else to do before its first barrier: the bonus, which the
  // token dot product needs, goes ahead of the tile there (RWKV6 5x8 heads 128x128, bf16
  // state: 4.42 -> 4.11 us).
  if constexpr (CF::BONUS && MODE == M_EAGER) uf = p.u[size_t(h) * DK + rl];
  sched_fence();

  const int cg = tid % NCG, rg = tid / NCG;
  TS* const Sh = static_cast<TS*>(S_) + sh * size_t(DK) * DV;
  const auto srs = state_rsrc(Sh, DK * DV * sizeof(TS));
  const uint32_t toff = uint32_t(rg * DV + 4 * cg) * sizeof(TS);   // lane's byte offset in a row block
  constexpr uint32_t kRowBlock = NRG * DV * sizeof(TS);             // bytes from row j to row j+1 of a lane
  StateQuad<TS> t[RPT];
#pragma unroll
  for (int j = 0; j < RPT; ++j) t[j].load(srs, toff, j * kRowBlock);
  if constexpr (CF::HAS_TOKEN) {
    if constexpr (CF::DECAY && DL == 1) lam = scalar_ld(p.lam + th);
    if constexpr (CF::BONUS && MODE != M_EAGER) uf = p.u[size_t(h) * DK + rl];
    if constexpr (MODE == M_EAGER) v4_raw.load(static_cast<const TIN*>(p.v) + th * DV + 4 * cg);
    else v_raw = (static_cast<const TIN*>(p.v) + th * DV)[cl];
    if constexpr (CF::DELTA) beta = scalar_ld(p.beta + th);
  }
  // Per-key snapshots of a (slot, head) are contiguous rows of dk values, [B,H,C,dk].
  // Scalar snapshots are entry-major, [B,C,H]: the H heads of a slot append entry L side by
  // side (one 128-byte line for 32 heads) instead of each writing 4 bytes into a sector of
  // its own.  Entry i of a (slot, head) is at Lb[i * LS].
  const size_t LS = DL == 1 ? size_t(H) : size_t(DL);
  const TIN* Kb = nullptr;
  const TU* Ub = nullptr;
  float* Lb = nullptr;
  if constexpr (CF::HAS_LOG) {
    Kb = static_cast<const TIN*>(p.k_log) + sh * size_t(C) * DK;
    Ub = static_cast<const TU*>(p.u_log) + sh * size_t(C) * DV;
    if constexpr (CF::DECAY)
      Lb = p.lam_log + (DL == 1 ? size_t(slot) * size_t(C) * H + h : sh * size_t(C) * DL);
    // The pointers' argument loads complete beside the live length's, not after it.
    asm volatile("" ::"s"(Kb), "s"(Ub), "s"(Lb));
  }
  sched_fence();

  const int L = __builtin_amdgcn_readfirstlane(L_raw);
  if (L < 0 || L > C) {                           // every address below is in bounds
    if (tid == 0 && p.err) atomicOr(p.err, 2);
    return;
  }
  // Log entries: lanes past the live length re-read entry L-1 (unused values); waves past
  // it load nothing.
  const int e_ = tid / LPE, c_ = tid % LPE;       // coefficient pass: entry, key-row run
  const int ew = w * EW;                          // ... the wave's first entry
  RawRun<TIN, RPL> kr_raw[NP];
  RawRun<float, DL == 1 ? 4 : RPL> lr_raw[NP];    // per-key snapshots (unused for DL == 1)
  float lr0[NP] = {};                             // scalar snapshots (DL == 1)
  Raw4<TU> u_raw[UQ];
  if constexpr (CF::HAS_LOG) {
#pragma unroll
    for (int a = 0; a < NP; ++a) {
      if (ew < EPP && a * EPP + ew < L) {         // uniform per wave
        const int i = min(a * EPP + e_, L - 1);
        kr_raw[a].load(Kb + size_t(i) * DK + c_ * RPL);
        if constexpr (CF::DECAY) {
          if constexpr (DL == 1) lr0[a] = Lb[size_t(i) * LS];
          else lr_raw[a].load(Lb + size_t(i) * DK + c_ * RPL);
        }
      }
    }
#pragma unroll
    for (int a = 0; a < UQ; ++a)
      if (a * NRG + w * GW < L)                   // uniform per wave
        u_raw[a].load(Ub + size_t(min(a * NRG + rg, L - 1)) * DV + 4 * cg);
  }
  sched_fence();
  // Does this (slot, head) materialise in this launch?  (Uniform per workgroup.)
  const bool merging = MODE == M_MERGE || MODE == M_EAGER || (MODE == M_STEP && L == C);

  // ---- 2. decay factors and the token dot product -------------------------------------
  // The cumulative log-decay equals the newest snapshot (Eq. 5 writes both with the same
  // value) or 0 with an empty log.  Readouts are of the decayed state (the delta-rule
  // correction, and the post-update output's base part), except RWKV6, which reads the
  // old state; READOUT takes the represented state as it stands.
  //
  // One decay per head scales whole sums, so every wave keeps it in a register (ell through
  // the scalar path: entry L-1 is not written by this launch) and multiplies the base
  // readout by it afterwards: neither the barrier below nor the readout waits for ell,
  // which is known a memory round trip after the live length.  Per-key factors go into
  // the vectors of the readout, in LDS.
  float lm1 = 0.f, er1 = 1.f;                     // l' and e^l' (= e^l), one per head
  if constexpr (DL == 1 && CF::DECAY) {
    if constexpr (CF::HAS_LOG) {
      if (L > 0) ell = scalar_ld(Lb + size_t(L - 1) * LS);
    }
    lm1 = ell + lam;
    er1 = dl_exp(lm1);
  }
  if (w < WK) {
    const float kf = to_f32(k_raw), qf = to_f32(q_raw);
    const int pr = CF::pos(tid);
    s_kf[pr] = kf;
    s_qf[pr] = qf;
    if constexpr (DL == 1) {
      s_x[tid] = make_float2(kf, qf);
    } else {
      if constexpr (CF::HAS_LOG) {
        if (L > 0) ell = Lb[size_t(L - 1) * LS + tid];
      }
      const float lm = ell + lam, lr = CF::BONUS ? ell : lm;
      const float er = dl_exp(lr);
      s_x[tid] = make_float2(er * kf, er * qf);
      s_em[tid] = dl_exp(lm);
      s_lr[pr] = lr;
      s_lm[pr] = lm;
    }
    if constexpr (CF::HAS_TOKEN) {
      // q.k (post-update readout of the new term) or r.(u*k) (RWKV6 bonus)
      float d = CF::BONUS ? qf * uf * kf : qf * kf;
      d = xor32_sum(xor16_sum(group_sum<16>(d)));
      if ((tid & 63) == 0) s_dotw[w] = d;
    }
  }
  __syncthreads();

  // ---- 3. base readout from the registers (the log entries may still be in flight) ------
  // bf16 rows are widened again for a merge, but kept by an eager step, which holds no log
  // (RWKV6 5x8 heads 128x128: 4.66 -> 4.42 us; 128x32 heads 64x128 23.09 -> 23.01).
  float4 cv = f4(0.f), ov = f4(0.f);
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const float2 x = s_x[rg + NRG * j];
    const float4 sj = t[j].get();
    if constexpr (CF::CAN_MERGE && MODE != M_EAGER) t[j].opaque();
    if constexpr (CF::NEEDS_C) cv = fma4(x.x, sj, cv);
    ov = fma4(x.y, sj, ov);
    if (CF::LEAN && j % 2 == 1) {
      if constexpr (CF::NEEDS_C) pin(cv);
      pin(ov);
    }
  }
  if constexpr (DL == 1 && CF::DECAY) {
    if constexpr (CF::NEEDS_C) cv = er1 * cv;
    ov = er1 * ov;
  }
  if constexpr (CF::NEEDS_C) pin(cv);
  pin(ov);

  // ---- 4. replay coefficients g_i(k), g_i(q) of the live entries ---------------------
  // A merging workgroup also writes the decayed keys K~_i[r] = e^(l'_r - Lam_i,r) K_i[r]
  // of the first chunk to LDS here, from the same loads (the merge decay l' equals the readout decay, except
  // for RWKV6, which reads at ell), zeros past the live length.
  if constexpr (CF::HAS_LOG) {
#pragma unroll
    for (int a = 0; a < NP; ++a) {
      const bool stage = CF::MERGES_LOG && merging && a * EPP < CF::CH;
      if (ew < EPP && (a * EPP + ew < L || stage)) {          // uniform per wave
        const int i = a * EPP + e_;
        const bool live = i < L;
        float ak = 0.f, aq = 0.f, wt = 1.f;
        if constexpr (DL == 1 && CF::DECAY) wt = live ? dl_exp(lm1 - lr0[a]) : 0.f;
#pragma unroll
        for (int x = 0; x < RPL; ++x) {
          const int pr = x * LPE + c_;
          float kx = kr_raw[a].at(x);
          if constexpr (DL != 1) kx *= dl_exp(s_lr[pr] - lr_raw[a].at(x));
          if constexpr (CF::NEEDS_C) ak = fmaf(kx, s_kf[pr], ak);
          aq = fmaf(kx, s_qf[pr], aq);
          if (DL != 1 && !CF::BONUS && stage) s_kt[pr * KTS + i] = live ? kx : 0.f;
          if (CF::LEAN && x % 2 == 1) {
            pin(ak);
            pin(aq);
          }
        }
        if constexpr (DL == 1 && CF::DECAY) {
          if constexpr (CF::NEEDS_C) ak *= wt;
          aq *= wt;
        }
        if ((DL == 1 || CF::BONUS) && stage) {
#pragma unroll
          for (int x = 0; x < RPL; ++x) {
            const int pr = x * LPE + c_;
            float kx = kr_raw[a].at(x);
            if constexpr (DL != 1) kx *= dl_exp(s_lm[pr] - lr_raw[a].at(x));
            else kx *= wt;
            s_kt[pr * KTS + i] = live ? kx : 0.f;
            if (CF::LEAN && x % 4 == 3) sched_fence();
          }
        }
        if constexpr (CF::NEEDS_C) ak = group_sum<LPE>(ak);   // the delta-rule correction only
        aq = group_sum<LPE>(aq);
        if (c_ == 0 && live) {
          if constexpr (CF::NEEDS_C) s_gk[i] = ak;
          s_gq[i] = aq;
        }
      }
    }
    __syncthreads();

    // ---- 5. log replay: each log value row is read by one row group --------------------
#pragma unroll
    for (int a = 0; a < UQ; ++a) {
      if (a * NRG + w * GW < L) {                 // uniform per wave
        const int i = a * NRG + rg, ic = min(i, L - 1);
        const float4 u = u_raw[a].get();
        const float gk = CF::NEEDS_C ? s_gk[ic] : 0.f, gq = s_gq[ic];
        if (i < L) {                              // lanes past the log add nothing: entry L-1
          if constexpr (CF::NEEDS_C) cv = fma4(gk, u, cv);   // may hold an infinity
          ov = fma4(gq, u, ov);
        }
      }
    }
  }

  float4 bv = f4(0.f);
  // ---- 6. sums over rows, update factors, output, append -----------------------------
  // Rows of one column group live in lanes NCG apart inside a wave, then across waves.
  // The sums of a column group's lanes are left one part per lane (see swap32_sum), and
  // each lane stores its part: c in lanes 0-31 and o in lanes 32-63, or halves of o.
  const int lane = tid & 63, hi = lane >> 5, odd = (lane >> 4) & 1;
  if constexpr (CF::NEEDS_C) {
    const float4 v = make_float4(swap32_sum(cv.x, ov.x), swap32_sum(cv.y, ov.y),
                                 swap32_sum(cv.z, ov.z), swap32_sum(cv.w, ov.w));
    float* const d = &s_red[(w * 2 + hi) * DV + 4 * cg];
    if constexpr (NCG == 32) st4(d, v);
    else *reinterpret_cast<float2*>(d + 2 * odd) =
        make_float2(swap16_sum(v.x, v.z), swap16_sum(v.y, v.w));
  } else {
    const float2 v = make_float2(swap32_sum(ov.x, ov.z), swap32_sum(ov.y, ov.w));
    float* const d = &s_red[(w * 2 + 1) * DV + 4 * cg + 2 * hi];
    if constexpr (NCG == 32) *reinterpret_cast<float2*>(d) = v;
    else d[odd] = swap16_sum(v.x, v.y);
  }
  __syncthreads();
  float dot = 0.f;
  if constexpr (CF::HAS_TOKEN) {
#pragma unroll
    for (int x = 0; x < WK; ++x) dot += s_dotw[x];
  }
  if constexpr (MODE == M_EAGER) {
    // Every workgroup goes on to its update: each thread sums its own quad (in the same
    // order), which saves a barrier and a trip through LDS.
    const float4* const q = reinterpret_cast<const float4*>(s_red) + cg;
    if constexpr (CF::NEEDS_C) cv = pair_sum<NW>([&](int x) { return q[x * 2 * NCG]; });
    ov = pair_sum<NW>([&](int x) { return q[(x * 2 + 1) * NCG]; });
    const float4 v = v4_raw.get();
    bv = CF::DELTA ? beta * (v - cv) : v;
    if (rg == 0) st4(p.o + th * DV + 4 * cg, fma4(dot, bv, ov));
  } else if (w < WV) {
    // One thread per value column (every thread summing its whole quad would read NRG
    // times as much LDS as there are partial sums).
    float c = 0.f, b = 0.f;
    if constexpr (CF::NEEDS_C) c = pair_sum<NW>([&](int x) { return s_red[x * 2 * DV + tid]; });
    float o = pair_sum<NW>([&](int x) { return s_red[(x * 2 + 1) * DV + tid]; });
    if constexpr (CF::HAS_TOKEN) {
      const float v = to_f32(v_raw);
      b = CF::DELTA ? beta * (v - c) : v;
      o = fmaf(dot, b, o);                      // post-update readout, or the RWKV6 bonus
    }
    p.o[th * DV + tid] = o;
    if constexpr (MODE == M_STEP) {
      if (L < C) {                              // Eq. 5
        TU* Ud = static_cast<TU*>(p.u_log) + (sh * size_t(C) + L) * DV;
        if constexpr (CF::DELTA) reinterpret_cast<float*>(Ud)[tid] = b;
        else Ud[tid] = v_raw;                   // bit-exact copy
      }
    }
    if constexpr (CF::CAN_MERGE) s_bv[tid] = b;
  }
  if constexpr (MODE == M_READOUT) return;
  if constexpr (MODE == M_STEP) {
    if (L < C) {
      if (w < WK) {
        static_cast<TIN*>(p.k_log)[(sh * size_t(C) + L) * DK + tid] = k_raw;
        if constexpr (CF::DECAY) {
          if constexpr (DL != 1) Lb[size_t(L) * LS + tid] = s_lm[CF::pos(tid)];
          else if (tid == 0) Lb[size_t(L) * LS] = lm1;
        }
        if (tid == 0) len[sh] = L + 1;
      }
      return;
    }
  }

  // ---- 7. materialise (Eq. 6 / Eq. 7 / Eq. 3) ------------------------------------------
  if constexpr (CF::CAN_MERGE) {
    constexpr bool kBvLds = CF::HAS_TOKEN && MODE != M_EAGER;
    if constexpr (kBvLds) __syncthreads();        // s_bv written, the partial sums read
    if constexpr (kBvLds) bv = *reinterpret_cast<const float4*>(&s_bv[4 * cg]);
    // Stage chunk c0 of the log: values from the replay's registers, keys (the first
    // chunk's are there already) from memory.  Zeros past the live length.
    [[maybe_unused]] auto stage_chunk = [&](int c0) {
      if (c0 > 0) {
#pragma unroll
        for (int a = 0; a < CF::CH / EPP; ++a) {
          if (ew < EPP) {
            const int e = a * EPP + e_, i = c0 + e, ic = min(i, L - 1);
            RawRun<TIN, RPL> kg;
            RawRun<float, DL == 1 ? 4 : RPL> lg;
            kg.load(Kb + size_t(ic) * DK + c_ * RPL);
            float wt = 1.f;
            if constexpr (DL != 1) lg.load(Lb + size_t(ic) * DK + c_ * RPL);
            else if constexpr (CF::DECAY) wt = dl_exp(lm1 - Lb[size_t(ic) * LS]);
#pragma unroll
            for (int x = 0; x < RPL; ++x) {
              const int pr = x * LPE + c_;
              if constexpr (DL != 1) wt = dl_exp(s_lm[pr] - lg.at(x));
              s_kt[pr * KTS + e] = i < L ? wt * kg.at(x) : 0.f;
            }
          }
        }
      }
#pragma unroll
      for (int a = 0; a < UQ; ++a) {
        const int i = a * NRG + rg, e = i - c0;
        if (e >= 0 && e < CF::CH) s_u[e * NCG + cg] = i < L ? u_raw[a].get() : f4(0.f);
      }
      __syncthreads();
    };
    if constexpr (CF::MERGES_LOG) {
      if (L > 0) stage_chunk(0);                  // uniform
    }
    // The live length is written before the rows, so that no register is written behind
    // the state stores.
    if constexpr (CF::HAS_LOG) {
      if (tid == 0) len[sh] = 0;                  // the cumulative log-decay restarts at 0
    }
    // Row blocks of four: an eager step stores each block as soon as it is formed (GDN
    // 128x32 heads 95.7 -> 91.8 us against two blocks at a time).  A merge forms two at a
    // time; all four together read each staged log value from LDS once instead of twice,
    // but their registers cost every append more (GLA 100x32 heads, bf16 state, one cycle
    // of M = 16: 411 us with two, 414 with four; 8 layers of 8 staggered GDN slots: 59.6
    // and 61.7).  The rank-L contraction runs on v_mfma_f32_4x4x1f32
    // (fp32 products and sums, twice the rate of plain FMAs) with the block's rows as the
    // accumulator: of its 16 independent 4 x 4 products, block l / 4 is that of lanes
    // 4 b .. 4 b + 3; lane l holds output column l % 4 of its block and all four rows,
    // i.e. with rows j = 0 .. 3 of the lane's own row group and component c of its own
    // column quad as the column, accumulator c is component c of the lane's four quads.
    // The B operand (U) is the lane's own quad; the A operand (K~) is the lane's row
    // cg % 4, the same for the NCG / 4 blocks of a row group, so each of those blocks
    // reads another entry and the instruction broadcasts one block's (cbsz, abid).
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    static_assert(CE <= 2 * CF::CH, "at most two chunks");
    constexpr int NRB = RPT / 4, RBG = MODE == M_EAGER ? 1 : NRB < 2 ? NRB : 2, NR = 4 * RBG;
#pragma unroll
    for (int g = 0; g < NRB; g += RBG) {
      float4 m[NR];
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const int r = rg + NRG * (4 * g + j);
        const float em = DL == 1 ? er1 : s_em[DL == 1 ? 0 : r];
        m[j] = em * t[4 * g + j].get();
        if constexpr (CF::HAS_TOKEN) m[j] = fma4(s_kf[CF::pos(r)], bv, m[j]);
      }
      if constexpr (CF::MERGES_LOG) {
        f32x4 acc[RBG][4];
        int a_off[RBG];
#pragma unroll
        for (int rb = 0; rb < RBG; ++rb) {
          a_off[rb] = CF::pos(rg + NRG * (4 * (g + rb) + (cg & 3))) * KTS + (cg >> 2);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float4 r = m[4 * rb + i];
            acc[rb][0][i] = r.x; acc[rb][1][i] = r.y; acc[rb][2][i] = r.z; acc[rb][3][i] = r.w;
          }
        }
        static_assert(CE == CF::CH || RBG == NRB, "chunks are staged once");
        constexpr int EB = NCG / 4;               // entries per read of the A operand
        constexpr int CB = EB == 8 ? 3 : 2;       // cbsz: log2 of the blocks per broadcast
        for (int i0 = 0; i0 < L; i0 += EB) {      // zeros past the live length
          if (CE > CF::CH && i0 == CF::CH) {      // the second chunk (one row group only)
            __syncthreads();                      // the first is consumed
            stage_chunk(i0);
          }
          const int e0 = CE > CF::CH && i0 >= CF::CH ? i0 - CF::CH : i0;
          float a[RBG];
#pragma unroll
          for (int rb = 0; rb < RBG; ++rb) a[rb] = s_kt[a_off[rb] + e0];
#define DL_MERGE_ENTRY(e)                                                                   \
  {                                                                                         \
    const float4 b = s_u[(e0 + e) * NCG + cg];                                              \
    _Pragma("unroll") for (int rb = 0; rb < RBG; ++rb) {                                    \
      acc[rb][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.x, acc[rb][0], CB, e, 0);    \
      acc[rb][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.y, acc[rb][1], CB, e, 0);    \
      acc[rb][2] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.z, acc[rb][2], CB, e, 0);    \
      acc[rb][3] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[rb], b.w, acc[rb][3], CB, e, 0);    \
    }                                                                                       \
  }
          DL_MERGE_ENTRY(0) DL_MERGE_ENTRY(1) DL_MERGE_ENTRY(2) DL_MERGE_ENTRY(3)
          if constexpr (EB == 8) {
            if (CF::LEAN) sched_fence();
            DL_MERGE_ENTRY(4) DL_MERGE_ENTRY(5) DL_MERGE_ENTRY(6) DL_MERGE_ENTRY(7)
          }
          if (CF::LEAN) sched_fence();
#undef DL_MERGE_ENTRY
        }
#pragma unroll
        for (int rb = 0; rb < RBG; ++rb) {
          // Wait states between the last MFMA and the first VALU read of its results, on
          // top of those the compiler inserts.
          asm volatile("s_nop 7\n\ts_nop 7"
                       : "+v"(acc[rb][0]), "+v"(acc[rb][1]), "+v"(acc[rb][2]), "+v"(acc[rb][3]));
#pragma unroll
          for (int i = 0; i < 4; ++i)
            m[4 * rb + i] = make_float4(acc[rb][0][i], acc[rb][1][i], acc[rb][2][i], acc[rb][3][i]);
        }
      }
      if constexpr (sizeof(TS) == 4) {
        // Every row is gathered into registers of its own and all of them stay allocated
        // until the last store has issued, with wait states before they are reused:
        // gathered into one reused set of four registers, each row's registers were
        // rewritten right behind its store, and on the GPU that store then wrote the next
        // row's value in lanes 12-15 of each 16-lane row now and then.
        u32x4 x[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) {
          x[j] = u32x4{__float_as_uint(m[j].x), __float_as_uint(m[j].y),
                       __float_as_uint(m[j].z), __float_as_uint(m[j].w)};
          asm volatile("" : "+v"(x[j]));
        }
#pragma unroll
        for (int j = 0; j < NR; ++j)
          __builtin_amdgcn_raw_buffer_store_b128(x[j], srs, toff, (4 * g + j) * kRowBlock,
                                                 kStateStorePolicy);
#pragma unroll
        for (int j = 0; j < NR; ++j) asm volatile("s_nop 0" ::"v"(x[j]));
      } else {
#pragma unroll
        for (int j = 0; j < NR; ++j)
          StateQuad<TS>::store(srs, toff, (4 * g + j) * kRowBlock, m[j]);
      }
    }
  }
}

}  // namespace dl
