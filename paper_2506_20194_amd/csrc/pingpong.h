// The main loop of the bf16 MFMA products (duo_linear, stage 1's Gram kernel):
// 512 threads, operands streamed global -> LDS directly, the two waves of every
// SIMD taking turns at the LDS and the matrix core.
//
// Each operand of the tile is split in two halves per wave (A0 / A1, B0 / B1); a
// unit of LDS is one half of one operand for all waves of one 64-deep stage, and
// two stages are resident.  A stage is four phases,
//   A0 B0, A0 B1, A1 B1, A1 B0,
// and each phase has a memory part (the fragment reads of its MFMAs, and the
// load of one unit that died two phases ago, for the stage after next) and a
// matrix part, with a barrier after each.  Waves 4-7 run one barrier behind waves
// 0-3, so that one wave of a SIMD is in its matrix part (with raised wave
// priority) while the other is in its memory part.
//
// Waits.  A unit first read in phase p is issued in the memory part of phase
// p - 6, and every wave waits for its own part of it at the end of the memory
// part of phase p - 1, before a barrier that all waves pass before any of them
// enters phase p: at most the five units issued since may then be in flight.
// Overwriting: a unit is overwritten (its successor issued) two phases after the
// one that last reads it, and by then every wave's reads of it have returned:
// waves 4-7 pass the barrier that lets waves 0-3 into phase p + 2 at the end of
// their memory part of phase p + 1.  The fragments that are used in the phase that
// reads them have been waited for by then.  B0 is read a phase before its first
// use (in phase 3 of the stage before), so phase 0's memory part waits for it.
#pragma once

#include "common.h"

namespace duo {
namespace pp {

// v_mfma_f32_16x16x32_bf16: lane l holds row l % 16 of A and column l % 16 of B,
// each as the 8 consecutive k of group l / 16; the accumulator's element r sits
// at row 4 (l / 16) + r, column l % 16
__device__ __forceinline__ f4 mma_bf16(const u32x4& a, const u32x4& b, f4 c) {
  bf16x8 av, bv;
  __builtin_memcpy(&av, &a, 16);
  __builtin_memcpy(&bv, &b, 16);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
}

// Workgroup barrier without the memory fence of __syncthreads, whose fence
// would wait for the global prefetches in flight; this wave's LDS traffic is
// drained first.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Wait until at most N of this wave's vector memory operations (the direct
// global -> LDS loads) are in flight; expcnt and lgkmcnt are not waited for.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Wait until at most N of this wave's LDS reads are in flight (they return in
// order).  No LDS read moves across it.
template <int N>
__device__ __forceinline__ void wait_lds() {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (N << 8));
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// Barrier between the parts of a phase: nothing moves across it, and nothing
// is waited for (the waits that matter stand before it or come with the uses).
__device__ __forceinline__ void phase_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// acc[HA hA + a][2 hB + b] += the products of nst >= 1 stages.  HA: 16-row blocks
// of an A half (a B half has two); LA, LB: loads per wave and unit of A, B.
//   issue(op, stage, parity)  the unit's loads (op 0..3: A0, A1, B0, B1); called for
//                             stages up to nst + 1: it clamps them (those units
//                             are not read)
//   read_a(parity, half, F), read_b(parity, half, F)  this wave's fragments,
//                             F[k-step][block]
// On return no load is in flight and the accumulators may be read; the waves
// are not synchronised.
template <int HA, int LA, int LB, class Issue, class ReadA, class ReadB>
__device__ __forceinline__ void pp_loop(int nst, f4 (&acc)[2 * HA][4], const Issue& issue, const ReadA& read_a,
                                        const ReadB& read_b) {
  const bool late = threadIdx.x >> 8;  // waves 4-7
  // end of the memory part of a phase; A and B units alternate (phases 0 and 2
  // issue an A one)
  auto mem_end = [&](int phase) {
    if (phase & 1)
      wait_vm<3 * LB + 2 * LA>();
    else
      wait_vm<3 * LA + 2 * LB>();
    phase_barrier();
  };
  auto mma = [&](int ha, int hb, const u32x4 (&Fa)[2][HA], const u32x4 (&Fb)[2][2]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int a = 0; a < HA; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[HA * ha + a][2 * hb + b] = mma_bf16(Fa[s2][a], Fb[s2][b], acc[HA * ha + a][2 * hb + b]);
    __builtin_amdgcn_s_setprio(0);
    phase_barrier();
  };
  issue(2, 0, 0);
  issue(0, 0, 0);
  issue(3, 0, 0);
  issue(1, 0, 0);
  issue(2, 1, 1);
  issue(0, 1, 1);
  issue(3, 1, 1);
  u32x4 fa[2][HA], fb1[2][2], xa[2][2], xb[2][2];
  mem_end(3);  // B0 and A0 of stage 0
  read_b(0, 0, xa);
  if (late) phase_barrier();
  // x0: B0 of stage t; nx takes B0 of stage t + 1
  auto stage = [&](int t, int par, const u32x4 (&x0)[2][2], u32x4 (&nx)[2][2]) {
    read_a(par, 0, fa);
    issue(1, t + 1, par ^ 1);
    wait_lds<2 * HA>();  // all but read_a's: B0 of this stage, whose successor the next phase issues
    mem_end(0);
    mma(0, 0, fa, x0);
    read_b(par, 1, fb1);
    issue(2, t + 2, par);
    mem_end(1);
    mma(0, 1, fa, fb1);
    read_a(par, 1, fa);
    issue(0, t + 2, par);
    mem_end(2);
    mma(1, 1, fa, fb1);
    read_b(par ^ 1, 0, nx);
    issue(3, t + 2, par);
    mem_end(3);
    mma(1, 0, fa, x0);
  };
  int t = 0;
  for (; t + 1 < nst; t += 2) {  // two stages per trip: static slots, and no copies of B0
    stage(t, 0, xa, xb);
    stage(t + 1, 1, xb, xa);
  }
  if (t < nst) stage(t, 0, xa, xb);
  if (!late) phase_barrier();
#pragma unroll
  for (int a = 0; a < 2 * HA; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) asm volatile("s_nop 1" : "+v"(acc[a][b]));  // the last products have been written
  wait_vm<0>();
}

}  // namespace pp
}  // namespace duo
