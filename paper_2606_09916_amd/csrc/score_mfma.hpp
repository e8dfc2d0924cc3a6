// What the matrix-core score passes share: types, direct global->LDS loads and the waits
// on them.
#pragma once

#include "ikv_internal.hpp"

namespace ikv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int MD = 128;          // head dimension of this path
constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// 16 bytes per lane from global memory straight into LDS at lds_base + 16 * lane.
// Issued from asm so that the compiler does not serialise LDS reads behind every
// outstanding load; the waits on these loads are placed by hand.
__device__ __forceinline__ void dma16(const void *g, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds_base), "v"(g)
               : "memory", "m0");
}
// The same with the non-temporal hint, for the key streams: a key row is read once
// per pass, and kept in L2 it would push out what the workgroups read again (the
// memory rows, which every workgroup of a head pair or unit reloads). Measured at
// Qwen3-8B 32k: first pass 443 -> 412 us, second pass 486 -> 435 us.
__device__ __forceinline__ void dma16_nt(const void *g, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt"
               :
               : "s"(lds_base), "v"(g)
               : "memory", "m0");
}

template <int N>
__device__ __forceinline__ void vm_wait_c() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// s_waitcnt vmcnt(n) for a wave-uniform n: exact for even n up to 12, otherwise a longer
// wait. Few cases, since the compares are part of a loop's serial chain (with 30 the first
// pass at 128 rows took 7% longer).
__device__ __forceinline__ void vm_wait(int n) {
  switch (n) {
    case 2: vm_wait_c<2>(); break;
    case 4: vm_wait_c<4>(); break;
    case 6: vm_wait_c<6>(); break;
    case 8: vm_wait_c<8>(); break;
    case 10: vm_wait_c<10>(); break;
    case 12: vm_wait_c<12>(); break;
    default: vm_wait_c<0>(); break;
  }
}

// ---- the position-major passes in narrow tiles (k_score_narrow.hip)
// Groups of 32 list entries per tile (1 or 2), 0 where the 128-entry passes run.
int narrow_tiles(const ScoreArgs &a);
// The second pass of the two-pass form, or with a.stash the one key pass.
hipError_t launch_score_narrow(const ScoreArgs &a, int lch, int ng, hipStream_t st);

}  // namespace ikv
