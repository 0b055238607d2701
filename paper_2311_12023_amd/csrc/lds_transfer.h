// Transfers from global memory straight into LDS.
#pragma once
#include <hip/hip_runtime.h>

namespace lq {

// Every lane moves 16 bytes from base + voff to LDS address lds + 16 * lane.  Counts in vmcnt; the caller waits before a
// barrier.  In inline assembly because the compiler, given the builtin, waits for all transfers before each LDS read.
// M0 (the LDS address) takes one wait state to reach the transfer, which the hardware does not insert and the compiler not
// inside an asm statement: hence the s_nop.
__device__ __forceinline__ void transfer_to_lds(const uint16_t* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}

}  // namespace lq
