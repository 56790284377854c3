// Asynchronous copies from memory straight into LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cnnsns {

// 16 bytes a lane from `from` (each lane its own address) to `to` + 16 lane; `to` is the same for the whole
// wavefront.  The caller waits with lds_copies_arrived() before the barrier after which the data is read.
//
// Not the builtin: with that, the compiler waits for every copy in flight before the wavefront's next LDS read,
// because it cannot tell the buffer being filled from the one being read, and a double-buffered copy hides nothing
// (an FP32 pass on 1531 x 1531 cells: 495 us with the builtin, 479 with this; at 4096 x 4096 2720
// and 2640; the classifier's wide layers for 300 particles: 58 and 46).  Nothing is loaded into registers, and the
// compiler's own waits count loads in order, so a copy it does not know of can only make them longer.  The place in LDS
// goes through M0: an operand, since the compiler allows no asm statement to overwrite that register.  It is read
// one wait state after it is written at the earliest.
__device__ __forceinline__ void lds_copy16(const void* from, void* to)
{
    const uint32_t at = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)to);
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "{m0}"(at), "v"(from) : "memory");
}

// Waits for every copy (and every other memory operation) of the wavefront.
__device__ __forceinline__ void lds_copies_arrived()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace cnnsns
