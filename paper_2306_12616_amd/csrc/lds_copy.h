// Memory to LDS without passing registers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace chebdm {

// 1 KB: 16 bytes a lane from base + voff into LDS at lds + 16 lane (lds: the wavefront's byte offset).  Counted
// by vmcnt.
__device__ __forceinline__ void copy_1k(uint32_t lds, uint32_t voff, const void* base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
                 : "memory", "m0");
}

}  // namespace chebdm
