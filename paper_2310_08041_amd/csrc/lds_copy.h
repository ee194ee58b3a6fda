// Internal to libqllm: a wavefront's copy from global memory into LDS.
#ifndef QLLM_LDS_COPY_H
#define QLLM_LDS_COPY_H

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace qllm_detail {

// 1 KB: lane l's 16 bytes at base + uniform_off + lane_off land at lds + 16 l.  base, bytes, uniform_off and lds are the
// wavefront's.  A lane whose place lies past base + bytes brings zeros.  Counted by vmcnt, in order.
__device__ __forceinline__ void copy_1k_to_lds(const uint8_t *base, uint32_t bytes, uint32_t lane_off, uint32_t uniform_off, uint8_t *lds)
{
#if defined(__HIP_DEVICE_COMPILE__) // the host pass has no such type and would drop the body of every kernel that names it
    const __amdgpu_buffer_rsrc_t memory = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(memory, (__attribute__((address_space(3))) void *)lds, 16, lane_off, uniform_off, 0, 0);
#else
    (void)base, (void)bytes, (void)lane_off, (void)uniform_off, (void)lds;
#endif
}

} // namespace qllm_detail

#endif
