// Coherent-at-device-scope accesses for partial results that one workgroup writes and another reads
// inside the same kernel (last-arriver reductions).  They bypass the per-XCD L2's non-coherent lines
// one access at a time, so no whole-cache write-back or invalidate is needed.  A region is addressed
// through a buffer descriptor (wavefront-uniform base) and a byte offset or the index of a 16-byte quad.
// Also the descriptor form for plain loads that several kernels share (Stretch, below).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace w4 {

typedef __amdgpu_buffer_rsrc_t PartialBuffer;
constexpr int kDeviceScope = 16;   // cache-policy bit sc1

__device__ __forceinline__ PartialBuffer partial_buffer(const float *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0x7FFFFFFF, 0x00020000);
}
__device__ __forceinline__ void store_partial(PartialBuffer b, int quad, float __attribute__((ext_vector_type(4))) v)
{
    typedef uint32_t u32x4_ __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_, v), b, quad * 16, 0, kDeviceScope);
}
__device__ __forceinline__ float __attribute__((ext_vector_type(4))) load_partial(PartialBuffer b, int quad)
{
    typedef float float4v_ __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(float4v_, __builtin_amdgcn_raw_buffer_load_b128(b, quad * 16, 0, kDeviceScope));
}
__device__ __forceinline__ void store_partial_f32(PartialBuffer b, int index, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), b, index * 4, 0, kDeviceScope);
}
__device__ __forceinline__ float load_partial_f32(PartialBuffer b, int index)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, index * 4, 0, kDeviceScope));
}


// A wavefront-uniform stretch of memory behind a buffer descriptor: loads address it with a 32-bit lane offset plus a
// scalar offset, so a moving base costs scalar arithmetic only and no 64-bit lane address occupies registers.
typedef __amdgpu_buffer_rsrc_t Stretch;
constexpr int kStreamed = 2;   // cache policy nt: read once
__device__ __forceinline__ Stretch stretch(const void *base, uint32_t bytes)
{
    const uint64_t v = reinterpret_cast<uint64_t>(base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((uint64_t)hi << 32) | lo), 0, (int)bytes, 0x00020000);
}
// 16 bytes per lane at lane offset + scalar offset; and the same straight into LDS, lane l's at lds + 16 l (lds
// wavefront-uniform; counted by vmcnt, and nothing but an explicit wait and a barrier orders it with reads of other wavefronts)
__device__ __forceinline__ uint32_t __attribute__((ext_vector_type(4))) stream_quad(Stretch s, uint32_t lane_offset, uint32_t offset)
{
    return __builtin_amdgcn_raw_buffer_load_b128(s, lane_offset, offset, kStreamed);
}
__device__ __forceinline__ void quad_to_lds(Stretch s, void *lds, uint32_t lane_offset, uint32_t offset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(s, (__attribute__((address_space(3))) void *)lds, 16, lane_offset, offset, 0, 0);
}

}  // namespace w4
