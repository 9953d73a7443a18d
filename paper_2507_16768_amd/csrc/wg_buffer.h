// Memory that is reached through a buffer descriptor (gfx950): by 16 bytes or a word at an offset from its beginning.  What lies
// behind its end reads as zero and is not written, so that a lane without anything to do needs no branch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wg {

typedef __amdgpu_buffer_rsrc_t Window;
typedef uint32_t FourWords __attribute__((ext_vector_type(4)));
constexpr uint32_t kNowhere = 0xFFFFFFF0u;           // an offset behind every window

// How the caches take an access: kStream, they need not keep it.
constexpr int kKeep = 0, kStream = 2;

// (p and bytes are the same for all lanes)
__device__ __forceinline__ Window window_of(const void *p, uint32_t bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000); }
template <int kPolicy = kKeep>
__device__ __forceinline__ uint4 block_at(Window w, uint32_t at)
{
    const FourWords x = __builtin_amdgcn_raw_buffer_load_b128(w, at, 0, kPolicy);
    return uint4{x.x, x.y, x.z, x.w};
}
__device__ __forceinline__ uint32_t word_at(Window w, uint32_t at) { return __builtin_amdgcn_raw_buffer_load_b32(w, at, 0, 0); }
template <int kPolicy = kKeep>
__device__ __forceinline__ void put_block(Window w, uint32_t at, const uint4 &v) { __builtin_amdgcn_raw_buffer_store_b128(FourWords{v.x, v.y, v.z, v.w}, w, at, 0, kPolicy); }

}  // namespace wg
