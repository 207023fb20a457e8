// Raw buffer access and scalar values, for kernels whose base addresses are
// the same in all lanes.
#pragma once
#include <hip/hip_runtime.h>

namespace fsic {

// Raw buffer access: a uniform resource (base, size) plus a 32-bit vector
// byte offset and a 32-bit scalar byte offset, so no per-lane 64-bit address
// arithmetic is needed.
// An index that is in range has to be so by construction; kDrop is not.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc make_rsrc(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}
template <class X> __device__ __forceinline__ X bld(Rsrc r, unsigned vidx, int sidx);
template <> __device__ __forceinline__ float bld<float>(Rsrc r, unsigned vidx, int sidx) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vidx * 4u, sidx * 4, 0));
}
template <> __device__ __forceinline__ double bld<double>(Rsrc r, unsigned vidx, int sidx) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vidx * 8u, sidx * 8, 0));
}
__device__ __forceinline__ void bst(Rsrc r, unsigned vidx, int sidx, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, vidx * 4u, sidx * 4, 0);
}
__device__ __forceinline__ void bst(Rsrc r, unsigned vidx, int sidx, double v) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, vidx * 8u, sidx * 8, 0);
}

// values that are the same in every lane, for scalar registers (the compiler
// cannot know that of loads beside stores, and a buffer resource in vector
// registers makes a loop of every access)
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni(long long v) {
    return (long long)((unsigned long long)(unsigned)uni((int)(v >> 32)) << 32 | (unsigned)uni((int)v));
}

// element index of a store that is to be dropped: beyond every buffer.  Stores
// are issued in any case, so that the number of stores behind a prefetch is
// known and waiting for the one does not wait for the others
constexpr unsigned kDrop = 0x1fffffffu;

}  // namespace fsic
