// Populations through a buffer descriptor (buffers below 4 GiB).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

// Populations of one run through a buffer descriptor: a 32-bit byte offset per
// lane plus a scalar one per direction, so that a load or store takes no
// address arithmetic in vector registers (the block is below 4 GiB).
template <typename S> struct PopBuf {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ explicit PopBuf(const S *base)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<S *>(base), 0, -1, 0x00020000))
    {
    }
    // `uni` is the same in every lane of the wave; read as a scalar, because a
    // uniform value that the compiler keeps in a vector register makes every
    // access a loop over the lanes' values
    __device__ __forceinline__ S load(uint32_t lane, uint32_t uni) const
    {
        uni = __builtin_amdgcn_readfirstlane(uni);
        if constexpr (sizeof(S) == 2)
            return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)lane, (int)uni, 0));
        else if constexpr (sizeof(S) == 4)
            return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)lane, (int)uni, 0));
        else
            return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)lane, (int)uni, 0));
    }
    // NT: non-temporal, for states that outgrow the cache they would be read from next
    template <bool NT = false> __device__ __forceinline__ void store(uint32_t lane, uint32_t uni, S v) const
    {
        constexpr int kAux = NT ? 2 : 0;
        uni = __builtin_amdgcn_readfirstlane(uni);
        if constexpr (sizeof(S) == 2)
            __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), rsrc, (int)lane, (int)uni, kAux);
        else if constexpr (sizeof(S) == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), rsrc, (int)lane, (int)uni, kAux);
        else {
            typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rsrc, (int)lane, (int)uni, kAux);
        }
    }
};

} // namespace lbm
