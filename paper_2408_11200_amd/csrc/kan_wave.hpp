// Cross-lane sums of the walk kernels, and the order of a wave's own LDS accesses.
#pragma once
#include "kan_device.hpp"

namespace KAN_NS {

typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Buffer loads by the compiler's intrinsics (hipcc 7.2 builds __builtin_amdgcn_raw_buffer_load_b64 as a load of 32 bits).
__device__ f32x4 buffer_load4(i32x4 rsrc, int off, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.load.v4f32");
__device__ f32x2 buffer_load2(i32x4 rsrc, int off, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.load.v2f32");
__device__ float buffer_load1(i32x4 rsrc, int off, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.load.f32");

// a buffer of `bytes` bytes at the wave-uniform address p: loads past its end return zeros
__device__ __forceinline__ i32x4 buffer_of(const float *p, unsigned bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return i32x4{(int)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), (int)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)),
                 (int)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
}

// value of the partner lane for the level that pairs lanes differing in bit D (for D = 4 the partner
// is lane ^ 7: it differs in bit 2, which is all the reduction below needs)
template <int D>
__device__ __forceinline__ float partner(float v)
{
    const int iv = __builtin_bit_cast(int, v);
    if constexpr (D >= 16) return __shfl_xor(v, D, 64);
    else if constexpr (D == 8) return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x128, 0xF, 0xF, true));
    else if constexpr (D == 4) return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x141, 0xF, 0xF, true));
    else if constexpr (D == 2) return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x4E, 0xF, 0xF, true));
    else return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0xB1, 0xF, 0xF, true));
}

// p[0..N) hold, per lane, partial sums of N quantities.  Sums them over groups of LPS lanes while
// halving the number of quantities a lane carries at each level (lanes whose bit D is set keep the
// upper half); once one is left the remaining levels are plain sums.  Returns the total of quantity
// number quantity_of<LPS>(lane).
template <int D, int N>
__device__ __forceinline__ float reduce_levels(float (&p)[N], int lane)
{
    if constexpr (N > 1 && D >= 16) {
        // lanes of the lower and upper half (of 32, or 16 of each 32) trade a quantity each
        float h[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const auto t = D == 32 ? __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, p[k]), __builtin_bit_cast(int, p[k + N / 2]), false, false)
                                   : __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, p[k]), __builtin_bit_cast(int, p[k + N / 2]), false, false);
            h[k] = __builtin_bit_cast(float, (int)t[0]) + __builtin_bit_cast(float, (int)t[1]);
        }
        return reduce_levels<D / 2, N / 2>(h, lane);
    } else if constexpr (N > 1) {
        const bool up = (lane & D) != 0;
        float h[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const float keep = up ? p[k + N / 2] : p[k];
            const float send = up ? p[k] : p[k + N / 2];
            h[k] = keep + partner<D>(send);
        }
        if constexpr (D > 1) return reduce_levels<D / 2, N / 2>(h, lane);
        else return h[0];
    } else {
        float v = p[0] + partner<D>(p[0]);
        if constexpr (D > 1) {
            float one[1] = {v};
            return reduce_levels<D / 2, 1>(one, lane);
        } else {
            return v;
        }
    }
}
// What lanes of this wave wrote to LDS before is read by lanes of this wave after it (a wave's LDS operations run in order;
// this keeps the compiler to that order).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace KAN_NS
