// Bit matrices in registers and ORs over a wave, for the kernels that hold the
// same component of many samples in one word (k_sparse.hip, k_eval.hip).
#pragma once

#include <type_traits>

#include "rsr_internal.h"

namespace rsr {
namespace bits {

// One step of the transpose: swaps the upper J-bit halves of the words k with
// the lower ones of the words k + J (k without bit J).
template <int J>
__device__ __forceinline__ void transpose_step(uint32_t (&a)[32]) {
    constexpr uint32_t m = J == 4 ? 0x0F0F0F0Fu : J == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int k = (i & (J - 1)) | ((i & ~(J - 1)) << 1);
        const uint32_t x = a[k], y = a[k + J];
        if (J == 16) {
            a[k] = __builtin_amdgcn_perm(y, x, 0x05040100u);
            a[k + J] = __builtin_amdgcn_perm(y, x, 0x07060302u);
        } else if (J == 8) {
            a[k] = __builtin_amdgcn_perm(y, x, 0x06020400u);
            a[k + J] = __builtin_amdgcn_perm(y, x, 0x07030501u);
        } else {
            a[k] = (x & m) | ((y << J) & ~m);
            a[k + J] = ((x >> J) & m) | (y & ~m);
        }
    }
}

// In place: bit i of a[k] becomes bit k of a[i].
__device__ __forceinline__ void transpose32(uint32_t (&a)[32]) {
    transpose_step<16>(a);
    transpose_step<8>(a);
    transpose_step<4>(a);
    transpose_step<2>(a);
    transpose_step<1>(a);
}

// OR of v over the lanes with this lane's number modulo 1 << lg (over the wave
// at lg = 0), in every lane: rotations within the rows of 16 lanes, then swaps
// of the rows and of the wave's halves.
__device__ __forceinline__ uint32_t or_rows(uint32_t v, int lg) {
    auto ror = [](uint32_t x, auto ctrl) {
        return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
            0, static_cast<int>(x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    if (lg < 1) v |= ror(v, std::integral_constant<int, 0x121>{});
    if (lg < 2) v |= ror(v, std::integral_constant<int, 0x122>{});
    if (lg < 3) v |= ror(v, std::integral_constant<int, 0x124>{});
    if (lg < 4) v |= ror(v, std::integral_constant<int, 0x128>{});
    const auto h = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = h[0] | h[1];
    const auto w = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return w[0] | w[1];
}

__device__ __forceinline__ uint64_t or_wave(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(or_rows(static_cast<uint32_t>(v), 0));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(or_rows(static_cast<uint32_t>(v >> 32), 0));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// The pointers of a job table are loaded from memory, so the compiler has to be
// told that they point to global memory.
template <class T>
__device__ __forceinline__ T* global_ptr(T* p) {
    return (T*)(__attribute__((address_space(1))) T*)p;
}

}  // namespace bits
}  // namespace rsr
