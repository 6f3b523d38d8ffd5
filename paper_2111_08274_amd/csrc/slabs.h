// Slabs of channels, element access and split weights shared by the convolution kernels that serve both element types.
#pragma once
#include "mfma_tiles.h"

namespace hadfl {
namespace tiles {

// channels per slab, LDS bytes per row of a slab, bytes of the same row in memory (weights), groups of a row that a thread
// stages at a time (32 bytes of float, 16 of bf16), planes
template <typename T> struct Slab;
template <> struct Slab<float> { static constexpr int channels = 32, row = 208, bytes = 192, groups = 4, planes = 3; };
template <> struct Slab<__bf16> { static constexpr int channels = 64, row = 144, bytes = 128, groups = 8, planes = 1; };

// four consecutive elements as floats
__device__ __forceinline__ f4 load4(const float* p) { return *reinterpret_cast<const f4*>(p); }
__device__ __forceinline__ f4 load4(const __bf16* p)
{
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
    return f4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
// stores v rounded to the element type and leaves the rounded values in v
__device__ __forceinline__ void store4(float* p, f4& v) { *reinterpret_cast<f4*>(p) = v; }
__device__ __forceinline__ void store4(__bf16* p, f4& v)
{
    const bf16x4 r = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    *reinterpret_cast<bf16x4*>(p) = r;
    v = f4{(float)r[0], (float)r[1], (float)r[2], (float)r[3]};
}
// The parts of a weight in its copy, of 2^24 times the weight as in split3.  A weight too large for that, or not finite, has a
// NaN for the first part, so that no tile that meets it keeps the products of parts, and its 32 bits in the other two.
__device__ __forceinline__ void split_weight(float x, __bf16& h, __bf16& m, __bf16& l)
{
    if (fabsf(x) < 0x1p103f) {
        const float y = x * kSplitScale;
        h = (__bf16)y;
        const float r = y - (float)h;
        m = (__bf16)r;
        l = (__bf16)(r - (float)m);
    } else {
        const unsigned bits = __builtin_bit_cast(unsigned, x);
        h = __builtin_bit_cast(__bf16, (unsigned short)0x7fc0);
        m = __builtin_bit_cast(__bf16, (unsigned short)(bits >> 16)); l = __builtin_bit_cast(__bf16, (unsigned short)bits);
    }
}
__device__ __forceinline__ float join_weight(__bf16 h, __bf16 m, __bf16 l)
{
    if ((float)h == (float)h) return (((float)l + (float)m) + (float)h) * (1.0f / kSplitScale);
    return __builtin_bit_cast(float, (unsigned)__builtin_bit_cast(unsigned short, m) << 16 | __builtin_bit_cast(unsigned short, l));
}

}  // namespace tiles
}  // namespace hadfl
