// Pieces shared by the tiled matrix-core kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace hadfl {
namespace tiles {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16 __attribute__((ext_vector_type(16)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

// Workgroups are handed to the eight accelerator dies in turn (workgroup i runs on die i % 8), and each die has its own
// L2.  With a one-dimensional grid of 8 * chunk workgroups, die d takes the consecutive logical items
// [d * chunk, (d + 1) * chunk): the tiles of one replica, which share its weights and activations, meet in one L2.
constexpr int kDies = 8;
__device__ __forceinline__ unsigned logical_block()
{
    const unsigned chunk = gridDim.x / kDies;
    return (blockIdx.x % kDies) * chunk + blockIdx.x / kDies;
}
inline unsigned die_grid(long long items) { return (unsigned)((items + kDies - 1) / kDies * kDies); }

__device__ __forceinline__ u4 ldg16(const char* base, unsigned off) { return *reinterpret_cast<const u4*>(base + off); }

// Three bf16 values whose sum is the float times 2^24: with y = 2^24 x, h = bf16(y), m = bf16(y - h), l = y - h - m.  The two
// differences are exact, and what is left for l fits bf16's eight significant bits; |m| <= 2^-9 |y|, |l| <= 2^-18 |y|.  The
// scale keeps l a normal number down to the smallest normal x: without it the lowest bits of |x| < 2^-107 are lost
// (relative error of a product 9e-6 at 2^-118, 6e-4 at 2^-124); it costs 1.0 to 1.4 % of a step of the fp32 residual and VGG
// networks and changes no bit of an ordinary result.  From 2^104 on y, and with it h, overflows.
// Four at a time in pairs: a conversion yields two bf16 in one register, whose floats are a shift and a mask away.
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr float kSplitScale = 0x1p24f, kProductScale = 0x1p-48f;   // of an operand; what takes a product of two back
__device__ __forceinline__ unsigned to_bf16x2(float x, float y)
{
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f2{x, y}), bf16x2));
}
__device__ __forceinline__ void split3(const f4& x, u2& h, u2& m, u2& l)
{
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        float a = x[2 * e] * kSplitScale, b = x[2 * e + 1] * kSplitScale;
        h[e] = to_bf16x2(a, b);
        a -= __builtin_bit_cast(float, h[e] << 16); b -= __builtin_bit_cast(float, h[e] & 0xffff0000u);
        m[e] = to_bf16x2(a, b);
        a -= __builtin_bit_cast(float, m[e] << 16); b -= __builtin_bit_cast(float, m[e] & 0xffff0000u);
        l[e] = to_bf16x2(a, b);
    }
}
// Loads through a buffer descriptor: an offset outside the tensor (kOutside, or anything from `bytes` on) yields zeros, so
// that padding costs a select instead of a branch.
constexpr unsigned kOutside = 0xfffffff0u;
typedef __amdgpu_buffer_rsrc_t Buffer;
__device__ __forceinline__ Buffer buffer(const void* base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ u4 ldb16(Buffer b, unsigned off) { return __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, 0, 0)); }
__device__ __forceinline__ u4 join8(const u2& x, const u2& y) { return u4{x[0], x[1], y[0], y[1]}; }

// Transposing LDS read: within a group of 16 lanes, lane i receives element (i % 4) of the 8 bytes addressed by lane
// 4*j + i/4, for j = 0..3.  Pointing lane L at row k0 + L/4, columns 4*(L%4).. of a 16-column block therefore hands lane i
// the four consecutive k of column i -- half of an MFMA operand.
typedef short s4v __attribute__((ext_vector_type(4)));
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s4v lds_s4v;
__device__ __forceinline__ bf16x8 lds_read_tr8(const char* base, unsigned off, unsigned row_pitch_bytes)
{
    // base + off addresses this lane's 8 bytes in row k0; rows k0+4.. supply the upper four k
    const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)(base + off));
    const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)(base + off + 4 * row_pitch_bytes));
    const s8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}

}  // namespace tiles
}  // namespace hadfl
