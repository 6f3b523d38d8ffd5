// Memory-bound layers of the local-training path, grouped over the active replicas: ReLU, 2x2 max-pool,
// residual add, global average pool, batch normalisation (training mode), softmax cross-entropy and the fused
// SGD/momentum update.  All reductions run in a fixed order (no floating-point atomics): results are repeatable.
#include "train_kernels.h"
#include "mfma_tiles.h"

namespace hadfl {
namespace {

constexpr float kBwdStatCond = 16.f;    // largest |beta / gamma| for which y determines xhat well enough (bn_finalize_kernel)
constexpr float kBnEps = 1e-5f;
constexpr float kBnStatMomentum = 0.1f;

// Activation tensors are fp32 or bf16 (the bf16 configuration); offsets and per-replica strides are always counted
// in 4-byte units, so a bf16 tensor occupies the first half of its slot.
template <typename T> __device__ __forceinline__ T* tptr(const void* base, long long rep, long long rep_stride)
{
    return (T*)((char*)base + rep * rep_stride * 4);
}
__device__ __forceinline__ float ldf(const float* p, long long i) { return p[i]; }
__device__ __forceinline__ float ldf(const __bf16* p, long long i) { return (float)p[i]; }
__device__ __forceinline__ void stf(float* p, long long i, float v) { p[i] = v; }
__device__ __forceinline__ void stf(__bf16* p, long long i, float v) { p[i] = (__bf16)v; }

__device__ __forceinline__ long long gtid() { return (long long)blockIdx.x * blockDim.x + threadIdx.x; }
__device__ __forceinline__ long long gstride() { return (long long)gridDim.x * blockDim.x; }

template <typename T>
__global__ __launch_bounds__(256) void relu_fwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* in = tptr<T>(p.in, rep, p.in_rep);
    T* out = tptr<T>(p.out, rep, p.out_rep);
    for (long long i = gtid(); i < p.count; i += gstride()) stf(out, i, fmaxf(ldf(in, i), 0.f));
}

template <typename T>
__global__ __launch_bounds__(256) void relu_bwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* x = tptr<T>(p.in, rep, p.in_rep);
    const T* dout = tptr<T>(p.in2, rep, p.in2_rep);
    T* din = tptr<T>(p.out, rep, p.out_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    for (long long i = gtid(); i < p.count; i += gstride()) {
        float g = ldf(x, i) > 0.f ? ldf(dout, i) : 0.f;
        if (mask && !(ldf(mask, i) > 0.f)) g = 0.f;
        stf(din, i, p.accumulate ? ldf(din, i) + g : g);
    }
}

// count = pooled elements; in is [B][H][W][C]
template <typename T>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* in = tptr<T>(p.in, rep, p.in_rep);
    T* out = tptr<T>(p.out, rep, p.out_rep);
    const int Ho = p.H / 2, Wo = p.W / 2;
    for (long long i = gtid(); i < p.count; i += gstride()) {
        const int c = (int)(i % p.C);
        long long t = i / p.C;
        const int xo = (int)(t % Wo); t /= Wo;
        const int yo = (int)(t % Ho);
        const int b = (int)(t / Ho);
        const long long q = (((long long)b * p.H + 2 * yo) * p.W + 2 * xo) * p.C + c;
        const long long rowp = (long long)p.W * p.C;
        stf(out, i, fmaxf(fmaxf(ldf(in, q), ldf(in, q + p.C)), fmaxf(ldf(in, q + rowp), ldf(in, q + rowp + p.C))));
    }
}

// the gradient goes to the first maximal element in (dy, dx) scan order; count = pooled elements
template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* x = tptr<T>(p.in, rep, p.in_rep);
    const T* dout = tptr<T>(p.in2, rep, p.in2_rep);
    T* din = tptr<T>(p.out, rep, p.out_rep);
    const int Ho = p.H / 2, Wo = p.W / 2;
    for (long long i = gtid(); i < p.count; i += gstride()) {
        const int c = (int)(i % p.C);
        long long t = i / p.C;
        const int xo = (int)(t % Wo); t /= Wo;
        const int yo = (int)(t % Ho);
        const int b = (int)(t / Ho);
        const long long base = (((long long)b * p.H + 2 * yo) * p.W + 2 * xo) * p.C + c;
        const long long rowp = (long long)p.W * p.C;
        const long long off[4] = {0, p.C, rowp, rowp + p.C};
        float m = ldf(x, base); int arg = 0;
#pragma unroll
        for (int j = 1; j < 4; ++j) { const float v = ldf(x, base + off[j]); if (v > m) { m = v; arg = j; } }
        const float g = ldf(dout, i);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // with p.mask set, x is a fused ReLU output: the gradient passes only where it is positive
            const float v = (j == arg && (!p.mask || m > 0.f)) ? g : 0.f;
            const long long d = base + off[j];
            stf(din, d, p.accumulate ? ldf(din, d) + v : v);
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void add_fwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* a = tptr<T>(p.in, rep, p.in_rep);
    const T* b = tptr<T>(p.in2, rep, p.in2_rep);
    T* out = tptr<T>(p.out, rep, p.out_rep);
    for (long long i = gtid(); i < p.count; i += gstride()) {
        const float v = ldf(a, i) + ldf(b, i);
        stf(out, i, p.relu ? fmaxf(v, 0.f) : v);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void pass_grad_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* dout = tptr<T>(p.in, rep, p.in_rep);
    T* din = tptr<T>(p.out, rep, p.out_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    for (long long i = gtid(); i < p.count; i += gstride()) {
        const float g = (!mask || ldf(mask, i) > 0.f) ? ldf(dout, i) : 0.f;
        stf(din, i, p.accumulate ? ldf(din, i) + g : g);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void zero_kernel(EwParams p)
{
    T* out = tptr<T>(p.out, p.order[blockIdx.y], p.out_rep);
    for (long long i = gtid(); i < p.count; i += gstride()) stf(out, i, 0.f);
}

// out[b][c] = mean over H*W; count = B*C
template <typename T>
__global__ __launch_bounds__(256) void gap_fwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* in = tptr<T>(p.in, rep, p.in_rep);
    T* out = tptr<T>(p.out, rep, p.out_rep);
    const int hw = p.H * p.W;
    for (long long i = gtid(); i < p.count; i += gstride()) {
        const int c = (int)(i % p.C);
        const long long b = i / p.C;
        float s = 0.f;
#pragma unroll 8
        for (int q = 0; q < hw; ++q) s += ldf(in, (b * hw + q) * p.C + c);
        stf(out, i, s / (float)hw);
    }
}

// din[b][q][c] (+)= dout[b][c] / (H*W); count = B*H*W*C
template <typename T>
__global__ __launch_bounds__(256) void gap_bwd_kernel(EwParams p)
{
    const int rep = p.order[blockIdx.y];
    const T* dout = tptr<T>(p.in, rep, p.in_rep);
    T* din = tptr<T>(p.out, rep, p.out_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    const int hw = p.H * p.W;
    for (long long i = gtid(); i < p.count; i += gstride()) {
        const int c = (int)(i % p.C);
        const long long b = i / ((long long)hw * p.C);
        float g = ldf(dout, b * p.C + c) / (float)hw;
        if (mask && !(ldf(mask, i) > 0.f)) g = 0.f;
        stf(din, i, p.accumulate ? ldf(din, i) + g : g);
    }
}

// ------------------------------------------------------------------------------------------------------
// Batch normalisation over rows = B*H*W per channel.  Two reduction passes (sum, then squared deviation from
// the mean) keep the variance accurate in fp32; every pass writes per-chunk partial sums that the next kernel
// adds in chunk order.
// Block = 256 threads = 64 channel lanes x 4 row lanes; grid = (chunks * ceil(C/64), n_active).
// ------------------------------------------------------------------------------------------------------
template <int PASS, typename T>   // 0: sum x   1: sum (x-mean)^2   2 (backward): sum dy and sum dy*xhat
__global__ __launch_bounds__(256) void bn_reduce_kernel(BnParams p)
{
    __shared__ float red[2][4][64];
    const int g = blockIdx.y, rep = p.order[g];
    const int cgroups = (p.C + 63) / 64;
    const int chunk = blockIdx.x / cgroups, cg = blockIdx.x % cgroups;
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
    const int c = cg * 64 + cl;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    float* part = p.partial + g * p.partial_rep;
    float mean = 0.f, istd = 0.f;
    if (PASS >= 1 && c < p.C) {
        if (PASS == 1) {
            float s = 0.f;
            for (int k = 0; k < p.chunks; ++k) s += part[((long long)k * 2 + 0) * p.C + c];
            mean = s / (float)p.rows;
        } else {
            const float* sv = p.saved + rep * p.saved_rep;
            mean = sv[c]; istd = sv[p.C + c];
        }
    }
    const int r0 = chunk * p.chunk_rows, r1 = min(p.rows, r0 + p.chunk_rows);
    float s0 = 0.f, s1 = 0.f;
    if (c < p.C) {
        const T* dy = (PASS == 2) ? tptr<T>(p.dy, rep, p.dy_rep) : nullptr;
        for (int r = r0 + rl; r < r1; r += 4) {
            const float v = ldf(x, (long long)r * p.C + c);
            if (PASS == 0) s0 += v;
            else if (PASS == 1) { const float d = v - mean; s1 += d * d; }
            else { const float d = ldf(dy, (long long)r * p.C + c); s0 += d; s1 += d * ((v - mean) * istd); }
        }
    }
    red[0][rl][cl] = s0; red[1][rl][cl] = s1;
    __syncthreads();
    if (rl == 0 && c < p.C) {
        const float t0 = (red[0][0][cl] + red[0][1][cl]) + (red[0][2][cl] + red[0][3][cl]);
        const float t1 = (red[1][0][cl] + red[1][1][cl]) + (red[1][2][cl] + red[1][3][cl]);
        if (PASS == 0) part[((long long)chunk * 2 + 0) * p.C + c] = t0;
        else if (PASS == 1) part[((long long)chunk * 2 + 1) * p.C + c] = t1;
        else { part[((long long)chunk * 2 + 0) * p.C + c] = t0; part[((long long)chunk * 2 + 1) * p.C + c] = t1; }
    }
}

// (fused explicitly: which of the two products is rounded would otherwise be the compiler's choice, kernel by kernel)
__device__ __forceinline__ float bn_running_mean(float old, float mean) { return __builtin_fmaf(1.f - kBnStatMomentum, old, kBnStatMomentum * mean); }

// The bias that the convolution in front left out of its outputs; it belongs to the running mean.  An Inf or NaN among the biases would
// have made the outputs NaN or Inf: added to the mean times zero, it makes that NaN, and with it all that is normalised.
__device__ __forceinline__ float bn_left_out(const BnParams& p, int rep, int c) { return p.left_out ? p.left_out[rep * p.left_out_rep + c] : 0.f; }

// y = gamma * (x - mean) * istd + beta; the blocks of chunk 0 also store mean / istd and update the running statistics
template <typename T>
__global__ __launch_bounds__(256) void bn_apply_fwd_kernel(BnParams p)
{
    const int g = blockIdx.y, rep = p.order[g];
    const int cgroups = (p.C + 63) / 64;
    const int chunk = blockIdx.x / cgroups, cg = blockIdx.x % cgroups;
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
    const int c = cg * 64 + cl;
    if (c >= p.C) return;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    T* y = tptr<T>(p.y, rep, p.y_rep);
    const float* part = p.partial + g * p.partial_rep;
    float* row = p.params + rep * p.row_stride;
    float s = 0.f, q = 0.f;
    for (int k = 0; k < p.chunks; ++k) { s += part[((long long)k * 2 + 0) * p.C + c]; q += part[((long long)k * 2 + 1) * p.C + c]; }
    const float mean = s / (float)p.rows, var = q / (float)p.rows;
    const float istd = 1.0f / sqrtf(var + kBnEps);
    const float gamma = row[p.w_off + c], beta = row[p.w_off + p.C + c];
    if (chunk == 0 && rl == 0) {
        float* sv = p.saved + rep * p.saved_rep;
        sv[c] = mean; sv[p.C + c] = istd;
        const float unb = p.rows > 1 ? q / (float)(p.rows - 1) : var;
        float* rm = row + p.stat_off;
        rm[c] = bn_running_mean(rm[c], mean);
        rm[p.C + c] = (1.f - kBnStatMomentum) * rm[p.C + c] + kBnStatMomentum * unb;
    }
    const int r0 = chunk * p.chunk_rows, r1 = min(p.rows, r0 + p.chunk_rows);
    for (int r = r0 + rl; r < r1; r += 4) {
        const long long i = (long long)r * p.C + c;
        const float v = gamma * ((ldf(x, i) - mean) * istd) + beta;
        stf(y, i, p.relu ? fmaxf(v, 0.f) : v);
    }
}

// dx = gamma*istd*(dy - sum(dy)/n - xhat*sum(dy*xhat)/n); chunk-0 blocks write dgamma, dbeta
template <typename T>
__global__ __launch_bounds__(256) void bn_apply_bwd_kernel(BnParams p)
{
    const int g = blockIdx.y, rep = p.order[g];
    const int cgroups = (p.C + 63) / 64;
    const int chunk = blockIdx.x / cgroups, cg = blockIdx.x % cgroups;
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
    const int c = cg * 64 + cl;
    if (c >= p.C) return;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* dy = tptr<T>(p.dy, rep, p.dy_rep);
    T* dx = tptr<T>(p.y, rep, p.y_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    const float* part = p.partial + g * p.partial_rep;
    const float* sv = p.saved + rep * p.saved_rep;
    float db = 0.f, dg = 0.f;
    for (int k = 0; k < p.chunks; ++k) { db += part[((long long)k * 2 + 0) * p.C + c]; dg += part[((long long)k * 2 + 1) * p.C + c]; }
    const float mean = sv[c], istd = sv[p.C + c];
    const float gamma = p.params[rep * p.row_stride + p.w_off + c];
    if (chunk == 0 && rl == 0) {
        float* gr = p.grads + rep * p.row_stride + p.w_off;
        gr[c] = dg; gr[p.C + c] = db;
    }
    const float inv_n = 1.0f / (float)p.rows, k1 = gamma * istd;
    const int r0 = chunk * p.chunk_rows, r1 = min(p.rows, r0 + p.chunk_rows);
    for (int r = r0 + rl; r < r1; r += 4) {
        const long long i = (long long)r * p.C + c;
        const float xh = (ldf(x, i) - mean) * istd;
        float v = k1 * (ldf(dy, i) - db * inv_n - xh * dg * inv_n);
        if (mask && !(ldf(mask, i) > 0.f)) v = 0.f;
        stf(dx, i, p.accumulate ? ldf(dx, i) + v : v);
    }
}

// ------------------------------------------------------------------------------------------------------
// Vectorised batch-norm kernels (channel count a multiple of 16 bytes' worth of elements): a thread owns a vector of
// VEC consecutive channels (one 16-byte access per row) and strides over rows; a workgroup is CVB channel vectors x
// 256/CVB row lanes.  The forward statistics take ONE pass: sums of d = x - x0 and d^2 with x0 the tensor's first
// row (a shift close to the mean keeps  E[d^2] - E[d]^2  well conditioned), so forward is 2 passes and backward 2.
// ------------------------------------------------------------------------------------------------------
template <typename T> struct VecOf { static constexpr int n = 16 / (int)sizeof(T); };
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ void ldv(const float* p, long long i, float (&o)[4])
{
    const f4v v = *reinterpret_cast<const f4v*>(p + i);
    o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3];
}
// (bf16 tensors of the large configuration are streamed once per pass and exceed the caches: non-temporal accesses
// measured 3 % faster over the BN kernels; the fp32 tensors of the smaller configurations measured slower with them)
__device__ __forceinline__ void ldv(const __bf16* p, long long i, float (&o)[8])
{
    const bf8v v = __builtin_nontemporal_load(reinterpret_cast<const bf8v*>(p + i));
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (float)v[e];
}
__device__ __forceinline__ void stv(float* p, long long i, const float (&o)[4])
{
    f4v v = {o[0], o[1], o[2], o[3]};
    *reinterpret_cast<f4v*>(p + i) = v;
}
__device__ __forceinline__ void stv(__bf16* p, long long i, const float (&o)[8])
{
    bf8v v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (__bf16)o[e];
    __builtin_nontemporal_store(v, reinterpret_cast<bf8v*>(p + i));
}

// Element-wise kernels with 16-byte accesses for counts that are a multiple of VEC (same results as the scalar ones).
template <typename T>
__global__ __launch_bounds__(256) void add_fwd_vec_kernel(EwParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int rep = p.order[blockIdx.y];
    const T* a = tptr<T>(p.in, rep, p.in_rep);
    const T* b = tptr<T>(p.in2, rep, p.in2_rep);
    T* out = tptr<T>(p.out, rep, p.out_rep);
    const long long nvec = p.count / VEC;
    for (long long i = gtid(); i < nvec; i += gstride()) {
        float u[VEC], w[VEC];
        ldv(a, i * VEC, u); ldv(b, i * VEC, w);
#pragma unroll
        for (int e = 0; e < VEC; ++e) { const float v = u[e] + w[e]; u[e] = p.relu ? fmaxf(v, 0.f) : v; }
        stv(out, i * VEC, u);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void pass_grad_vec_kernel(EwParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int rep = p.order[blockIdx.y];
    const T* dout = tptr<T>(p.in, rep, p.in_rep);
    T* din = tptr<T>(p.out, rep, p.out_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    const long long nvec = p.count / VEC;
    for (long long i = gtid(); i < nvec; i += gstride()) {
        float g[VEC];
        ldv(dout, i * VEC, g);
        if (mask) {
            float mk[VEC];
            ldv(mask, i * VEC, mk);
#pragma unroll
            for (int e = 0; e < VEC; ++e) if (!(mk[e] > 0.f)) g[e] = 0.f;
        }
        if (p.accumulate) {
            float old[VEC];
            ldv(din, i * VEC, old);
#pragma unroll
            for (int e = 0; e < VEC; ++e) g[e] = old[e] + g[e];
        }
        stv(din, i * VEC, g);
    }
}

// 2 x 2 max pooling, one thread per pooled pixel and group of VEC channels (16-byte accesses); count = pooled elements.
// Same results as the scalar kernels above, which stay for channel counts that are not a multiple of VEC.
template <typename T>
__global__ __launch_bounds__(256) void maxpool_fwd_vec_kernel(EwParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int rep = p.order[blockIdx.y];
    const T* in = tptr<T>(p.in, rep, p.in_rep);
    T* out = tptr<T>(p.out, rep, p.out_rep);
    const int Ho = p.H / 2, Wo = p.W / 2, CV = p.C / VEC;
    const long long nvec = p.count / VEC;
    const long long rowp = (long long)p.W * p.C;
    for (long long i = gtid(); i < nvec; i += gstride()) {
        const int cv = (int)(i % CV);
        long long t = i / CV;
        const int xo = (int)(t % Wo); t /= Wo;
        const int yo = (int)(t % Ho);
        const int b = (int)(t / Ho);
        const long long q = (((long long)b * p.H + 2 * yo) * p.W + 2 * xo) * p.C + cv * VEC;
        float a0[VEC], a1[VEC], a2[VEC], a3[VEC];
        ldv(in, q, a0); ldv(in, q + p.C, a1); ldv(in, q + rowp, a2); ldv(in, q + rowp + p.C, a3);
#pragma unroll
        for (int e = 0; e < VEC; ++e) a0[e] = fmaxf(fmaxf(a0[e], a1[e]), fmaxf(a2[e], a3[e]));
        stv(out, i * VEC, a0);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_vec_kernel(EwParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int rep = p.order[blockIdx.y];
    const T* x = tptr<T>(p.in, rep, p.in_rep);
    const T* dout = tptr<T>(p.in2, rep, p.in2_rep);
    T* din = tptr<T>(p.out, rep, p.out_rep);
    const int Ho = p.H / 2, Wo = p.W / 2, CV = p.C / VEC;
    const long long nvec = p.count / VEC;
    const long long rowp = (long long)p.W * p.C;
    for (long long i = gtid(); i < nvec; i += gstride()) {
        const int cv = (int)(i % CV);
        long long t = i / CV;
        const int xo = (int)(t % Wo); t /= Wo;
        const int yo = (int)(t % Ho);
        const int b = (int)(t / Ho);
        const long long base = (((long long)b * p.H + 2 * yo) * p.W + 2 * xo) * p.C + cv * VEC;
        const long long off[4] = {0, p.C, rowp, rowp + p.C};
        float v[4][VEC], g[VEC];
#pragma unroll
        for (int j = 0; j < 4; ++j) ldv(x, base + off[j], v[j]);
        ldv(dout, i * VEC, g);
        int arg[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float m = v[0][e]; arg[e] = 0;
#pragma unroll
            for (int j = 1; j < 4; ++j) if (v[j][e] > m) { m = v[j][e]; arg[e] = j; }     // first maximum in scan order
            // with p.mask set, x is a fused ReLU output: the gradient passes only where it is positive
            if (p.mask && !(m > 0.f)) arg[e] = -1;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float o[VEC];
            if (p.accumulate) ldv(din, base + off[j], o);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const float w = (arg[e] == j) ? g[e] : 0.f;
                o[e] = p.accumulate ? o[e] + w : w;
            }
            stv(din, base + off[j], o);
        }
    }
}

struct BnGeo { int cvb, rl_count, cgroups, chunk, cv, rl, c; bool live; };
__device__ __forceinline__ BnGeo bn_geo(const BnParams& p, int vec)
{
    BnGeo g;
    const int CV = p.C / vec;
    g.cvb = p.cvb; g.rl_count = 256 / g.cvb;
    g.cgroups = (CV + g.cvb - 1) / g.cvb;
    g.chunk = blockIdx.x / g.cgroups;
    g.cv = (blockIdx.x % g.cgroups) * g.cvb + (threadIdx.x % g.cvb);
    g.rl = threadIdx.x / g.cvb;
    g.c = g.cv * vec;
    g.live = g.cv < CV;
    return g;
}

// MODE 0 (forward): partial[chunk][0] = sum(x - x0), [1] = sum((x - x0)^2)
// MODE 1 (backward): partial[chunk][0] = sum(dy), [1] = sum(dy * xhat)
template <int MODE, typename T>
__global__ __launch_bounds__(256) void bn_sums_vec_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    __shared__ float red[256][2 * VEC + 1];
    const int gi = blockIdx.y, rep = p.order[gi];
    const BnGeo g = bn_geo(p, VEC);
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* dy = (MODE == 1) ? tptr<T>(p.dy, rep, p.dy_rep) : nullptr;
    float s0[VEC], s1[VEC], a[VEC], b[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) { s0[e] = 0.f; s1[e] = 0.f; a[e] = 0.f; b[e] = 1.f; }
    if (g.live) {
        if (MODE == 0) ldv(x, g.c, a);                       // the shift: first row of the tensor
        else {
            const float* sv = p.saved + rep * p.saved_rep;
#pragma unroll
            for (int e = 0; e < VEC; ++e) { a[e] = sv[g.c + e]; b[e] = sv[p.C + g.c + e]; }
        }
        const int r0 = g.chunk * p.chunk_rows, r1 = min(p.rows, r0 + p.chunk_rows);
#pragma unroll 4
        for (int r = r0 + g.rl; r < r1; r += g.rl_count) {
            float v[VEC];
            ldv(x, (long long)r * p.C + g.c, v);
            if (MODE == 0) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) { const float d = v[e] - a[e]; s0[e] += d; s1[e] += d * d; }
            } else {
                float d[VEC];
                ldv(dy, (long long)r * p.C + g.c, d);
#pragma unroll
                for (int e = 0; e < VEC; ++e) { s0[e] += d[e]; s1[e] += d[e] * ((v[e] - a[e]) * b[e]); }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) { red[threadIdx.x][e] = s0[e]; red[threadIdx.x][VEC + e] = s1[e]; }
    __syncthreads();
    for (int w = g.rl_count / 2; w > 0; w >>= 1) {           // fixed-order tree over the row lanes
        if (g.rl < w) {
#pragma unroll
            for (int e = 0; e < 2 * VEC; ++e) red[threadIdx.x][e] += red[threadIdx.x + w * g.cvb][e];
        }
        __syncthreads();
    }
    if (g.rl == 0 && g.live) {
        float* part = p.partial + gi * p.partial_rep + (long long)g.chunk * 2 * p.C;
#pragma unroll
        for (int e = 0; e < VEC; ++e) { part[g.c + e] = red[threadIdx.x][e]; part[p.C + g.c + e] = red[threadIdx.x][VEC + e]; }
    }
}

struct PoolWin { long long q[4]; long long o; };
__device__ __forceinline__ PoolWin pool_window(const BnParams& p, int w, int c)
{
    const int Wo = p.W / 2, Ho = p.H / 2;
    const int xo = w % Wo; int t = w / Wo;
    const int yo = t % Ho, b = t / Ho;
    PoolWin r;
    r.q[0] = (((long long)b * p.H + 2 * yo) * p.W + 2 * xo) * p.C + c;
    r.q[1] = r.q[0] + p.C; r.q[2] = r.q[0] + (long long)p.W * p.C; r.q[3] = r.q[2] + p.C;
    r.o = (long long)w * p.C + c;
    return r;
}

// A workgroup takes 32 channels; eight threads per channel add the per-chunk partial sums (chunks k, k+8, ..) and a
// fixed-order tree over the eight joins them.
// Scale and shift of the normalisation and the stored output of one element.  The kernels of a batch norm with a
// folded max-pool do not keep the full-resolution output: the backward ones form a window's four outputs again from x.
// Both directions go through these two functions -- explicit fused multiply-adds, the rounding of the stored type --
// so the values compared for the window's maximum are bit for bit the ones the forward pass took the maximum of.
__device__ __forceinline__ void bn_scale_shift(float mean, float istd, float gamma, float beta, float& sc, float& sh)
{
    sc = gamma * istd;
    sh = __builtin_fmaf(-mean, sc, beta);
}
__device__ __forceinline__ float bn_value(float x, float sc, float sh, bool relu)
{
    const float t = __builtin_fmaf(x, sc, sh);
    return relu ? fmaxf(t, 0.f) : t;
}
template <typename T> __device__ __forceinline__ float bn_stored_value(float x, float sc, float sh, bool relu)
{
    return (float)(T)bn_value(x, sc, sh, relu);
}

// Mean and 1 / sqrt(var + eps) of a channel from its sums s and q of d = x - x0 and d^2; `keeps`: the thread that leaves them for the backward pass
// and updates the running statistics.
__device__ __forceinline__ void bn_statistics(const BnParams& p, int rep, int c, float s, float q, float x0, float left_out, bool keeps, float& mean, float& istd)
{
    const float n = (float)p.rows;
    const float md = s / n + 0.f * left_out;                  // mean of the shifted values
    const float cen = fmaxf(q - s * md, 0.f);                 // sum of squared deviations from the mean
    const float var = cen / n;
    mean = x0 + md; istd = 1.0f / sqrtf(var + kBnEps);
    if (!keeps) return;
    float* sv = p.saved + rep * p.saved_rep;
    sv[c] = mean; sv[p.C + c] = istd;
    const float unb = p.rows > 1 ? cen / (n - 1.f) : var;
    float* rm = p.params + rep * p.row_stride + p.stat_off;
    rm[c] = bn_running_mean(rm[c], mean + left_out);
    rm[p.C + c] = (1.f - kBnStatMomentum) * rm[p.C + c] + kBnStatMomentum * unb;
}

// Batch norms whose sums have few entries: every workgroup of the apply kernel adds those of its own channels, in the order of
// bn_finalize_kernel, whose launch is saved; `finish` makes two numbers per channel of the totals (one thread a channel), which all threads
// get in u and v.
template <int VEC> struct BnFold { float part[8][32][2 * VEC + 1]; float done[32][2 * VEC]; };
template <int VEC, typename F>
__device__ __forceinline__ void bn_fold(const BnParams& p, const BnGeo& g, int gi, int entries, BnFold<VEC>& lds, F&& finish, float (&u)[VEC], float (&v)[VEC])
{
    const int cl = threadIdx.x % g.cvb;
    if (g.rl < 8 && g.live) {                                 // (a workgroup has at least eight row lanes)
        float a[2 * VEC];
#pragma unroll
        for (int e = 0; e < 2 * VEC; ++e) a[e] = 0.f;
        const float* part = p.partial + gi * p.partial_rep + g.c;
#pragma unroll 4
        for (int k = g.rl; k < entries; k += 8)
#pragma unroll
            for (int e = 0; e < VEC; ++e) { a[e] += part[(long long)k * 2 * p.C + e]; a[VEC + e] += part[(long long)k * 2 * p.C + p.C + e]; }
#pragma unroll
        for (int e = 0; e < 2 * VEC; ++e) lds.part[g.rl][cl][e] = a[e];
    }
    __syncthreads();
    const int tc = threadIdx.x / VEC, te = threadIdx.x % VEC, c = (g.cv - cl + tc) * VEC + te;      // this thread's channel
    if (tc < g.cvb && c < p.C) {
        auto total = [&](int e) {
            const auto at = [&](int k) { return lds.part[k][tc][e]; };
            return ((at(0) + at(4)) + (at(2) + at(6))) + ((at(1) + at(5)) + (at(3) + at(7)));
        };
        finish(c, total(te), total(VEC + te), lds.done[tc][te], lds.done[tc][VEC + te]);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < VEC; ++e) { u[e] = lds.done[cl][e]; v[e] = lds.done[cl][VEC + e]; }
}

// MODE 0: mean and 1/sqrt(var+eps) -> saved, running statistics updated.  x0 is the shift used by the sums pass.
// MODE 1: totals of dy and dy*xhat -> gradient of beta and gamma, and into chunk 0 of the partial buffer.
template <int MODE, typename T>
__global__ __launch_bounds__(256) void bn_finalize_kernel(BnParams p)
{
    __shared__ float red[8][32][2];
    const int gi = blockIdx.y, rep = p.order[gi];
    const int cl = threadIdx.x & 31, kl = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + cl;
    const bool live = c < p.C;
    float* part = p.partial + gi * p.partial_rep;
    const int nk = ((MODE == 0 && p.stats_done) || (MODE == 1 && p.bwd_stats_done)) ? p.stat_entries : p.chunks;
    const float left_out = MODE == 0 && live ? bn_left_out(p, rep, c) : 0.f;          // (on its way beside the sums)
    float s = 0.f, q = 0.f;
    // Backward sums left by the data gradient above are s = sum g and q = sum g * y, y = gamma * xhat + beta the stored
    // (bf16) output, so that  sum g * xhat = (q - beta * s) / gamma.  The bf16 rounding of y enters xhat multiplied by
    // |y / gamma| <= |xhat| + |beta / gamma|: harmless while |beta| <= kBwdStatCond * |gamma| (every trained net's
    // case; the rounding errors of the terms are independent and average out in the sum), useless when gamma is zero
    // or tiny beside beta.  Channels outside that range are summed again from x and the gradient, exactly as the sums
    // kernels do, by the whole workgroup, one channel after the other (slow, and rare).
    float gamma = 1.f, beta = 0.f;
    bool direct = false;
    if (MODE == 1) {
        __shared__ int s_direct[32];
        __shared__ float s_sum[32][2];
        __shared__ float s_red[256][2];
        if (p.bwd_stats_done == 1 && live) {
            const float* row = p.params + rep * p.row_stride + p.w_off;
            gamma = row[c]; beta = row[p.C + c];
            direct = gamma == 0.f || !(fabsf(beta) <= kBwdStatCond * fabsf(gamma));
        }
        if (kl == 0) s_direct[cl] = direct ? 1 : 0;
        const int any = __syncthreads_or(direct);
        for (int j = 0; any && j < 32; ++j) {
            if (!s_direct[j]) continue;                       // uniform over the workgroup
            const int cj = blockIdx.x * 32 + j;
            const T* x = tptr<T>(p.x, rep, p.x_rep);
            const float* sv = p.saved + rep * p.saved_rep;
            const float mean = sv[cj], istd = sv[p.C + cj];
            float ts = 0.f, tq = 0.f;
            if (!p.pool) {
                const T* dy = tptr<T>(p.dy, rep, p.dy_rep);
                for (int r = threadIdx.x; r < p.rows; r += 256) {
                    const float d = ldf(dy, (long long)r * p.C + cj);
                    ts += d; tq += d * ((ldf(x, (long long)r * p.C + cj) - mean) * istd);
                }
            } else {
                const T* pg = tptr<T>(p.pool_g, rep, p.pool_g_rep);
                const float* row = p.params + rep * p.row_stride + p.w_off;
                float sc, sh;
                bn_scale_shift(mean, istd, row[cj], row[p.C + cj], sc, sh);
                for (int w = threadIdx.x; w < p.rows / 4; w += 256) {
                    const PoolWin pw = pool_window(p, w, cj);
                    float xw[4];
                    for (int t = 0; t < 4; ++t) xw[t] = ldf(x, pw.q[t]);
                    float m = bn_stored_value<T>(xw[0], sc, sh, p.relu != 0), xs = xw[0];
                    for (int t = 1; t < 4; ++t) {             // first maximum of the window's (recomputed) outputs
                        const float v = bn_stored_value<T>(xw[t], sc, sh, p.relu != 0);
                        if (v > m) { m = v; xs = xw[t]; }
                    }
                    if (p.relu && !(m > 0.f)) continue;       // the fused ReLU passes nothing there
                    const float d = ldf(pg, pw.o);
                    ts += d; tq += d * ((xs - mean) * istd);
                }
            }
            s_red[threadIdx.x][0] = ts; s_red[threadIdx.x][1] = tq;
            __syncthreads();
            for (int w = 128; w > 0; w >>= 1) {               // fixed-order tree
                if ((int)threadIdx.x < w) { s_red[threadIdx.x][0] += s_red[threadIdx.x + w][0]; s_red[threadIdx.x][1] += s_red[threadIdx.x + w][1]; }
                __syncthreads();
            }
            if (threadIdx.x == 0) { s_sum[j][0] = s_red[0][0]; s_sum[j][1] = s_red[0][1]; }
            __syncthreads();
        }
        if (direct && kl == 0) { s = s_sum[cl][0]; q = s_sum[cl][1]; }
    }
    if (live && !direct) {
        // (up to a thousand entries per lane after a convolution with small tiles: keep many loads in flight; the
        // additions stay in ascending order)
#pragma unroll 16
        for (int k = kl; k < nk; k += 8) { s += part[(long long)k * 2 * p.C + c]; q += part[(long long)k * 2 * p.C + p.C + c]; }
    }
    red[kl][cl][0] = s; red[kl][cl][1] = q;
    __syncthreads();
    for (int w = 4; w > 0; w >>= 1) {
        if (kl < w) { red[kl][cl][0] += red[kl + w][cl][0]; red[kl][cl][1] += red[kl + w][cl][1]; }
        __syncthreads();
    }
    if (kl != 0 || !live) return;
    s = red[0][cl][0]; q = red[0][cl][1];
    if (MODE == 0) {
        // the shift the sums were taken with: the producing convolution's bias, or the tensor's first row
        const float x0 = p.stats_done ? (p.stat_shift ? p.stat_shift[rep * p.stat_shift_rep + c] : 0.f)
                                      : ldf(tptr<T>(p.x, rep, p.x_rep), c);
        float mean, istd;
        bn_statistics(p, rep, c, s, q, x0, left_out, true, mean, istd);
    } else {
        if (p.bwd_stats_done == 1 && !direct) q = (q - beta * s) / gamma;
        if (p.bwd_stats_done == 2) q = q * p.saved[rep * p.saved_rep + p.C + c];
        float* gr = p.grads + rep * p.row_stride + p.w_off;
        gr[c] = q; gr[p.C + c] = s;
        part[c] = s; part[p.C + c] = q;
    }
}

// Scale and shift of a thread's channels, with the statistics of bn_finalize_kernel<0> or (FOLD, all threads of the workgroup) formed here
template <typename T, bool FOLD>
__device__ __forceinline__ void bn_forward_scales(const BnParams& p, const BnGeo& g, int gi, int rep, const T* x, float (&sc)[VecOf<T>::n], float (&sh)[VecOf<T>::n])
{
    constexpr int VEC = VecOf<T>::n;
    const float* row = p.params + rep * p.row_stride;
    if constexpr (FOLD) {
        __shared__ BnFold<VEC> lds;
        bn_fold<VEC>(p, g, gi, p.stats_done ? p.stat_entries : p.chunks, lds, [&](int c, float s, float q, float& scale, float& shift) {
            const float x0 = p.stats_done ? (p.stat_shift ? p.stat_shift[rep * p.stat_shift_rep + c] : 0.f) : ldf(x, c);
            float mean, istd;
            bn_statistics(p, rep, c, s, q, x0, bn_left_out(p, rep, c), g.chunk == 0, mean, istd);
            bn_scale_shift(mean, istd, row[p.w_off + c], row[p.w_off + p.C + c], scale, shift);
        }, sc, sh);
    } else {
        const float* sv = p.saved + rep * p.saved_rep;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const int c = g.c + e;
            bn_scale_shift(sv[c], sv[p.C + c], row[p.w_off + c], row[p.w_off + p.C + c], sc[e], sh[e]);
        }
    }
}

// Means of dy and of dy xhat over the batch, for a thread's channels: of the totals that bn_finalize_kernel<1> left in chunk 0, or (FOLD)
// formed here, and the gradients of beta and gamma with them
template <int VEC, bool FOLD>
__device__ __forceinline__ void bn_backward_means(const BnParams& p, const BnGeo& g, int gi, int rep, float (&kb)[VEC], float (&kg)[VEC])
{
    const float inv_n = 1.0f / (float)p.rows;
    if constexpr (FOLD) {
        __shared__ BnFold<VEC> lds;
        bn_fold<VEC>(p, g, gi, p.bwd_stats_done ? p.stat_entries : p.chunks, lds, [&](int c, float s, float q, float& b, float& w) {
            if (p.bwd_stats_done == 2) q = q * p.saved[rep * p.saved_rep + p.C + c];
            if (g.chunk == 0) {
                float* gr = p.grads + rep * p.row_stride + p.w_off;
                gr[c] = q; gr[p.C + c] = s;
            }
            b = s * inv_n; w = q * inv_n;
        }, kb, kg);
    } else {
        const float* part = p.partial + gi * p.partial_rep;
#pragma unroll
        for (int e = 0; e < VEC; ++e) { kb[e] = part[g.c + e] * inv_n; kg[e] = part[p.C + g.c + e] * inv_n; }
    }
}

template <typename T, bool FOLD>
__global__ __launch_bounds__(256) void bn_apply_fwd_vec_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int gi = blockIdx.y, rep = p.order[gi];
    const BnGeo g = bn_geo(p, VEC);
    if (!FOLD && !g.live) return;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    T* y = tptr<T>(p.y, rep, p.y_rep);
    const T* add = p.add ? tptr<T>(p.add, rep, p.add_rep) : nullptr;
    float sc[VEC], sh[VEC];
    bn_forward_scales<T, FOLD>(p, g, gi, rep, x, sc, sh);
    if (!g.live) return;
    const int r0 = g.chunk * p.chunk_rows, r1 = min(p.rows, r0 + p.chunk_rows);
#pragma unroll 4
    for (int r = r0 + g.rl; r < r1; r += g.rl_count) {
        float v[VEC];
        const long long i = (long long)r * p.C + g.c;
        ldv(x, i, v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = bn_value(v[e], sc[e], sh[e], p.relu != 0);
        if (add) {                                        // the sum of two tensors that follows, with its ReLU
            float w[VEC];
            ldv(add, i, w);
#pragma unroll
            for (int e = 0; e < VEC; ++e) { const float u = (float)(T)v[e] + w[e]; v[e] = p.add_relu ? fmaxf(u, 0.f) : u; }
        }
        stv(y, i, v);
    }
}

template <typename T, bool FOLD>
__global__ __launch_bounds__(256) void bn_apply_bwd_vec_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int gi = blockIdx.y, rep = p.order[gi];
    const BnGeo g = bn_geo(p, VEC);
    if (!FOLD && !g.live) return;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* dy = tptr<T>(p.dy, rep, p.dy_rep);
    T* dx = tptr<T>(p.y, rep, p.y_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    const float* sv = p.saved + rep * p.saved_rep;
    float mean[VEC], istd[VEC], k1[VEC], kb[VEC], kg[VEC];
    const int c0 = g.live ? g.c : 0;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        mean[e] = sv[c0 + e]; istd[e] = sv[p.C + c0 + e];
        k1[e] = p.params[rep * p.row_stride + p.w_off + c0 + e] * istd[e];
    }
    bn_backward_means<VEC, FOLD>(p, g, gi, rep, kb, kg);
    if (!g.live) return;
    const int r0 = g.chunk * p.chunk_rows, r1 = min(p.rows, r0 + p.chunk_rows);
#pragma unroll 4
    for (int r = r0 + g.rl; r < r1; r += g.rl_count) {
        const long long i = (long long)r * p.C + g.c;
        float v[VEC], d[VEC], o[VEC];
        ldv(x, i, v); ldv(dy, i, d);
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[e] = k1[e] * (d[e] - kb[e] - ((v[e] - mean[e]) * istd[e]) * kg[e]);
        if (mask) {
            float mk[VEC];
            ldv(mask, i, mk);
#pragma unroll
            for (int e = 0; e < VEC; ++e) if (!(mk[e] > 0.f)) o[e] = 0.f;
        }
        if (p.accumulate) {
            float old[VEC];
            ldv(dx, i, old);
#pragma unroll
            for (int e = 0; e < VEC; ++e) o[e] += old[e];
        }
        stv(dx, i, o);
    }
}

// ------------------------------------------------------------------------------------------------------
// Batch norm whose (ReLU'd) output feeds a 2x2/stride-2 max-pool only: the pool is folded into the BN kernels.
// A thread walks 2x2 windows instead of single rows.  Forward: it normalises the four pixels, stores them and their
// maximum (one pass less over the full-resolution tensor than a separate pool).  Backward: the gradient of a pixel
// is the pooled gradient where the pixel is the window's first maximum in scan order and is positive, else zero; it
// is formed on the fly from the stored output and the pooled gradient, so the full-resolution gradient tensor is
// neither written nor read (two passes less).  Window w of chunk c: [c * chunk_windows, (c + 1) * chunk_windows).
// ------------------------------------------------------------------------------------------------------
template <typename T, bool FOLD>
__global__ __launch_bounds__(256) void bn_apply_fwd_pool_vec_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int gi = blockIdx.y, rep = p.order[gi];
    const BnGeo g = bn_geo(p, VEC);
    if (!FOLD && !g.live) return;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    T* po = tptr<T>(p.pool_out, rep, p.pool_out_rep);
    float sc[VEC], sh[VEC];
    bn_forward_scales<T, FOLD>(p, g, gi, rep, x, sc, sh);
    if (!g.live) return;
    const int windows = p.rows / 4, cw = (windows + p.chunks - 1) / p.chunks;
    const int w0 = g.chunk * cw, w1 = min(windows, w0 + cw);
#pragma unroll 2
    for (int w = w0 + g.rl; w < w1; w += g.rl_count) {
        const PoolWin pw = pool_window(p, w, g.c);
        float v[4][VEC], m[VEC];
#pragma unroll
        for (int j = 0; j < 4; ++j) ldv(x, pw.q[j], v[j]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) v[j][e] = bn_value(v[j][e], sc[e], sh[e], p.relu != 0);
        }                                                     // (the four outputs themselves are not stored)
#pragma unroll
        for (int e = 0; e < VEC; ++e) m[e] = fmaxf(fmaxf(v[0][e], v[1][e]), fmaxf(v[2][e], v[3][e]));
        stv(po, pw.o, m);
    }
}

// which of the window's four pixels receives the pooled gradient (per channel), or -1
template <int VEC>
__device__ __forceinline__ void pool_argmax(const float (&yv)[4][VEC], bool relu, int (&arg)[VEC])
{
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        float m = yv[0][e]; arg[e] = 0;
#pragma unroll
        for (int j = 1; j < 4; ++j) if (yv[j][e] > m) { m = yv[j][e]; arg[e] = j; }     // first maximum in scan order
        if (relu && !(m > 0.f)) arg[e] = -1;                                             // the fused ReLU passes nothing there
    }
}

template <typename T>
__global__ __launch_bounds__(256) void bn_sums_pool_vec_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    __shared__ float red[256][2 * VEC + 1];
    const int gi = blockIdx.y, rep = p.order[gi];
    const BnGeo g = bn_geo(p, VEC);
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* pg = tptr<T>(p.pool_g, rep, p.pool_g_rep);
    float s0[VEC], s1[VEC], a[VEC], b[VEC], sc[VEC], sh[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) { s0[e] = 0.f; s1[e] = 0.f; a[e] = 0.f; b[e] = 1.f; sc[e] = 0.f; sh[e] = 0.f; }
    if (g.live) {
        const float* sv = p.saved + rep * p.saved_rep;
        const float* row = p.params + rep * p.row_stride + p.w_off;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            a[e] = sv[g.c + e]; b[e] = sv[p.C + g.c + e];
            bn_scale_shift(a[e], b[e], row[g.c + e], row[p.C + g.c + e], sc[e], sh[e]);
        }
        const int windows = p.rows / 4, cw = (windows + p.chunks - 1) / p.chunks;
        const int w0 = g.chunk * cw, w1 = min(windows, w0 + cw);
#pragma unroll 2
        for (int w = w0 + g.rl; w < w1; w += g.rl_count) {
            const PoolWin pw = pool_window(p, w, g.c);
            float yv[4][VEC], xv[4][VEC], gv[VEC];
            int arg[VEC];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ldv(x, pw.q[j], xv[j]);
#pragma unroll
                for (int e = 0; e < VEC; ++e) yv[j][e] = bn_stored_value<T>(xv[j][e], sc[e], sh[e], p.relu != 0);
            }
            ldv(pg, pw.o, gv);
            pool_argmax<VEC>(yv, p.relu != 0, arg);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                float xs = xv[0][e];
#pragma unroll
                for (int j = 1; j < 4; ++j) xs = arg[e] == j ? xv[j][e] : xs;
                const float d = arg[e] >= 0 ? gv[e] : 0.f;
                s0[e] += d; s1[e] += d * ((xs - a[e]) * b[e]);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) { red[threadIdx.x][e] = s0[e]; red[threadIdx.x][VEC + e] = s1[e]; }
    __syncthreads();
    for (int w = g.rl_count / 2; w > 0; w >>= 1) {           // fixed-order tree over the row lanes
        if (g.rl < w) {
#pragma unroll
            for (int e = 0; e < 2 * VEC; ++e) red[threadIdx.x][e] += red[threadIdx.x + w * g.cvb][e];
        }
        __syncthreads();
    }
    if (g.rl == 0 && g.live) {
        float* part = p.partial + gi * p.partial_rep + (long long)g.chunk * 2 * p.C;
#pragma unroll
        for (int e = 0; e < VEC; ++e) { part[g.c + e] = red[threadIdx.x][e]; part[p.C + g.c + e] = red[threadIdx.x][VEC + e]; }
    }
}

template <typename T, bool FOLD>
__global__ __launch_bounds__(256) void bn_apply_bwd_pool_vec_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    const int gi = blockIdx.y, rep = p.order[gi];
    const BnGeo g = bn_geo(p, VEC);
    if (!FOLD && !g.live) return;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* pg = tptr<T>(p.pool_g, rep, p.pool_g_rep);
    T* dx = tptr<T>(p.y, rep, p.y_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    const float* sv = p.saved + rep * p.saved_rep;
    float mean[VEC], istd[VEC], k1[VEC], kb[VEC], kg[VEC], sc[VEC], sh[VEC];
    bn_backward_means<VEC, FOLD>(p, g, gi, rep, kb, kg);
    if (!g.live) return;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const int c = g.c + e;
        const float* row = p.params + rep * p.row_stride + p.w_off;
        mean[e] = sv[c]; istd[e] = sv[p.C + c];
        k1[e] = row[c] * istd[e];
        bn_scale_shift(mean[e], istd[e], row[c], row[p.C + c], sc[e], sh[e]);
    }
    const int windows = p.rows / 4, cw = (windows + p.chunks - 1) / p.chunks;
    const int w0 = g.chunk * cw, w1 = min(windows, w0 + cw);
#pragma unroll 2
    for (int w = w0 + g.rl; w < w1; w += g.rl_count) {
        const PoolWin pw = pool_window(p, w, g.c);
        float yv[4][VEC], xv[4][VEC], gv[VEC];
        int arg[VEC];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ldv(x, pw.q[j], xv[j]);
#pragma unroll
            for (int e = 0; e < VEC; ++e) yv[j][e] = bn_stored_value<T>(xv[j][e], sc[e], sh[e], p.relu != 0);
        }
        ldv(pg, pw.o, gv);
        pool_argmax<VEC>(yv, p.relu != 0, arg);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float o[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const float d = arg[e] == j ? gv[e] : 0.f;
                o[e] = k1[e] * (d - kb[e] - ((xv[j][e] - mean[e]) * istd[e]) * kg[e]);
            }
            if (mask) {
                float mk[VEC];
                ldv(mask, pw.q[j], mk);
#pragma unroll
                for (int e = 0; e < VEC; ++e) if (!(mk[e] > 0.f)) o[e] = 0.f;
            }
            if (p.accumulate) {
                float old[VEC];
                ldv(dx, pw.q[j], old);
#pragma unroll
                for (int e = 0; e < VEC; ++e) o[e] += old[e];
            }
            stv(dx, pw.q[j], o);
        }
    }
}

// Sixteen bytes of a tensor as they lie, and their values
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ u4v ldraw(const T* p, long long i) { return *reinterpret_cast<const u4v*>(p + i); }
__device__ __forceinline__ void values(const u4v& r, float (&v)[4])
{
    const f4v f = __builtin_bit_cast(f4v, r);                 // (of the whole: of an element, the compiler takes the first for each)
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = f[e];
}
__device__ __forceinline__ void values(const u4v& r, float (&v)[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = __builtin_bit_cast(float, e & 1 ? r[e >> 1] & 0xffff0000u : r[e >> 1] << 16);
}

// ---- batch norm of a small tensor in one launch ----
// A workgroup of 1024 threads owns 4 channel vectors of one replica over all rows: sums, statistics and the normalised output
// (backward: sums, gradients and the data gradient).  A thread has at most eight rows of its vector: they are fetched first of all, beside
// the sums that the convolution left, and kept in registers for the second pass (80 channels on 1250 rows, 1 to 5 replicas: forward 9.0-11.4 us and backward 9.0-10.3 when
// the second pass read them again; 7.3-10.5 and 7.2-9.0 here).  Three dependent launches of 5 to 6 us each are what such a layer's
// backward pass otherwise costs, two its forward pass where the convolution left the sums.  512 channels on 1024 rows, 4 replicas, 2 M
// values: 29 us, no better than three launches, hence the limit in bn_small().
constexpr int kBnSmallThreads = 1024, kBnSmallWaves = kBnSmallThreads / 64, kBnSmallRows = 8;      // (kBnSmallRows: of a thread)

// Totals over the row lanes of one channel vector, in every thread: xor-shuffles inside the waves, the waves in order by one
// thread per value.
constexpr int kBnSmallCvb = 4;                                // channel vectors per workgroup: 64 bytes of a row
template <int N>
__device__ __forceinline__ void bn_small_total(float (&v)[N], float (*red)[kBnSmallCvb][N], int cvb)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cv = threadIdx.x % cvb;
    for (int off = cvb; off < 64; off <<= 1)
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] += __shfl_xor(v[e], off, 64);
    if (lane < cvb)
#pragma unroll
        for (int e = 0; e < N; ++e) red[wave][cv][e] = v[e];
    __syncthreads();
    if ((int)threadIdx.x < cvb * N) {
        const int c = threadIdx.x / N, e = threadIdx.x % N;
        float t = red[0][c][e];
#pragma unroll
        for (int w = 1; w < kBnSmallWaves; ++w) t += red[w][c][e];
        red[0][c][e] = t;                                     // (read by this thread only until the barrier)
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < N; ++e) v[e] = red[0][cv][e];
}

template <typename T>
__global__ __launch_bounds__(kBnSmallThreads) void bn_small_fwd_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    __shared__ __attribute__((aligned(16))) float red[kBnSmallWaves][kBnSmallCvb][2 * VEC];
    const int gi = blockIdx.y, rep = p.order[gi];
    const int CV = p.C / VEC, cv = blockIdx.x * p.cvb + threadIdx.x % p.cvb, rl = threadIdx.x / p.cvb, lanes = kBnSmallThreads / p.cvb;
    const bool live = cv < CV;
    const int c0 = live ? cv * VEC : 0;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    u4v xr[kBnSmallRows];
#pragma unroll
    for (int q = 0; q < kBnSmallRows; ++q) xr[q] = ldraw(x, (long long)min(rl + q * lanes, p.rows - 1) * p.C + c0);
    float x0[VEC], t[2 * VEC];                                // the shift the sums are taken with; sums of d and d^2
#pragma unroll
    for (int e = 0; e < 2 * VEC; ++e) t[e] = 0.f;
    if (p.stats_done) {
        const float* part = p.partial + gi * p.partial_rep;
#pragma unroll
        for (int e = 0; e < VEC; ++e) x0[e] = p.stat_shift ? p.stat_shift[rep * p.stat_shift_rep + c0 + e] : 0.f;
        if (live)
            for (int k = rl; k < p.stat_entries; k += lanes)
#pragma unroll
                for (int e = 0; e < VEC; ++e) { t[e] += part[(long long)k * 2 * p.C + c0 + e]; t[VEC + e] += part[(long long)k * 2 * p.C + p.C + c0 + e]; }
    } else {
        ldv(x, c0, x0);
#pragma unroll
        for (int q = 0; q < kBnSmallRows; ++q) {
            if (!live || rl + q * lanes >= p.rows) continue;
            float v[VEC];
            values(xr[q], v);
#pragma unroll
            for (int e = 0; e < VEC; ++e) { const float d = v[e] - x0[e]; t[e] += d; t[VEC + e] += d * d; }
        }
    }
    float* row = p.params + rep * p.row_stride;
    float gamma[VEC], beta[VEC], left_out[VEC] = {};          // (on their way beside the totals)
#pragma unroll
    for (int e = 0; e < VEC; ++e) { gamma[e] = row[p.w_off + c0 + e]; beta[e] = row[p.w_off + p.C + c0 + e]; }
    if (p.left_out) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) left_out[e] = p.left_out[rep * p.left_out_rep + c0 + e];
    }
    bn_small_total(t, red, p.cvb);
    if (!live) return;
    const float n = (float)p.rows;
    float sc[VEC], sh[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {                           // as in bn_finalize_kernel<0>
        const int c = c0 + e;
        const float md = t[e] / n + 0.f * left_out[e], cen = fmaxf(t[VEC + e] - t[e] * md, 0.f), mean = x0[e] + md, var = cen / n, istd = 1.0f / sqrtf(var + kBnEps);
        if (rl == 0) {
            float* sv = p.saved + rep * p.saved_rep;
            sv[c] = mean; sv[p.C + c] = istd;
            const float unb = p.rows > 1 ? cen / (n - 1.f) : var;
            float* rm = row + p.stat_off;
            rm[c] = bn_running_mean(rm[c], mean + left_out[e]);
            rm[p.C + c] = (1.f - kBnStatMomentum) * rm[p.C + c] + kBnStatMomentum * unb;
        }
        bn_scale_shift(mean, istd, gamma[e], beta[e], sc[e], sh[e]);
    }
    T* y = tptr<T>(p.y, rep, p.y_rep);
    const T* add = p.add ? tptr<T>(p.add, rep, p.add_rep) : nullptr;
#pragma unroll
    for (int q = 0; q < kBnSmallRows; ++q) {
        const int r = rl + q * lanes;
        if (r >= p.rows) break;
        const long long i = (long long)r * p.C + c0;
        float v[VEC];
        values(xr[q], v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = bn_value(v[e], sc[e], sh[e], p.relu != 0);
        if (add) {
            float w[VEC];
            ldv(add, i, w);
#pragma unroll
            for (int e = 0; e < VEC; ++e) { const float u = (float)(T)v[e] + w[e]; v[e] = p.add_relu ? fmaxf(u, 0.f) : u; }
        }
        stv(y, i, v);
    }
}

template <typename T>
__global__ __launch_bounds__(kBnSmallThreads) void bn_small_bwd_kernel(BnParams p)
{
    constexpr int VEC = VecOf<T>::n;
    __shared__ __attribute__((aligned(16))) float red[kBnSmallWaves][kBnSmallCvb][2 * VEC];
    const int gi = blockIdx.y, rep = p.order[gi];
    const int CV = p.C / VEC, cv = blockIdx.x * p.cvb + threadIdx.x % p.cvb, rl = threadIdx.x / p.cvb, lanes = kBnSmallThreads / p.cvb;
    const bool live = cv < CV;
    const int c0 = live ? cv * VEC : 0;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* dy = tptr<T>(p.dy, rep, p.dy_rep);
    u4v xr[kBnSmallRows], dr[kBnSmallRows];
#pragma unroll
    for (int q = 0; q < kBnSmallRows; ++q) {
        const long long i = (long long)min(rl + q * lanes, p.rows - 1) * p.C + c0;
        xr[q] = ldraw(x, i); dr[q] = ldraw(dy, i);
    }
    const float* sv = p.saved + rep * p.saved_rep;
    const float* const gamma = p.params + rep * p.row_stride + p.w_off + c0;
    float mean[VEC], istd[VEC], k1[VEC], t[2 * VEC];          // sums of dy and dy * xhat
    constexpr bool kEarly = VEC == 4;                         // (beside the sums; eight more registers a thread does not have)
    if constexpr (kEarly)
#pragma unroll
        for (int e = 0; e < VEC; ++e) k1[e] = gamma[e];
#pragma unroll
    for (int e = 0; e < VEC; ++e) { mean[e] = sv[c0 + e]; istd[e] = sv[p.C + c0 + e]; t[e] = 0.f; t[VEC + e] = 0.f; }
#pragma unroll
    for (int q = 0; q < kBnSmallRows; ++q) {
        if (!live || rl + q * lanes >= p.rows) continue;
        float v[VEC], d[VEC];
        values(xr[q], v); values(dr[q], d);
#pragma unroll
        for (int e = 0; e < VEC; ++e) { t[e] += d[e]; t[VEC + e] += d[e] * ((v[e] - mean[e]) * istd[e]); }
    }
    bn_small_total(t, red, p.cvb);
    if (!live) return;
    const float inv_n = 1.0f / (float)p.rows;
    float kb[VEC], kg[VEC];
    float* gr = p.grads + rep * p.row_stride + p.w_off;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        if (rl == 0) { gr[c0 + e] = t[VEC + e]; gr[p.C + c0 + e] = t[e]; }
        k1[e] = (kEarly ? k1[e] : gamma[e]) * istd[e];
        kb[e] = t[e] * inv_n; kg[e] = t[VEC + e] * inv_n;
    }
    T* dx = tptr<T>(p.y, rep, p.y_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
#pragma unroll
    for (int q = 0; q < kBnSmallRows; ++q) {
        const int r = rl + q * lanes;
        if (r >= p.rows) break;
        const long long i = (long long)r * p.C + c0;
        float v[VEC], d[VEC], o[VEC];
        values(xr[q], v); values(dr[q], d);
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[e] = k1[e] * (d[e] - kb[e] - ((v[e] - mean[e]) * istd[e]) * kg[e]);
        if (mask) {
            float mk[VEC];
            ldv(mask, i, mk);
#pragma unroll
            for (int e = 0; e < VEC; ++e) if (!(mk[e] > 0.f)) o[e] = 0.f;
        }
        if (p.accumulate) {
            float old[VEC];
            ldv(dx, i, old);
#pragma unroll
            for (int e = 0; e < VEC; ++e) o[e] += old[e];
        }
        stv(dx, i, o);
    }
}

// One workgroup per replica, one thread per sample: softmax, loss, d(loss)/d(logits); loss summed by an LDS tree.
template <typename T>
__global__ __launch_bounds__(1024) void softmax_ce_kernel(LossParams p)
{
    __shared__ float red[1024];
    const int rep = p.order[blockIdx.x];
    const int b = threadIdx.x;
    float li = 0.f;
    if (b < p.batch) {
        const long long first = ((p.cursor[rep] + p.ahead) * (long long)p.batch) % p.n_samples;
        const int label = p.y[(long long)rep * p.n_samples + first + b];
        const T* z = tptr<T>(p.logits, rep, p.logits_rep) + (long long)b * p.n_classes;
        T* dz = tptr<T>(p.dlogits, rep, p.dlogits_rep) + (long long)b * p.n_classes;
        float m = ldf(z, 0);
        for (int j = 1; j < p.n_classes; ++j) m = fmaxf(m, ldf(z, j));
        float s = 0.f;
        for (int j = 0; j < p.n_classes; ++j) s += expf(ldf(z, j) - m);
        li = (logf(s) + m - ldf(z, label)) / (float)p.batch;
        const float inv = 1.0f / s;
        for (int j = 0; j < p.n_classes; ++j)
            stf(dz, j, (expf(ldf(z, j) - m) * inv - (j == label ? 1.f : 0.f)) / (float)p.batch);
    }
    red[b] = li;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (b < w) red[b] += red[b + w];
        __syncthreads();
    }
    if (b == 0) p.loss[rep] = red[0];
}

typedef float f4 __attribute__((ext_vector_type(4)));

// buf = momentum*buf + g; w = w - lr*buf (local-update equation; momentum 0 is the paper's form).
__global__ __launch_bounds__(256) void sgd_kernel(SgdParams p)
{
    const int rep = p.order[blockIdx.y];
    float* const w = p.w + rep * p.row_stride;
    const float* const g = p.g + rep * p.row_stride;
    float* const buf = p.buf ? p.buf + rep * p.row_stride : nullptr;
    long long n4 = 0;
    for (int k = 0; k < p.n_seg; ++k) n4 += p.count[k] / 4;
    for (long long i = gtid(); i < n4; i += gstride()) {
        long long j = i; int k = 0;
        while (j >= p.count[k] / 4) { j -= p.count[k] / 4; ++k; }       // piece k, vector j of it
        const long long o = p.first[k] + 4 * j;
        f4 d = *reinterpret_cast<const f4*>(g + o);
        if (buf) { d = *reinterpret_cast<const f4*>(buf + o) * p.momentum + d; *reinterpret_cast<f4*>(buf + o) = d; }
        *reinterpret_cast<f4*>(w + o) = *reinterpret_cast<const f4*>(w + o) - d * p.lr;
    }
}

__global__ __launch_bounds__(256) void advance_kernel(const int* steps, int* versions, long long* cursor, int n)
{
    for (int k = gtid(); k < n; k += gstride()) { versions[k] = steps[k]; cursor[k] += steps[k]; }
}

// Narrow dense layer (the classifier: out <= 16): one workgroup per sample row; threads stride over the input
// features, keep `out` partial sums each and combine them with a fixed butterfly and a fixed LDS order.  Too small
// for the matrix cores.  For long rows, whose weights come from beyond the die's L2 (the update has just written them): what
// bounds it is the latency of a thread's loads, four features of which are in flight, two weights a load where they are even.  4096 features,
// 10 outputs, 64 rows on 2 / 4 / 6 / 8 replicas, us: 20 20 26 30 one feature after another, 14 14 16 18 here (eight features: the same;
// weights through LDS, fetched a piece of 256 features ahead: 22 23 24 27); dense_rows_fwd_kernel takes 40, but 5 on 512 features.
typedef float f2 __attribute__((ext_vector_type(2)));
template <int NMAX, typename T>
__global__ __launch_bounds__(256) void dense_small_fwd_kernel(DenseSmallParams p)
{
    __shared__ float red[4][NMAX];
    const int rep = p.order[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blockIdx.x;
    const T* x = tptr<T>(p.x, rep, p.x_rep) + (long long)m * p.K;
    const float* w = p.w + rep * p.w_rep;
    constexpr bool kRoundW = sizeof(T) == 2;      // bf16 configuration: weights take part rounded to bf16
    float acc[NMAX];
#pragma unroll
    for (int n = 0; n < NMAX; ++n) acc[n] = 0.f;
    // (rows of an even number of weights start at multiples of eight bytes)
    constexpr int kAhead = 4;                     // features whose loads are in flight together
    const bool pairs = p.N % 2 == 0;
    for (int k0 = threadIdx.x; k0 < p.K; k0 += 256 * kAhead) {
        float xv[kAhead], wv[kAhead][NMAX];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int k = min(k0 + 256 * u, p.K - 1);         // (beyond the last: not used)
            xv[u] = ldf(x, k);
            const float* const wr = w + (long long)k * p.N;
            if (pairs) {
#pragma unroll
                for (int n = 0; n < NMAX; n += 2)
                    if (n < p.N) { const f2 v = *reinterpret_cast<const f2*>(wr + n); wv[u][n] = v[0]; wv[u][n + 1] = v[1]; }
            } else {
#pragma unroll
                for (int n = 0; n < NMAX; ++n) if (n < p.N) wv[u][n] = wr[n];
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (k0 + 256 * u >= p.K) break;
#pragma unroll
            for (int n = 0; n < NMAX; ++n) if (n < p.N) acc[n] += xv[u] * (kRoundW ? (float)(__bf16)wv[u][n] : wv[u][n]);
        }
    }
#pragma unroll
    for (int n = 0; n < NMAX; ++n) {
        if (n >= p.N) continue;
        float v = acc[n];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) red[wave][n] = v;
    }
    __syncthreads();
    if (threadIdx.x < p.N) {
        const int n = threadIdx.x;
        T* o = tptr<T>(p.out, rep, p.out_rep) + (long long)m * p.N;
        stf(o, n, ((red[0][n] + red[1][n]) + (red[2][n] + red[3][n])) + (p.has_bias ? w[(long long)p.K * p.N + n] : 0.f));
    }
}

// Forward of a dense layer with few rows: classifiers and layers on the data set.  A workgroup owns 32 rows x 32 outputs and its
// sixteen waves share the contraction: a step is eight features, of which instruction e multiplies features e and 4 + e
// (lanes of half 0 and half 1), so a lane's operand of a step is one 16-byte piece of its row; the weights are read as they
// lie in the master.  Nothing passes through LDS but the waves' sums, added in wave order.  What bounds it is the latency of
// K / 128 steps: 784 x 128 on 32 rows 5 us (generic tile kernel, one workgroup walking all of K: 77 us).
// SRC: type of x; float for T = __bf16 is the data set, rounded to bf16 like every operand of that configuration.
template <typename T, typename SRC>
__global__ __launch_bounds__(1024) void dense_rows_fwd_kernel(DenseRowsParams p)
{
    typedef float f16v __attribute__((ext_vector_type(16)));
    constexpr bool kRound = sizeof(T) == 2;
    __shared__ float red[16][16][64];
    const int rep = p.order[blockIdx.z];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5;
    const int m0 = blockIdx.x * 32, n0 = blockIdx.y * 32, m = m0 + (lane & 31), n = n0 + (lane & 31);
    const SRC* x;
    if (p.cursor) {
        const long long first = ((p.cursor[rep] + p.ahead) * (long long)p.batch) % p.n_samples;
        x = reinterpret_cast<const SRC*>(p.x) + ((long long)rep * p.n_samples + first) * p.K;
    } else {
        x = tptr<SRC>(p.x, rep, p.x_rep);
    }
    x += (long long)m0 * p.K;
    const float* const w = p.w + rep * p.w_rep;
    const bool m_ok = m < p.rows, n_ok = n < p.N, vec = p.K % 4 == 0;
    f16v acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    // The loads of kAhead steps are in flight together: through buffer descriptors, which give zeros for what lies outside, there is no
    // branch between them.
    constexpr int kAhead = 8;
    constexpr unsigned ES = sizeof(SRC), kAll = tiles::kOutside;
    const unsigned xoff = ((unsigned)(lane & 31) * (unsigned)p.K + 4u * h) * ES, woff = (4u * h * (unsigned)p.N + (unsigned)n) * 4u;
    for (int k8 = wave * 8; k8 < p.K; k8 += 128 * kAhead) {
        float a[kAhead][4], b[kAhead][4];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int ku = k8 + 128 * u, k = ku + 4 * h;
            if (ku >= p.K) break;
            const tiles::Buffer xb = tiles::buffer(x + ku, kAll), wb = tiles::buffer(w + (long long)ku * p.N, kAll);
            if (vec) {
                const unsigned o = m_ok && k < p.K ? xoff : kAll;
                if constexpr (sizeof(SRC) == 4) {
                    const tiles::f4 v = __builtin_bit_cast(tiles::f4, tiles::ldb16(xb, o));
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[u][e] = v[e];
                } else {
                    const tiles::bf16x4 v = __builtin_bit_cast(tiles::bf16x4, __builtin_amdgcn_raw_buffer_load_b64(xb, (int)o, 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[u][e] = (float)v[e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned o = m_ok && k + e < p.K ? xoff + e * ES : kAll;
                    if constexpr (sizeof(SRC) == 4) a[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xb, (int)o, 0, 0));
                    else a[u][e] = __builtin_bit_cast(float, (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(xb, (int)o, 0, 0) << 16);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                b[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wb, (int)(n_ok && k + e < p.K ? woff + (unsigned)(e * p.N) * 4u : kAll), 0, 0));
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (k8 + 128 * u >= p.K) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (kRound) { a[u][e] = (float)(__bf16)a[u][e]; b[u][e] = (float)(__bf16)b[u][e]; }
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][e], b[u][e], acc, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
    __syncthreads();
    // thread (v, lane) finishes output row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
    const int v = threadIdx.x >> 6, row = m0 + 8 * (v >> 2) + 4 * h + (v & 3);
    if (row < p.rows && n_ok) {
        float r = red[0][v][lane];
#pragma unroll
        for (int k = 1; k < 16; ++k) r += red[k][v][lane];
        if (p.has_bias) r += w[(long long)p.K * p.N + n];
        if (p.relu) r = fmaxf(r, 0.f);
        stf(tptr<T>(p.out, rep, p.out_rep), (long long)row * p.N + n, r);
    }
}

// Backward of the narrow dense layer in one pass: data gradient, weight and bias gradient and their update.  Nothing but
// launch latency and one read of x bounds it (10 outputs on 512 features, batch 64: three generic launches of 7-13 us and the
// gradient's way through memory before).  A workgroup owns 64 input features, a lane one of them and a wave every fourth
// sample: the lane keeps the feature's weights and its N partial gradients in registers, the samples' dY rows come from LDS at
// a wave-uniform address.  The four waves' partial gradients are added in wave order, and since no other workgroup reads
// these features' weights, the update (buf = momentum*buf + g; w -= lr*buf) follows on the spot.
// The classifier of a network also forms its dY, the gradient of the softmax cross-entropy, a thread per sample: again in every
// workgroup, some 2 us where a launch of its own (softmax_ce_kernel) takes 6, and its reader waits for it.
template <int NMAX, typename T>
__global__ __launch_bounds__(256) void dense_small_bwd_kernel(DenseSmallParams p)
{
    constexpr int ROWS = 256;                     // samples staged at a time
    __shared__ __attribute__((aligned(16))) float sdy[ROWS][NMAX];
    __shared__ float red[4][64][NMAX + 1];
    __shared__ float losses[256];
    __shared__ float redb[4][NMAX];
    const int rep = p.order[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k0 = blockIdx.x * 64, k = k0 + lane;
    const bool on = k < p.K;
    const T* x = tptr<T>(p.x, rep, p.x_rep);
    const T* dy = tptr<T>(p.dy, rep, p.dy_rep);
    T* dx = tptr<T>(p.dx, rep, p.dx_rep);
    const T* mask = p.mask ? tptr<T>(p.mask, rep, p.mask_rep) : nullptr;
    float* const w = p.w + rep * p.w_rep;
    float* const buf = p.buf ? p.buf + rep * p.w_rep : nullptr;
    constexpr bool kRoundW = sizeof(T) == 2;
    float wv[NMAX], acc[NMAX], accb = 0.f;
#pragma unroll
    for (int n = 0; n < NMAX; ++n) {
        acc[n] = 0.f;
        wv[n] = on && n < p.N ? w[(long long)k * p.N + n] : 0.f;
        if (kRoundW) wv[n] = (float)(__bf16)wv[n];
    }
    // The weights to update and the first of a wave's rows of x are on their way while dY is formed.  (A row or feature beyond the last
    // is the last again.)
    constexpr int kRows = 8, kMine = 64 * NMAX / 256;
    const int cnt = min(64, p.K - k0) * p.N;
    const long long u0 = (long long)k0 * p.N;
    float wu[kMine], bu[kMine];
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const long long o = u0 + min((int)threadIdx.x + q * 256, cnt - 1);
        wu[q] = w[o];
        bu[q] = buf ? buf[o] : 0.f;
    }
    const int kc = min(k, p.K - 1);
    float xv[kRows], mv[kRows], old[kRows];
    auto load_rows = [&](int first) {                         // rows first + wave, first + wave + 4, ...
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            const long long o = (long long)min(first + wave + 4 * q, p.rows - 1) * p.K + kc;
            xv[q] = ldf(x, o);
            mv[q] = !mask ? 1.f : mask == x ? xv[q] : ldf(mask, o);
            old[q] = p.accumulate ? ldf(dx, o) : 0.f;
        }
    };
    load_rows(0);
    for (int r0 = 0; r0 < p.rows; r0 += ROWS) {
        const int nr = min(ROWS, p.rows - r0);
        __syncthreads();
        if (p.criterion.loss) {                   // (the launcher checks that there is one round, and n_classes = N)
            const LossParams& c = p.criterion;
            const int r = threadIdx.x;
            float li = 0.f;
            if (r < nr) {
                const long long first = ((c.cursor[rep] + c.ahead) * (long long)c.batch) % c.n_samples;
                const int label = c.y[(long long)rep * c.n_samples + first + r];
                const T* z = tptr<T>(c.logits, rep, c.logits_rep) + (long long)r * p.N;
                // as in softmax_ce_kernel, in registers
                float v[NMAX], m, sum = 0.f, own = 0.f;
#pragma unroll
                for (int n = 0; n < NMAX; ++n) v[n] = ldf(z, min(n, p.N - 1));
                m = v[0];
#pragma unroll
                for (int n = 1; n < NMAX; ++n) m = fmaxf(m, v[n]);           // (the last value again does not change it)
#pragma unroll
                for (int n = 0; n < NMAX; ++n) {
                    if (n == label) own = v[n];
                    v[n] = n < p.N ? expf(v[n] - m) : 0.f;
                    sum += v[n];
                }
                li = (logf(sum) + m - own) / (float)c.batch;
                const float inv = 1.0f / sum;
#pragma unroll
                for (int n = 0; n < NMAX; ++n)                               // rounded as it would be stored
                    sdy[r][n] = n < p.N ? (float)(T)((v[n] * inv - (n == label ? 1.f : 0.f)) / (float)c.batch) : 0.f;
            }
            losses[threadIdx.x] = li;
        } else {
            for (int i = threadIdx.x; i < nr * NMAX; i += 256) {
                const int r = i / NMAX, n = i % NMAX;
                sdy[r][n] = n < p.N ? ldf(dy, (long long)(r0 + r) * p.N + n) : 0.f;
            }
        }
        __syncthreads();
        for (int rb = 0; rb < nr; rb += 4 * kRows) {
            if (r0 + rb > 0) load_rows(r0 + rb);
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
                const int r = rb + wave + 4 * q;
                if (r >= nr) break;
                float g[NMAX], d = 0.f;
#pragma unroll
                for (int n = 0; n < NMAX; ++n) g[n] = sdy[r][n];
#pragma unroll
                for (int n = 0; n < NMAX; ++n) { d += g[n] * wv[n]; acc[n] += xv[q] * g[n]; }
                if (!(mv[q] > 0.f)) d = 0.f;
                if (p.accumulate) d += old[q];
                if (on) stf(dx, (long long)(r0 + r) * p.K + k, d);
            }
        }
        if (blockIdx.x == 0 && lane < NMAX)
            for (int r = wave; r < nr; r += 4) accb += sdy[r][lane];
    }
#pragma unroll
    for (int n = 0; n < NMAX; ++n) red[wave][lane][n] = acc[n];
    if (lane < NMAX) redb[wave][lane] = accb;
    __syncthreads();
    if (p.criterion.loss && blockIdx.x == 0) {    // (the order of softmax_ce_kernel)
        for (int i = 128; i > 0; i >>= 1) {
            if ((int)threadIdx.x < i) losses[threadIdx.x] += losses[threadIdx.x + i];
            __syncthreads();
        }
        if (threadIdx.x == 0) p.criterion.loss[rep] = losses[0];
    }
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const int i = threadIdx.x + q * 256, kk = i / p.N, n = i - kk * p.N;
        if (i >= cnt) break;
        float d = ((red[0][kk][n] + red[1][kk][n]) + red[2][kk][n]) + red[3][kk][n];
        if (buf) { d = bu[q] * p.momentum + d; buf[u0 + i] = d; }
        w[u0 + i] = wu[q] - d * p.lr;
    }
    if (blockIdx.x == 0 && p.has_bias && threadIdx.x < p.N) {
        const int n = threadIdx.x;
        float d = ((redb[0][n] + redb[1][n]) + redb[2][n]) + redb[3][n];
        const long long o = (long long)p.K * p.N + n;
        if (buf) { d = buf[o] * p.momentum + d; buf[o] = d; }
        w[o] -= d * p.lr;
    }
}

dim3 ew_grid(long long count, int n_active)
{
    long long b = (count + 255) / 256;
    if (b > 2048) b = 2048;
    if (b < 1) b = 1;
    return dim3((unsigned)b, (unsigned)n_active);
}

}  // namespace

#define HADFL_EW_LAUNCH(fn, kern) \
    hipError_t fn(const EwParams& p, int n_active, hipStream_t s) { \
        if (n_active < 1 || p.count < 1) return hipSuccess; \
        if (p.bf16) hipLaunchKernelGGL(kern<__bf16>, ew_grid(p.count, n_active), dim3(256), 0, s, p); \
        else hipLaunchKernelGGL(kern<float>, ew_grid(p.count, n_active), dim3(256), 0, s, p); \
        return hipGetLastError(); }
HADFL_EW_LAUNCH(launch_relu_fwd, relu_fwd_kernel)
HADFL_EW_LAUNCH(launch_relu_bwd, relu_bwd_kernel)
HADFL_EW_LAUNCH(launch_gap_fwd, gap_fwd_kernel)
HADFL_EW_LAUNCH(launch_gap_bwd, gap_bwd_kernel)
#undef HADFL_EW_LAUNCH

#define HADFL_EW_VEC_LAUNCH(fn, vkern, kern) \
    hipError_t fn(const EwParams& p, int n_active, hipStream_t s) { \
        if (n_active < 1 || p.count < 1) return hipSuccess; \
        const int vec = p.bf16 ? 8 : 4; \
        if (p.count % vec == 0) { \
            if (p.bf16) hipLaunchKernelGGL(vkern<__bf16>, ew_grid(p.count / vec, n_active), dim3(256), 0, s, p); \
            else hipLaunchKernelGGL(vkern<float>, ew_grid(p.count / vec, n_active), dim3(256), 0, s, p); \
        } else { \
            if (p.bf16) hipLaunchKernelGGL(kern<__bf16>, ew_grid(p.count, n_active), dim3(256), 0, s, p); \
            else hipLaunchKernelGGL(kern<float>, ew_grid(p.count, n_active), dim3(256), 0, s, p); \
        } \
        return hipGetLastError(); }
HADFL_EW_VEC_LAUNCH(launch_add_fwd, add_fwd_vec_kernel, add_fwd_kernel)
HADFL_EW_VEC_LAUNCH(launch_pass_grad, pass_grad_vec_kernel, pass_grad_kernel)

hipError_t launch_zero(const EwParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.count < 1) return hipSuccess;
    if (p.bf16) hipLaunchKernelGGL(zero_kernel<__bf16>, ew_grid(p.count, n_active), dim3(256), 0, s, p);
    else hipLaunchKernelGGL(zero_kernel<float>, ew_grid(p.count, n_active), dim3(256), 0, s, p);
    return hipGetLastError();
}
#undef HADFL_EW_VEC_LAUNCH

hipError_t launch_maxpool_fwd(const EwParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.count < 1) return hipSuccess;
    const int vec = p.bf16 ? 8 : 4;
    if (p.C % vec == 0) {
        if (p.bf16) hipLaunchKernelGGL(maxpool_fwd_vec_kernel<__bf16>, ew_grid(p.count / vec, n_active), dim3(256), 0, s, p);
        else hipLaunchKernelGGL(maxpool_fwd_vec_kernel<float>, ew_grid(p.count / vec, n_active), dim3(256), 0, s, p);
    } else {
        if (p.bf16) hipLaunchKernelGGL(maxpool_fwd_kernel<__bf16>, ew_grid(p.count, n_active), dim3(256), 0, s, p);
        else hipLaunchKernelGGL(maxpool_fwd_kernel<float>, ew_grid(p.count, n_active), dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_maxpool_bwd(const EwParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.count < 1) return hipSuccess;
    const int vec = p.bf16 ? 8 : 4;
    if (p.C % vec == 0) {
        if (p.bf16) hipLaunchKernelGGL(maxpool_bwd_vec_kernel<__bf16>, ew_grid(p.count / vec, n_active), dim3(256), 0, s, p);
        else hipLaunchKernelGGL(maxpool_bwd_vec_kernel<float>, ew_grid(p.count / vec, n_active), dim3(256), 0, s, p);
    } else {
        if (p.bf16) hipLaunchKernelGGL(maxpool_bwd_kernel<__bf16>, ew_grid(p.count, n_active), dim3(256), 0, s, p);
        else hipLaunchKernelGGL(maxpool_bwd_kernel<float>, ew_grid(p.count, n_active), dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_dense_small_fwd(const DenseSmallParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.rows < 1) return hipSuccess;
    if (p.bf16) hipLaunchKernelGGL((dense_small_fwd_kernel<16, __bf16>), dim3((unsigned)p.rows, (unsigned)n_active), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((dense_small_fwd_kernel<16, float>), dim3((unsigned)p.rows, (unsigned)n_active), dim3(256), 0, s, p);
    return hipGetLastError();
}

// Offsets of the rows of a workgroup from its first are 32-bit byte offsets, of floats at most, the last piece of the last row included.
bool dense_rows_supported(int rows, long long K) { return ((std::min(rows, 32) - 1) * K + 8) * 4 <= tiles::kOutside; }

hipError_t launch_dense_rows_fwd(const DenseRowsParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.rows < 1) return hipSuccess;
    if (!dense_rows_supported(p.rows, p.K)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((p.rows + 31) / 32), (unsigned)((p.N + 31) / 32), (unsigned)n_active), block(1024);
    if (!p.bf16) hipLaunchKernelGGL((dense_rows_fwd_kernel<float, float>), grid, block, 0, s, p);
    else if (p.cursor) hipLaunchKernelGGL((dense_rows_fwd_kernel<__bf16, float>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((dense_rows_fwd_kernel<__bf16, __bf16>), grid, block, 0, s, p);
    return hipGetLastError();
}

hipError_t launch_dense_small_bwd(const DenseSmallParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.rows < 1) return hipSuccess;
    if (p.N > 16 || (p.criterion.loss && (p.rows > 256 || p.criterion.batch != p.rows || p.criterion.n_classes != p.N))) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((p.K + 63) / 64), (unsigned)n_active);
    if (p.bf16) hipLaunchKernelGGL((dense_small_bwd_kernel<16, __bf16>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((dense_small_bwd_kernel<16, float>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

namespace {
// channel vectors per workgroup: the largest power of two that is at most min(C / vec, 32)
int bn_cvb(int C, int vec) { int cv = C / vec, b = 1; while (b * 2 <= cv && b * 2 <= 32) b *= 2; return b; }
// One launch for the whole layer: as many rows as a workgroup's registers hold, and a tensor that the few workgroups can move in that time
bool bn_small(const BnParams& p, int n_active) { return !p.pool && p.rows <= kBnSmallRows * (kBnSmallThreads / kBnSmallCvb) && (long long)p.rows * p.C * n_active <= (1 << 20); }
dim3 bn_small_grid(BnParams& p, int vec, int n_active)
{
    p.cvb = std::min(kBnSmallCvb, bn_cvb(p.C, vec));
    return dim3((unsigned)((p.C / vec + p.cvb - 1) / p.cvb), (unsigned)n_active);
}
}  // namespace

bool bn_backward_in_one_launch(const BnParams& p, int n_active) { return p.C % (p.bf16 ? 8 : 4) == 0 && bn_small(p, n_active); }

// Sums with few entries are added by the apply kernel's workgroups, each for its own channels, in place of a launch.  Finalize and apply, us, with
// that launch and folded: 512 channels on 1024 rows (8 to 32 entries), fp32, 3 / 8 / 16 replicas forward 16 18 23 and 13 14 18, backward 13
// 17 23 and 10 13 19; 256 channels on 4096 rows (16 to 64 entries) 19 25 37 and 13 21 33, 16 24 40 and 11 20 35.  Beyond some 64 entries,
// or 64 MB that all workgroups read together, the launch is the shorter way (bf16, 128 channels on 32768 rows, 128 entries, 7 / 32
// replicas forward 18 59 and 19 71).  With a max-pool folded in the same: a network of 13 such layers, five with a pool, three of
// those below the limit, fp32, 4 replicas 7.52 -> 7.44 ms.
namespace {
constexpr int kFoldEntries = 64;
constexpr long long kFoldBytes = 64 << 20;
bool bn_folds(const BnParams& p, int vec, int entries, long long workgroups) { return entries <= kFoldEntries && workgroups * entries * 2 * p.cvb * vec * 4 <= kFoldBytes; }

// (finalize and) apply kernels
template <typename T> void bn_apply_fwd(const BnParams& p, bool fold, dim3 grid, dim3 fgrid, hipStream_t s)
{
    const dim3 block(256);
    if (!fold) hipLaunchKernelGGL((bn_finalize_kernel<0, T>), fgrid, block, 0, s, p);
    if (p.pool && fold) hipLaunchKernelGGL((bn_apply_fwd_pool_vec_kernel<T, true>), grid, block, 0, s, p);
    else if (p.pool) hipLaunchKernelGGL((bn_apply_fwd_pool_vec_kernel<T, false>), grid, block, 0, s, p);
    else if (fold) hipLaunchKernelGGL((bn_apply_fwd_vec_kernel<T, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((bn_apply_fwd_vec_kernel<T, false>), grid, block, 0, s, p);
}
template <typename T> void bn_apply_bwd(const BnParams& p, bool fold, dim3 grid, dim3 fgrid, hipStream_t s)
{
    const dim3 block(256);
    if (!fold) hipLaunchKernelGGL((bn_finalize_kernel<1, T>), fgrid, block, 0, s, p);
    if (p.pool && fold) hipLaunchKernelGGL((bn_apply_bwd_pool_vec_kernel<T, true>), grid, block, 0, s, p);
    else if (p.pool) hipLaunchKernelGGL((bn_apply_bwd_pool_vec_kernel<T, false>), grid, block, 0, s, p);
    else if (fold) hipLaunchKernelGGL((bn_apply_bwd_vec_kernel<T, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((bn_apply_bwd_vec_kernel<T, false>), grid, block, 0, s, p);
}
}  // namespace

hipError_t launch_bn_fwd(const BnParams& p0, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    BnParams p = p0;
    const int vec = p.bf16 ? 8 : 4;
    const dim3 block(256);
    if (p.C % vec == 0 && bn_small(p, n_active)) {
        const dim3 grid = bn_small_grid(p, vec, n_active);
        if (p.bf16) hipLaunchKernelGGL(bn_small_fwd_kernel<__bf16>, grid, dim3(kBnSmallThreads), 0, s, p);
        else hipLaunchKernelGGL(bn_small_fwd_kernel<float>, grid, dim3(kBnSmallThreads), 0, s, p);
        return hipGetLastError();
    }
    if (p.C % vec == 0) {
        p.cvb = bn_cvb(p.C, vec);
        const int cgroups = (p.C / vec + p.cvb - 1) / p.cvb;
        const dim3 grid((unsigned)(p.chunks * cgroups), (unsigned)n_active), fgrid((unsigned)((p.C + 31) / 32), (unsigned)n_active);
        if (p.pool && (p.H % 2 != 0 || p.W % 2 != 0 || p.rows % 4 != 0 || !p.pool_out)) return hipErrorInvalidValue;
        const bool fold = bn_folds(p, vec, p.stats_done ? p.stat_entries : p.chunks, (long long)grid.x * n_active);
        if (p.bf16) {
            if (!p.stats_done) hipLaunchKernelGGL((bn_sums_vec_kernel<0, __bf16>), grid, block, 0, s, p);
            bn_apply_fwd<__bf16>(p, fold, grid, fgrid, s);
        } else {
            if (!p.stats_done) hipLaunchKernelGGL((bn_sums_vec_kernel<0, float>), grid, block, 0, s, p);
            bn_apply_fwd<float>(p, fold, grid, fgrid, s);
        }
        return hipGetLastError();
    }
    if (p.pool || p.stats_done || p.add || p.left_out) return hipErrorInvalidValue;  // the caller asks for these only where the vector kernels apply
    const dim3 grid((unsigned)(p.chunks * ((p.C + 63) / 64)), (unsigned)n_active);
    if (p.bf16) {
        hipLaunchKernelGGL((bn_reduce_kernel<0, __bf16>), grid, block, 0, s, p);
        hipLaunchKernelGGL((bn_reduce_kernel<1, __bf16>), grid, block, 0, s, p);
        hipLaunchKernelGGL(bn_apply_fwd_kernel<__bf16>, grid, block, 0, s, p);
    } else {
        hipLaunchKernelGGL((bn_reduce_kernel<0, float>), grid, block, 0, s, p);
        hipLaunchKernelGGL((bn_reduce_kernel<1, float>), grid, block, 0, s, p);
        hipLaunchKernelGGL(bn_apply_fwd_kernel<float>, grid, block, 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_bn_bwd(const BnParams& p0, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    BnParams p = p0;
    const int vec = p.bf16 ? 8 : 4;
    const dim3 block(256);
    if (p.C % vec == 0 && !p.bwd_stats_done && bn_small(p, n_active)) {
        const dim3 grid = bn_small_grid(p, vec, n_active);
        if (p.bf16) hipLaunchKernelGGL(bn_small_bwd_kernel<__bf16>, grid, dim3(kBnSmallThreads), 0, s, p);
        else hipLaunchKernelGGL(bn_small_bwd_kernel<float>, grid, dim3(kBnSmallThreads), 0, s, p);
        return hipGetLastError();
    }
    if (p.C % vec == 0) {
        p.cvb = bn_cvb(p.C, vec);
        const int cgroups = (p.C / vec + p.cvb - 1) / p.cvb;
        const dim3 grid((unsigned)(p.chunks * cgroups), (unsigned)n_active), fgrid((unsigned)((p.C + 31) / 32), (unsigned)n_active);
        if (p.pool && (p.H % 2 != 0 || p.W % 2 != 0 || p.rows % 4 != 0 || !p.pool_g)) return hipErrorInvalidValue;
        if (p.pool && p.bwd_stats_done == 2) return hipErrorInvalidValue;
        // (sums of the stored output need the finalize kernel's second look at the scales)
        const bool fold = p.bwd_stats_done != 1 && bn_folds(p, vec, p.bwd_stats_done ? p.stat_entries : p.chunks, (long long)grid.x * n_active);
        if (p.bf16) {
            if (p.bwd_stats_done) {}                                  // the data gradient above left the sums
            else if (p.pool) hipLaunchKernelGGL(bn_sums_pool_vec_kernel<__bf16>, grid, block, 0, s, p);
            else hipLaunchKernelGGL((bn_sums_vec_kernel<1, __bf16>), grid, block, 0, s, p);
            bn_apply_bwd<__bf16>(p, fold, grid, fgrid, s);
        } else {
            if (p.bwd_stats_done == 1) return hipErrorInvalidValue;  // (of the stored output: only the bf16 data-gradient kernels leave those)
            if (p.bwd_stats_done) {}
            else if (p.pool) hipLaunchKernelGGL(bn_sums_pool_vec_kernel<float>, grid, block, 0, s, p);
            else hipLaunchKernelGGL((bn_sums_vec_kernel<1, float>), grid, block, 0, s, p);
            bn_apply_bwd<float>(p, fold, grid, fgrid, s);
        }
        return hipGetLastError();
    }
    if (p.pool || p.bwd_stats_done) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(p.chunks * ((p.C + 63) / 64)), (unsigned)n_active);
    if (p.bf16) {
        hipLaunchKernelGGL((bn_reduce_kernel<2, __bf16>), grid, block, 0, s, p);
        hipLaunchKernelGGL(bn_apply_bwd_kernel<__bf16>, grid, block, 0, s, p);
    } else {
        hipLaunchKernelGGL((bn_reduce_kernel<2, float>), grid, block, 0, s, p);
        hipLaunchKernelGGL(bn_apply_bwd_kernel<float>, grid, block, 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_softmax_ce(const LossParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    int threads = 64;
    while (threads < p.batch) threads *= 2;      // power of two for the tree; batch <= 1024 is checked at init
    if (p.bf16) hipLaunchKernelGGL(softmax_ce_kernel<__bf16>, dim3((unsigned)n_active), dim3((unsigned)threads), 0, s, p);
    else hipLaunchKernelGGL(softmax_ce_kernel<float>, dim3((unsigned)n_active), dim3((unsigned)threads), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_sgd(const SgdParams& p, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    if (p.n_seg < 0 || p.n_seg > kMaxSgdSegments) return hipErrorInvalidValue;
    long long n4 = 0;
    for (int k = 0; k < p.n_seg; ++k) {
        if (p.count[k] % 4 != 0 || p.first[k] % 4 != 0 || p.count[k] < 0) return hipErrorInvalidValue;
        n4 += p.count[k] / 4;
    }
    if (n4 < 1) return hipSuccess;
    hipLaunchKernelGGL(sgd_kernel, ew_grid(n4, n_active), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_advance(const int* steps, int* versions, long long* cursor, int n, hipStream_t s)
{
    hipLaunchKernelGGL(advance_kernel, dim3((unsigned)std::min((n + 255) / 256, 64)), dim3(256), 0, s, steps, versions, cursor, n);
    return hipGetLastError();
}

}  // namespace hadfl
