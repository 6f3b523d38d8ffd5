// Networks of two dense layers (data set -> hidden, ReLU -> classes): the end of one local step and the beginning of the next in
// one launch (paper Sec. 2.1, Sec. 2.2).
//
// Layer by layer a step of such a network is four dependent launches of 5 to 10 us that compute for one or two.  A workgroup
// here owns sixteen hidden units of a replica through the whole step: their column of the first layer's weights and row of
// the second's are read and updated by nobody else, so all that the workgroups of a replica have to exchange are their shares of
// the logits.  The kernel boundary is that exchange, through two buffers that steps take in turn: a launch reads the shares that the one before
// it wrote, of all workgroups of a replica, and writes its own for the next where none of this launch reads, since nothing orders its workgroups:
//   end of a step     logits = sum of the shares; loss and its gradient; the gradient of the own hidden units; both weight
//                     gradients and their updates;
//   begin of a step   the own hidden units of the next batch, from the weights just updated, still in registers; their share of
//                     the logits.
// Eight waves share the contraction over the input features, sixteen at a time: wave w takes blocks w, w + 8, ...  The
// accumulator of a weight gradient (four features of one unit a lane) is after its update the operand of the next forward
// product as it lies: instruction v of a block multiplies features 4 g + v of the four lane groups g.
// Arithmetic as in the kernels of the single layers: the forward product on the fp32 matrix instruction (bf16: of rounded operands),
// the weight gradient on split floats (conv_general.hip; bf16: on the operands as they are), with the same second pass on
// the fp32 instruction where a block's result is not finite.
// What bounds it: a chain of dependent steps (shares of the logits from the L2, loss, gradient, product, product, sums over the waves through
// LDS), with both batches of rows and the weights on their way from the start; beyond 64 samples the rows, which every
// workgroup reads for itself (some 7 us per 32 samples).  784 features, 128 hidden units, batch 32, 4 replicas: 19 us a step, 30 layer by
// layer (other sizes: dense_pair_net); four replicas of 1, 2, 3 and 4 steps with selection and aggregate 128 -> 78 us.
#include "train_kernels.h"
#include "mfma_tiles.h"
#include "slabs.h"

namespace hadfl {
namespace {

using namespace tiles;

constexpr int kUnits = 16, kWaves = 8, kThreads = 64 * kWaves, kBlocks = 8;    // kBlocks: blocks of sixteen features per wave
constexpr int kMaxRows = 128, kMaxClasses = 16;
constexpr int kPitch = 2 * kMaxRows + 16;                  // bytes of a unit's gradients in one plane

__device__ __forceinline__ float ld32(Buffer b, unsigned off) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, 0)); }

template <typename T>
__global__ __launch_bounds__(kThreads, 2) void dense_pair_kernel(DensePairParams p)
{
    constexpr bool kSplit = sizeof(T) == 4;
    constexpr int PL = kSplit ? 3 : 1;
    __shared__ __attribute__((aligned(16))) char s_planes[PL][kUnits][kPitch];      // gradient of the hidden units, in parts
    __shared__ float s_d[kMaxRows][kUnits + 1];            // the same as floats
    __shared__ float s_h[kMaxRows][kUnits + 1], s_dy[kMaxRows][kMaxClasses + 1];
    __shared__ float s_w2[kUnits][kMaxClasses + 1], s_b1[kUnits], s_b2[kMaxClasses];
    __shared__ float s_red[kWaves][2][4][64];
    const int J = p.H / kUnits;
    const unsigned item = logical_block();
    if (item >= (unsigned)(J * max(p.n_end, p.n_begin))) return;
    const int slot = (int)item / J, j = (int)item - slot * J, rep = p.order[slot];
    const bool ends = slot < p.n_end, begins = slot < p.n_begin;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4, B = p.batch, u0 = j * kUnits;
    const int blocks = p.K / 16;
    float* const w1 = p.w1 + rep * p.w_rep;
    float* const w2 = p.w2 + rep * p.w_rep;
    float* const m1 = p.m1 ? p.m1 + rep * p.w_rep : nullptr;
    float* const m2 = p.m2 ? p.m2 + rep * p.w_rep : nullptr;
    T* const hidden = reinterpret_cast<T*>(p.hidden + rep * p.act_rep) + u0;
    const float* const share_in = p.share_in + rep * p.act_rep;
    float* const share_out = p.share_out + rep * p.act_rep;
    const long long bias1 = (long long)p.K * p.H + u0, bias2 = (long long)p.H * p.N;

    // the own weights: 16 features x 16 units a block
    float w[kBlocks][4], m[kBlocks][4];
    const unsigned wofs = (unsigned)((4 * g) * p.H + u0 + c);
#pragma unroll
    for (int u = 0; u < kBlocks; ++u) {
        const int t = wave + kWaves * u;
        if (t >= blocks) break;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const unsigned o = wofs + (unsigned)((16 * t + v) * p.H);
            w[u][v] = w1[o];
            m[u][v] = ends && m1 ? m1[o] : 0.f;
        }
    }
    // thread 256 + 16 a + n: unit a, class n of the second layer
    const int a2 = (tid & 255) >> 4, n2 = tid & 15;
    const bool own2 = tid >= 256 && n2 < p.N;
    const long long o2 = (long long)(u0 + a2) * p.N + n2;
    float w2v = own2 ? w2[o2] : 0.f;
    if (tid >= 256) s_w2[a2][n2] = kSplit ? w2v : (float)(__bf16)w2v;
    if (tid < kUnits) s_b1[tid] = p.has_bias1 ? w1[bias1 + tid] : 0.f;
    if (tid < kMaxClasses) s_b2[tid] = p.has_bias2 && j == 0 && tid < p.N ? w2[bias2 + tid] : 0.f;      // (the first workgroup's alone, which updates it)
    // the rows of the step that ends and of the one that begins (n_samples is a multiple of the batch)
    long long row = ((p.cursor[rep] + p.ahead - (ends ? 1 : 0)) * (long long)B) % p.n_samples;
    const float* const data = p.x + (long long)rep * p.n_samples * p.K;

    if (ends) {
        const Buffer xb = buffer(data + row * p.K, (unsigned)(B * p.K) * 4u);
        f4 x[kBlocks][2];                                  // 16 features x 32 samples a block: feature c, samples 8 g ... 8 g + 7
        auto load_rows = [&](int u, int r0) {              // (zeros beyond the batch)
#pragma unroll
            for (int e = 0; e < 8; ++e) x[u][e >> 2][e & 3] = ld32(xb, (unsigned)((r0 + 8 * g + e) * p.K + 16 * (wave + kWaves * u) + c) * 4u);
        };
#pragma unroll
        for (int u = 0; u < kBlocks; ++u) {                // on their way while the gradient of the loss is formed
            if (wave + kWaves * u >= blocks) break;
            load_rows(u, 0);
        }
        const int label = tid < B ? p.y[(long long)rep * p.n_samples + row + tid] : 0;
        for (int i = tid; i < B * kUnits; i += kThreads) {
            const int r = i >> 4, n = i & 15;
            float z = 0.f;
            for (int q = 0; q < J; ++q) z += share_in[(q * B + r) * 16 + n];
            s_dy[r][n] = (float)(T)z;                      // the logits as they would be stored
            s_h[r][n] = (float)hidden[(long long)r * p.H + n];
        }
        __syncthreads();
        float li = 0.f;
        if (tid < B) {                                     // as in dense_small_bwd_kernel
            float v[kMaxClasses], top, sum = 0.f, own = 0.f;
#pragma unroll
            for (int n = 0; n < kMaxClasses; ++n) v[n] = s_dy[tid][min(n, p.N - 1)];
            top = v[0];
#pragma unroll
            for (int n = 1; n < kMaxClasses; ++n) top = fmaxf(top, v[n]);
#pragma unroll
            for (int n = 0; n < kMaxClasses; ++n) {
                if (n == label) own = v[n];
                v[n] = n < p.N ? expf(v[n] - top) : 0.f;
                sum += v[n];
            }
            li = (logf(sum) + top - own) / (float)B;
            const float inv = 1.0f / sum;
#pragma unroll
            for (int n = 0; n < kMaxClasses; ++n) s_dy[tid][n] = n < p.N ? (float)(T)((v[n] * inv - (n == label ? 1.f : 0.f)) / (float)B) : 0.f;
        }
        float* const losses = &s_red[0][0][0][0];
        if (tid < 256) losses[tid] = li;
        __syncthreads();
        if (j == 0) {                                      // (the order of softmax_ce_kernel)
            for (int i = 128; i > 0; i >>= 1) {
                if (tid < i) losses[tid] += losses[tid + i];
                __syncthreads();
            }
            if (tid == 0) p.loss[rep] = losses[0];
        }
        // gradient of the own hidden units (zeros in the rows that fill the last 32)
        for (int i = tid; i < (B + 31) / 32 * 32 * kUnits; i += kThreads) {
            const int r = i >> 4, a = i & 15;
            float d = 0.f;
            if (r < B) {
#pragma unroll
                for (int n = 0; n < kMaxClasses; ++n) d += s_dy[r][n] * s_w2[a][n];
                if (!(s_h[r][a] > 0.f)) d = 0.f;
            }
            if constexpr (kSplit) {
                __bf16 q[3];
                float y = d * kSplitScale;
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    q[s] = (__bf16)y;
                    y -= (float)q[s];
                    *reinterpret_cast<__bf16*>(&s_planes[s][a][2 * r]) = q[s];
                }
                s_d[r][a] = d;
            } else {
                *reinterpret_cast<__bf16*>(&s_planes[0][a][2 * r]) = (__bf16)d;
                s_d[r][a] = (float)(__bf16)d;
            }
        }
        __syncthreads();
        // second layer and the biases: four chains of samples, as in dense_small_bwd_kernel
        auto update = [&](float grad, float& wv, float* mv) {
            if (mv) { grad = *mv * p.momentum + grad; *mv = grad; }
            wv = wv - grad * p.lr;
        };
        if (tid >= 256) {
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            for (int r = 0; r < B; r += 4)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r + q < B) s[q] += s_h[r + q][a2] * s_dy[r + q][n2];
            if (own2) {
                update(((s[0] + s[1]) + s[2]) + s[3], w2v, m2 ? m2 + o2 : nullptr);
                w2[o2] = w2v;
                s_w2[a2][n2] = kSplit ? w2v : (float)(__bf16)w2v;
            }
        } else if (wave >= 2 && lane < 16) {               // wave 3: bias of the own hidden units; wave 2 of the first workgroup: of the classes
            const float (*const src)[17] = wave == 3 ? s_d : s_dy;
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            for (int r = 0; r < B; r += 4)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (r + q < B) s[q] += src[r + q][lane];
            const float grad = ((s[0] + s[1]) + s[2]) + s[3];
            if (wave == 3 && p.has_bias1) {
                float b = s_b1[lane];
                update(grad, b, m1 ? m1 + bias1 + lane : nullptr);
                w1[bias1 + lane] = b; s_b1[lane] = b;
            } else if (wave == 2 && p.has_bias2 && j == 0 && lane < p.N) {
                float b = s_b2[lane];
                update(grad, b, m2 ? m2 + bias2 + lane : nullptr);
                w2[bias2 + lane] = b; s_b2[lane] = b;
            }
        }
        // first layer
        f4 acc[kBlocks], low[kSplit ? kBlocks : 1];
#pragma unroll
        for (int u = 0; u < kBlocks; ++u) {
            acc[u] = f4{0.f, 0.f, 0.f, 0.f};
            if constexpr (kSplit) low[u] = acc[u];
        }
        for (int r0 = 0; r0 < B; r0 += 32) {
            bf16x8 d[PL];
#pragma unroll
            for (int s = 0; s < PL; ++s) d[s] = *reinterpret_cast<const bf16x8*>(&s_planes[s][c][2 * (r0 + 8 * g)]);
#pragma unroll
            for (int u = 0; u < kBlocks; ++u) {
                if (wave + kWaves * u >= blocks) break;
                if constexpr (kSplit) {
                    u2 h0, q0, l0, h1, q1, l1;
                    split3(x[u][0], h0, q0, l0);
                    split3(x[u][1], h1, q1, l1);
                    const bf16x8 a[3] = {__builtin_bit_cast(bf16x8, join8(h0, h1)), __builtin_bit_cast(bf16x8, join8(q0, q1)), __builtin_bit_cast(bf16x8, join8(l0, l1))};
                    constexpr int SA[5] = {0, 2, 1, 0, 1}, SB[5] = {2, 0, 1, 1, 0};
#pragma unroll
                    for (int s = 0; s < 5; ++s) low[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[SA[s]], d[SB[s]], low[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], d[0], acc[u], 0, 0, 0);
                } else {
                    bf16x8 a;
#pragma unroll
                    for (int e = 0; e < 8; ++e) a[e] = (__bf16)x[u][e >> 2][e & 3];
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, d[0], acc[u], 0, 0, 0);
                }
                if (r0 + 32 < B) load_rows(u, r0 + 32);
            }
        }
#pragma unroll
        for (int u = 0; u < kBlocks; ++u) {
            const int t = wave + kWaves * u;
            if (t >= blocks) break;
            if constexpr (kSplit) {
                float bad = 0.f;
                acc[u] = (acc[u] + low[u]) * kProductScale;
#pragma unroll
                for (int v = 0; v < 4; ++v) bad = __builtin_fmaf(acc[u][v], 0.f, bad);
                if (__ballot(bad != 0.f)) {                // (NaN != 0) something is not finite: the block again, with the fp32 instruction
                    acc[u] = f4{0.f, 0.f, 0.f, 0.f};
                    for (int r = g; r < (B + 3) / 4 * 4; r += 4)
                        acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ld32(xb, (unsigned)(r * p.K + 16 * t + c) * 4u), r < B ? s_d[r][c] : 0.f, acc[u], 0, 0, 0);
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const unsigned o = wofs + (unsigned)((16 * t + v) * p.H);
                float d = acc[u][v];
                if (m1) { d = m[u][v] * p.momentum + d; m1[o] = d; }
                w[u][v] = w[u][v] - d * p.lr;
                w1[o] = w[u][v];
            }
        }
        row += B;
        if (row >= p.n_samples) row -= p.n_samples;
    }
    if (!begins) return;

    const Buffer xb = buffer(data + row * p.K, (unsigned)(B * p.K) * 4u);
    f4 x[kBlocks][2];                                      // samples c and 16 + c of 32, features 4 g ... 4 g + 3 of a block
    auto load_rows = [&](int u, int r0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) x[u][q] = __builtin_bit_cast(f4, ldb16(xb, (unsigned)((r0 + 16 * q + c) * p.K + 16 * (wave + kWaves * u) + 4 * g) * 4u));
    };
#pragma unroll
    for (int u = 0; u < kBlocks; ++u) {
        if (wave + kWaves * u >= blocks) break;
        load_rows(u, 0);
    }
    for (int r0 = 0; r0 < B; r0 += 32) {
        f4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int u = 0; u < kBlocks; ++u) {
            if (wave + kWaves * u >= blocks) break;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(kSplit ? x[u][q][v] : (float)(__bf16)x[u][q][v], kSplit ? w[u][v] : (float)(__bf16)w[u][v], acc[q], 0, 0, 0);
            if (r0 + 32 < B) load_rows(u, r0 + 32);
        }
        __syncthreads();                                   // s_red has been read
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) s_red[wave][q][v][lane] = acc[q][v];
        __syncthreads();
        const int r = tid >> 4, n = tid & 15;              // row of the 32, unit (class)
        float h = s_red[0][r >> 4][r & 3][((r & 15) >> 2) * 16 + n];
#pragma unroll
        for (int k = 1; k < kWaves; ++k) h += s_red[k][r >> 4][r & 3][((r & 15) >> 2) * 16 + n];
        h = (float)(T)fmaxf(h + s_b1[n], 0.f);
        s_h[r0 + r][n] = h;
        if (r0 + r < B) hidden[(long long)(r0 + r) * p.H + n] = (T)h;
        __syncthreads();
        float z = j == 0 ? s_b2[n] : 0.f;
#pragma unroll
        for (int k = 0; k < kUnits; ++k) z += s_h[r0 + r][k] * s_w2[k][n];
        if (r0 + r < B) share_out[(j * B + r0 + r) * 16 + n] = z;
    }
}

}  // namespace

// Offsets inside a replica's weights and batch are 32-bit.
bool dense_pair_supported(int batch, int K, int H, int N)
{
    return batch <= kMaxRows && K % 16 == 0 && K <= 16 * kWaves * kBlocks && H % kUnits == 0 && H <= 4096 && N <= kMaxClasses;
}

hipError_t launch_dense_pair(const DensePairParams& p, hipStream_t s)
{
    const int n = p.n_end > p.n_begin ? p.n_end : p.n_begin;
    if (n < 1) return hipSuccess;
    if (p.batch < 1 || p.N < 1 || p.K < 16 || p.H < kUnits || !dense_pair_supported(p.batch, p.K, p.H, p.N) || p.n_samples % p.batch != 0) return hipErrorInvalidValue;
    if (p.n_end > 0 && p.n_begin > 0 && p.share_in == p.share_out) return hipErrorInvalidValue;
    const dim3 grid(die_grid((long long)n * (p.H / kUnits)));
    if (p.bf16) hipLaunchKernelGGL((dense_pair_kernel<__bf16>), grid, dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL((dense_pair_kernel<float>), grid, dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace hadfl
