// fp32 stride-1 "same" convolutions whose sums run along K in one chain (paper Sec. 2.1), forward and data gradient: the sums of gemm.hip,
// product by product in the same order on the same instruction, v_mfma_f32_32x32x2_f32, and so the same bits.
//
// igemm_kernel fetches an activation once per tap, sixteen channels at a time, one slab ahead of the matrix cores: a workgroup
// alone on its compute unit takes 3400 clocks for the 1024 that a slab's matrix instructions need.  Here a workgroup loads all channels of
// its tile's pixels and of the border around it once; pixels stay in memory order, so a tap is a row offset into that patch
// (a tap outside the image reads a row of zeros: its products are formed, as there).  What is left in the loop is the weights, read as they lie
// in the master, two groups of sixteen k ahead.  Rows of C + 2 floats: two lanes of a wave never meet in a bank.
// What bounds it: the matrix cores (31 us of the 57 below at their rate), and the patch and the stores of all workgroups at once before
// and behind them.  Images of 16 x 16, batch 64, 2 / 4 / 6 / 8 replicas, us, igemm_kernel and this: 32 to 64 channels forward 29 42 53 66 and 21
// 33 45 57, 64 to 32 channels data gradient 36 47 59 72 and 25 37 54 58.
//
// Convolutions on the data set whose footprint R S C fits 32 (igemm_chain_first_kernel): a lane gathers its pixel's values of every second k
// straight into the operand, the next tile's while the present one is multiplied; the weights stay in registers for all tiles of a
// wave.  Nothing passes through LDS.  3 to 32 channels, images of 32 x 32, batch 64: 20 34 44 58 and 12
// 18 25 31 (stores of 67 MB: 14).
#include "train_kernels.h"
#include "mfma_tiles.h"

namespace hadfl {
namespace {

using namespace tiles;

// (kOutside: zero, and nothing stored; a branch around an access would wait for all before it)
__device__ __forceinline__ float ld32(Buffer b, unsigned off) { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, 0)); }
__device__ __forceinline__ void st32(Buffer b, unsigned off, float v) { __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, (int)off, 0, 0); }

// WM x WN waves of 32 TM pixels x 32 outputs each.  Lane: column lane & 31, rows 8 (v / 4) + 4 (lane / 32) + v % 4 of a block.
template <int TM, int WM, int WN, bool DGRAD>
__global__ __launch_bounds__(64 * WM * WN) void igemm_chain_kernel(GemmParams p)
{
    constexpr int NT = 64 * WM * WN, BM = 32 * TM * WM, BN = 32 * WN, AHEAD = 2;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN, half = lane >> 5;
    const unsigned tiles = (unsigned)(p.tiles_m * p.tiles_n), item = logical_block();
    if (item >= tiles * (unsigned)p.n_active) return;
    const int rep = p.order[item / tiles];
    const int m0 = (int)(item % tiles) / p.tiles_n * BM, n0 = (int)(item % tiles) % p.tiles_n * BN;
    const int C = DGRAD ? p.Cout : p.Cin, N = DGRAD ? p.Cin : p.Cout;     // channels of the source, outputs
    const int hw = p.H * p.W, M = p.B * hw, halo = p.pad * (p.W + 1), rows = BM + 2 * halo, pitch = C + 2, taps = p.R * p.S;
    const float* const w = p.w + (long long)rep * p.w_rep;

    // weights: step j of a group of sixteen k has k = 2 j + half of it
    const int n = n0 + wn * 32 + (lane & 31), nc = n < N ? n : N - 1;      // (columns beyond the last: the last again, never stored)
    float b[AHEAD][8];
    int f_tap = 0, f_c = 0;                                               // the group that is fetched next
    auto fetch = [&](int d) {
        if constexpr (DGRAD) {
            const float* const src = w + ((long long)f_tap * N + nc) * C + f_c;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f4 v = *reinterpret_cast<const f4*>(src + 4 * q);
                b[d][2 * q] = half ? v[1] : v[0];
                b[d][2 * q + 1] = half ? v[3] : v[2];
            }
        } else {
            const float* const src = w + ((long long)f_tap * C + f_c + half) * N + nc;
#pragma unroll
            for (int j = 0; j < 8; ++j) b[d][j] = src[2 * j * N];
        }
        f_c += 16;
        if (f_c == C) { f_c = 0; f_tap = f_tap + 1 < taps ? f_tap + 1 : 0; }      // (beyond the last group: the first ones again, not used)
    };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) fetch(d);

    {   // the patch: rows m0 - halo ... of the source, zeros outside the batch, and a row of zeros behind them
        const Buffer src = buffer(p.a + (long long)rep * p.a_rep, (unsigned)M * (unsigned)C * 4u);
        const int per = C / 4, total = rows * per;
        constexpr int kLoads = 8;
        for (int i0 = tid; i0 < total; i0 += NT * kLoads) {
            u4 v[kLoads];
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const int i = i0 + q * NT, r = i / per;
                const int m = m0 - halo + r;
                v[q] = ldb16(src, i < total && m >= 0 && m < M ? (unsigned)(m * C + (i - r * per) * 4) * 4u : kOutside);
            }
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const int i = i0 + q * NT, r = i / per;
                if (i >= total) break;
                float* const o = smem + r * pitch + (i - r * per) * 4;
                *reinterpret_cast<u2*>(o) = u2{v[q][0], v[q][1]};
                *reinterpret_cast<u2*>(o + 2) = u2{v[q][2], v[q][3]};
            }
        }
        for (int i = tid; i < pitch; i += NT) smem[rows * pitch + i] = 0.f;
    }
    int rd[TM]; unsigned inside[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int lr = (wm * TM + i) * 32 + (lane & 31), m = m0 + lr, pos = m % hw, y = pos / p.W, x = pos - y * p.W;
        rd[i] = (lr + halo) * pitch + half;
        inside[i] = 0;
        for (int t = 0; t < taps; ++t) {
            const int r = t / p.S, s = t - r * p.S, yy = DGRAD ? y + p.pad - r : y + r - p.pad, xx = DGRAD ? x + p.pad - s : x + s - p.pad;
            if (m < M && yy >= 0 && yy < p.H && xx >= 0 && xx < p.W) inside[i] |= 1u << t;
        }
    }
    f16 acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    __syncthreads();

    int tap = 0, c = 0, at[TM];
    auto aim = [&]() {
        const int r = tap / p.S, s = tap - r * p.S, shift = ((r - p.pad) * p.W + s - p.pad) * pitch;
#pragma unroll
        for (int i = 0; i < TM; ++i) at[i] = tap < taps && (inside[i] >> tap) & 1u ? rd[i] + (DGRAD ? -shift : shift) : rows * pitch + half;
    };
    aim();
    const int groups = taps * (C / 16);
    auto multiply = [&](int d) {
        float a[TM][8];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) a[i][j] = smem[at[i] + c + 2 * j];
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][j], b[d][j], acc[i], 0, 0, 0);
        fetch(d);
        c += 16;
        if (c == C) { c = 0; ++tap; aim(); }
    };
    for (int g = groups / AHEAD; g > 0; --g)
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) multiply(d);
#pragma unroll
    for (int d = 0; d < AHEAD - 1; ++d)
        if (d < groups % AHEAD) multiply(d);

    const Buffer out = buffer(p.out + (long long)rep * p.out_rep, (unsigned)M * (unsigned)N * 4u);
    const Buffer mask = buffer(DGRAD && p.mask ? p.mask + (long long)rep * p.mask_rep : p.out, (unsigned)M * (unsigned)N * 4u);
    const float bv = !DGRAD && p.has_bias ? w[(long long)p.K * N + nc] : 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        unsigned o[16]; float mk[16], old[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + (wm * TM + i) * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
            o[v] = m < M && n < N ? (unsigned)(m * N + n) * 4u : kOutside;
            if constexpr (DGRAD) {
                mk[v] = p.mask ? ld32(mask, o[v]) : 1.f;
                old[v] = p.accumulate ? ld32(out, o[v]) : 0.f;
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float r = acc[i][v];
            if constexpr (DGRAD) {
                if (!(mk[v] > 0.f)) r = 0.f;
                if (p.accumulate) r += old[v];
            } else {
                r += bv;
                if (p.relu) r = fmaxf(r, 0.f);
            }
            st32(out, o[v], r);
        }
    }
}

constexpr int kFirstTiles = 4;                       // blocks of 32 pixels a wave, one after another
template <int STEPS>                                 // of two k each
__global__ __launch_bounds__(256) void igemm_chain_first_kernel(GemmParams p)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
    const unsigned tiles = (unsigned)(p.tiles_m * p.tiles_n), item = logical_block();
    if (item >= tiles * (unsigned)p.n_active) return;
    const int rep = p.order[item / tiles];
    const int tile = (int)(item % tiles) / p.tiles_n, n = (int)(item % tiles) % p.tiles_n * 32 + (lane & 31), N = p.Cout, nc = n < N ? n : N - 1;
    const int hw = p.H * p.W, M = p.B * hw;
    const long long first = ((p.cursor[rep] + p.ahead) * (long long)p.batch) % p.n_samples;
    const Buffer src = buffer(p.a + ((long long)rep * p.n_samples + first) * p.sample_sz, (unsigned)M * (unsigned)p.Cin * 4u);
    const float* const w = p.w + (long long)rep * p.w_rep;
    // this lane's k of every step, 2 j + half: weight, place in the source relative to the pixel, tap
    float b[STEPS]; int off[STEPS]; int tap[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int k = 2 * j + half;
        const bool on = k < p.K;
        const int t = k / p.Cin, r = t / p.S, s = t - r * p.S;
        b[j] = on ? w[(long long)k * N + nc] : 0.f;
        off[j] = (((r - p.pad) * p.W + s - p.pad) * p.Cin + k - t * p.Cin) * 4;
        tap[j] = on ? t : 31;                        // (no footprint has so many taps: never inside)
    }
    const float bv = p.has_bias ? w[(long long)p.K * N + nc] : 0.f;
    const Buffer out = buffer(p.out + (long long)rep * p.out_rep, (unsigned)M * (unsigned)N * 4u);
    float a[2][STEPS];
    auto block = [&](int t) { return ((tile * kFirstTiles + t) * 4 + wave) * 32; };
    auto gather = [&](float (&v)[STEPS], int t) {
        const int m = block(t) + (lane & 31), pos = m % hw, y = pos / p.W, x = pos - y * p.W;
        const unsigned cols = ((1u << min(p.S, p.W + p.pad - x)) - 1u) & ~((1u << max(0, p.pad - x)) - 1u);
        unsigned inside = 0;
        for (int r = 0; r < p.R; ++r) inside |= m < M && y + r - p.pad >= 0 && y + r - p.pad < p.H ? cols << (r * p.S) : 0u;
        const int at = m * p.Cin * 4;
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            v[j] = ld32(src, (inside >> tap[j]) & 1u ? (unsigned)(at + off[j]) : kOutside);
        }
    };
    gather(a[0], 0);
#pragma unroll
    for (int t = 0; t < kFirstTiles; ++t) {
        if (t + 1 < kFirstTiles) gather(a[(t + 1) & 1], t + 1);
        f16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
        for (int j = 0; j < STEPS; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t & 1][j], b[j], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = block(t) + 8 * (v >> 2) + 4 * half + (v & 3);
            float r = acc[v] + bv;
            if (p.relu) r = fmaxf(r, 0.f);
            st32(out, m < M && n < N ? (unsigned)(m * N + n) * 4u : kOutside, r);
        }
    }
}

template <int TM, int WM, int WN, bool DGRAD>
hipError_t launch_t(GemmParams& p, int n_active, hipStream_t s)
{
    constexpr int BM = 32 * TM * WM, BN = 32 * WN;
    const int C = DGRAD ? p.Cout : p.Cin, N = DGRAD ? p.Cin : p.Cout;
    const size_t lds = (size_t)(BM + 2 * p.pad * (p.W + 1) + 1) * (C + 2) * 4;
    if (lds > 65536) {
        static const bool ok = hipFuncSetAttribute((const void*)igemm_chain_kernel<TM, WM, WN, DGRAD>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess;
        if (!ok) return hipErrorInvalidValue;
    }
    p.tiles_m = (int)(((long long)p.B * p.H * p.W + BM - 1) / BM);
    p.tiles_n = (N + BN - 1) / BN;
    hipLaunchKernelGGL((igemm_chain_kernel<TM, WM, WN, DGRAD>), dim3(die_grid((long long)p.tiles_m * p.tiles_n * n_active)), dim3(64 * WM * WN), lds, s, p);
    return hipGetLastError();
}

constexpr int kTallest = 256;
}  // namespace

// A patch of the tallest tile with all channels fits LDS twice; offsets inside a batch are 32-bit byte offsets.
bool conv_chain_supported(int B, int H, int W, int C, int N, int k)
{
    const long long rows = kTallest + 2ll * (k / 2) * (W + 1) + 1;
    return k % 2 == 1 && k * k <= 32 && C % 16 == 0 && N % 4 == 0 && rows * (C + 2) * 4 <= 80 * 1024 && (long long)B * H * W * (C > N ? C : N) * 4 < 1ll << 31;
}
bool conv_chain_first_supported(int B, int H, int W, int C, int N, int k)
{
    return k % 2 == 1 && (long long)k * k * C <= 32 && k * k < 31 && (long long)B * H * W * (C > N ? C : N) * 4 < 1ll << 31;
}

hipError_t launch_conv_chain(const GemmParams& p0, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    GemmParams p = p0;
    p.n_active = n_active;
    if (p.stride != 1 || p.R != p.S || 2 * p.pad != p.R - 1 || p.Ho != p.H || p.Wo != p.W || (p.mode != kFwd && p.mode != kDgrad)) return hipErrorInvalidValue;
    const bool dgrad = p.mode == kDgrad;
    if (p.cursor) {
        if (dgrad || !conv_chain_first_supported(p.B, p.H, p.W, p.Cin, p.Cout, p.R) || p.sample_sz != (long long)p.H * p.W * p.Cin) return hipErrorInvalidValue;
        constexpr int BM = 32 * 4 * kFirstTiles;
        p.tiles_m = (int)(((long long)p.B * p.H * p.W + BM - 1) / BM);
        p.tiles_n = (p.Cout + 31) / 32;
        const dim3 grid(die_grid((long long)p.tiles_m * p.tiles_n * n_active));
        if (p.K <= 28) hipLaunchKernelGGL(igemm_chain_first_kernel<14>, grid, dim3(256), 0, s, p);
        else hipLaunchKernelGGL(igemm_chain_first_kernel<16>, grid, dim3(256), 0, s, p);
        return hipGetLastError();
    }
    const int N = dgrad ? p.Cin : p.Cout;
    // Tiles of 256 pixels where they give every compute unit a workgroup: 64 to 32 channels, 4 / 6 / 8 replicas (256 / 384 / 512 of them) 37 54 58 us, tiles
    // of 128 pixels 43 62 82; 2 replicas 35 and 25.
    if (!conv_chain_supported(p.B, p.H, p.W, dgrad ? p.Cout : p.Cin, N, p.R)) return hipErrorInvalidValue;
    const long long blocks = ((long long)p.B * p.H * p.W + 255) / 256 * n_active;       // 256 pixels each
    if (N > 32) return dgrad ? launch_t<2, 2, 2, true>(p, n_active, s) : launch_t<2, 2, 2, false>(p, n_active, s);
    if (blocks >= 256) return dgrad ? launch_t<2, 4, 1, true>(p, n_active, s) : launch_t<2, 4, 1, false>(p, n_active, s);
    return dgrad ? launch_t<1, 4, 1, true>(p, n_active, s) : launch_t<1, 4, 1, false>(p, n_active, s);
}

}  // namespace hadfl
