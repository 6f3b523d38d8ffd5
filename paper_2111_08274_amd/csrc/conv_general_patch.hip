// Stride-1 "same" convolutions, forward and data gradient of every local step (paper Sec. 2.1).  The arithmetic is that of
// conv_general.hip: fp32 as six bf16 products of split floats with an accumulator for the large ones and one for the small
// ones, bf16 as it is; what differs is how the operands reach the matrix cores.
//
// conv_general_kernel fetches an activation once per tap, and splits and writes it to LDS each time; both operands pass through
// LDS, whose writes (some 70 bytes a clock) and reads cost as much as the matrix instructions.  Here
//   * a workgroup loads the pixels of its tile and of the border around it ONCE per slab of channels.  Pixels stay
//     in memory order, so tap (dy, dx) of pixel q is the row q + dy W + dx of that patch, whatever the image's size: the patch is
//     the tile's BMT pixels and W + 1 (3 x 3 filters) before and behind them, none when the tile holds whole images.  A tap
//     outside the image reads a row of zeros.
//   * the weights never enter LDS: the copies (weight_copy_kernel) hold them in the order in which the lanes of a matrix
//     instruction take them, 1 KiB per 32 outputs x 16 channels and plane, one coalesced 16-byte load per lane.  A fragment
//     is fetched into the registers of the one just used, a tap ahead.
// Per 16 channels of a tap a wave with a 128 x 32 tile then reads 4 KiB of LDS per plane and 1 KiB of memory for its 24 (bf16: 4)
// matrix instructions, and a slab's barriers come once per R * S taps.
// fp32, 3 x 3, batch 64, forward with statistics, us (conv_general_kernel / this; TFLOP/s of fp32 products; the six bf16 products of
// 240 TFLOP/s are 1.44 PFLOP/s, of some 2.0 that pure matrix instructions reach):
//   64 channels, 32 x 32 images:   1 replica 46 / 32,  4 replicas 138 / 98,  16 replicas 523 / 398 (194 TFLOP/s)
//   128 channels, 16 x 16:         46 / 30,  105 / 89,  424 / 340 (227)
//   256 channels, 8 x 8:           49 / 30,  105 / 91,  377 / 325 (238)
//   512 channels, 4 x 4:           78 / 31,  138 / 89,  356 / 316 (245)
#include <algorithm>
#include <type_traits>

#include "train_kernels.h"
#include "conv_stats.h"
#include "mfma_tiles.h"
#include "slabs.h"

namespace hadfl {
namespace {

using namespace tiles;
using conv_stats::store_column_stats;
using conv_stats::kStatLdsBytes;

// KG groups of WGM x WGN waves share a tile of BMT = 32 TM WGM pixels x 32 WGN outputs (wave tile 32 TM x 32): group kg multiplies
// slabs kg, kg + KG, ... from a patch of its own, and the groups' sums are joined in group order through LDS at the end.
// Q: passes of a group's threads over a patch (the launcher checks that they cover it).  D: taps that the weights are fetched ahead.
// SORTED: the tile holds whole images and its rows are ordered by position, the positions sorted by their set of taps inside the
// image (p.perm), so that a block of 32 rows leaves out the taps that none of its positions has: 5 of 9 on a 2 x 2 image.
// EPI 0: + bias, optional ReLU, optional statistics;  EPI 1: optional mask, optional accumulate, (bf16) optional statistics
template <typename T, int TM, int WGM, int WGN, int KG, int Q, int D, int EPI, bool SORTED>
__global__ __launch_bounds__(WGM * WGN * KG * 64, 2) void conv_general_patch_kernel(GeneralConvParams p)
{
    constexpr bool kSplit = std::is_same<T, float>::value;
    constexpr int kSlab = Slab<T>::channels, kRow = Slab<T>::row, GR = Slab<T>::groups, PL = Slab<T>::planes, KS = kSlab / 16;
    constexpr unsigned ES = sizeof(T);
    constexpr int NW = WGM * WGN, NT = NW * 64, BMT = 32 * TM * WGM, BN = 32 * WGN, STEP = NT / GR;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x % NT, lane = tid & 63;
    const int kg = KG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int rows = BMT + 2 * p.halo, zero = rows * kRow;    // (LDS row `rows`: zeros)
    char* const patch = smem + kg * (zero + kRow);
    // logical item = (slot, column tile, row tile), row tiles fastest
    const int hw = p.H * p.W, M = p.B * hw;
    const unsigned tiles_m = (unsigned)p.tiles_m, tiles_n = (unsigned)(p.N + BN - 1) / BN;
    const unsigned item = logical_block();
    if (item >= tiles_m * tiles_n * (unsigned)p.n_active) return;
    const int slot = (int)(item / (tiles_m * tiles_n));
    const int rep = p.order[slot];
    const int m0 = (int)(item % tiles_m) * BMT, n0 = (int)((item / tiles_m) % tiles_n) * BN;
    const int ntap = p.R * p.S, cs = (p.C + kSlab - 1) / kSlab;

    // patch slots of this thread: rows arow + q STEP, 16-byte group ag of a plane
    const int ag = tid % GR, arow = tid / GR;
    const unsigned aoff = (unsigned)((m0 - p.halo + arow) * p.C + ag * (kSplit ? 4 : 8)) * ES;    // (rows before the batch wrap to far beyond it)
    const Buffer abuf = buffer(p.a + (long long)rep * p.a_rep, (unsigned)M * (unsigned)p.C * ES);
    f4 ra[Q][kSplit ? 2 : 1];                                 // the next slab's patch on its way (bf16: eight elements)
    auto load_patch = [&](int slab) {
        const int c0 = slab * kSlab + ag * (kSplit ? 4 : 8);
        const bool in0 = c0 < p.C, in1 = c0 + 16 < p.C;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool ok = arow + q * STEP < rows;
            const unsigned o = aoff + (unsigned)(q * STEP * p.C + slab * kSlab) * ES;
            ra[q][0] = __builtin_bit_cast(f4, ldb16(abuf, ok && in0 ? o : kOutside));
            if constexpr (kSplit) ra[q][1] = __builtin_bit_cast(f4, ldb16(abuf, ok && in1 ? o + 64u : kOutside));
        }
    };
    auto store_patch = [&]() {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (arow + q * STEP >= rows) break;
            char* const o = patch + (arow + q * STEP) * kRow + ag * 16;
            if constexpr (kSplit) {
                u2 h0, m0_, l0, h1, m1, l1;
                split3(ra[q][0], h0, m0_, l0);
                split3(ra[q][1], h1, m1, l1);
                *reinterpret_cast<u4*>(o) = join8(h0, h1);
                *reinterpret_cast<u4*>(o + 64) = join8(m0_, m1);
                *reinterpret_cast<u4*>(o + 128) = join8(l0, l1);
            } else {
                *reinterpret_cast<f4*>(o) = ra[q][0];
            }
        }
    };

    // this lane's rows of the tile: LDS address of the pixel's own row, taps inside the image
    const int half = lane >> 5, images = SORTED ? BMT / hw : 1;
    auto local_row = [&](int i) {
        const int r = (i * WGM + wm) * 32 + (lane & 31);
        if constexpr (!SORTED) return r;
        const int ps = r / images;
        return (r - ps * images) * hw + p.perm[ps];
    };
    int rd[TM]; unsigned inside[TM], block[TM];               // (block: taps that some row of the block has)
    const int base = SORTED ? 0 : m0 % hw;
    unsigned taps = SORTED ? 0u : ntap >= 32 ? 0xffffffffu : (1u << ntap) - 1u;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int lr = local_row(i), far = base + lr, pos = far - (int)__umulhi((unsigned)far, p.inv_hw) * hw;
        const int y = (int)__umulhi((unsigned)pos, p.inv_w), x = pos - y * p.W;
        rd[i] = (lr + p.halo) * kRow + half * 16;
        inside[i] = 0; block[i] = 0;
        const unsigned cols = ((1u << min(p.S, p.W + p.pad - x)) - 1u) & ~((1u << max(0, p.pad - x)) - 1u);
        if (m0 + lr < M)
            for (int r = 0; r < p.R; ++r)
                if (y + r - p.pad >= 0 && y + r - p.pad < p.H) inside[i] |= cols << (r * p.S);
        if constexpr (SORTED) {
            const int r0 = (i * WGM + wm) * 32;
            for (int ps = r0 / images; ps <= (r0 + 31) / images; ++ps) block[i] |= p.posmask[ps];
            taps |= block[i];
        }
    }

    // weights: fragments [32 outputs][slab][tap][ks][plane][lane], fetched D taps ahead of their use
    const int cols32 = (p.N + 31) / 32;
    const char* const wbase = (const char*)(p.wmat + (long long)rep * p.wmat_rep) + (long long)min(n0 / 32 + wn, cols32 - 1) * cs * ntap * (KS * PL * 1024);
    int fslab = kg; unsigned fleft = taps;                    // the slab and the taps of it that are still to be fetched
    const char* fptr = nullptr;
    auto aim = [&]() { fptr = wbase + (fslab * ntap + __builtin_ctz(fleft)) * (KS * PL * 1024); };
    auto next_tap = [&]() {
        fleft &= fleft - 1u;
        if (!fleft && fslab + KG < cs) { fslab += KG; fleft = taps; }
        if (fleft) aim();                                     // (beyond the last tap: the last fragment again, not used)
    };
    u4 b[D][KS][PL];
    auto fetch = [&](int d, int ks) {
#pragma unroll
        for (int s = 0; s < PL; ++s) b[d][ks][s] = *reinterpret_cast<const u4*>(fptr + (ks * PL + s) * 1024 + lane * 16);
    };

    f16 acc[TM], low[kSplit ? TM : 1];                        // sums of the large and of the small products
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[i][v] = 0.f; if constexpr (kSplit) low[i][v] = 0.f; }
    };
    const int inv_s = (65536 + p.S - 1) / p.S;                // tap / S for taps below 32
    auto tap_shift = [&](int tap) {
        const int r = (tap * inv_s) >> 16, s = tap - r * p.S;
        return ((r - p.pad) * p.W + s - p.pad) * kRow;
    };
    auto multiply = [&](int tap, int d) {
        const int shift = tap_shift(tap);
        int at[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) at[i] = (inside[i] >> tap) & 1u ? rd[i] + shift : zero + half * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (SORTED && !((block[i] >> tap) & 1u)) continue;
                bf16x8 a[PL];
#pragma unroll
                for (int s = 0; s < PL; ++s) a[s] = *reinterpret_cast<const bf16x8*>(patch + at[i] + s * 64 + ks * 32);
                // operands swapped: the accumulator holds the transposed tile.  Small products in ascending size.
                if constexpr (kSplit) {
                    constexpr int SA[5] = {0, 2, 1, 0, 1}, SB[5] = {2, 0, 1, 1, 0};
#pragma unroll
                    for (int t = 0; t < 5; ++t)
                        low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[d][ks][SB[t]]), a[SA[t]], low[i], 0, 0, 0);
                }
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[d][ks][0]), a[0], acc[i], 0, 0, 0);
            }
            fetch(d, ks);
        }
    };

    const int rounds = (cs + KG - 1) / KG;
    clear();
    if (tid < kRow / 16) *reinterpret_cast<u4*>(patch + zero + tid * 16) = u4{0u, 0u, 0u, 0u};
    if (kg < cs) {
        load_patch(kg);
        aim();
#pragma unroll
        for (int d = 0; d < D; ++d) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) fetch(d, ks);
            next_tap();
        }
    }
    unsigned left = 0;                                        // taps of the present slab that are still to be multiplied
    int staged = 0;
    for (bool more = true; more;) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (!left) {
                if (staged == rounds) { more = false; break; }
                const int slab = staged++ * KG + kg;
                __syncthreads();                              // every wave is done reading the previous patch
                if (slab < cs) store_patch();
                __syncthreads();
                if (slab + KG < cs) load_patch(slab + KG);
                if (slab >= cs) { more = false; break; }      // (the last round, which this group sits out)
                left = taps;
            }
            multiply(__builtin_ctz(left), d);
            next_tap();
            left &= left - 1u;
        }
    }
    if constexpr (kSplit) {
        float bad = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            acc[i] = (acc[i] + low[i]) * kProductScale;
#pragma unroll
            for (int v = 0; v < 16; ++v) bad = __builtin_fmaf(acc[i][v], 0.f, bad);
        }
        if (__syncthreads_or(bad != 0.f)) {                   // (NaN != 0) something is not finite: the tile again, with the fp32 instruction
            clear();
            for (int t = 0; t < rounds; ++t) {
                const int slab = t * KG + kg;
                __syncthreads();
                if (slab < cs) {
                    load_patch(slab);
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        if (arow + q * STEP >= rows) break;
                        char* const o = patch + (arow + q * STEP) * kRow + ag * 32;
                        *reinterpret_cast<f4*>(o) = ra[q][0];
                        *reinterpret_cast<f4*>(o + 16) = ra[q][kSplit ? 1 : 0];
                    }
                }
                __syncthreads();
                for (int tap = 0; slab < cs && tap < ntap; ++tap) {
                    const char* const w = wbase + (slab * ntap + tap) * (KS * PL * 1024) + lane * 16;
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 f[PL];
#pragma unroll
                        for (int s = 0; s < PL; ++s) f[s] = *reinterpret_cast<const bf16x8*>(w + (ks * PL + s) * 1024);
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const char* const src = patch + ((inside[i] >> tap) & 1u ? rd[i] + tap_shift(tap) : zero + half * 16) + ks * 64 + half * 16;
#pragma unroll
                            for (int e = 0; e < 8; ++e)       // (both halves of the lanes: eight channels each, one per instruction)
                                acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(join_weight(f[0][e], f[PL > 1 ? 1 : 0][e], f[PL > 2 ? 2 : 0][e]),
                                                                              *reinterpret_cast<const float*>(src + e * 4), acc[i], 0, 0, 0);
                        }
                    }
                }
            }
            __syncthreads();
        }
    } else {
        __syncthreads();                                      // nobody reads a patch any more
    }
    if constexpr (KG > 1) {                                   // (behind the barriers above)
        float* const part = reinterpret_cast<float*>(smem);
        if (kg > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) part[((((kg - 1) * NW + wave) * TM + i) * 16 + v) * 64 + lane] = acc[i][v];
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int g = 0; g < KG - 1; ++g)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][v] += part[(((g * NW + wave) * TM + i) * 16 + v) * 64 + lane];
        }
    }

    // ---- epilogue: lane holds output row (lane & 31) and channels 8*g + 4*(lane >> 5) + {0..3}, g = 0..3 ----
    const bool stats = (EPI == 0 || !kSplit) && p.stat != nullptr;        // per-channel sums of the outputs for a batch norm
    float ss[1][16], qq[1][16];
#pragma unroll
    for (int k = 0; k < 16; ++k) { ss[0][k] = 0.f; qq[0][k] = 0.f; }
    if (kg == 0) {
        T* const obase = reinterpret_cast<T*>(p.out + (long long)rep * p.out_rep);
        const float* bias = (EPI == 0 && p.bias) ? p.bias + (long long)rep * p.bias_rep : nullptr;
        const T* mask = (EPI == 1 && p.mask) ? reinterpret_cast<const T*>(p.mask + (long long)rep * p.mask_rep) : nullptr;
        // data gradient with statistics: values of the tensor whose gradient this is (see FastConvParams::stat_y)
        const T* ysrc = (EPI == 1 && stats) ? reinterpret_cast<const T*>(p.stat_y + (long long)rep * p.stat_y_rep) : nullptr;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mm = m0 + local_row(i);
            if (mm >= M) continue;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + wn * 32 + 8 * g + 4 * half;
                if (n >= p.N) continue;
                const unsigned o = (unsigned)mm * (unsigned)p.N + (unsigned)n;
                f4 v = {acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
                f4 sh = {0.f, 0.f, 0.f, 0.f}, mk = {};        // sh: what the statistics are centred on, the bias
                if constexpr (EPI == 0) {
                    if (bias) { sh = *reinterpret_cast<const f4*>(bias + n); v += sh; }
                    if (p.relu) { v[0] = fmaxf(v[0], 0.f); v[1] = fmaxf(v[1], 0.f); v[2] = fmaxf(v[2], 0.f); v[3] = fmaxf(v[3], 0.f); }
                } else {
                    if (mask) {
                        mk = load4(mask + o);
#pragma unroll
                        for (int e = 0; e < 4; ++e) if (!(mk[e] > 0.f)) v[e] = 0.f;
                    }
                    if (p.accumulate) v += load4(obase + o);
                }
                store4(obase + o, v);
                if (stats) {
                    if constexpr (EPI == 0) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) { const float f = v[e] - sh[e]; ss[0][4 * g + e] += f; qq[0][4 * g + e] += f * f; }
                    } else {
                        const f4 yv = ysrc == mask ? mk : load4(ysrc + o);          // (the mask of a fused ReLU is that very tensor)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float f = (p.stat_relu && !(yv[e] > 0.f)) ? 0.f : v[e];
                            ss[0][4 * g + e] += f; qq[0][4 * g + e] += f * yv[e];
                        }
                    }
                }
            }
        }
    }
    if (stats) {                                              // (the launcher asks for the larger of the K loop's LDS and kStatLdsBytes)
        __syncthreads();                                      // every wave is past its last read of LDS
        if (kg == 0)
            store_column_stats<1, WGM, WGN>(ss, qq, reinterpret_cast<float*>(smem), wave, lane, p.stat + (long long)slot * p.stat_rep,
                                            m0 / BMT, n0 + wn * 32, p.N);
        else
            __syncthreads();                                  // the barrier inside store_column_stats
    }
}

constexpr size_t kMaxLds = 159 * 1024;               // (__syncthreads_or has a little of its own)

// LDS bytes of a launch with tiles of 32 TM WGM pixels, and the tile's border
template <typename T, int TM, int WGM, int WGN, int KG> size_t patch_lds(int halo)
{
    const size_t loop = (size_t)KG * (32 * TM * WGM + 2 * halo + 1) * Slab<T>::row, join = (size_t)(KG - 1) * WGM * WGN * TM * 16 * 64 * 4;
    return std::max(std::max(loop, join), kStatLdsBytes<1, WGM, WGN>);
}

template <typename T, int TM, int WGM, int WGN, int KG, int Q, int D, int EPI, bool SORTED>
hipError_t launch_t(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    constexpr int BMT = 32 * TM * WGM;
    const size_t lds = patch_lds<T, TM, WGM, WGN, KG>(p.halo);
    if (lds > 65536) {
        static const bool ok = hipFuncSetAttribute((const void*)conv_general_patch_kernel<T, TM, WGM, WGN, KG, Q, D, EPI, SORTED>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds) == hipSuccess;
        if (!ok) return hipErrorInvalidValue;
    }
    if (p.W < 2 || lds > kMaxLds || (BMT + 2 * p.halo) * Slab<T>::groups > Q * WGM * WGN * 64) return hipErrorInvalidValue;
    if (stat_rows) *stat_rows = BMT;
    p.tiles_m = (p.B * p.H * p.W + BMT - 1) / BMT;
    p.inv_hw = 0xffffffffu / (unsigned)(p.H * p.W) + 1u; p.inv_w = 0xffffffffu / (unsigned)p.W + 1u;     // x / d for x d < 2^32, d > 1
    const dim3 grid(die_grid((long long)p.tiles_m * ((p.N + 32 * WGN - 1) / (32 * WGN)) * n_active)), block(WGM * WGN * KG * 64);
    hipLaunchKernelGGL((conv_general_patch_kernel<T, TM, WGM, WGN, KG, Q, D, EPI, SORTED>), grid, block, lds, s, p);
    return hipGetLastError();
}

template <typename T, int EPI>
hipError_t launch_patch(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    // Per tap of a slab, in us: `alone` for a workgroup that has its compute unit to itself, `full` with one on every unit, `share` the
    // unit's time per workgroup under load; about three taps' time goes into the first loads and the epilogue.  Measured on 3 x 3
    // layers of 64 to 512 channels, batch 64, 1 to 16 replicas, and fitted to within some 10 %.
    struct Tile { int m, n, groups, rows; float alone, full, share; };
    static constexpr Tile kTile[] = {
        {128, 128, 1, 256, 1.14f, 1.38f, 1.12f}, {256, 64, 1, 384, 1.14f, 1.50f, 1.13f}, {128, 64, 1, 256, 0.69f, 0.82f, 0.61f},
        {64, 64, 2, 160, 0.75f, 0.82f, 0.64f}, {64, 64, 4, 160, 1.18f, 1.35f, 1.30f}, {64, 32, 8, 96, 1.40f, 1.50f, 1.45f},
        {32, 64, 4, 96, 0.75f, 0.86f, 0.92f}};
    const int hw = p.H * p.W, border = p.pad * (p.W + 1), cs = (p.C + Slab<T>::channels - 1) / Slab<T>::channels, taps = p.R * p.S;
    const long long M = (long long)p.B * hw;
    const bool sorted = p.perm && hw <= 16 && 64 % hw == 0;
    int best = -1;
    float best_t = 0.f;
    for (int i = 0; i < (int)(sizeof(kTile) / sizeof(kTile[0])); ++i) {
        const Tile& t = kTile[i];
        const int halo = t.m % hw == 0 ? 0 : border, rows = t.m + 2 * halo;
        if (rows > t.rows || (size_t)t.groups * (rows + 1) * Slab<T>::row > kMaxLds) continue;
        if (p.tile_hint == 1) { if (best < 0 || i == 1) best = p.N <= 64 && i == 1 ? 1 : best < 0 ? i : best; continue; }
        const long long wgs = (M + t.m - 1) / t.m * ((p.N + t.n - 1) / t.n) * n_active;
        const float step = wgs <= 128 ? t.alone : wgs <= 256 ? t.full : std::max(t.full, (float)((wgs + 255) / 256) * t.share);
        const bool skips = sorted && (i == 0 || i == 2 || i == 5);          // (tiles with a variant for sorted rows)
        const float kept = !skips ? 1.0f : hw <= 4 ? 0.55f : i == 0 ? 0.93f : 1.0f;
        const float idle = cs < t.groups ? 0.5f + 0.5f * (float)cs / (float)t.groups : 1.0f;         // groups without a slab
        const float time = ((float)((cs + t.groups - 1) / t.groups * taps) * kept + 3.0f) * step * idle;
        if (best < 0 || time < best_t) { best = i; best_t = time; }
    }
    if (best < 0) return hipErrorInvalidValue;
    p.halo = kTile[best].m % hw == 0 ? 0 : border;
    const bool skip = sorted && (hw <= 4 || best == 0);
    if (!skip) p.perm = nullptr;
    switch (best) {
    case 0: return skip ? launch_t<T, 4, 1, 4, 1, 2, 1, EPI, true>(p, n_active, s, stat_rows) : launch_t<T, 4, 1, 4, 1, 4, 1, EPI, false>(p, n_active, s, stat_rows);
    case 1: return launch_t<T, 4, 2, 2, 1, 6, 1, EPI, false>(p, n_active, s, stat_rows);
    case 2: return skip ? launch_t<T, 2, 2, 2, 1, 2, 2, EPI, true>(p, n_active, s, stat_rows) : launch_t<T, 2, 2, 2, 1, 4, 1, EPI, false>(p, n_active, s, stat_rows);
    case 3: return launch_t<T, 2, 1, 2, 2, 5, 2, EPI, false>(p, n_active, s, stat_rows);
    case 4: return launch_t<T, 2, 1, 2, 4, 5, 2, EPI, false>(p, n_active, s, stat_rows);
    case 5: return skip ? launch_t<T, 2, 1, 1, 8, 4, 2, EPI, true>(p, n_active, s, stat_rows) : launch_t<T, 2, 1, 1, 8, 6, 2, EPI, false>(p, n_active, s, stat_rows);
    default: return launch_t<T, 1, 1, 2, 4, 3, 2, EPI, false>(p, n_active, s, stat_rows);
    }
}

}  // namespace

// The patch of 128 pixels has room for 64 pixels of border on either side: 3 x 3 filters on images up to 63 pixels wide.  Layers of
// up to 32 channels stay with conv_general_kernel, whose tiles have 32 columns.
bool conv_patch_supported(int bf16, int H, int W, int C, int N, int k)
{
    const int unit = bf16 ? 8 : 4;
    return !bf16 && k > 1 && k % 2 == 1 && k * k <= 32 && W >= 2 && H * W >= 4 && k / 2 * (W + 1) <= 64 && C % unit == 0 && N % unit == 0 && std::min(C, N) > 32;
}

hipError_t launch_conv_general_patch(const GeneralConvParams& p0, int epi, int n_active, hipStream_t s, int* stat_rows)
{
    if (n_active < 1) return hipSuccess;
    GeneralConvParams p = p0;
    p.n_active = n_active;
    if (p.cursor || p.classes != 1 || p.sstride != 1 || p.Ho != p.H || p.Wo != p.W || p.R != p.S || 2 * p.pad != p.R - 1 ||
        !conv_patch_supported(p.bf16, p.H, p.W, p.C, p.N, p.R)) return hipErrorInvalidValue;
    return epi == 0 ? launch_patch<float, 0>(p, n_active, s, stat_rows) : launch_patch<float, 1>(p, n_active, s, stat_rows);
}

}  // namespace hadfl
