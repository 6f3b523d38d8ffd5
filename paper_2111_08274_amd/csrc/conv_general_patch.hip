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
// matrix instructions, and a slab's barriers come once per R * S taps.  In bf16 that is all that LDS can deliver (1 KiB per
// instruction and wave), so the large bf16 tiles give a wave 64 columns: half as much.
// fp32, 3 x 3, batch 64, forward with statistics, us (conv_general_kernel / this; TFLOP/s of fp32 products; the six bf16 products of
// 240 TFLOP/s are 1.44 PFLOP/s, of some 2.0 that pure matrix instructions reach):
//   64 channels, 32 x 32 images:   1 replica 46 / 32,  4 replicas 138 / 98,  16 replicas 523 / 398 (194 TFLOP/s)
//   128 channels, 16 x 16:         46 / 30,  105 / 89,  424 / 340 (227)
//   256 channels, 8 x 8:           49 / 30,  105 / 91,  377 / 325 (238)
//   512 channels, 4 x 4:           78 / 31,  138 / 89,  356 / 316 (245)
// bf16, 3 x 3, batch 128, us, forward with statistics and data gradient with mask and statistics (earlier kernels, which passed the
// weights through LDS and stored 8 bytes a lane / this):
//   64 channels, 32 x 32 images:   1 replica 20 / 19, 26 / 19,  4 replicas 58 / 59, 77 / 62,  16 replicas 243 / 226, 337 / 268
//   128 channels, 16 x 16:         25 / 16, 36 / 17,  44 / 42, 55 / 44,  155 / 144 (1.07 PFLOP/s), 225 / 170
//   256 channels, 8 x 8:           37 / 16, 43 / 17,  54 / 40, 61 / 41,  150 / 126 (1.23), 173 / 131
//   512 channels, 4 x 4:           64 / 17, 69 / 17,  68 / 41, 72 / 42,  128 / 116 (1.33), 139 / 117
//   512 channels, 2 x 2:           34 / 11, 40 / 12,  35 / 16, 40 / 17,  38 / 32, 44 / 32
#include <algorithm>
#include <type_traits>

#include "train_kernels.h"
#include "mfma_tiles.h"
#include "slabs.h"

namespace hadfl {
namespace {

using namespace tiles;

// sixteen bytes of a tensor
template <typename T> struct Vec;
template <> struct Vec<float> {
    u4 bits;
    __device__ __forceinline__ void load(const float* p) { bits = *reinterpret_cast<const u4*>(p); }
    __device__ __forceinline__ float at(int e) const { return __builtin_bit_cast(f4, bits)[e]; }
    __device__ __forceinline__ void round(const float (&v)[4]) { bits = __builtin_bit_cast(u4, f4{v[0], v[1], v[2], v[3]}); }
};
template <> struct Vec<__bf16> {
    u4 bits;
    __device__ __forceinline__ void load(const __bf16* p) { bits = *reinterpret_cast<const u4*>(p); }
    __device__ __forceinline__ float at(int e) const { return __builtin_bit_cast(float, e & 1 ? bits[e >> 1] & 0xffff0000u : bits[e >> 1] << 16); }
    __device__ __forceinline__ void round(const float (&v)[8]) { bits = u4{to_bf16x2(v[0], v[1]), to_bf16x2(v[2], v[3]), to_bf16x2(v[4], v[5]), to_bf16x2(v[6], v[7])}; }
};
// Exchange between the lanes of one wave through LDS: what was written before can be read after
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// KG groups of WGM x WGN waves share a tile of BMT = 32 TM WGM pixels x 32 TN WGN outputs (wave tile 32 TM x 32 TN): group kg multiplies
// slabs kg, kg + KG, ... from a patch of its own, and the groups' sums are joined in group order through LDS at the end.
// Q: passes of a group's threads over a patch (the launcher checks that they cover it).  D: taps that the weights are fetched ahead.
// SORTED: the tile holds whole images and its rows are ordered by position, the positions sorted by their set of taps inside the
// image (p.perm), so that a block of 32 rows leaves out the taps that none of its positions has: 5 of 9 on a 2 x 2 image.
// EPI 0: + bias, optional ReLU, optional statistics;  EPI 1: optional mask, optional accumulate, optional statistics
template <typename T, int TM, int WGM, int WGN, int KG, int Q, int D, int EPI, bool SORTED, int TN>
__global__ __launch_bounds__(WGM * WGN * KG * 64, 2) void conv_general_patch_kernel(GeneralConvParams p)
{
    constexpr bool kSplit = std::is_same<T, float>::value;
    constexpr int kSlab = Slab<T>::channels, kRow = Slab<T>::row, GR = Slab<T>::groups, PL = Slab<T>::planes, KS = kSlab / 16;
    constexpr unsigned ES = sizeof(T);
    constexpr int NW = WGM * WGN, NT = NW * 64, BMT = 32 * TM * WGM, BN = 32 * TN * WGN, STEP = NT / GR;
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
    const int images = SORTED ? BMT / hw : 1, image_bits = __builtin_ctz(images);       // (SORTED: powers of two)
    // LDS row of a pixel: the memory order, or (SORTED) position by position, so that lanes on the same pixel of neighbouring images
    // read neighbouring rows (16 pixels apart they would all meet in the same banks)
    auto lds_row = [&](int row) {
        if constexpr (!SORTED) return row;
        const int image = (int)__umulhi((unsigned)row, p.inv_hw);
        return (row - image * hw) * images + image;
    };
    auto store_patch = [&]() {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (arow + q * STEP >= rows) break;
            char* const o = patch + lds_row(arow + q * STEP) * kRow + ag * 16;
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
    const int half = lane >> 5;
    auto pixel = [&](int r) {                                 // of the tile, in row r
        if constexpr (!SORTED) return r;
        return (r & (images - 1)) * hw + p.perm[r >> image_bits];
    };
    int rd[TM]; unsigned inside[TM], block[TM];               // (block: taps that some row of the block has)
    const int base = SORTED ? 0 : m0 % hw;
    unsigned taps = SORTED ? 0u : ntap >= 32 ? 0xffffffffu : (1u << ntap) - 1u;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int lr = pixel((i * WGM + wm) * 32 + (lane & 31)), far = base + lr, pos = far - (int)__umulhi((unsigned)far, p.inv_hw) * hw;
        const int y = (int)__umulhi((unsigned)pos, p.inv_w), x = pos - y * p.W;
        rd[i] = (SORTED ? lds_row(lr) : lr + p.halo) * kRow + half * 16;
        inside[i] = 0; block[i] = 0;
        const unsigned cols = ((1u << min(p.S, p.W + p.pad - x)) - 1u) & ~((1u << max(0, p.pad - x)) - 1u);
        if (m0 + lr < M)
            for (int r = 0; r < p.R; ++r)
                if (y + r - p.pad >= 0 && y + r - p.pad < p.H) inside[i] |= cols << (r * p.S);
        if constexpr (SORTED) {
            const int r0 = (i * WGM + wm) * 32;
            for (int ps = r0 >> image_bits; ps <= (r0 + 31) >> image_bits; ++ps) block[i] |= p.posmask[ps];
            taps |= block[i];
        }
    }

    // weights: fragments [32 outputs][slab][tap][ks][plane][lane], fetched D taps ahead of their use
    const int cols32 = (p.N + 31) / 32;
    const char* const wbase = (const char*)(p.wmat + (long long)rep * p.wmat_rep);
    unsigned col[TN];                                         // (columns beyond the last: the last again, never stored)
#pragma unroll
    for (int j = 0; j < TN; ++j) col[j] = (unsigned)min(n0 / 32 + wn * TN + j, cols32 - 1) * (unsigned)(cs * ntap) * (unsigned)(KS * PL * 1024) + (unsigned)lane * 16u;
    int fslab = kg; unsigned fleft = taps;                    // the slab and the taps of it that are still to be fetched
    const char* fptr = nullptr;
    auto aim = [&]() { fptr = wbase + (fslab * ntap + __builtin_ctz(fleft)) * (KS * PL * 1024); };
    auto next_tap = [&]() {
        fleft &= fleft - 1u;
        if (!fleft && fslab + KG < cs) { fslab += KG; fleft = taps; }
        if (fleft) aim();                                     // (beyond the last tap: the last fragment again, not used)
    };
    u4 b[D][KS][TN][PL];
    auto fetch = [&](int d, int ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int s = 0; s < PL; ++s) b[d][ks][j][s] = *reinterpret_cast<const u4*>(fptr + (ks * PL + s) * 1024 + col[j]);
    };

    f16 acc[TM][TN], low[kSplit ? TM : 1][TN];                // sums of the large and of the small products
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) { acc[i][j][v] = 0.f; if constexpr (kSplit) low[i][j][v] = 0.f; }
    };
    const int inv_s = (65536 + p.S - 1) / p.S;                // tap / S for taps below 32
    auto tap_shift = [&](int tap) {
        const int r = (tap * inv_s) >> 16, s = tap - r * p.S;
        return ((r - p.pad) * p.W + s - p.pad) * images * kRow;
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
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (kSplit) {
                        constexpr int SA[5] = {0, 2, 1, 0, 1}, SB[5] = {2, 0, 1, 1, 0};
#pragma unroll
                        for (int t = 0; t < 5; ++t)
                            low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[d][ks][j][SB[t]]), a[SA[t]], low[i][j], 0, 0, 0);
                    }
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[d][ks][j][0]), a[0], acc[i][j], 0, 0, 0);
                }
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
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                acc[i][j] = (acc[i][j] + low[i][j]) * kProductScale;
#pragma unroll
                for (int v = 0; v < 16; ++v) bad = __builtin_fmaf(acc[i][j][v], 0.f, bad);
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
                        char* const o = patch + lds_row(arow + q * STEP) * kRow + ag * 32;
                        *reinterpret_cast<f4*>(o) = ra[q][0];
                        *reinterpret_cast<f4*>(o + 16) = ra[q][kSplit ? 1 : 0];
                    }
                }
                __syncthreads();
                for (int tap = 0; slab < cs && tap < ntap; ++tap) {
                    const char* const w = wbase + (slab * ntap + tap) * (KS * PL * 1024);
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 f[TN][PL];
#pragma unroll
                        for (int j = 0; j < TN; ++j)
#pragma unroll
                            for (int s = 0; s < PL; ++s) f[j][s] = *reinterpret_cast<const bf16x8*>(w + (ks * PL + s) * 1024 + col[j]);
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const char* const src = patch + ((inside[i] >> tap) & 1u ? rd[i] + tap_shift(tap) : zero + half * 16) + ks * 64 + half * 16;
#pragma unroll
                            for (int e = 0; e < 8; ++e)       // (both halves of the lanes: eight channels each, one per instruction)
#pragma unroll
                                for (int j = 0; j < TN; ++j)
                                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(join_weight(f[j][0][e], f[j][PL > 1 ? 1 : 0][e], f[j][PL > 2 ? 2 : 0][e]),
                                                                                     *reinterpret_cast<const float*>(src + e * 4), acc[i][j], 0, 0, 0);
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
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) part[(((((kg - 1) * NW + wave) * TM + i) * TN + j) * 16 + v) * 64 + lane] = acc[i][j][v];
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int g = 0; g < KG - 1; ++g)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[i][j][v] += part[((((g * NW + wave) * TM + i) * TN + j) * 16 + v) * 64 + lane];
        }
        __syncthreads();                                      // the epilogue's areas lie over the sums
    }

    // ---- epilogue ----
    // The accumulator has a pixel per lane (lane & 31) and channels 8 g + 4 (lane >> 5) + {0..3}: stored as it lies, every instruction
    // would touch 32 lines for 8 bytes (bf16) or 16 of each.  A block of 32 pixels goes through an area of LDS of the wave's own
    // instead, and lane c of the L lanes that share a pixel takes its c-th 16 bytes: whole runs of a line per instruction, in
    // stores and in the loads of the mask and of what is added to, and a lane keeps the sums of one group of channels.
    constexpr int VE = 16 / (int)ES, L = 32 * TN / VE, ST = L / 2, P = 32 * TN + 4;      // (ST: passes over a block)
    const bool stats = p.stat != nullptr;                     // per-channel sums of the outputs for a batch norm, forward or backward
    float ss[VE], qq[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) { ss[e] = 0.f; qq[e] = 0.f; }
    const int nl = (lane % L) * VE, n = n0 + wn * (32 * TN) + nl;         // this lane's channels
    if (kg == 0) {
        float* const area = reinterpret_cast<float*>(smem) + wave * (32 * P);
        T* const obase = reinterpret_cast<T*>(p.out + (long long)rep * p.out_rep);
        const float* bias = (EPI == 0 && p.bias) ? p.bias + (long long)rep * p.bias_rep : nullptr;
        const T* const added = p.addend ? reinterpret_cast<const T*>(p.addend + (long long)rep * p.addend_rep) : obase;
        const T* mask = (EPI == 1 && p.mask) ? reinterpret_cast<const T*>(p.mask + (long long)rep * p.mask_rep) : nullptr;
        // data gradient with statistics: values of the tensor whose gradient this is (see FastConvParams::stat_y), or of the batch norm's input
        const T* ysrc = (EPI == 1 && stats) ? reinterpret_cast<const T*>(p.stat_y + (long long)rep * p.stat_y_rep) : nullptr;
        auto offset = [&](int i, int t, unsigned& o) {                    // pass t of block i: this lane's place in the tensors
            const int mm = m0 + pixel((i * WGM + wm) * 32 + t * (64 / L) + lane / L);
            o = (unsigned)mm * (unsigned)p.N + (unsigned)n;
            return mm < M && n < p.N;
        };
        float sh[VE] = {};                                                // what the statistics are centred on: the bias
        if (EPI == 0 && bias && n < p.N) {
#pragma unroll
            for (int e = 0; e < VE; e += 4) *reinterpret_cast<f4*>(sh + e) = *reinterpret_cast<const f4*>(bias + n + e);
        }
        const bool centred = EPI == 1 && stats && p.stat_mean;            // (or that input's mean)
        if (centred && n < p.N) {
#pragma unroll
            for (int e = 0; e < VE; e += 4) *reinterpret_cast<f4*>(sh + e) = *reinterpret_cast<const f4*>(p.stat_mean + (long long)rep * p.stat_mean_rep + n + e);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            Vec<T> mk[EPI == 1 ? ST : 1], old[EPI == 1 ? ST : 1], xv[EPI == 1 && kSplit ? ST : 1];
            if constexpr (EPI == 1) {
#pragma unroll
                for (int t = 0; t < ST; ++t) {
                    unsigned o;
                    if (!offset(i, t, o)) continue;
                    if (mask) mk[t].load(mask + o);
                    if (p.accumulate) old[t].load(added + o);
                    if constexpr (kSplit) if (stats) xv[t].load(ysrc + o);
                }
            }
            wave_lds_fence();                                 // the block before has been read
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<f4*>(area + (lane & 31) * P + j * 32 + 8 * g + 4 * half) =
                        f4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
            wave_lds_fence();
#pragma unroll
            for (int t = 0; t < ST; ++t) {
                unsigned o;
                if (!offset(i, t, o)) continue;
                float v[VE];
#pragma unroll
                for (int e = 0; e < VE; e += 4) *reinterpret_cast<f4*>(v + e) = *reinterpret_cast<const f4*>(area + (t * (64 / L) + lane / L) * P + nl + e);
                if constexpr (EPI == 0) {
#pragma unroll
                    for (int e = 0; e < VE; ++e) {
                        if (bias) v[e] += sh[e];
                        if (p.relu) v[e] = fmaxf(v[e], 0.f);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < VE; ++e) {
                        if (p.accumulate) v[e] += old[t].at(e);
                        if (mask && !(mk[t].at(e) > 0.f)) v[e] = 0.f;
                    }
                }
                Vec<T> out;
                out.round(v);
                *reinterpret_cast<u4*>(obase + o) = out.bits;
                if (stats) {
                    if constexpr (EPI == 0) {
#pragma unroll
                        for (int e = 0; e < VE; ++e) { const float f = out.at(e) - sh[e]; ss[e] += f; qq[e] += f * f; }
                    } else {
                        Vec<T> yv = kSplit ? xv[kSplit ? t : 0] : mk[t];      // (the mask of a fused ReLU is the output)
                        if (!kSplit && ysrc != mask) yv.load(ysrc + o);
#pragma unroll
                        for (int e = 0; e < VE; ++e) {
                            const float f = (!kSplit && p.stat_relu && !(yv.at(e) > 0.f)) ? 0.f : out.at(e);
                            ss[e] += f; qq[e] += f * (yv.at(e) - sh[e]);
                        }
                    }
                }
            }
        }
    }
    if (stats) {
        // totals of a wave by shuffles, of the tile's waves above each other in wave order
        float* const cross = reinterpret_cast<float*>(smem) + NW * (32 * P);             // [wave][2][32 TN]
        if (kg == 0) {
#pragma unroll
            for (int e = 0; e < VE; ++e) {
#pragma unroll
                for (int d = L; d < 64; d *= 2) { ss[e] += __shfl_xor(ss[e], d); qq[e] += __shfl_xor(qq[e], d); }
            }
            if (lane < L) {
#pragma unroll
                for (int e = 0; e < VE; ++e) { cross[(wave * 2) * (32 * TN) + nl + e] = ss[e]; cross[(wave * 2 + 1) * (32 * TN) + nl + e] = qq[e]; }
            }
        }
        __syncthreads();
        float* const entry = p.stat + (long long)slot * p.stat_rep + (long long)(m0 / BMT) * 2 * p.N;
        for (int i = threadIdx.x; i < 2 * BN; i += NT * KG) {
            const int which = i / BN, c = i % BN;
            float t = 0.f;
#pragma unroll
            for (int r = 0; r < WGM; ++r) t += cross[((r * WGN + c / (32 * TN)) * 2 + which) * (32 * TN) + c % (32 * TN)];
            if (n0 + c < p.N) entry[which * p.N + n0 + c] = t;
        }
    }
}

constexpr int kMaxTile = 256;                        // pixels of the tallest tile

// x / d as umulhi(x, inverse(d)), d > 1: inverse(d) d is 2^32 + e with e < d (0 for powers of two), which adds x e / (d 2^32) to the quotient,
// less than the 1 / d that would take it to the next whole number while x e < 2^32.
unsigned inverse(unsigned d) { return 0xffffffffu / d + 1u; }
bool exact_quotients(unsigned d, unsigned long long largest) { return d > 1 && largest * ((unsigned long long)inverse(d) * d - (1ull << 32)) < 1ull << 32; }
// Those of a pixel's number by the image and of its place in the image by the width
bool exact_places(long long H, long long W) { return H * W < 1ll << 31 && exact_quotients((unsigned)(H * W), H * W - 1 + kMaxTile) && exact_quotients((unsigned)W, H * W - 1); }

constexpr size_t kMaxLds = 159 * 1024;               // (__syncthreads_or has a little of its own)

// LDS bytes of a launch with tiles of 32 TM WGM pixels, and the tile's border
template <typename T, int TM, int TN, int WGM, int WGN, int KG> size_t patch_lds(int halo)
{
    const size_t loop = (size_t)KG * (32 * TM * WGM + 2 * halo + 1) * Slab<T>::row, join = (size_t)(KG - 1) * WGM * WGN * TM * TN * 16 * 64 * 4;
    constexpr size_t epilogue = (size_t)WGM * WGN * (32 * (32 * TN + 4) + 2 * 32 * TN) * 4;
    return std::max(std::max(loop, join), epilogue);
}

template <typename T, int TM, int WGM, int WGN, int KG, int Q, int D, int EPI, bool SORTED, int TN>
hipError_t launch_t(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    constexpr int BMT = 32 * TM * WGM;
    const size_t lds = patch_lds<T, TM, TN, WGM, WGN, KG>(p.halo);
    if (lds > 65536) {
        static const bool ok = hipFuncSetAttribute((const void*)conv_general_patch_kernel<T, TM, WGM, WGN, KG, Q, D, EPI, SORTED, TN>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds) == hipSuccess;
        if (!ok) return hipErrorInvalidValue;
    }
    static_assert(BMT <= kMaxTile, "");
    if (!exact_places(p.H, p.W) || lds > kMaxLds || (BMT + 2 * p.halo) * Slab<T>::groups > Q * WGM * WGN * 64) return hipErrorInvalidValue;
    if (stat_rows) *stat_rows = BMT;
    p.tiles_m = (p.B * p.H * p.W + BMT - 1) / BMT;
    p.inv_hw = inverse(p.H * p.W); p.inv_w = inverse(p.W);
    const dim3 grid(die_grid((long long)p.tiles_m * ((p.N + 32 * TN * WGN - 1) / (32 * TN * WGN)) * n_active)), block(WGM * WGN * KG * 64);
    hipLaunchKernelGGL((conv_general_patch_kernel<T, TM, WGM, WGN, KG, Q, D, EPI, SORTED, TN>), grid, block, lds, s, p);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_split(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    typedef float T;
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
    case 0: return skip ? launch_t<T, 4, 1, 4, 1, 2, 1, EPI, true, 1>(p, n_active, s, stat_rows) : launch_t<T, 4, 1, 4, 1, 4, 1, EPI, false, 1>(p, n_active, s, stat_rows);
    case 1: return launch_t<T, 4, 2, 2, 1, 6, 1, EPI, false, 1>(p, n_active, s, stat_rows);
    case 2: return skip ? launch_t<T, 2, 2, 2, 1, 2, 2, EPI, true, 1>(p, n_active, s, stat_rows) : launch_t<T, 2, 2, 2, 1, 4, 1, EPI, false, 1>(p, n_active, s, stat_rows);
    case 3: return launch_t<T, 2, 1, 2, 2, 5, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    case 4: return launch_t<T, 2, 1, 2, 4, 5, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    case 5: return skip ? launch_t<T, 2, 1, 1, 8, 4, 2, EPI, true, 1>(p, n_active, s, stat_rows) : launch_t<T, 2, 1, 1, 8, 6, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    default: return launch_t<T, 1, 1, 2, 4, 3, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    }
}

// Pixels of border before and behind a tile that the bf16 launches have room for: 3 x 3 filters on images up to 32 pixels wide.  A patch on
// its way is in registers, 11 loads of 16 bytes a thread for the 256 + 66 pixels of the largest tiles; more was not measured, and
// wider images stay in the earlier kernels.
constexpr int kBorderBf16 = 33;

template <int EPI>
hipError_t launch_bf16(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    typedef __bf16 T;
    // As above; `extra` is what the first loads and the epilogue take, in taps.  Fitted to 3 x 3 and 1 x 1 layers of 64 to 512 channels,
    // 2 x 2 to 32 x 32 images, batch 128, 1 to 16 replicas, both directions: over those 108 launches the choice takes 1.1 % longer than
    // the best of these tiles.  The last entry has its rows sorted by position (2 x 2 images, 9 taps: its times are those of the taps
    // it visits); on 4 x 4 images sorted rows gain 2 % in the forward pass and lose 3 % in the data gradient, and are not used.
    struct Tile { int m, n, groups; float alone, full, share, extra; };
    static constexpr Tile kTile[] = {
        {256, 128, 1, 0.90f, 0.99f, 0.68f, 12.5f}, {256, 64, 1, 0.69f, 0.88f, 0.40f, 11.5f}, {128, 256, 1, 0.81f, 0.91f, 0.64f, 13.6f},
        {128, 128, 1, 0.55f, 0.64f, 0.375f, 12.3f}, {128, 64, 1, 0.44f, 0.52f, 0.194f, 13.8f}, {64, 64, 2, 0.48f, 0.48f, 0.193f, 16.1f},
        {64, 64, 4, 0.43f, 0.43f, 0.37f, 22.1f}, {32, 64, 4, 0.36f, 0.43f, 0.17f, 22.6f}, {128, 64, 1, 0.29f, 0.32f, 0.22f, 1.4f}};
    const int hw = p.H * p.W, border = p.pad * (p.W + 1), cs = (p.C + Slab<T>::channels - 1) / Slab<T>::channels, taps = p.R * p.S;
    const long long M = (long long)p.B * hw;
    const bool sorted = p.perm && hw == 4 && taps > 1;
    int best = p.N <= 64 ? 1 : 0;
    float best_t = 0.f;
    for (int i = 0; i < 9 && p.tile_hint != 1; ++i) {
        const Tile& t = kTile[i];
        if ((i == 8 && !sorted) || (t.n > 64 && t.n / 2 >= p.N)) continue;
        const long long wgs = (M + t.m - 1) / t.m * ((p.N + t.n - 1) / t.n) * n_active;
        const float step = wgs <= 128 ? t.alone : wgs <= 256 ? t.full : std::max(t.full, (float)((wgs + 255) / 256) * t.share);
        const float idle = cs < t.groups ? 0.5f + 0.5f * (float)cs / (float)t.groups : 1.0f;         // groups without a slab
        const float time = ((float)((cs + t.groups - 1) / t.groups * taps) + t.extra) * step * idle;
        if (best_t == 0.f || time < best_t) { best = i; best_t = time; }
    }
    p.halo = kTile[best].m % hw == 0 ? 0 : border;
    if (best != 8) p.perm = nullptr;
    switch (best) {
    case 0: return launch_t<T, 4, 2, 2, 1, 11, 1, EPI, false, 2>(p, n_active, s, stat_rows);
    case 1: return launch_t<T, 4, 2, 2, 1, 11, 1, EPI, false, 1>(p, n_active, s, stat_rows);
    case 2: return launch_t<T, 4, 1, 4, 1, 7, 1, EPI, false, 2>(p, n_active, s, stat_rows);
    case 3: return launch_t<T, 2, 2, 2, 1, 7, 1, EPI, false, 2>(p, n_active, s, stat_rows);
    case 4: return launch_t<T, 2, 2, 2, 1, 7, 1, EPI, false, 1>(p, n_active, s, stat_rows);
    case 5: return launch_t<T, 2, 1, 2, 2, 9, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    case 6: return launch_t<T, 2, 1, 2, 4, 9, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    case 7: return launch_t<T, 1, 1, 2, 4, 7, 2, EPI, false, 1>(p, n_active, s, stat_rows);
    default: return launch_t<T, 1, 4, 1, 1, 4, 1, EPI, true, 2>(p, n_active, s, stat_rows);
    }
}

}  // namespace

// fp32: the patch of 128 pixels has room for 64 pixels of border on either side, 3 x 3 filters on images up to 63 pixels wide; layers of
// up to 32 channels stay with conv_general_kernel, whose tiles have 32 columns.  1 x 1 filters have one tap for each patch: in fp32
// conv_general_kernel, which splits as much there, keeps them; in bf16 they run here (64 channels, 32 x 32 images, batch 128, 16
// replicas 152 -> 123 us forward, 282 -> 163 us data gradient against the kernels of conv_bf16_fast.hip).  Images of some 65 thousand pixels
// and more whose quotients would not be exact stay with the earlier kernels.
bool conv_patch_supported(int bf16, int H, int W, int C, int N, int k)
{
    const int unit = bf16 ? 8 : 4, border = k / 2 * (W + 1);
    return k % 2 == 1 && k * k <= 32 && (bf16 ? border <= kBorderBf16 : k > 1 && border <= 64) && (long long)H * W >= 4 && exact_places(H, W) &&
           C % unit == 0 && N % unit == 0 && std::min(C, N) > 32;
}

hipError_t launch_conv_general_patch(const GeneralConvParams& p0, int epi, int n_active, hipStream_t s, int* stat_rows)
{
    if (n_active < 1) return hipSuccess;
    GeneralConvParams p = p0;
    p.n_active = n_active;
    if (p.cursor || p.classes != 1 || p.sstride != 1 || p.Ho != p.H || p.Wo != p.W || p.R != p.S || 2 * p.pad != p.R - 1 ||
        !conv_patch_supported(p.bf16, p.H, p.W, p.C, p.N, p.R)) return hipErrorInvalidValue;
    if (p.bf16) return epi == 0 ? launch_bf16<0>(p, n_active, s, stat_rows) : launch_bf16<1>(p, n_active, s, stat_rows);
    return epi == 0 ? launch_split<0>(p, n_active, s, stat_rows) : launch_split<1>(p, n_active, s, stat_rows);
}

}  // namespace hadfl
