// Convolutions and dense layers of any geometry, forward, data gradient and weight gradient of every local step (paper Sec. 2.1),
// on the bf16 matrix cores: the fp32 configuration (T = float) without giving up fp32 accuracy, and the layers of the bf16
// configuration (T = __bf16) that the lean kernels of conv_bf16_fast.hip do not take (strides, ragged channel counts, odd images).
//
// T = float.  The fp32 matrix instruction runs at a sixteenth of the bf16 rate (157 against 2500 TFLOP/s).  A float is the exact sum
// of three bf16 numbers, x = xh + xm + xl, so a product is the sum of nine bf16 products, and the six of them that are
// not below 2^-26 of it,
//       xh*yh  +  (xh*ym + xm*yh + xm*ym + xh*yl + xl*yh),
// cost 6 / 16 of the fp32 instruction's time.  Every bf16 product is exact in fp32; what rounds is the accumulation.
// The large products xh*yh have an accumulator of their own and the five small ones another, joined once at the end:
// the small ones are then never rounded to the size of the running sum, and the large accumulator rounds once per
// sixteen products where the fp32 instruction rounds after each.  Root-mean-square error against 64 bits, 32 x 32 products of
// length K, in units of the products' 2-norm (fp32 instruction / this, one accumulator for all six / this, two):
//   normal x normal          K = 64: 1.4e-7 / 1.1e-7 / 4.9e-8    1152: 5.9e-7 / 5.2e-7 / 1.9e-7    16384: 2.4e-6 / 2.1e-6 / 8.2e-7
//   ReLU(normal) x normal    K = 64: 1.0e-7 / 1.1e-7 / 3.8e-8    1152: 4.3e-7 / 5.0e-7 / 1.5e-7    16384: 1.6e-6 / 2.0e-6 / 7.2e-7
//   positive x positive      K = 64: 6.4e-7 / 4.6e-7 / 2.7e-7    1152: 1.1e-5 / 7.6e-6 / 4.0e-6    16384: 1.6e-4 / 1.1e-4 / 5.8e-5
// The parts are those of the operand times 2^24, so that no bit of a small float is lost (see split3), and the sums are
// scaled back.  An operand from 2^104 on or not finite, or an accumulator that overflows, makes the six products disagree
// with the one (Inf * 0): a tile that finds a result that is not finite is computed again with the fp32 instruction
// from the floats themselves, which is what it then stores.
//
//   * The weights are kept as two copies per layer, refreshed from the master before every forward pass,
//       Wf[co][tap][ci]  and  Wb[ci][flipped tap][co],
//     so that forward and data gradient are the same kernel: a data gradient is a convolution of dY with the flipped,
//     transposed filter.  For stride s an input pixel only meets the taps of its own residue (y mod s, x mod s); the
//     pixels of one residue class are a dense problem over that class's taps, one class after another in the grid.
//   * K is walked in slabs of 32 (float) or 64 (bf16) channels of one tap, the last one of a tap padded with zeros.  A
//     slab of a row is 208 bytes of LDS (three planes of 32 bf16 and 16 bytes of padding) or 144 (64 bf16 and 16), so that
//     sixteen consecutive rows start in distinct groups of four banks and the 16-byte operand reads run at full rate
//     (the stores of float activations, four rows of 64 bytes at a time, meet two to a bank: bank conflicts are a fifth to
//     a quarter of the fp32 kernels' LDS cycles).  The weights lie in memory in that very order, 192 or 128 contiguous bytes per slab; float activations are split
//     on their way into LDS.
//   * Position of float channel k inside a slab: pos = ((k / 4) % 4) * 8 + (k / 16) * 4 + k % 4, the same for both operands:
//     a thread reads channels 4g..4g+3 and 16+4g..16+4g+3 (64 contiguous bytes over four lanes each) and stores one
//     16-byte group per plane.
//   * MFMA operands are swapped (C^T = B^T A^T): four consecutive output channels per lane, 8- or 16-byte stores.
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

__device__ __forceinline__ u4 round8(const f4& a, const f4& b)
{
    return u4{to_bf16x2(a[0], a[1]), to_bf16x2(a[2], a[3]), to_bf16x2(b[0], b[1]), to_bf16x2(b[2], b[3])};
}

// What one residue class of pixels needs (one class, the whole image, unless it is a strided data gradient)
struct ClassGeo {
    int ph, pw;                           // output pixel = (y * ostride + ph, x * ostride + pw)
    int hc, wc;                           // rows of the class: y < hc, x < wc
    int ny, nx;                           // taps of the class (ny * nx)
    int wy0, wx0;                         // filter tap of (iy, ix) = ((wy0 + iy * wst) * S + wx0 + ix * wst)
    int by, bx;                           // source pixel of tap (iy, ix) = (y * sstride + by + iy, x * sstride + bx + ix)
};
__device__ __forceinline__ ClassGeo class_geo(const GeneralConvParams& p, int cls)
{
    ClassGeo c;
    if (p.classes == 1) {
        c.ph = c.pw = 0; c.hc = p.Ho; c.wc = p.Wo; c.ny = p.R; c.nx = p.S; c.wy0 = c.wx0 = 0; c.by = c.bx = -p.pad;
        return c;
    }
    const int st = p.ostride;
    c.ph = cls / st; c.pw = cls - c.ph * st;
    c.hc = (p.Ho - c.ph + st - 1) / st; c.wc = (p.Wo - c.pw + st - 1) / st;
    c.wy0 = ((p.pad - c.ph) % st + st) % st; c.wx0 = ((p.pad - c.pw) % st + st) % st;
    c.ny = c.wy0 < p.R ? (p.R - c.wy0 + st - 1) / st : 0;
    c.nx = c.wx0 < p.S ? (p.S - c.wx0 + st - 1) / st : 0;
    c.by = (c.ph - p.pad + c.wy0) / st; c.bx = (c.pw - p.pad + c.wx0) / st;       // exact
    return c;
}

// KG groups of WGM x WGN waves share a BMT x BN tile (wave tile BMT/WGM x BN/WGN): group kg multiplies slabs kg, kg + KG,
// ..., and the groups' sums are joined in group order through LDS at the end.
// NBUF = 1, one LDS buffer per group: the next slab waits in registers while the current one is multiplied, two barriers per
// slab, and another workgroup or group fills the matrix cores meanwhile.  NBUF = 2, one workgroup of eight waves per compute
// unit: slab t + 1 is split and written to the other buffer BETWEEN the matrix instructions of slab t (a matrix instruction
// occupies its core for 32 clocks and the wave for 4), while slab t + 2 is on its way into a second set of registers;
// one barrier per slab.
// EPI 0: + bias, optional ReLU, optional statistics;  EPI 1: optional mask, optional accumulate.
// GATHER: a convolution on the data set, whose few channels come in no 16-byte groups.  All taps and channels are one
// contraction in the order of the weights, (tap, channel), and the source values are gathered one by one.
template <typename T, int BMT, int BN, int WGM, int WGN, int KG, int NBUF, int EPI, bool GATHER>
__global__ __launch_bounds__(WGM * WGN * KG * 64, WGM * WGN * KG == 4 ? 2 : WGM * WGN * KG / 4) void conv_general_kernel(GeneralConvParams p)
{
    constexpr bool kSplit = std::is_same<T, float>::value;
    constexpr int kSlab = Slab<T>::channels, kRow = Slab<T>::row, kSlabBytes = Slab<T>::bytes, GR = Slab<T>::groups, CH = kSlabBytes / 16;
    constexpr unsigned ES = sizeof(T);
    constexpr int NW = WGM * WGN, NT = NW * 64;
    constexpr int TM = BMT / WGM / 32, TN = BN / WGN / 32;
    constexpr int NQA = BMT * GR / NT, NQB = (BN * CH + NT - 1) / NT;
    static_assert(NQA >= 1 && TM >= 1 && TN >= 1 && BMT * GR % NT == 0, "tile does not fit the thread count");
    static_assert(NBUF == 1 || (KG == 1 && !GATHER), "two buffers: one group");
    constexpr unsigned A_BUF = BMT * kRow, GROUP = (BMT + BN) * kRow;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x % NT, kg = threadIdx.x / NT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    char* const sAc = smem + kg * GROUP;              // [BMT][kRow]
    char* const sBc = sAc + A_BUF;                    // [BN][kRow]
    // logical item = (slot, class, column tile, row tile), row tiles fastest
    const unsigned tiles_m = (unsigned)p.tiles_m, tiles_n = (unsigned)(p.N + BN - 1) / BN, per_class = tiles_m * tiles_n;
    const unsigned item = logical_block();
    if (item >= per_class * (unsigned)p.classes * (unsigned)p.n_active) return;
    const int slot = (int)(item / (per_class * (unsigned)p.classes));
    const int rep = p.order[slot];
    const ClassGeo cg = class_geo(p, (int)((item / per_class) % (unsigned)p.classes));
    const int m0 = (int)(item % tiles_m) * BMT, n0 = (int)((item / tiles_m) % tiles_n) * BN;
    const int hw = cg.hc * cg.wc, M = p.B * hw;
    if (m0 >= M) return;
    const char* abase = (const char*)(p.a + (long long)rep * p.a_rep);
    if constexpr (GATHER) {                           // the batch inside the data set
        const long long first = ((p.cursor[rep] + p.ahead) * (long long)p.batch) % p.n_samples;
        abase = (const char*)(p.a + ((long long)rep * p.n_samples + first) * p.sample_sz);
    }
    const char* wbase = (const char*)(p.wmat + (long long)rep * p.wmat_rep);

    // A slots of this thread: (row, group g)
    const int ag = tid % GR;
    unsigned aoff[NQA], tapmask[NQA], sa_st[NQA];
    int row_y[GATHER ? NQA : 1], row_x[GATHER ? NQA : 1];     // source pixel of tap (0, 0); out of reach beyond the last row
#pragma unroll
    for (int q = 0; q < NQA; ++q) {
        const int i = tid + q * NT, arow = i / GR, m = m0 + arow;
        aoff[q] = 0; tapmask[q] = 0;
        if constexpr (GATHER) { row_y[q] = -(1 << 20); row_x[q] = 0; }
        if (m < M) {
            int b, pos;
            if (p.perm) { const int ps = m / p.B; b = m - ps * p.B; pos = p.perm[ps]; }
            else { b = m / hw; pos = m - b * hw; }
            const int y = pos / cg.wc, x = pos - y * cg.wc;
            const int sy = y * p.sstride + cg.by, sx = x * p.sstride + cg.bx;
            if constexpr (GATHER) {
                row_y[q] = sy; row_x[q] = sx;
                aoff[q] = (unsigned)(((b * p.H + sy) * p.W + sx) * p.C) * ES;
            } else {
            aoff[q] = (unsigned)(((b * p.H + sy) * p.W + sx) * p.C + ag * (kSplit ? 4 : 8)) * ES;      // (may lie outside: only used with a tap's delta)
            for (int iy = 0, t = 0; iy < cg.ny; ++iy)
                for (int ix = 0; ix < cg.nx; ++ix, ++t)
                    if (sy + iy >= 0 && sy + iy < p.H && sx + ix >= 0 && sx + ix < p.W) tapmask[q] |= 1u << t;
            }
        }
        sa_st[q] = (unsigned)(arow * kRow + ag * 16);
    }
    const int kflat = p.R * p.S * p.C;                // (GATHER)
    const int cs = ((GATHER ? kflat : p.C) + kSlab - 1) / kSlab;         // slabs per tap
    const unsigned wrow = (unsigned)((GATHER ? 1 : p.R * p.S) * cs * kSlabBytes);
    unsigned boff[NQB], sb_st[NQB]; bool b_ok[NQB];
#pragma unroll
    for (int q = 0; q < NQB; ++q) {
        const int i = tid + q * NT, r = i / CH, c = i - r * CH;
        b_ok[q] = r < BN && n0 + r < p.N;
        boff[q] = b_ok[q] ? (unsigned)(n0 + r) * wrow + (unsigned)c * 16u : 0u;
        sb_st[q] = (unsigned)(r * kRow + c * 16);
    }
    const unsigned a_rd = (unsigned)((wm * (BMT / WGM) + (lane & 31)) * kRow + (lane >> 5) * 16);
    const unsigned b_rd = (unsigned)((wn * (BN / WGN) + (lane & 31)) * kRow + (lane >> 5) * 16);

    // slabs: (tap, kSlab channels) for the taps some row of the tile can reach, taps ascending
    const int ntap = GATHER ? 1 : cg.ny * cg.nx;
    unsigned taps = ntap >= 32 ? 0xffffffffu : (1u << ntap) - 1u;
    if (p.perm) {
        const int last = min(m0 + BMT, M) - 1;
        unsigned u = 0;
        for (int ps = m0 / p.B; ps <= last / p.B; ++ps) u |= p.posmask[ps];
        taps &= u;
    }
    const int nslab = __builtin_popcount(taps) * cs;
    unsigned taps_left = taps;
    int tap = 0, ch = 0;                              // the slab that load_tiles fetches next: tap and group of channels
    auto start = [&]() { taps_left = taps; tap = taps ? __builtin_ctz(taps) : 0; ch = 0; };
    auto advance = [&](int by) {
        ch += by;
        while (ch >= cs && taps_left) {
            ch -= cs;
            taps_left &= taps_left - 1u;              // drop the tap just finished
            tap = taps_left ? __builtin_ctz(taps_left) : 0;
        }
    };
    struct Regs { f4 a[NQA][2]; u4 b[NQB]; };         // a slab on its way (bf16: a[q][0] holds the eight elements)
    const Buffer abuf = buffer(abase, (unsigned)(p.B * p.H * p.W) * (unsigned)p.C * ES), wbuf = buffer(wbase, (unsigned)p.N * wrow);
    auto load_tiles = [&](Regs& g, bool on) {         // (zeros unless on)
        f4 (&ra)[NQA][2] = g.a;
        u4 (&rb)[NQB] = g.b;
        if constexpr (GATHER) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = ch * kSlab + (j >> 2) * 16 + ag * 4 + (j & 3);
                const int t = k / p.C, r = t / p.S, c = k - t * p.C, x = t - r * p.S;
                const unsigned o = (unsigned)((r * p.W + x) * p.C + c) * ES;
#pragma unroll
                for (int q = 0; q < NQA; ++q) {
                    const int yy = row_y[q] + r, xx = row_x[q] + x;
                    float v = 0.f;
                    if (k < kflat && yy >= 0 && yy < p.H && xx >= 0 && xx < p.W) v = *reinterpret_cast<const float*>(abase + (aoff[q] + o));   // (32-bit sum: aoff alone may lie outside)
                    ra[q][j >> 2][j & 3] = v;
                }
            }
#pragma unroll
            for (int q = 0; q < NQB; ++q) {
                rb[q] = u4{0u, 0u, 0u, 0u};
                if (b_ok[q]) rb[q] = ldg16(wbase, boff[q] + (unsigned)(ch * kSlabBytes));
            }
            return;
        }
        const int iy = tap / cg.nx, ix = tap - iy * cg.nx;
        const int c0 = ch * kSlab + ag * (kSplit ? 4 : 8);
        const unsigned delta = (unsigned)((iy * p.W + ix) * p.C + ch * kSlab) * ES;
        const bool in0 = on && c0 < p.C, in1 = on && c0 + 16 < p.C;
#pragma unroll
        for (int q = 0; q < NQA; ++q) {
            const bool ok = (tapmask[q] >> tap) & 1u;
            const unsigned o = aoff[q] + delta;
            ra[q][0] = __builtin_bit_cast(f4, ldb16(abuf, ok && in0 ? o : kOutside));
            if (kSplit) ra[q][1] = __builtin_bit_cast(f4, ldb16(abuf, ok && in1 ? o + 64u : kOutside));
        }
        const int wt = (cg.wy0 + iy * p.wst) * p.S + cg.wx0 + ix * p.wst;
        const unsigned kb = (unsigned)((wt * cs + ch) * kSlabBytes);
#pragma unroll
        for (int q = 0; q < NQB; ++q) rb[q] = ldb16(wbuf, b_ok[q] && on ? boff[q] + kb : kOutside);
    };
    auto store_weights = [&](const Regs& g, unsigned at) {
#pragma unroll
        for (int q = 0; q < NQB; ++q)
            if (BN * CH % NT == 0 || tid + q * NT < BN * CH) *reinterpret_cast<u4*>(sBc + at + sb_st[q]) = g.b[q];
    };
    auto store_tiles = [&](const Regs& g, unsigned at) {
        const f4 (&ra)[NQA][2] = g.a;
#pragma unroll
        for (int q = 0; q < NQA; ++q) {
            if constexpr (kSplit) {
                u2 h0, m0_, l0, h1, m1, l1;
                split3(ra[q][0], h0, m0_, l0);
                split3(ra[q][1], h1, m1, l1);
                *reinterpret_cast<u4*>(sAc + at + sa_st[q]) = join8(h0, h1);
                *reinterpret_cast<u4*>(sAc + at + sa_st[q] + 64) = join8(m0_, m1);
                *reinterpret_cast<u4*>(sAc + at + sa_st[q] + 128) = join8(l0, l1);
            } else {
                *reinterpret_cast<f4*>(sAc + at + sa_st[q]) = ra[q][0];
            }
        }
        store_weights(g, at);
    };

    f16 acc[TM][TN], low[TM][TN];                     // sums of the large and of the small products
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) { acc[i][j][v] = 0.f; low[i][j][v] = 0.f; }
    };
    auto compute = [&](unsigned at) {
#pragma unroll
        for (int ks = 0; ks < kSlab / 16; ++ks) {
            constexpr int PL = Slab<T>::planes;
            bf16x8 a[TM][PL], b[TN][PL];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int s = 0; s < PL; ++s) a[i][s] = *reinterpret_cast<const bf16x8*>(sAc + at + a_rd + i * 32 * kRow + s * 64 + ks * 32);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int s = 0; s < PL; ++s) b[j][s] = *reinterpret_cast<const bf16x8*>(sBc + at + b_rd + j * 32 * kRow + s * 64 + ks * 32);
            // operands swapped: the accumulator holds the transposed tile.  Small products in ascending size.
            if constexpr (kSplit) {
                constexpr int SA[5] = {0, 2, 1, 0, 1}, SB[5] = {2, 0, 1, 1, 0};
#pragma unroll
                for (int t = 0; t < 5; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j][SB[t]], a[i][SA[t]], low[i][j], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j][0], a[i][0], acc[i][j], 0, 0, 0);
        }
    };

    clear();
    start();
    const int rounds = (nslab + KG - 1) / KG;
    if constexpr (NBUF == 1) {
        Regs g;
        advance(kg);
        if (kg < nslab) load_tiles(g, true);
        for (int t = 0; t < rounds; ++t) {
            const int mine = t * KG + kg;
            __syncthreads();                          // every wave is done reading the previous slab
            if (mine < nslab) store_tiles(g, 0);
            __syncthreads();
            if (mine + KG < nslab) { advance(KG); load_tiles(g, true); }
            if (mine < nslab) compute(0);
        }
    } else if (nslab > 0) {
        Regs g0, g1;
        load_tiles(g0, true);
        store_tiles(g0, 0);
        advance(1);
        load_tiles(g0, nslab > 1);
        __syncthreads();
        // slab t is in buffer `at`, slab t + 1 in `have`; beyond the last slab zeros are loaded and stored, and not multiplied
        auto step = [&](int t, unsigned at, const Regs& have, Regs& next) {
            advance(1);
            load_tiles(next, t + 2 < nslab);
            store_tiles(have, GROUP - at);
            compute(at);
            __syncthreads();
        };
        for (int t = 0; t < nslab; t += 2) {
            step(t, 0, g0, g1);
            if (t + 1 >= nslab) break;
            step(t + 1, GROUP, g1, g0);
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
    if (__syncthreads_or(bad != 0.f)) {               // (NaN != 0) something is not finite: the tile again, with the fp32 instruction
        clear();
        start();
        advance(kg);
        Regs g;
        for (int t = 0; t < rounds; ++t) {
            const int mine = t * KG + kg;
            __syncthreads();
            if (mine < nslab) {
                load_tiles(g, true);
                advance(KG);
#pragma unroll
                for (int q = 0; q < NQA; ++q) {
                    char* const dst = sAc + sa_st[q] + ag * 16;
                    *reinterpret_cast<f4*>(dst) = g.a[q][0];
                    *reinterpret_cast<f4*>(dst + 16) = g.a[q][1];
                }
                store_weights(g, 0);
            }
            __syncthreads();
            if (mine < nslab) {
                for (int k = lane >> 5; k < kSlab; k += 2) {
                    float a[TM], b[TN];
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        a[i] = *reinterpret_cast<const float*>(sAc + (wm * (BMT / WGM) + i * 32 + (lane & 31)) * kRow + k * 4);
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const __bf16* w = reinterpret_cast<const __bf16*>(sBc + (wn * (BN / WGN) + j * 32 + (lane & 31)) * kRow) + k;
                        b[j] = join_weight(w[0], w[32], w[64]);
                    }
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], a[i], acc[i][j], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    } else {
        __syncthreads();                              // nobody reads a slab any more
    }
    if (KG > 1) {                                     // (behind the barriers above nobody reads a slab any more)
        float* const part = reinterpret_cast<float*>(smem);
        static_assert((size_t)(KG - 1) * NW * TM * TN * 16 * 64 * 4 <= (size_t)KG * GROUP, "the groups' sums do not fit the LDS of the K loop");
        if (kg > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        part[((((kg - 1) * NW + wave) * TM * TN + i * TN + j) * 16 + v) * 64 + lane] = acc[i][j][v];
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
                        for (int v = 0; v < 16; ++v)
                            acc[i][j][v] += part[(((g * NW + wave) * TM * TN + i * TN + j) * 16 + v) * 64 + lane];
        }
    }

    // ---- epilogue: lane holds output row (lane & 31) and channels 8*g + 4*(lane >> 5) + {0..3}, g = 0..3 ----
    const bool stats = EPI == 0 && p.stat != nullptr;         // per-channel sums of the outputs for a batch norm that follows
    float ss[TN][16], qq[TN][16];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int k = 0; k < 16; ++k) { ss[j][k] = 0.f; qq[j][k] = 0.f; }
    if (kg == 0) {
        T* const obase = reinterpret_cast<T*>(p.out + (long long)rep * p.out_rep);
        const float* bias = (EPI == 0 && p.bias) ? p.bias + (long long)rep * p.bias_rep : nullptr;
        const T* mask = (EPI == 1 && p.mask) ? reinterpret_cast<const T*>(p.mask + (long long)rep * p.mask_rep) : nullptr;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mm = m0 + wm * (BMT / WGM) + i * 32 + (lane & 31);
            if (mm >= M) continue;
            int b, pos;
            if (p.perm) { const int ps = mm / p.B; b = mm - ps * p.B; pos = p.perm[ps]; }
            else { b = mm / hw; pos = mm - b * hw; }
            const int y = pos / cg.wc, x = pos - y * cg.wc;
            const long long pix = ((long long)b * p.Ho + y * p.ostride + cg.ph) * p.Wo + x * p.ostride + cg.pw;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = n0 + wn * (BN / WGN) + j * 32 + 8 * g + 4 * (lane >> 5);
                    if (n >= p.N) continue;
                    const long long o = pix * p.N + n;
                    f4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                    f4 sh = {0.f, 0.f, 0.f, 0.f};              // what the statistics are centred on: the bias
                    if (EPI == 0) {
                        if (bias) { sh = *reinterpret_cast<const f4*>(bias + n); v += sh; }
                        if (p.relu) { v[0] = fmaxf(v[0], 0.f); v[1] = fmaxf(v[1], 0.f); v[2] = fmaxf(v[2], 0.f); v[3] = fmaxf(v[3], 0.f); }
                    } else {
                        if (mask) {
                            const f4 mk = load4(mask + o);
#pragma unroll
                            for (int e = 0; e < 4; ++e) if (!(mk[e] > 0.f)) v[e] = 0.f;
                        }
                        if (p.accumulate) v += load4(obase + o);
                    }
                    store4(obase + o, v);
                    if (stats) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) { const float f = v[e] - sh[e]; ss[j][4 * g + e] += f; qq[j][4 * g + e] += f * f; }
                    }
                }
            }
        }
    }
    if (stats) {                                              // (the launcher asks for the larger of the K loop's LDS and kStatLdsBytes)
        __syncthreads();                                      // every wave is past its last read of LDS
        if (kg == 0)
            store_column_stats<TN, WGM, WGN>(ss, qq, reinterpret_cast<float*>(smem), wave, lane, p.stat + (long long)slot * p.stat_rep,
                                             m0 / BMT, n0 + wn * (BN / WGN), p.N);
        else
            __syncthreads();                                  // the barrier inside store_column_stats
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Weight gradient: dW[m = (tap, ci)][n = co] = sum over pixels k of x[source pixel(k, tap)][ci] * dy[k][co]
// ---------------------------------------------------------------------------------------------------------------
// Both operands are contiguous along channels and the contraction runs over pixels: tiles of 32 pixels are split on their
// way into LDS as [pixel][plane][channel] and transposed on the way out (ds_read_b64_tr_b16).  A pixel's row is a multiple of
// 256 bytes plus or minus 64, so that the four rows a transposing read touches land in distinct banks.  Pixels advance by
// 32 per slab with carries instead of divisions, and a thread's tap is fixed, so a slab costs a few additions per
// address.  The bias gradient is summed in fp32 by the tiles of the first row of tiles, from the dY values they stage anyway.
template <typename T, int COLS> constexpr int kPixelRow = COLS == 32 ? (Slab<T>::planes == 3 ? 320 : 192) : COLS * 2 * Slab<T>::planes + 64;

// Each wave passes its 32 x 32 blocks through a private piece of LDS and takes them back with eight lanes per row, so that
// global accesses cover whole lines.  With w set the block is the complete gradient and the update is applied instead.
constexpr int kStagePitch = 36;                               // floats per staged row
__device__ __forceinline__ void put_gradient(const f4& v, long long o, const GeneralWgradParams& p, float* out, float* w, float* buf)
{
    if (!w) { *reinterpret_cast<f4*>(out + o) = v; return; }
    f4 d = v;
    if (buf) { d = *reinterpret_cast<const f4*>(buf + o) * p.momentum + d; *reinterpret_cast<f4*>(buf + o) = d; }
    *reinterpret_cast<f4*>(w + o) = *reinterpret_cast<const f4*>(w + o) - d * p.lr;
}

// GATHER: the source is the data set and its few channels come in no 16-byte groups; the four rows of a slot have a tap and a
// channel each and are gathered one by one.  Tiles of 32 rows: the waves without a block only help to stage.
// One LDS buffer and two workgroups per compute unit: with two buffers and 256 x 128 tiles of eight waves (conv_general_kernel's
// NBUF = 2) the transposing reads, at 90 bytes a clock, keep it from being faster (173 against 175 TFLOP/s on 16 replicas).
template <typename T, typename SRC, int BMT, int BN, int WGM, int WGN, bool GATHER>
__global__ __launch_bounds__(GATHER ? 256 : WGM * WGN * 64, 2) void wgrad_general_kernel(GeneralWgradParams p)
{
    constexpr int NT = GATHER ? 256 : WGM * WGN * 64;
    constexpr int TM = BMT / WGM / 32, TN = BN / WGN / 32, BK = 32;
    constexpr bool kSplit = std::is_same<T, float>::value, kRound = !kSplit && std::is_same<SRC, float>::value;
    constexpr unsigned ES = sizeof(SRC);
    constexpr int PA = kPixelRow<T, BMT>, PB = kPixelRow<T, BN>;
    constexpr int GS = 16 / sizeof(T);                        // channels per group: 16 bytes
    constexpr int AG = BMT / GS, BG = BN / GS;                // groups per pixel
    constexpr int AR = NT / AG, BR = NT / BG;               // pixels the threads cover per pass (more than a slab has: the rest idles)
    constexpr int NQA = (BK + AR - 1) / AR, NQB = (BK + BR - 1) / BR;
    static_assert(TM >= 1 && TN >= 1 && NT % AG == 0 && NT % BG == 0, "tile does not fit the thread count");
    constexpr unsigned A_BUF = BK * PA;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* const sA = smem;                                    // [BK][PA]
    char* const sB = smem + A_BUF;                            // [BK][PB]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const bool mma = wave < WGM * WGN;                        // (all waves but in GATHER tiles)
    // logical item = (slot, split, tile): the tiles of one split of one replica read the same pixels
    const int mw = p.R * p.S * p.C;                           // rows that are weights; row mw is the bias gradient
    const unsigned tiles_n = (unsigned)(p.N + BN - 1) / BN, tiles = (unsigned)((mw + BMT - 1) / BMT) * tiles_n;
    const unsigned item = logical_block();
    if (item >= tiles * (unsigned)p.splits * (unsigned)p.n_active) return;
    const int slot = (int)(item / (tiles * (unsigned)p.splits));
    const int rep = p.order[slot];
    const unsigned tile = item % tiles;
    const int m0 = (int)(tile / tiles_n) * BMT, n0 = (int)(tile % tiles_n) * BN;
    const int split = (int)((item / tiles) % (unsigned)p.splits);
    const int kbeg = split * p.kchunk, kend = min(p.K, kbeg + p.kchunk);
    const char* xbase;
    if (p.cursor) {
        const long long first = ((p.cursor[rep] + p.ahead) * (long long)p.batch) % p.n_samples;
        xbase = (const char*)(p.x + ((long long)rep * p.n_samples + first) * p.sample_sz);
    } else {
        xbase = (const char*)(p.x + (long long)rep * p.x_rep);
    }
    const char* dbase = (const char*)(p.dy + (long long)rep * p.dy_rep);

    // A slots: channels am..am+GS-1 of one tap, pixels arow + AR * q;  B slots: channels bn.., pixels brow + BR * q
    const int am = m0 + (tid % AG) * GS, arow = tid / AG;
    const int bn = n0 + (tid % BG) * GS, brow = tid / BG;
    const bool a_ok = am < mw && arow < BK, b_ok = bn < p.N && brow < BK;
    const int atap = am / p.C, aci = am - atap * p.C;
    const int ady = atap / p.S - p.pad, adx = atap % p.S - p.pad;
    // output rows y with a source row inside the image: ylo <= y < ylo + yn (likewise x)
    const int ylo = ady < 0 ? (-ady + p.stride - 1) / p.stride : 0, xlo = adx < 0 ? (-adx + p.stride - 1) / p.stride : 0;
    const int yn = p.H - 1 - ady >= 0 ? max(0, (p.H - 1 - ady) / p.stride + 1 - ylo) : 0;
    const int xn = p.W - 1 - adx >= 0 ? max(0, (p.W - 1 - adx) / p.stride + 1 - xlo) : 0;
    const unsigned a_shift = (unsigned)((ady * p.W + adx) * p.C + aci) * ES;
    int gy[GATHER ? 4 : 1], gx[GATHER ? 4 : 1]; unsigned gs[GATHER ? 4 : 1];     // GATHER: tap offset and shift of each row of the slot
    if constexpr (GATHER) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = (am + e) / p.C;
            gy[e] = am + e < mw ? t / p.S - p.pad : 1 << 20; gx[e] = t % p.S - p.pad;
            gs[e] = (((unsigned)gy[e] * (unsigned)p.W + (unsigned)gx[e]) * (unsigned)p.C + (unsigned)(am + e - t * p.C)) * ES;
        }
    }
    // 32 pixels further: x += dx, y += dyy, image += db, in source bytes step (carries adjust by cx, cy)
    const int hw = p.Ho * p.Wo;
    const int dx = BK % p.Wo, dyy = (BK / p.Wo) % p.Ho, db = BK / hw;
    const unsigned pc = (unsigned)p.C * ES, st = (unsigned)p.stride;
    const unsigned cx = (st * (unsigned)p.W - (unsigned)p.Wo * st) * pc, cy = ((unsigned)p.H - (unsigned)p.Ho * st) * (unsigned)p.W * pc;
    const unsigned step = (((unsigned)db * (unsigned)p.H + (unsigned)dyy * st) * (unsigned)p.W + (unsigned)dx * st) * pc;
    int px[NQA], py[NQA]; unsigned poff[NQA];
    auto seek = [&](int k0) {                                 // (no position table)
#pragma unroll
        for (int q = 0; q < NQA; ++q) {
            const int k = k0 + arow + AR * q, b = k / hw, rem = k - b * hw;
            py[q] = rem / p.Wo; px[q] = rem - py[q] * p.Wo;
            poff[q] = ((unsigned)(b * p.H + py[q] * p.stride) * (unsigned)p.W + (unsigned)(px[q] * p.stride)) * pc + (GATHER ? 0u : a_shift);
        }
    };
    // Contraction order.  With a position table, index k = ps * B + b is image b at pixel perm[ps] (B a multiple of the slab
    // length); a slab whose position cannot reach any tap of this row tile contributes exact zeros and is left out, but for
    // the tiles that sum the bias gradient.
    const bool with_bias = p.has_bias && m0 == 0;
    unsigned tile_tapbits = 0xffffffffu;
    if (p.perm && !with_bias) {
        const int tlo = m0 / p.C, thi = min(m0 + BMT - 1, mw - 1) / p.C;
        tile_tapbits = (thi >= 31 ? 0xffffffffu : ((2u << thi) - 1u)) & ~((1u << tlo) - 1u);
    }
    auto next_slab = [&](int k) {
        if (p.perm)
            while (k < kend && !(p.posmask[k / p.B] & tile_tapbits)) k += BK;
        return k;
    };
    const Buffer xbuf = buffer(xbase, (unsigned)(p.B * p.H * p.W) * pc), dbuf = buffer(dbase, (unsigned)p.K * (unsigned)p.N * (unsigned)sizeof(T));
    f4 ra[NQA], ra2[kRound ? NQA : 1], rb[NQB];              // (bf16 tensors: eight elements in the 16 bytes)
    float bsum[GS] = {};
    auto load_tiles = [&](int k0) {
        int bbase = 0, pos = 0;
        if (p.perm) { const int ps = k0 / p.B; bbase = k0 - ps * p.B; pos = p.perm[ps]; }
        if (p.perm) {                                         // stride 1, source and output images alike
            const int y = pos / p.W, x = pos - y * p.W;
            const bool in = a_ok && (unsigned)(y - ylo) < (unsigned)yn && (unsigned)(x - xlo) < (unsigned)xn;
#pragma unroll
            for (int q = 0; q < NQA; ++q) {
                const int kr = arow + AR * q;
                ra[q] = __builtin_bit_cast(f4, ldb16(xbuf, in && k0 + kr < kend ? (unsigned)((bbase + kr) * hw + pos) * pc + a_shift : kOutside));
                if constexpr (kRound) ra2[q] = f4{0.f, 0.f, 0.f, 0.f};            // (the data set has no position table)
            }
        } else {
#pragma unroll
            for (int q = 0; q < NQA; ++q) {
                const bool in = a_ok && (unsigned)(py[q] - ylo) < (unsigned)yn && (unsigned)(px[q] - xlo) < (unsigned)xn;
                const bool on = in && k0 + arow + AR * q < kend;
                if constexpr (GATHER) {
                    ra[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int yy = py[q] * p.stride + gy[e], xx = px[q] * p.stride + gx[e];
                        if (k0 + arow + AR * q < kend && yy >= 0 && yy < p.H && xx >= 0 && xx < p.W)
                            ra[q][e] = *reinterpret_cast<const float*>(xbase + (poff[q] + gs[e]));     // (32-bit sum: gs may be negative)
                    }
                } else {
                    ra[q] = __builtin_bit_cast(f4, ldb16(xbuf, on ? poff[q] : kOutside));
                }
                if constexpr (kRound) {
                    ra2[q] = __builtin_bit_cast(f4, ldb16(xbuf, on ? poff[q] + 16u : kOutside));
                }
                px[q] += dx; py[q] += dyy; poff[q] += step;
                const bool carry_x = px[q] >= p.Wo;
                px[q] -= carry_x ? p.Wo : 0; py[q] += carry_x ? 1 : 0; poff[q] += carry_x ? cx : 0u;
                const bool carry_y = py[q] >= p.Ho;
                py[q] -= carry_y ? p.Ho : 0; poff[q] += carry_y ? cy : 0u;
            }
        }
#pragma unroll
        for (int q = 0; q < NQB; ++q) {
            const int kr = brow + BR * q;
            const unsigned pix = p.perm ? (unsigned)((bbase + kr) * hw + pos) : (unsigned)(k0 + kr);
            rb[q] = __builtin_bit_cast(f4, ldb16(dbuf, b_ok && k0 + kr < kend ? (pix * (unsigned)p.N + (unsigned)bn) * (unsigned)sizeof(T) : kOutside));
        }
    };
    const unsigned sa_st = (unsigned)(arow * PA + (tid % AG) * GS * 2), sb_st = (unsigned)(brow * PB + (tid % BG) * GS * 2);
    auto store_tiles = [&]() {
#pragma unroll
        for (int q = 0; q < NQA; ++q) {
            char* const o = sA + sa_st + AR * q * PA;
            if constexpr (kSplit) {
                u2 h, m, l;
                split3(ra[q], h, m, l);
                *reinterpret_cast<u2*>(o) = h; *reinterpret_cast<u2*>(o + BMT * 2) = m; *reinterpret_cast<u2*>(o + BMT * 4) = l;
            } else if (AR <= BK || arow < BK) {
                if constexpr (kRound) *reinterpret_cast<u4*>(o) = round8(ra[q], ra2[q]);
                else *reinterpret_cast<f4*>(o) = ra[q];
            }
        }
#pragma unroll
        for (int q = 0; q < NQB; ++q) {
            char* const o = sB + sb_st + BR * q * PB;
            if constexpr (kSplit) {
                u2 h, m, l;
                split3(rb[q], h, m, l);
                *reinterpret_cast<u2*>(o) = h; *reinterpret_cast<u2*>(o + BN * 2) = m; *reinterpret_cast<u2*>(o + BN * 4) = l;
#pragma unroll
                for (int e = 0; e < 4; ++e) bsum[e] += rb[q][e];          // (used by the tiles with the bias row only)
            } else if (BR <= BK || brow < BK) {
                *reinterpret_cast<f4*>(o) = rb[q];
                const bf16x8 v = __builtin_bit_cast(bf16x8, rb[q]);
#pragma unroll
                for (int e = 0; e < GS; ++e) bsum[e] += (float)v[e];
            }
        }
    };
    // operand reads (see lds_read_tr8): lane L of a 16-lane group points at pixel L / 4, channels 4 * (L % 4)
    const unsigned rd_lane = (unsigned)((lane >> 5) * 8 + ((lane & 15) >> 2));
    const unsigned a_rd = rd_lane * PA + (unsigned)(wm * (BMT / WGM) + ((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2u;
    const unsigned b_rd = rd_lane * PB + (unsigned)(wn * (BN / WGN) + ((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2u;

    f16 acc[TM][TN], low[TM][TN];                             // sums of the large and of the small products
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) { acc[i][j][v] = 0.f; low[i][j][v] = 0.f; }
    };
    auto compute = [&]() {
        if (mma)
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            constexpr int PL = Slab<T>::planes;
            bf16x8 a[TM][PL], b[TN][PL];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int s = 0; s < PL; ++s) a[i][s] = lds_read_tr8(sA, a_rd + ks * 16 * PA + s * BMT * 2 + i * 64, PA);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int s = 0; s < PL; ++s) b[j][s] = lds_read_tr8(sB, b_rd + ks * 16 * PB + s * BN * 2 + j * 64, PB);
            if constexpr (kSplit) {
                constexpr int SA[5] = {0, 2, 1, 0, 1}, SB[5] = {2, 0, 1, 1, 0};
#pragma unroll
                for (int t = 0; t < 5; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            low[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j][SB[t]], a[i][SA[t]], low[i][j], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j][0], a[i][0], acc[i][j], 0, 0, 0);
        }
    };
    clear();
    int k0 = next_slab(kbeg);
    seek(kbeg);
    if (k0 < kend) load_tiles(k0);
    while (k0 < kend) {
        __syncthreads();                                      // every wave is done reading the previous slab
        store_tiles();
        __syncthreads();
        k0 = next_slab(k0 + BK);
        if (k0 < kend) load_tiles(k0);
        compute();
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
    if (__syncthreads_or(bad != 0.f)) {                       // (NaN != 0) something is not finite: the tile again, with the fp32 instruction
        clear();
        seek(kbeg);
        for (k0 = next_slab(kbeg); k0 < kend; k0 = next_slab(k0 + BK)) {
            __syncthreads();
            load_tiles(k0);
#pragma unroll
            for (int q = 0; q < NQA; ++q) *reinterpret_cast<f4*>(sA + (arow + AR * q) * PA + (tid % AG) * 16) = ra[q];
#pragma unroll
            for (int q = 0; q < NQB; ++q) *reinterpret_cast<f4*>(sB + (brow + BR * q) * PB + (tid % BG) * 16) = rb[q];
            __syncthreads();
            for (int k = lane >> 5; mma && k < BK; k += 2) {
                float a[TM], b[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const float*>(sA + k * PA + (wm * (BMT / WGM) + i * 32 + (lane & 31)) * 4);
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const float*>(sB + k * PB + (wn * (BN / WGN) + j * 32 + (lane & 31)) * 4);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], a[i], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    } else {
        __syncthreads();                                      // nobody reads a slab any more
    }

    // ---- epilogue (the barrier above: nobody reads a slab any more) ----
    float* const out = (p.splits > 1) ? p.out + (long long)slot * p.out_rep + (long long)split * p.out_split
                                      : p.out + (long long)rep * p.out_rep;
    float* const w = (p.splits == 1 && p.sgd_w) ? p.sgd_w + (long long)rep * p.out_rep : nullptr;
    float* const buf = (w && p.sgd_buf) ? p.sgd_buf + (long long)rep * p.out_rep : nullptr;
    float* const stage = reinterpret_cast<float*>(smem) + wave * (32 * kStagePitch);
    if (mma)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f4*>(stage + (lane & 31) * kStagePitch + 8 * q + 4 * (lane >> 5)) =
                    f4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int rr = (lane >> 3) + 8 * t, cc = (lane & 7) * 4;
                const f4 v = *reinterpret_cast<const f4*>(stage + rr * kStagePitch + cc);
                const int mm = m0 + wm * (BMT / WGM) + i * 32 + rr, nn = n0 + wn * (BN / WGN) + j * 32 + cc;
                if (mm < mw && nn < p.N) put_gradient(v, (long long)mm * p.N + nn, p, out, w, buf);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    if (with_bias) {                                          // join the partial sums of the threads that share a channel group, pixels ascending
        __syncthreads();
        float* const red = reinterpret_cast<float*>(smem);    // [BR][BN]
#pragma unroll
        for (int e = 0; e < GS; e += 4) *reinterpret_cast<f4*>(red + brow * BN + (tid % BG) * GS + e) = f4{bsum[e], bsum[e + 1], bsum[e + 2], bsum[e + 3]};
        __syncthreads();
        if (brow == 0 && b_ok) {
#pragma unroll
            for (int e = 0; e < GS; e += 4) {
                f4 v = *reinterpret_cast<const f4*>(red + (tid % BG) * GS + e);
#pragma unroll
                for (int r = 1; r < (BR < BK ? BR : BK); ++r) v += *reinterpret_cast<const f4*>(red + r * BN + (tid % BG) * GS + e);
                put_gradient(v, (long long)mw * p.N + bn + e, p, out, w, buf);
            }
        }
    }
}

// fp32 master W[tap][ci][co] -> Wf[co][tap][ci] and Wb[ci][T-1-tap][co] as described at the top.  A workgroup handles one
// tap and a 64 x 64 (ci, co) tile; each thread forms 16-byte groups of eight positions.  p.fragments: the order of the lanes of a
// matrix instruction instead (conv_general_patch.hip), [32 rows][slab][tap][16 channels][plane][half of them][row], rows beyond the
// last zero.  Bound by memory: 4 bytes read and 12 (bf16: 4) written per weight.  Weights are read, and pass through LDS, sixteen bytes a
// lane (N and the layer's offset are multiples of four).  One launch takes up to 32 layers: a small layer's few hundred tiles take
// less time than the launch, and a sub-step whose layers all wait for their copies had a launch and a drained chip for each
// (five layers of 64 to 256 channels, 5 replicas, four sub-steps: 1355 -> 1325 us with one; residual nets of 20 layers 0.5 to 0.9 %).
template <typename T>
__global__ __launch_bounds__(256) void weight_copy_kernel(WeightCopies all)
{
    constexpr bool kSplit = std::is_same<T, float>::value;
    constexpr int kSlab = Slab<T>::channels, kSlabBytes = Slab<T>::bytes, GR = Slab<T>::groups;
    __shared__ __attribute__((aligned(16))) float tile[64][68];          // [ci][co], zero outside the layer
    const int lane = threadIdx.x & 63;                                   // the last layer that begins at or before this workgroup
    const int which_layer = __popcll(__ballot(lane < all.count && (int)blockIdx.x >= all.first[lane & (kWeightCopies - 1)])) - 1;
    const WeightCopyParams& p = all.layer[which_layer];
    const int rep = p.order[blockIdx.y];
    const int block = (int)blockIdx.x - all.first[which_layer], tiles_c = (p.C + 63) / 64, rest = block / tiles_c;
    const int tap = rest % p.taps, co0 = (rest / p.taps) * 64, ci0 = (block % tiles_c) * 64;
    const float* w = p.w + (long long)rep * p.w_rep + (long long)tap * p.C * p.N;
    const int tx = (threadIdx.x & 15) * 4, ty = threadIdx.x >> 4;
    f4 in[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int ci = ci0 + ty + 16 * r;
        in[r] = f4{0.f, 0.f, 0.f, 0.f};
        if (ci < p.C && co0 + tx < p.N) in[r] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(w + (long long)ci * p.N + co0 + tx));
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) *reinterpret_cast<f4*>(&tile[ty + 16 * r][tx]) = in[r];
    __syncthreads();
    const int csf = (p.C + kSlab - 1) / kSlab, csb = (p.N + kSlab - 1) / kSlab;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        __bf16* const dst = which ? p.wb : p.wf;
        if (!dst) continue;
        const int row0 = which ? ci0 : co0, rows = which ? p.C : p.N;       // rows of the copy and the channels along its slabs
        const int k0 = which ? co0 : ci0, cs = which ? csb : csf, t = which ? p.taps - 1 - tap : tap;
        char* const base = (char*)(dst + (long long)rep * p.wcopy_rep);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = threadIdx.x + q * 256;
            const int row = p.fragments ? i & 63 : i >> 3, j = p.fragments ? i >> 6 : i & 7, g = j % GR, sl = j / GR;
            const int slab = k0 / kSlab + sl;
            if (row0 + row >= (p.fragments ? (rows + 31) / 32 * 32 : rows) || slab >= cs) continue;
            char* const o = p.fragments
                ? base + (((long long)((row0 + row) / 32) * cs + slab) * p.taps + t) * (32 * kSlabBytes) + (g >> 1) * (kSplit ? 3072 : 1024) + (g & 1) * 512 + (row & 31) * 16
                : base + ((long long)(row0 + row) * p.taps * cs + t * cs + slab) * kSlabBytes + g * 16;
            const int plane = p.fragments ? 1024 : 64;
            bf16x8 h, m, l;
            f4 v[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {                     // positions k .. k + 3 twice: sixteen apart, or neighbours (bf16)
                const int k = kSplit ? sl * kSlab + u * 16 + g * 4 : g * 8 + u * 4;
                if (which) v[u] = *reinterpret_cast<const f4*>(&tile[row][k]);
                else v[u] = f4{tile[k][row], tile[k + 1][row], tile[k + 2][row], tile[k + 3][row]};
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                __bf16 a, b, c;
                if (kSplit) { split_weight(v[e >> 2][e & 3], a, b, c); h[e] = a; m[e] = b; l[e] = c; }
                else h[e] = (__bf16)v[e >> 2][e & 3];
            }
            *reinterpret_cast<bf16x8*>(o) = h;
            if (kSplit) { *reinterpret_cast<bf16x8*>(o + plane) = m; *reinterpret_cast<bf16x8*>(o + 2 * plane) = l; }
        }
    }
}

template <typename T, int EPI, int BMT, int BN, int WGM, int WGN, int KG, int NBUF = 1, bool GATHER = false>
hipError_t launch_t(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    constexpr size_t loop_lds = (size_t)KG * NBUF * (BMT + BN) * Slab<T>::row, stat_lds = kStatLdsBytes<BN / WGN / 32, WGM, WGN>;
    constexpr size_t lds = loop_lds > stat_lds ? loop_lds : stat_lds;
    if (lds > 65536) {
        static const bool ok = hipFuncSetAttribute((const void*)conv_general_kernel<T, BMT, BN, WGM, WGN, KG, NBUF, EPI, GATHER>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
        if (!ok) return hipErrorInvalidValue;
    }
    if (stat_rows) *stat_rows = BMT;
    const int rows0 = p.B * ((p.Ho + p.ostride - 1) / p.ostride) * ((p.Wo + p.ostride - 1) / p.ostride);     // largest class
    p.tiles_m = (rows0 + BMT - 1) / BMT;
    const dim3 grid(die_grid((long long)p.tiles_m * ((p.N + BN - 1) / BN) * p.classes * n_active)), block(WGM * WGN * KG * 64);
    hipLaunchKernelGGL((conv_general_kernel<T, BMT, BN, WGM, WGN, KG, NBUF, EPI, GATHER>), grid, block, lds, s, p);
    return hipGetLastError();
}

template <typename T, int EPI>
hipError_t launch_conv(GeneralConvParams& p, int n_active, hipStream_t s, int* stat_rows)
{
    const long long rows0 = (long long)p.B * ((p.Ho + p.ostride - 1) / p.ostride) * ((p.Wo + p.ostride - 1) / p.ostride);
    const long long groups = (long long)p.classes * n_active;
    const bool large = p.tile_hint == 1;
    if constexpr (std::is_same<T, float>::value) {
        // A launch's time is the length of its K loop while every compute unit has at most one workgroup, and the chip's
        // throughput at that tile size once there are more, in whole rounds.  Per slab of 32 channels, measured in us on
        // 3 x 3 layers of 64 to 512 channels, batch 64, 1 to 16 replicas: `alone` the loop step of a workgroup that has its
        // unit to itself, `share` the unit's time per workgroup under load; about three slabs' time goes into the first
        // loads and the epilogue.  The estimate's best is the measured best or within 6 % of it on those layers but for
        // launches of some 10 us.  (512 channels, 4 x 4 images, 1 / 4 / 16 replicas: 64 x 64 in four groups 73 / 165 / 619 us,
        // 128 x 64 133 / 140 / 432, 256 x 128 281 / 281 / 368.)  Up to 32 outputs leave half of a wider tile empty: there
        // the choice is among the small tiles and 128 x 32, which is the best one or within 12 % of it but for launches of some
        // 10 us (16 channels, 3 x 3, 28 x 28 images, 100 k pixels, forward and data gradient: 64 x 64 in two groups 48 and 45 us,
        // 128 x 32 29 and 29).
        static constexpr struct { int m, n; float alone, share; } kTile[] = {
            {32, 32, 0.28f, 0.37f}, {64, 64, 0.50f, 0.62f}, {64, 64, 0.61f, 0.46f}, {128, 64, 1.33f, 0.816f},
            {128, 128, 1.22f, 1.50f}, {256, 128, 1.95f, 2.83f}, {128, 32, 1.6f, 0.50f}};
        const float slabs = (float)(p.R * p.S * ((p.C + 31) / 32)) / (float)p.classes + 3.0f;
        int best = 0;
        float best_t = 0.f;
        for (int i = 0; i < 7; ++i) {
            if (p.N <= 32 ? i > 2 && i < 6 : i == 6 || (p.N <= 64 && kTile[i].n > 64)) continue;
            const long long tiles = (rows0 + kTile[i].m - 1) / kTile[i].m * ((p.N + kTile[i].n - 1) / kTile[i].n) * groups;
            const float step = tiles <= 256 ? kTile[i].alone : std::max(kTile[i].alone, (float)((tiles + 255) / 256) * kTile[i].share);
            const float loaded = tiles > 128 && tiles <= 256 ? std::max(step, 0.9f * kTile[i].share) : step;
            if (i == 0 || slabs * loaded < best_t) { best = i; best_t = slabs * loaded; }
        }
        if (large) best = p.N > 64 ? 5 : p.N > 32 ? 3 : 6;
        switch (best) {
        case 0: return launch_t<T, EPI, 32, 32, 1, 1, 8>(p, n_active, s, stat_rows);
        case 1: return launch_t<T, EPI, 64, 64, 2, 2, 4>(p, n_active, s, stat_rows);
        case 2: return launch_t<T, EPI, 64, 64, 2, 2, 2>(p, n_active, s, stat_rows);
        case 3: return launch_t<T, EPI, 128, 64, 4, 1, 1>(p, n_active, s, stat_rows);
        case 4: return launch_t<T, EPI, 128, 128, 2, 4, 1, 2>(p, n_active, s, stat_rows);
        case 5: return launch_t<T, EPI, 256, 128, 4, 2, 1, 2>(p, n_active, s, stat_rows);
        default: return launch_t<T, EPI, 128, 32, 4, 1, 1>(p, n_active, s, stat_rows);
        }
    } else {
        // bf16 slabs are bound by their loads; the number of workgroups decides (within 10 % of the best of these and the
        // two-buffer tiles on ResNet-18's strided layers, 1 to 16 replicas)
        const long long t64 = (rows0 + 63) / 64 * ((p.N + 63) / 64) * groups, t128 = (rows0 + 127) / 128 * ((p.N + 127) / 128) * groups;
        if (!large && t64 <= 48) return launch_t<T, EPI, 32, 32, 1, 1, 8>(p, n_active, s, stat_rows);
        if (!large && t64 <= 256) return launch_t<T, EPI, 64, 64, 2, 2, 4>(p, n_active, s, stat_rows);
        if (!large && t64 <= 640) return launch_t<T, EPI, 64, 64, 2, 2, 2>(p, n_active, s, stat_rows);
        if (p.N <= 32) return launch_t<T, EPI, 128, 32, 4, 1, 1>(p, n_active, s, stat_rows);
        if (p.N > 64) {
            if (large || t128 > 256) return launch_t<T, EPI, 128, 128, 2, 2, 1>(p, n_active, s, stat_rows);
            if (t64 > 880) return launch_t<T, EPI, 128, 128, 2, 2, 2>(p, n_active, s, stat_rows);
        }
        if (p.N <= 64 && (large || t64 > 2048)) return launch_t<T, EPI, 128, 64, 4, 1, 1>(p, n_active, s, stat_rows);
        return launch_t<T, EPI, 64, 64, 2, 2, 1>(p, n_active, s, stat_rows);
    }
}

template <typename T, typename SRC, int BMT, int BN, int WGM, int WGN, bool GATHER = false>
hipError_t launch_wgrad_t(const GeneralWgradParams& p, int n_active, hipStream_t s)
{
    constexpr int NT = GATHER ? 256 : WGM * WGN * 64, GS = 16 / sizeof(T);
    constexpr size_t loop_lds = (size_t)32 * (kPixelRow<T, BMT> + kPixelRow<T, BN>);
    constexpr size_t stage_lds = std::max<size_t>((size_t)NT / 64 * 32 * kStagePitch * 4, (size_t)NT / (BN / GS) * BN * 4);
    constexpr size_t lds = std::max(loop_lds, stage_lds);
    if (lds > 65536) {
        static const bool ok = hipFuncSetAttribute((const void*)wgrad_general_kernel<T, SRC, BMT, BN, WGM, WGN, GATHER>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
        if (!ok) return hipErrorInvalidValue;
    }
    const long long tiles = (long long)((p.R * p.S * p.C + BMT - 1) / BMT) * ((p.N + BN - 1) / BN);
    const dim3 grid(die_grid(tiles * p.splits * n_active)), block(NT);
    hipLaunchKernelGGL((wgrad_general_kernel<T, SRC, BMT, BN, WGM, WGN, GATHER>), grid, block, lds, s, p);
    return hipGetLastError();
}

template <typename T, typename SRC>
hipError_t launch_wgrad(const GeneralWgradParams& p, int n_active, hipStream_t s)
{
    const bool gather = p.cursor && p.gather;
    if constexpr (std::is_same<T, float>::value) {
        if (gather && p.N <= 32) return launch_wgrad_t<T, SRC, 32, 32, 1, 1, true>(p, n_active, s);
        if (gather) return launch_wgrad_t<T, SRC, 32, 64, 1, 2, true>(p, n_active, s);
    }
    if (p.small_tiles) return launch_wgrad_t<T, SRC, 64, 64, 2, 2>(p, n_active, s);
    if (p.N > 64) return launch_wgrad_t<T, SRC, 128, 128, 2, 2>(p, n_active, s);
    if (p.N > 32) return launch_wgrad_t<T, SRC, 128, 64, 4, 1>(p, n_active, s);
    return launch_wgrad_t<T, SRC, 128, 32, 4, 1>(p, n_active, s);
}

}  // namespace

long long weight_copy_units(int bf16, int rows, int taps, int channels)
{
    const int per = bf16 ? Slab<__bf16>::channels : Slab<float>::channels, bytes = bf16 ? Slab<__bf16>::bytes : Slab<float>::bytes;
    return (long long)rows * taps * ((channels + per - 1) / per) * (bytes / 2);
}

long long weight_fragment_units(int bf16, int rows, int taps, int channels)
{
    return weight_copy_units(bf16, (rows + 31) / 32 * 32, taps, channels);
}

hipError_t launch_conv_general(const GeneralConvParams& p0, int epi, int n_active, hipStream_t s, int* stat_rows)
{
    if (n_active < 1) return hipSuccess;
    GeneralConvParams p = p0;
    p.n_active = n_active;
    const int unit = p.bf16 ? 8 : 4;
    if (p.cursor) {
        // one slab or a few: the tiles are bound by their loads and stores, so the small ones only serve launches that would
        // leave units idle
        if (p.bf16 || epi != 0 || p.N % 4 != 0 || p.perm || p.classes != 1) return hipErrorInvalidValue;
        const long long rows = (long long)p.B * p.Ho * p.Wo;
        if (p.N <= 32) return launch_t<float, 0, 128, 32, 4, 1, 1, 1, true>(p, n_active, s, stat_rows);
        if (rows / 128 * ((p.N + 63) / 64) * n_active < 512) return launch_t<float, 0, 64, 64, 2, 2, 1, 1, true>(p, n_active, s, stat_rows);
        return launch_t<float, 0, 128, 64, 4, 1, 1, 1, true>(p, n_active, s, stat_rows);
    }
    if (p.C % unit != 0 || p.N % 4 != 0 || p.R * p.S > 32 || (p.perm && p.classes != 1)) return hipErrorInvalidValue;
    if (!p.bf16) return epi == 0 ? launch_conv<float, 0>(p, n_active, s, stat_rows) : launch_conv<float, 1>(p, n_active, s, stat_rows);
    return epi == 0 ? launch_conv<__bf16, 0>(p, n_active, s, stat_rows) : launch_conv<__bf16, 1>(p, n_active, s, stat_rows);
}

// Tile and split-K factor of a weight gradient: the estimate of the launch's time with the least.  A workgroup walks K / s
// pixels in slabs of 32 (and about three slabs' time of first loads and epilogue); per slab of a 128 x 128 tile 2.2 us when it
// has its compute unit to itself, 2.7 when two share one, and 1.3 of the unit's time per workgroup in launches of more than
// two per unit, which end with half a workgroup's time of partly filled units; smaller tiles in proportion.  The partial
// sums move 8 bytes per weight and split at 4 TB/s.  64 x 64 tiles win where the larger ones leave compute units idle at
// every split.  (Measured in us, 3 x 3, batch 64.  128 channels on 16 x 16 images, 16 replicas, s = 1 2 4 8 16 32: 1082 664 598
// 477 426 441; 1 replica, s = 28 51 64: 49 41 49 and with 64 x 64 tiles 45 51 45; 64 channels on 32 x 32 images, 1 replica,
// s = 32 64: 110 67 and 82 55; 80 channels on 5 x 5 images, batch 50, 3 replicas: 21 and 16.)
WgradPlan wgrad_general_plan(int rows, int N, int K, int n_active, int gather)
{
    struct { int m, n; float f; } tile[2] = {{128, N > 64 ? 128 : N > 32 ? 64 : 32, N > 64 ? 1.0f : N > 32 ? 0.68f : 0.45f}, {64, 64, 0.35f}};
    if (gather) tile[0] = {32, N > 32 ? 64 : 32, 0.25f};
    const float moved = (float)rows * (float)N * (float)n_active * 8.0f / 4e6f;
    WgradPlan best{1, 0};
    float best_t = 0.f;
    for (int v = 0; v < (gather || N <= 32 ? 1 : 2); ++v) {
        const float wgs = (float)((rows + tile[v].m - 1) / tile[v].m) * (float)((N + tile[v].n - 1) / tile[v].n) * (float)n_active;
        for (int s = 1; s <= std::min(256, std::max(1, K / 128)); ++s) {
            if (s > 1 && moved * (float)(s + 1) >= best_t) break;        // (and any further split moves more)
            const float steps = ((float)K / (32.0f * (float)s) + 3.0f) * tile[v].f, w = wgs * (float)s;
            float t = w <= 256.f ? steps * 2.2f : w <= 512.f ? steps * 2.7f : w * steps * 1.3f / 256.f + 0.5f * steps * 2.2f;
            if (s > 1) t += moved * (float)(s + 1);
            if ((v == 0 && s == 1) || t < best_t) { best = {s, v}; best_t = t; }
        }
    }
    best.time = best_t;
    return best;
}

hipError_t launch_wgrad_general(const GeneralWgradParams& p0, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    GeneralWgradParams p = p0;
    p.n_active = n_active;
    const int unit = p.bf16 ? 8 : 4;
    if (p.gather && (!p.cursor || p.bf16)) return hipErrorInvalidValue;
    if ((p.C % unit != 0 && !p.gather) || p.N % unit != 0 || (p.splits > 1 && p.kchunk % 32 != 0)) return hipErrorInvalidValue;
    if (p.perm && (p.B % 32 != 0 || p.stride != 1 || p.R * p.S > 32 || p.cursor)) return hipErrorInvalidValue;
    if (!p.bf16) return launch_wgrad<float, float>(p, n_active, s);
    return p.cursor ? launch_wgrad<__bf16, float>(p, n_active, s) : launch_wgrad<__bf16, __bf16>(p, n_active, s);
}

hipError_t launch_weight_copies(WeightCopies& p, int n_active, hipStream_t s)
{
    if (n_active < 1 || p.count < 1) return hipSuccess;
    if (p.count > kWeightCopies) return hipErrorInvalidValue;
    long long tiles = 0;
    for (int i = 0; i < p.count; ++i) {
        const WeightCopyParams& l = p.layer[i];
        p.first[i] = (int)tiles;
        tiles += (long long)((l.C + 63) / 64) * ((l.N + 63) / 64) * l.taps;
        if (l.bf16 != p.layer[0].bf16 || tiles > 0x7fffffff / 256) return hipErrorInvalidValue;
    }
    const dim3 grid((unsigned)tiles, (unsigned)n_active), block(256);
    if (p.layer[0].bf16) hipLaunchKernelGGL(weight_copy_kernel<__bf16>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(weight_copy_kernel<float>, grid, block, 0, s, p);
    return hipGetLastError();
}

}  // namespace hadfl
