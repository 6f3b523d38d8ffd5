// Weight gradient of the fp32 3 x 3 stride-1 "same" convolutions of every local step (paper Sec. 2.1), on split floats like
// conv_general.hip:  dW[tap][ci][co] = sum over images and positions of x[image][position + tap][ci] * dy[image][position][co].
//
// wgrad_general_kernel walks pixels in memory order with one tap per row of its tile: every x is fetched, split and written to LDS
// once per tap, both operands lie in LDS by pixel and are transposed on the way out by reads of some 90 bytes a clock.  Here
// the order of the contraction is turned round: sixteen IMAGES at one position make the sixteen elements of a matrix
// instruction.  Then
//   * a tap moves whole operands: x at position + tap is another operand in LDS, for any image size, and a tap outside the
//     image is a matrix instruction less (31 % of them on 4 x 4 images, 56 % on 2 x 2);
//   * a lane fetches one channel of eight images, eight 4-byte loads that a wave makes as lines of 128 bytes, splits
//     them and has its sixteen bytes of an operand per plane: LDS holds operands in lane order, written and read without
//     transposition or conflict.
// A workgroup owns all nine taps of 64 input against 64 output channels and walks positions along the rows of sixteen images.  A
// step multiplies one position: of x it needs the 3 x 3 positions around it, the columns to the left of which came with the steps
// before, so a step fetches one column of three (six operands of 32 channels) and the position's dy (two): one for each of the
// eight waves.  Two steps make a pair with one barrier: within it the waves of a SIMD drift apart, so that one's splits and
// LDS traffic lie beside the other's matrix instructions (a barrier after each step, 16 / 4 replicas: 14.94 / 2.67 ms of these launches
// in ResNet-18 / VGG-16; a pair 14.24 / 2.60).  Columns are numbered along the walk, and x and dy have a ring of six places each, 144 of
// the 160 KiB together (a seventh place, 24 KiB, does not fit): the pair of t and t + 1 reads the columns t - 1 to t + 2 and, ahead, dy of t + 2 (in front of
// the first pair that of t too) while those of t + 3 and t + 4 are written.  Operands are fetched two steps before they are written, beside
// the matrix instructions.
// Waves 0 to 3 multiply the corner taps and the middle one, waves 4 to 7 the four others, each for a block of 32 x 32 channels: on a
// SIMD, which has one of either, that is nine.  Per step: 54 matrix instructions a SIMD (1728 clocks), some 130 KiB of LDS read
// (600 at the measured 220 bytes a clock), 24 KiB written (350 at 70), a wave's eight loads and some 90 vector instructions.
// 3 x 3, batch 64, us with the reduction of the split sums (wgrad_general_kernel / this, with a barrier after each step: pairs take some
// 4 % less; TFLOP/s of fp32 products):
//   64 channels, 32 x 32 images:   1 replica 67 / 46,  4 replicas 207 / 117,  16 replicas 629 / 414 (187 TFLOP/s)
//   128 channels, 16 x 16:         64 / 47,  128 / 108,  481 / 382 (207)
//   256 channels, 8 x 8:           67 / 49,  139 / 110,  525 / 339 (224)
//   512 channels, 4 x 4:           58 / 53,  157 / 92,  442 / 327 (233)
#include <algorithm>

#include "train_kernels.h"
#include "mfma_tiles.h"
#include "slabs.h"

namespace hadfl {
namespace {

using namespace tiles;

constexpr int kImages = 16;                                   // a step's contraction
constexpr int kOperand = 3 * 1024, kColumn = 6 * kOperand;    // bytes: 32 channels x 16 images; three positions x 64 channels
constexpr int kPlaces = 6, kRing = kPlaces * kColumn, kStepLds = kRing + kPlaces * 2 * kOperand;
// taps 0, 2, 4, 6, 8 of the corner waves, 1, 3, 5, 7 of the others (and a fifth that is not multiplied)
constexpr int kCornerRow[5] = {0, 0, 1, 2, 2}, kCornerCol[5] = {0, 2, 1, 0, 2}, kEdgeRow[5] = {0, 1, 1, 2, 1}, kEdgeCol[5] = {1, 0, 2, 1, 1};
// (The first of either reads a column that was written before the last pair, so that its operands can be read before the barrier.)
constexpr int kStagePitch = 36;                               // floats per staged row

// A 32 x 32 block or a bias: stored, or (w set: it is the complete gradient) applied as the update
template <typename V> __device__ __forceinline__ void put(const V& v, long long o, const GeneralWgradParams& p, float* out, float* w, float* buf)
{
    if (!w) { *reinterpret_cast<V*>(out + o) = v; return; }
    V d = v;
    if (buf) { d = *reinterpret_cast<const V*>(buf + o) * p.momentum + d; *reinterpret_cast<V*>(buf + o) = d; }
    *reinterpret_cast<V*>(w + o) = *reinterpret_cast<const V*>(w + o) - d * p.lr;
}

__global__ __launch_bounds__(512, 2) void wgrad_general_position_kernel(GeneralWgradParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int corners = wave < 4, cib = (wave >> 1) & 1, cob = wave & 1;
    // logical item = (slot, split, tile): the tiles of one split of one replica read the same positions
    const unsigned tiles_n = (unsigned)(p.N + 63) / 64, tiles = (unsigned)((p.C + 63) / 64) * tiles_n;
    const unsigned item = logical_block();
    if (item >= tiles * (unsigned)p.splits * (unsigned)p.n_active) return;
    const int slot = (int)(item / (tiles * (unsigned)p.splits)), rep = p.order[slot], split = (int)((item / tiles) % (unsigned)p.splits);
    const int c0 = (int)((item % tiles) / tiles_n) * 64, n0 = (int)((item % tiles) % tiles_n) * 64;
    const int hw = p.H * p.W, steps = (p.B + kImages - 1) / kImages * hw;
    const int per = (steps + p.splits - 1) / p.splits, t0 = min(steps, split * per), t1 = min(steps, t0 + per);

    // What this wave fetches for a column: waves 0 to 5 the channels of x in row `up` of the three, waves 6 and 7 those of dy.
    // (Channels beyond the last are the last again: their sums are not stored.)
    const bool is_x = wave < 6;
    const int up = is_x ? (wave >> 1) - 1 : 0, block = wave & 1, channels = is_x ? p.C : p.N;
    const int ch = min((is_x ? c0 : n0) + block * 32 + (lane & 31), channels - 1);
    const Buffer src = buffer(is_x ? p.x + (long long)rep * p.x_rep : p.dy + (long long)rep * p.dy_rep, (unsigned)(p.B * hw) * (unsigned)channels * 4u);
    const unsigned image = (unsigned)(hw * channels) * 4u;    // bytes; images beyond the batch lie outside the buffer: zeros
    const unsigned at = (unsigned)(lane >> 5) * 8u * image + (unsigned)ch * 4u;
    constexpr int kPair = 2, lead = kPair + 1;                // positions a barrier; steps between writing an operand and multiplying it
    int lt, lg, ly, lx;                                       // the column that is fetched next
    auto seek = [&](int t) { lt = t; lg = t / hw; ly = (t - lg * hw) / p.W; lx = t - lg * hw - ly * p.W; };
    auto fetch = [&](f4 (&v)[2]) {
        const int y = ly + up;
        const unsigned o = at + ((unsigned)(lg * kImages * hw + y * p.W + lx) * (unsigned)channels) * 4u;
        if ((unsigned)y < (unsigned)p.H && lt >= 0)           // (no tap reads an operand from outside the image)
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i >> 2][i & 3] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src, (int)(o + (unsigned)i * image), 0, 0));
        ++lt; ++lx;
        if (lx == p.W) { lx = 0; ++ly; }
        if (ly == p.H) { ly = 0; ++lg; }
    };
    int ring[kPlaces];                                        // places of the columns t - 1 to t + 4, t the first position of a pair
#pragma unroll
    for (int k = 0; k < kPlaces; ++k) ring[k] = k;
    auto place = [&](int at) { return smem + (is_x ? at * kColumn + wave * kOperand : kRing + (at * 2 + block) * kOperand); };
    auto write = [&](const f4 (&v)[2], int at) {
        u2 h0, m0, l0, h1, m1, l1;
        split3(v[0], h0, m0, l0);
        split3(v[1], h1, m1, l1);
        char* const o = place(at) + lane * 16;
        *reinterpret_cast<u4*>(o) = join8(h0, h1);
        *reinterpret_cast<u4*>(o + 1024) = join8(m0, m1);
        *reinterpret_cast<u4*>(o + 2048) = join8(l0, l1);
    };
    const bool with_bias = p.has_bias && c0 == 0 && !is_x;
    float bias = 0.f;                                         // sum of this lane's dy

    f16 acc[5], low[5];                                       // sums of the large and of the small products, a tap each
    auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < 5; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[j][v] = 0.f; low[j][v] = 0.f; }
    };
    const bool mine = c0 + cib * 32 < p.C && n0 + cob * 32 < p.N;
    int y, x;                                                 // position of the present step
    auto column = [&](int at, int r) { return smem + at * kColumn + (r * 2 + cib) * kOperand; };
    auto has_tap = [&](int j) {
        const int r = corners ? kCornerRow[j] : kEdgeRow[j], s = corners ? kCornerCol[j] : kEdgeCol[j];
        return (j < 4 || corners) && (unsigned)(y + r - 1) < (unsigned)p.H && (unsigned)(x + s - 1) < (unsigned)p.W;
    };
    bf16x8 a[2][3], b[2][3];                                  // read a tap ahead, the first of a step before the barrier (of a tap outside the image whatever is there)
    auto read_x = [&](bf16x8 (&o)[3], int d, int j) {         // of position t + d
        const char* const from = column(corners ? ring[d + kCornerCol[j]] : ring[d + kEdgeCol[j]], corners ? kCornerRow[j] : kEdgeRow[j]) + lane * 16;
#pragma unroll
        for (int q = 0; q < 3; ++q) o[q] = *reinterpret_cast<const bf16x8*>(from + q * 1024);
    };
    auto read_dy = [&](bf16x8 (&o)[3], int d) {
#pragma unroll
        for (int q = 0; q < 3; ++q) o[q] = *reinterpret_cast<const bf16x8*>(smem + kRing + (ring[d + 1] * 2 + cob) * kOperand + q * 1024 + lane * 16);
    };
    auto multiply = [&](int d) {
        if (!mine) return;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            if (j == 4) { read_x(a[(d + 1) & 1], d + 1, 0); read_dy(b[(d + 1) & 1], d + 1); }
            else if (j < 3 || corners) read_x(a[(d + j + 1) & 1], d, j + 1);
            if (!has_tap(j)) continue;
            const bf16x8 (&u)[3] = a[(d + j) & 1], (&v)[3] = b[d & 1];
            // operands swapped: the accumulator holds the transposed block.  Small products in ascending size.
            constexpr int SA[5] = {0, 2, 1, 0, 1}, SB[5] = {2, 0, 1, 1, 0};
#pragma unroll
            for (int q = 0; q < 5; ++q) low[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[SB[q]], u[SA[q]], low[j], 0, 0, 0);
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[0], u[0], acc[j], 0, 0, 0);
        }
    };
    auto next_position = [&]() { if (++x == p.W) { x = 0; if (++y == p.H) y = 0; } };

    clear();
    y = t0 % hw / p.W; x = t0 % hw % p.W;
    if (t0 < t1) {
        f4 v[kPair][2] = {};                                  // columns on their way
        auto sum8 = [&](const f4 (&u)[2]) { return ((u[0][0] + u[0][1]) + (u[0][2] + u[0][3])) + ((u[1][0] + u[1][1]) + (u[1][2] + u[1][3])); };
        seek(is_x ? t0 - 1 : t0);
        {
            f4 u[4][2] = {};
            fetch(u[0]); fetch(u[1]); fetch(u[2]);
            if (is_x) fetch(u[3]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (is_x) write(u[k], ring[k]);
                else if (k < 3) { write(u[k], ring[k + 1]); if (t0 + k < t1) bias += sum8(u[k]); }
            }
        }
#pragma unroll
        for (int d = 0; d < kPair; ++d) fetch(v[d]);          // columns t0 + 3, t0 + 4
        __syncthreads();
        read_x(a[0], 0, 0);
        read_dy(b[0], 0);
        for (int t = t0; t < t1; t += kPair) {
#pragma unroll
            for (int d = 0; d < kPair; ++d) {
                const int now = t + d;
                if (now >= t1) break;
                write(v[d], ring[d + lead + 1]);
                if (with_bias && now + lead < t1) bias += sum8(v[d]);
                fetch(v[d]);
                multiply(d);
                next_position();
            }
            __syncthreads();
            const int u0 = ring[0], u1 = ring[1];
#pragma unroll
            for (int k = 0; k + kPair < kPlaces; ++k) ring[k] = ring[k + kPair];
            ring[kPlaces - 2] = u0; ring[kPlaces - 1] = u1;
        }
    }
    float bad = 0.f;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        acc[j] = (acc[j] + low[j]) * kProductScale;
#pragma unroll
        for (int v = 0; v < 16; ++v) bad = __builtin_fmaf(acc[j][v], 0.f, bad);
    }
    if (__syncthreads_or(bad != 0.f)) {                       // (NaN != 0) something is not finite: again, with the fp32 instruction
        clear();
        y = t0 % hw / p.W; x = t0 % hw % p.W;
        for (int t = t0; t < t1; ++t) {
            f4 v[2] = {};
            seek(is_x ? t - 1 : t);
            for (int q = 0; q < (is_x ? 3 : 1); ++q) {
                const int at = lt - t + 1;
                fetch(v);
                char* const o = place(at) + lane * 32;
                *reinterpret_cast<f4*>(o) = v[0];
                *reinterpret_cast<f4*>(o + 16) = v[1];
            }
            __syncthreads();
            const float* const b = reinterpret_cast<const float*>(smem + kRing + (1 * 2 + cob) * kOperand + lane * 32);
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                const int r = corners ? kCornerRow[j] : kEdgeRow[j], s = corners ? kCornerCol[j] : kEdgeCol[j];
                    if (!has_tap(j)) continue;
                const float* const a = reinterpret_cast<const float*>(column(s, r) + lane * 32);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[e], a[e], acc[j], 0, 0, 0);
            }
            next_position();
            __syncthreads();
        }
    }

    // ---- epilogue (behind a barrier: nobody reads an operand any more): blocks through LDS, so that global accesses cover whole lines ----
    float* const out = p.splits > 1 ? p.out + (long long)slot * p.out_rep + (long long)split * p.out_split : p.out + (long long)rep * p.out_rep;
    float* const w = (p.splits == 1 && p.sgd_w) ? p.sgd_w + (long long)rep * p.out_rep : nullptr;
    float* const buf = (w && p.sgd_buf) ? p.sgd_buf + (long long)rep * p.out_rep : nullptr;
    float* const stage = reinterpret_cast<float*>(smem) + wave * (32 * kStagePitch);
    if (mine)
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            if (j == 4 && !corners) break;
            const int tap = corners ? 2 * j : 2 * j + 1;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f4*>(stage + (lane & 31) * kStagePitch + 8 * q + 4 * (lane >> 5)) = f4{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int rr = (lane >> 3) + 8 * q, cc = (lane & 7) * 4;
                const f4 v = *reinterpret_cast<const f4*>(stage + rr * kStagePitch + cc);
                const int ci = c0 + cib * 32 + rr, co = n0 + cob * 32 + cc;
                if (ci < p.C && co < p.N) put(v, ((long long)tap * p.C + ci) * p.N + co, p, out, w, buf);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    if (with_bias) {                                          // images 0..7 of the sixteen, then 8..15
        const float other = __shfl_xor(bias, 32);
        const int co = n0 + block * 32 + lane;
        if (lane < 32 && co < p.N) put(bias + other, (long long)9 * p.C * p.N + co, p, out, w, buf);
    }
}

}  // namespace

// Tiles of 64 x 64 channels, at most a third of them empty; offsets of the sixteen images of a step, the last ones beyond the batch,
// fit 32 bits.
bool wgrad_positions_supported(int B, int H, int W, int C, int N)
{
    const double padded = (double)((C + 63) / 64 * 64) * ((N + 63) / 64 * 64);
    const double numel = (double)H * W * std::max(C, N) * 4.0;
    return C % 4 == 0 && N % 4 == 0 && padded <= 1.34 * C * N && (B + 2 * kImages) * numel < 4.0e9;
}

// The split with the least estimated cost: a step takes 1.5 us, less the taps outside the image; a workgroup's first columns and its
// epilogue 10 us, and one workgroup is resident per compute unit, whose registers it fills; the partial sums move 8 bytes per weight
// and split at 4 TB/s.  The launch runs beside the data gradients of the layers below, which get the units that it leaves: what counts
// is its own duration (whole rounds of units) with 0.4 and the time it takes from the chip (its workgroups' time over all units) with
// 0.6.  Weights 1 / 0.7 / 0.5 / 0.3 / 0.1 of the duration: ResNet-18 on 4 replicas 17.4 17.0 17.0 17.0 17.5 ms, VGG-16 on 4
// 8.03 7.89 7.84 7.68 8.33, ResNet-18 on 16 59.9 59.9 59.9 59.9 59.4.
WgradPlan wgrad_positions_plan(int B, int H, int W, int C, int N, int n_active)
{
    const int steps = (B + kImages - 1) / kImages * H * W;
    const float step = 1.5f * (float)((3 * H - 2) * (3 * W - 2)) / (float)(9 * H * W);
    const float tiles = (float)((C + 63) / 64 * ((N + 63) / 64)) * (float)n_active, moved = 9.0f * (float)C * (float)N * (float)n_active * 8.0f / 4e6f;
    WgradPlan best{1, 0};
    for (int s = 1; s <= std::min(256, std::max(1, steps / 4)); ++s) {
        if (s > 1 && moved * (float)(s + 1) >= best.time) break;         // (and any further split moves more)
        const int per = (steps + s - 1) / s;
        if ((steps + per - 1) / per < s) continue;            // (a split without a step)
        const float rounds = (float)(int)((tiles * (float)s + 255.f) / 256.f), share = tiles * (float)s / 256.f;
        float t = (0.4f * rounds + 0.6f * share) * ((float)per * step + 10.0f);
        if (s > 1) t += moved * (float)(s + 1);
        if (s == 1 || t < best.time) { best.splits = s; best.time = t; }
    }
    best.positions = 1;
    return best;
}

hipError_t launch_wgrad_positions(const GeneralWgradParams& p0, int n_active, hipStream_t s)
{
    if (n_active < 1) return hipSuccess;
    GeneralWgradParams p = p0;
    p.n_active = n_active;
    if (p.bf16 || p.cursor || p.stride != 1 || p.R != 3 || p.S != 3 || p.pad != 1 || p.Ho != p.H || p.Wo != p.W ||
        !wgrad_positions_supported(p.B, p.H, p.W, p.C, p.N)) return hipErrorInvalidValue;
    static const bool ok = hipFuncSetAttribute((const void*)wgrad_general_position_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kStepLds) == hipSuccess;
    if (!ok) return hipErrorInvalidValue;
    const dim3 grid(die_grid((long long)((p.C + 63) / 64) * ((p.N + 63) / 64) * p.splits * n_active)), block(512);
    hipLaunchKernelGGL(wgrad_general_position_kernel, grid, block, kStepLds, s, p);
    return hipGetLastError();
}

}  // namespace hadfl
