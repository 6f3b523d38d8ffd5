// Probability-based replica selection (paper Sec. 3.3): one wavefront, or one workgroup above 64 replicas.
// Built with -ffp-contract=off: every fp64 operation below is rounded on its own, so the result is a
// function of the inputs alone and any IEEE-754 implementation of the same written steps gives the same bits.
#include <climits>
#include <mutex>
#include <type_traits>

#include "kernels.h"

// Working memory of hadfl_select_static, the selection for callers that cannot allocate device memory: the selection
// function's values f[kMaxReplicas] (fp64), then the ascending list of the selected replicas and their weights.
// Every GPU the library runs on holds its own copy until the process ends.  Host code never passes this name to a
// kernel: it is a host-side stand-in, the device address comes from hipGetSymbolAddress (static_scratch below).
constexpr size_t kStaticScratchBytes = hadfl::kMaxReplicas * (sizeof(double) + sizeof(int32_t) + sizeof(float));
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace hadfl {
namespace {

struct U4 { uint32_t x, y, z, w; };

// Philox4x32-10 (Salmon et al., SC'11).
__device__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
        const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
        c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return c;
}

// exp(x), x in [-690, 0]: n = nearest integer to x*log2(e); r = (x - n*ln2_hi) - n*ln2_lo (two-constant
// reduction, n*ln2_hi exact); Taylor polynomial of degree 13 by Horner; multiply by 2^n built in the exponent field.
__device__ double exp_neg(double x)
{
    const double c[14] = {1.0, 1.0, 1.0 / 2.0, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0, 1.0 / 5040.0,
                          1.0 / 40320.0, 1.0 / 362880.0, 1.0 / 3628800.0, 1.0 / 39916800.0,
                          1.0 / 479001600.0, 1.0 / 6227020800.0};
    const double n = __builtin_rint(x * 0x1.71547652b82fep+0);
    const double r = (x - n * 0x1.62e42feep-1) - n * 0x1.a39ef35793c76p-33;
    double p = c[13];
#pragma unroll
    for (int i = 12; i >= 0; --i) p = p * r + c[i];
    const long long e = (long long)n + 1023;
    if (e < 1) return 0.0;
    return p * __longlong_as_double(e << 52);
}

// value held by lane k of the wavefront (k is wave-uniform at every call site)
__device__ __forceinline__ double lane_value(double v, int k)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), k);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ long long uniform_key(long long v)
{
    return ((long long)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((int)v);
}

// Inclusive sums along the lanes of a row of 16, and along the whole wavefront.  One rounding per step of a tree of depth 4
// (6): not the sums of the rule, which add one value after another, but within kSumError of them.
template <int kCtrl, int kRows> __device__ __forceinline__ double lanes_below(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRows, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRows, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_sums(double v)
{
    v = v + lanes_below<0x111, 0xf>(v);                    // row_shr:1, 2, 4, 8
    v = v + lanes_below<0x112, 0xf>(v);
    v = v + lanes_below<0x114, 0xf>(v);
    return v + lanes_below<0x118, 0xf>(v);
}
__device__ __forceinline__ double wave_sums(double v)
{
    v = row_sums(v);
    v = v + lanes_below<0x142, 0xa>(v);                    // row_bcast:15 into the second and fourth row
    return v + lanes_below<0x143, 0xc>(v);                 // row_bcast:31 into the upper half
}

// A draw picks the first replica whose running sum R_i, added one value after another with a rounding each, exceeds
// fl(u * R_N).  That chain of N dependent additions need not be run to know the pick.  Let A_i be a sum of the same values
// formed by a tree, less what was picked since, and `total` the sum of all values when the tree was formed.  No value is negative, so
// a rounding is at most 2^-53 total: R_i has fewer than N <= 1024 of them, A_i at most ten for the tree and two for every one of
// up to 1024 picks, the threshold one more than its sum.  |A_i - R_i| and the difference of the thresholds are each below 3100 *
// 2^-53 total, so where A_i is further than kSumError * total from the threshold, R_i is on the same side.  Where it is not
// (some N * 2^-40 of all draws, and more of them as the picks leave little of the total), the tree is formed anew, and where that is not
// enough either, the chain decides.  NaN compares false, on neither side.
constexpr double kSumError = 0x1p-40;
struct Sides { unsigned long long above, below; };         // lanes whose running sum exceeds the threshold, lanes whose does not
__device__ __forceinline__ Sides sides(double sum, double thr, double error)
{
    const double d = sum - thr;
    return Sides{__ballot(d > error), __ballot(d < -error)};
}

template <typename V> __device__ __forceinline__ const V* versions_of(const SelectArgs& a);
template <> __device__ __forceinline__ const int* versions_of<int>(const SelectArgs& a) { return a.versions; }
template <> __device__ __forceinline__ const double* versions_of<double>(const SelectArgs& a) { return a.versions_f64; }

// the uniform of draw t: counter (cycle_lo, cycle_hi, draw, 0), key = seed, 53 bits of the first two words
__device__ __forceinline__ double draw_uniform(const SelectArgs& a, int t)
{
    const U4 o = philox4x32_10(U4{(uint32_t)a.cycle, (uint32_t)(a.cycle >> 32), (uint32_t)t, 0u},
                               (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
    const unsigned long long bits = ((unsigned long long)o.y << 32) | o.x;
    return (double)(bits >> 11) * 0x1.0p-53;
}

// the Gaussian selection function of Sec. 3.3, its exponent clamped so that no available replica has probability 0
__device__ __forceinline__ double selection_function(double v, double mu)
{
    const double d = v - mu;
    double e = -(d * d) * 0.5;
    if (e < -690.0) e = -690.0;
    return exp_neg(e);
}

// Selection among at most 64 replicas, one wavefront, a replica a lane.
// V = int: versions are step counters; V = double: forecast (real-valued) versions (Sec. 3.2 feeding Sec. 3.3)
//
// The draws are sequential (draw t renormalises over the replicas that remain).  A wavefront on its own issues a dependent
// instruction only every 5 to 8 clocks, so what counts is the number of instructions on the path, and straight-line code that
// runs once is paid for in instruction fetches.  A draw is a tree of sums over the lanes (six steps, where the running
// sums of the rule are N dependent additions: see kSumError), a product, two ballots; uniforms and f are computed up
// front.  64 replicas and 8 draws, with the launch: 5.7 us with the chain of additions in every draw, 4.2 here; forecast versions, 24
// replicas and 12 draws: 11.0 and 6.3.
template <typename V>
__global__ __launch_bounds__(64) void select_kernel(SelectArgs a)
{
    constexpr bool kIntVersions = std::is_same<V, int>::value;
    __shared__ double s_sorted[64];
    __shared__ long long s_key[kIntVersions ? 64 : 1];
    __shared__ double s_v[kIntVersions ? 1 : 64];
    const int lane = threadIdx.x, N = a.n;

    // a rank-counting sort of the available versions: rank(i) = #{available j : v_j < v_i or (v_j == v_i and j < i)}
    const bool on = lane < N && (!a.avail || a.avail[lane]);
    const V vi = lane < N ? versions_of<V>(a)[lane] : V(0);
    // step counters: (version, index) pairs are ordered by one integer key, version * 1024 + index; a replica
    // that is not available, or beyond N, gets the largest key and is counted before nobody.  Real-valued versions: such a
    // replica is a NaN, which is before nobody either.
    if constexpr (kIntVersions) s_key[lane] = on ? (long long)vi * kMaxReplicas + lane : LLONG_MAX;
    else s_v[lane] = on ? (double)vi : __builtin_nan("");
    // the uniform of every draw, lane t's for draw t (n_select <= N <= 64)
    const double my_u = draw_uniform(a, lane);
    __syncthreads();
    const unsigned long long avail = __ballot(on);
    const int na = __popcll(avail);
    int rank = 0;
    // every lane compares its own version with all, read from LDS at a wave-uniform address (a broadcast)
    if constexpr (kIntVersions) {
        const long long mine = s_key[lane];
        for (int j = 0; j < N; j += 16) {
#pragma unroll
            for (int u = 0; u < 16; ++u) rank += s_key[j + u] < mine ? 1 : 0;
        }
    } else {
        for (int j = 0; j < N; j += 16) {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double vj = s_v[j + u];
                rank += (int)(vj < vi) | ((int)(vj == vi) & (int)(j + u < lane));
            }
        }
    }
    if (on) s_sorted[rank] = (double)vi;
    __syncthreads();
    // third quartile: linear interpolation at 0.75*(na-1)
    const double pos = 0.75 * (double)(na - 1);
    const int lo = na > 0 ? (int)__builtin_floor(pos) : 0;
    const double frac = pos - (double)lo;
    double mu = s_sorted[lo];
    if (lo + 1 < na) mu = s_sorted[lo] + frac * (s_sorted[lo + 1] - s_sorted[lo]);

    const double f = on ? selection_function((double)vi, mu) : 0.0;
    if (lane < N) a.f[lane] = f;

    // Sequential draws: draw t picks the first live replica whose running sum of f exceeds u_t * S, S the total over
    // the live replicas; dead replicas (picked, unavailable, or beyond N) add +0.0, which leaves a sum unchanged.
    double g = f;                                          // f while the replica can still be drawn
    unsigned long long livemask = __ballot(f > 0.0);
    const unsigned long long could = livemask;
    int my_pick = -1;
    double sum = wave_sums(g), error = kSumError * lane_value(sum, 63);
    for (int t = 0; t < a.n_select; ++t) {
        const double u = lane_value(my_u, t);
        Sides at = sides(sum, u * lane_value(sum, 63), error);
        unsigned long long hit = at.above;
        if ((at.above | at.below) != ~0ull || !hit) {
            sum = wave_sums(g);
            error = kSumError * lane_value(sum, 63);
            at = sides(sum, u * lane_value(sum, 63), error);
            hit = at.above;
            if ((at.above | at.below) != ~0ull || !hit) {  // the sums of the rule
                double run = 0.0, mine = 0.0;
                for (int k = 0; k < 64; ++k) {
                    run = run + lane_value(g, k);
                    mine = lane == k ? run : mine;
                }
                hit = __ballot(mine > u * run) & livemask;
            }
        }
        int pick = -1;
        if (hit) pick = __ffsll((long long)hit) - 1;
        else if (livemask) pick = 63 - __clzll(livemask);   // stays -1 only if no replica is left to draw from
        pick = __builtin_amdgcn_readfirstlane(pick);
        if (lane == t) my_pick = pick;
        if (pick >= 0) {
            const double gone = lane_value(g, pick);
            if (lane >= pick) sum = sum - gone;
            if (lane == pick) g = 0.0;
            livemask &= ~(1ull << pick);
        }
    }
    if (lane < a.n_select) a.selected[lane] = my_pick;

    // aggregation weights a_k and the ascending list the aggregate kernel walks.  With unit terms the denominator is
    // the count itself (a sum of ones is exact); with f-weighted terms it adds the selected replicas' f in
    // ascending index, one after another.
    const unsigned long long picked = could & ~livemask;
    double denom = (double)__popcll(picked);
    if (a.weight_mode == 1) {
        denom = 0.0;
        for (unsigned long long m = picked; m; m &= m - 1) denom = denom + lane_value(f, __ffsll((long long)m) - 1);
    }
    if (lane < N) {
        const bool sel = (picked >> lane) & 1ull;
        float w = 0.f;
        if (sel) {
            w = (float)(((a.weight_mode == 1) ? f : 1.0) / denom);
            const int at = __popcll(picked & ((1ull << lane) - 1ull));
            a.sel_sorted[at] = lane;
            a.sel_weight[at] = w;
        }
        a.flag[lane] = sel ? 1 : 0;
        a.weights[lane] = w;
    }
}

// ---- selection among 65 to kMaxReplicas replicas ----
constexpr int kManyThreads = 256;

// A version as an integer of the same order, and back
__device__ __forceinline__ long long order_key(int v) { return v; }
__device__ __forceinline__ long long order_key(double v)
{
    const long long b = __double_as_longlong(v);
    return b ^ ((b >> 63) & LLONG_MAX);
}
template <typename V> __device__ __forceinline__ double key_value(long long k)
{
    return std::is_same<V, int>::value ? (double)k : __longlong_as_double(k ^ ((k >> 63) & LLONG_MAX));
}

// One workgroup of four wavefronts; the draws are wavefront 0's alone, the rest is shared.  A lane
// keeps the running sum after a segment of sixteen values; a draw is bound by its chain of dependent instructions: the segment's
// values from LDS, sums along them (four steps), the pick out of the running sums.  1000 replicas, 100 draws: 245-255 us with
// the chain of the rule in every draw, 41 here (0.31 us a draw; 11.5 us with one draw); 65 replicas and one draw: 8 us.
template <typename V>
__global__ __launch_bounds__(kManyThreads) void select_many_kernel(SelectArgs a)
{
    constexpr int kPer = kMaxReplicas / 64;                // values per lane of wavefront 0
    __shared__ double s_g[kMaxReplicas];                   // f of the replicas still to be drawn from, else +0.0
    __shared__ double s_f[kMaxReplicas];
    __shared__ double s_u[kMaxReplicas];
    __shared__ long long s_key[kMaxReplicas];
    __shared__ unsigned char s_flag[kMaxReplicas];
    __shared__ double s_mu;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, N = a.n;
    const int chunks = (N + 63) / 64;

    for (int i = tid; i < chunks * 64; i += kManyThreads) {
        const bool on = i < N && (!a.avail || a.avail[i]);
        s_key[i] = on ? order_key(versions_of<V>(a)[i]) : LLONG_MAX;      // (no version maps to the largest key)
        s_flag[i] = on ? 1 : 0;                            // until f is known: available
        if (i < a.n_select) s_u[i] = draw_uniform(a, i);
    }
    __syncthreads();
    // Third quartile, linear interpolation at 0.75 * (na - 1): two neighbouring order statistics, found by bisection of
    // the keys' range with a count per step (no sort).
    if (wave == 0) {
        long long key[kPer], kmin = LLONG_MAX, kmax = LLONG_MIN;
        int na = 0;
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            key[r] = r < chunks ? s_key[r * 64 + lane] : LLONG_MAX;
            na += __popcll(__ballot(key[r] != LLONG_MAX));
            kmin = key[r] < kmin ? key[r] : kmin;
            if (key[r] != LLONG_MAX) kmax = key[r] > kmax ? key[r] : kmax;
        }
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {
            const long long x = __shfl_xor(kmin, w), y = __shfl_xor(kmax, w);
            kmin = x < kmin ? x : kmin; kmax = y > kmax ? y : kmax;
        }
        const double pos = 0.75 * (double)(na - 1);
        const int lo = (int)__builtin_floor(pos);
        const double frac = pos - (double)lo;
        // smallest key with more than `lo` keys at or below it
        long long b0 = uniform_key(kmin), b1 = uniform_key(kmax);
        while (b0 < b1) {
            const long long mid = b0 + (long long)(((unsigned long long)b1 - (unsigned long long)b0) >> 1);
            int at_most = 0;
#pragma unroll
            for (int r = 0; r < kPer; ++r) at_most += __popcll(__ballot(key[r] <= mid));
            if (at_most > lo) b1 = mid; else b0 = mid + 1;
        }
        double mu = key_value<V>(b0);
        if (lo + 1 < na) {
            int at_most = 0;
            long long above = LLONG_MAX;                   // smallest key above b0
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                at_most += __popcll(__ballot(key[r] <= b0));
                if (key[r] > b0) above = key[r] < above ? key[r] : above;
            }
#pragma unroll
            for (int w = 32; w > 0; w >>= 1) { const long long x = __shfl_xor(above, w); above = x < above ? x : above; }
            const double next = at_most > lo + 1 ? mu : key_value<V>(above);
            mu = mu + frac * (next - mu);
        }
        if (lane == 0) s_mu = mu;
    }
    __syncthreads();
    const double mu = s_mu;
    for (int i = tid; i < chunks * 64; i += kManyThreads) {
        const double f = s_flag[i] ? selection_function(key_value<V>(s_key[i]), mu) : 0.0;
        s_f[i] = f;
        s_g[i] = f > 0.0 ? f : 0.0;
        s_flag[i] = 0;                                     // from here on: picked
        if (i < N) a.f[i] = f;
    }
    __syncthreads();

    // Sequential draws: draw t picks the first replica whose running sum exceeds u_t * S (it is a live one: a dead one
    // leaves the sum where it was).
    if (wave == 0) {
        const int e = lane & 15;
        auto segment_sums = [&]() {                         // of the lane's segment, elements 16 lane ... 16 lane + 15
            double part = 0.0;
            for (int r = 0; r < 4 * chunks; r += 4) {       // four segments at a time, a row of lanes each
                const double v = row_sums(s_g[r * 16 + lane]);
#pragma unroll
                for (int k = 0; k < 4; ++k) part = lane == r + k ? lane_value(v, 16 * k + 15) : part;
            }
            return part;
        };
        double sum = wave_sums(segment_sums()), error = kSumError * lane_value(sum, 63);
        int t = 0;
        double next_u = s_u[0];
        for (; t < a.n_select; ++t) {
            const double u = next_u;
            next_u = s_u[min(t + 1, a.n_select - 1)];       // (a read of LDS ahead)
            int seg, pick;
            double v;
            // the segment of the pick, its values and the pick, if the sums tell
            auto draw = [&]() {
                const double thr = u * lane_value(sum, 63);
                const unsigned long long over = __ballot(sum > thr);
                seg = over ? __builtin_amdgcn_readfirstlane(__ffsll((long long)over) - 1) : 0;
                v = s_g[seg * 16 + e];
                double below = lane_value(sum, max(seg, 1) - 1);
                below = seg > 0 ? below : 0.0;
                const Sides at = sides(below + row_sums(v), thr, error);
                pick = seg * 16 + __ffsll((long long)at.above) - 1;
                return (at.above | at.below) == ~0ull && at.above && thr - below > error;
            };
            bool known = draw();
            if (__builtin_expect(!known, 0)) {
                sum = wave_sums(segment_sums());
                error = kSumError * lane_value(sum, 63);
                known = draw();
            }
            if (__builtin_expect(!known, 0)) {              // the sums of the rule
                double run = 0.0, rec = 0.0;                // lane L of rec: after its segment
                for (int r = 0; r < 4 * chunks; ++r) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) run = run + s_g[r * 16 + k];
                    rec = lane == r ? run : rec;
                }
                const double limit = u * run;
                const unsigned long long hit = __ballot(rec > limit);
                if (!hit) break;                            // no replica is left to draw from (S = 0), nor in later draws
                seg = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1);
                v = s_g[seg * 16 + e];
                double q = seg > 0 ? lane_value(rec, seg - 1) : 0.0, mine = 0.0;
                for (int k = 0; k < 16; ++k) {
                    q = q + lane_value(v, k);
                    mine = e == k ? q : mine;
                }
                pick = seg * 16 + __ffsll((long long)__ballot(mine > limit)) - 1;
            }
            pick = __builtin_amdgcn_readfirstlane(pick);
            const double gone = lane_value(v, pick & 15);
            if (lane >= seg) sum = sum - gone;
            if (lane == 0) { s_g[pick] = 0.0; s_flag[pick] = 1; a.selected[t] = pick; }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        for (t += lane; t < a.n_select; t += 64) a.selected[t] = -1;
    }
    __syncthreads();

    // aggregation weights a_k and the ascending list the aggregate kernel walks (see select_kernel)
    unsigned long long picked[kPer];
    int count = 0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        picked[r] = __ballot(r < chunks && s_flag[r * 64 + lane]);
        count += __popcll(picked[r]);
    }
    double denom = (double)count;
    if (a.weight_mode == 1) {                              // the selected replicas' f, ascending, one after another (the others add +0.0)
        denom = 0.0;
#pragma unroll
        for (int r = 0; r < kPer; ++r)
            for (unsigned long long m = picked[r]; m; m &= m - 1) denom = denom + s_f[r * 64 + __ffsll((long long)m) - 1];
    }
    int before = 0;                                        // selected replicas in earlier chunks
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int idx = r * 64 + lane;
        if (r % (kManyThreads / 64) == wave && idx < N) {
            const bool on = (picked[r] >> lane) & 1ull;
            float w = 0.f;
            if (on) {
                w = (float)(((a.weight_mode == 1) ? s_f[idx] : 1.0) / denom);
                const int at = before + __popcll(picked[r] & ((1ull << lane) - 1ull));
                a.sel_sorted[at] = idx;
                a.sel_weight[at] = w;
            }
            a.flag[idx] = on ? 1 : 0;
            a.weights[idx] = w;
        }
        before += __popcll(picked[r]);
    }
}

// Version forecast (Sec. 3.2): double exponential smoothing of every replica's version series.
//   s1 <- alpha*v + (1-alpha)*s1;  s2 <- alpha*s1 + (1-alpha)*s2   (both start at the first observation)
//   forecast(m) = (2*s1 - s2) + alpha/(1-alpha)*(s1 - s2)*m
__global__ __launch_bounds__(64) void predict_kernel(const int32_t* versions, double* s1, double* s2, double* out, int n,
                                                     double alpha, int m, int first)
{
    for (int i = threadIdx.x; i < n; i += 64) {
        const double v = (double)versions[i];
        double a1, a2;
        if (first) { a1 = v; a2 = v; }
        else {
            a1 = alpha * v + (1.0 - alpha) * s1[i];
            a2 = alpha * a1 + (1.0 - alpha) * s2[i];
        }
        s1[i] = a1; s2[i] = a2;
        const double level = 2.0 * a1 - a2;
        const double trend = alpha / (1.0 - alpha) * (a1 - a2);
        out[i] = level + trend * (double)m;
    }
}

}  // namespace

hipError_t launch_predict(const int32_t* versions, double* s1, double* s2, double* out, int n, double alpha, int m,
                          int first, hipStream_t s)
{
    hipLaunchKernelGGL(predict_kernel, dim3(1), dim3(64), 0, s, versions, s1, s2, out, n, alpha, m, first);
    return hipGetLastError();
}

// Device address of this GPU's copy of `scratch`, looked up once per device with that device current.
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

hipError_t static_scratch(unsigned char** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<unsigned char*>(g_scratch_ptr[dev]);
    return hipSuccess;
}
}  // namespace

hipError_t launch_select_static(SelectArgs a, hipStream_t s)
{
    if (a.n < 1 || a.n > kMaxReplicas || a.n_select < 1 || a.n_select > a.n) return hipErrorInvalidValue;
    unsigned char* base = nullptr;
    const hipError_t e = static_scratch(&base);
    if (e != hipSuccess) return e;
    // the kernel writes every entry of these three before it reads it, so nothing has to be cleared between calls
    a.f = reinterpret_cast<double*>(base);
    a.sel_sorted = reinterpret_cast<int32_t*>(base + kMaxReplicas * sizeof(double));
    a.sel_weight = reinterpret_cast<float*>(base + kMaxReplicas * (sizeof(double) + sizeof(int32_t)));
    return launch_select(a, s);
}

hipError_t launch_select(const SelectArgs& a, hipStream_t s)
{
    // up to 64 replicas are a lane each and need no LDS in a draw (64 replicas, 8 draws 4.2 us; 65, 11 draws in the other 9.9)
    if (a.n <= 64) {
        if (a.versions_f64) hipLaunchKernelGGL(select_kernel<double>, dim3(1), dim3(64), 0, s, a);
        else hipLaunchKernelGGL(select_kernel<int>, dim3(1), dim3(64), 0, s, a);
    } else {
        if (a.versions_f64) hipLaunchKernelGGL(select_many_kernel<double>, dim3(1), dim3(kManyThreads), 0, s, a);
        else hipLaunchKernelGGL(select_many_kernel<int>, dim3(1), dim3(kManyThreads), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace hadfl
