// Stand-in for the HIP runtime under libhadfl.so, for host-only tests: "device" memory is host memory, copies are memcpy and
// a kernel launch is looked at instead of run.  From its parameters every launch declares which bytes it reads or writes and
// what they are for, and the checks are
//   * every range lies inside one of the buffers the caller gave to the library;
//   * ranges of different purposes (activations and their gradients, weight copies, split-K partial sums, batch-norm partial sums,
//     parameters, gradients, momentum, position tables, small state) never share a byte;
//   * the partial sums a batch norm reads are those that were left for it: no other launch has written the region since;
//   * the shares of the logits that the workgroups of a network of two dense layers read of each other are the launch before's, and
//     no workgroup of the launch writes to them.
// Loaded ahead of libhadfl.so with RTLD_GLOBAL, so that its symbols are found first.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../paper_2111_08274_amd/csrc/train_kernels.h"

using namespace hadfl;

namespace {

enum Kind { kData, kAct, kCopy, kSplit, kPartial, kParam, kGrad, kMom, kTable, kState, kKinds };
const char* const kKindName[kKinds] = {"data set", "activations", "weight copies", "split-K sums", "batch-norm sums", "parameters",
                                       "gradients", "momentum", "position tables", "state"};
typedef unsigned long long Addr;
struct Buf { Addr base, bytes; };
std::vector<Buf> g_bufs;
std::map<Addr, Addr> g_used[kKinds];                  // start -> end, merged
std::map<const void*, std::string> g_names;
std::string g_report, g_trace;
int g_errors = 0;
struct { const void* of; int entries; long long rep; } g_sums = {nullptr, 0, 0};      // what the batch-norm sums region holds
struct { const float* of; int n; } g_shares = {nullptr, 0};      // dense_pair_kernel: shares of the logits that the launch before wrote, of how many replicas
const void* g_mom = nullptr;                          // (parameters, gradients and momentum have one stride and one layout)

void error(const std::string& kernel, const std::string& what)
{
    if (g_errors++ < 20) g_report += kernel + ": " + what + "\n";
}

void use(const std::string& kernel, Kind kind, const void* p, long long bytes)
{
    if (bytes <= 0) return;
    Addr a = (Addr)p, b = a + (Addr)bytes;
    bool inside = false;
    for (const Buf& u : g_bufs) inside = inside || (a >= u.base && b <= u.base + u.bytes);
    if (!inside) { error(kernel, std::string(kKindName[kind]) + " outside the caller's buffers"); return; }
    for (int k = 0; k < kKinds; ++k) {
        if (k == kind) continue;
        auto it = g_used[k].lower_bound(b);
        if (it != g_used[k].begin() && (--it)->second > a)
            error(kernel, std::string(kKindName[kind]) + " of " + std::to_string(bytes) + " bytes run into " + kKindName[k]);
    }
    auto& m = g_used[kind];
    auto it = m.upper_bound(a);
    if (it != m.begin()) { auto q = it; --q; if (q->second >= a) { a = q->first; b = std::max(b, q->second); m.erase(q); } }
    for (it = m.lower_bound(a); it != m.end() && it->first <= b;) { b = std::max(b, it->second); it = m.erase(it); }
    m[a] = b;
}

std::vector<int> ints_of(const std::string& name)     // the integer template arguments of a mangled name
{
    std::vector<int> v;
    for (size_t i = 0; (i = name.find("Li", i)) != std::string::npos; ++i) v.push_back(std::atoi(name.c_str() + i + 2));
    return v;
}

struct Launch {
    std::string name;
    const int* order;
    int n;
    long long es;                                     // bytes per activation
    void tensor(Kind k, const void* p, long long rep_floats, long long bytes) const
    {
        if (p) for (int g = 0; g < n; ++g) use(name, k, (const float*)p + order[g] * rep_floats, bytes);
    }
    void act(const void* p, long long rep, long long elems) const { tensor(kAct, p, rep, elems * es); }
    void slots(Kind k, const void* p, long long rep_floats, long long floats) const
    {
        if (p) for (int g = 0; g < n; ++g) use(name, k, (const float*)p + g * rep_floats, floats * 4);
    }
    void data(const float* x, int n_samples, long long batch, long long sample) const
    {
        for (int g = 0; g < n; ++g) use(name, kData, x + (long long)order[g] * n_samples * sample, batch * sample * 4);
    }
    void sums(const float* p, long long rep, int entries, int channels, const void* of) const
    {
        slots(kPartial, p, rep, (long long)entries * 2 * channels);
        g_sums = {of, entries, rep};
    }
    void check_sums(const float* p, long long rep, int entries, int channels, const void* of) const
    {
        slots(kPartial, p, rep, (long long)entries * 2 * channels);
        if (g_sums.of != of || g_sums.entries != entries || g_sums.rep != rep) error(name, "reads sums that were left for another layer");
    }
};

bool has(const std::string& s, const char* part) { return s.find(part) != std::string::npos; }

void conv_general(Launch l, const GeneralConvParams& p, const std::vector<int>& t)
{
    l.order = p.order; l.n = p.n_active; l.es = p.bf16 ? 2 : 4;
    const long long out = (long long)p.B * p.Ho * p.Wo;
    if (p.cursor) l.data(p.a, p.n_samples, p.B, p.sample_sz);
    else l.act(p.a, p.a_rep, (long long)p.B * p.H * p.W * p.C);
    l.act(p.out, p.out_rep, out * p.N);
    l.act(p.mask, p.mask_rep, out * p.N);
    l.act(p.addend, p.addend_rep, out * p.N);
    const bool patch = has(l.name, "patch");
    const long long units = patch ? weight_fragment_units(p.bf16, p.N, p.R * p.S, p.C)
                                  : weight_copy_units(p.bf16, p.N, p.cursor ? 1 : p.R * p.S, p.cursor ? p.R * p.S * p.C : p.C);
    const int rows = patch ? 32 * t[0] * t[1] : t[0];
    l.act(p.stat_y, p.stat_y_rep, p.stat ? out * p.N : 0);
    for (int g = 0; g < l.n; ++g) use(l.name, kCopy, p.wmat + l.order[g] * p.wmat_rep, units * 2);
    l.tensor(kParam, p.bias, p.bias_rep, p.N * 4);
    if (p.perm) { use(l.name, kTable, p.perm, p.H * p.W * 4); use(l.name, kTable, p.posmask, p.H * p.W * 4); }
    if (p.stat) l.sums(p.stat, p.stat_rep, (int)((out + rows - 1) / rows), p.N, p.out);
}

void conv_fast(Launch l, const FastConvParams& p, int rows)
{
    l.order = p.order; l.n = p.n_active; l.es = 2;
    l.act(p.a, p.a_rep, (long long)p.M * p.C);
    l.act(p.out, p.out_rep, (long long)p.M * p.N);
    l.act(p.mask, p.mask_rep, (long long)p.M * p.N);
    l.act(p.stat_y, p.stat_y_rep, p.stat ? (long long)p.M * p.N : 0);
    for (int g = 0; g < l.n; ++g) use(l.name, kCopy, p.wmat + l.order[g] * p.wmat_rep, (long long)p.N * p.K * 2);
    l.tensor(kParam, p.bias, p.bias_rep, p.N * 4);
    if (p.perm) { use(l.name, kTable, p.perm, p.H * p.W * 4); use(l.name, kTable, p.posmask, p.H * p.W * 4); g_trace += "(its_rows_sorted)\n"; }
    if (p.stat) l.sums(p.stat, p.stat_rep, (p.M + rows - 1) / rows, p.N, p.out);
}

// weight gradient of `count` parameters: partial sums, or the gradient row, or the parameters with their momentum
void gradient(const Launch& l, float* out, long long out_rep, long long out_split, int splits, long long count, float* w, float* buf)
{
    if (splits > 1) { l.slots(kSplit, out, out_rep, (splits - 1) * out_split + count); return; }
    if (!w) { l.tensor(kGrad, out, out_rep, count * 4); return; }
    l.tensor(kParam, w, out_rep, count * 4);
    l.tensor(kMom, buf, out_rep, count * 4);
}

void batch_norm(Launch l, const BnParams& p, int n)
{
    l.order = p.order; l.n = n; l.es = p.bf16 ? 2 : 4;
    const long long all = (long long)p.rows * p.C;
    const bool bwd = has(l.name, "bwd") || has(l.name, "finalize_kernelILi1") || has(l.name, "sums_vec_kernelILi1") ||
                     has(l.name, "sums_pool") || has(l.name, "reduce_kernelILi2");
    l.act(p.x, p.x_rep, all);
    l.act(p.saved, p.saved_rep, 0);
    if (has(l.name, "apply") || has(l.name, "small")) {
        if (!p.pool || bwd) l.act(p.y, p.y_rep, all);
        l.act(p.pool_out, p.pool_out_rep, all / 4);
        l.act(p.add, p.add_rep, all);
        if (!p.pool) l.act(p.dy, p.dy_rep, bwd ? all : 0);
        l.act(p.pool_g, p.pool_g_rep, all / 4);
        l.act(p.mask, p.mask_rep, bwd ? all : 0);
    }
    l.tensor(kParam, p.params + p.w_off, p.row_stride, 2 * p.C * 4);
    if (!bwd) l.tensor(kParam, p.params + p.stat_off, p.row_stride, 2 * p.C * 4);
    else l.tensor(kGrad, p.grads + p.w_off, p.row_stride, 2 * p.C * 4);
    if (has(l.name, "sums") || has(l.name, "reduce")) l.sums(p.partial, p.partial_rep, p.chunks, p.C, p.x);
    else if (bwd ? p.bwd_stats_done : p.stats_done) {
        if (has(l.name, "finalize") || has(l.name, "small") || has(l.name, "Lb1E"))
            l.check_sums(p.partial, p.partial_rep, p.stat_entries, p.C, !bwd ? (const void*)p.x : p.pool ? (const void*)p.pool_g : (const void*)p.dy);
    } else if (has(l.name, "finalize") || has(l.name, "Lb1E")) l.check_sums(p.partial, p.partial_rep, p.chunks, p.C, p.x);
}

// Shares of the logits: what a launch reads of a step that ends is what the launch before it wrote of it, and it writes to none of
// that, nor to the hidden units of that step, whatever its workgroups' order.
void shares(const Launch& l, const DensePairParams& p)
{
    const long long bytes = (long long)p.H * p.batch * 4;
    if (p.n_end > 0) {
        l.tensor(kAct, p.share_in, p.act_rep, bytes);
        if (g_shares.of != p.share_in || g_shares.n < p.n_end) error(l.name, "reads shares that the launch before did not write");
    }
    g_shares = {nullptr, 0};
    if (p.n_begin < 1) return;
    l.tensor(kAct, p.share_out, p.act_rep, bytes);
    g_shares = {p.share_out, p.n_begin};
    const auto apart = [](const void* a, long long na, const void* b, long long nb) { return (Addr)a + (Addr)na <= (Addr)b || (Addr)b + (Addr)nb <= (Addr)a; };
    for (int g = 0; g < p.n_begin; ++g) {
        const float* const out = p.share_out + l.order[g] * p.act_rep;
        if (!apart(out, bytes, p.hidden + l.order[g] * p.act_rep, (long long)p.batch * p.H * l.es)) error(l.name, "writes shares over hidden units");
        for (int o = 0; o < p.n_end; ++o)
            if (!apart(out, bytes, p.share_in + l.order[o] * p.act_rep, bytes)) { error(l.name, "writes shares that another workgroup of the launch may still read"); return; }
    }
}

void look(const std::string& name, dim3 grid, void** args)
{
    Launch l{name, nullptr, 0, 4};
    const std::vector<int> t = ints_of(name);
    if (has(name, "conv_general_kernel") || has(name, "conv_general_patch_kernel")) conv_general(l, *(GeneralConvParams*)args[0], t);
    else if (has(name, "11conv_kernel")) conv_fast(l, *(FastConvParams*)args[0], t[0]);
    else if (has(name, "wgrad_general_kernel") || has(name, "wgrad_general_position_kernel")) {
        const GeneralWgradParams& p = *(GeneralWgradParams*)args[0];
        l.order = p.order; l.n = p.n_active; l.es = p.bf16 ? 2 : 4;
        if (p.cursor) l.data(p.x, p.n_samples, p.B, p.sample_sz); else l.act(p.x, p.x_rep, (long long)p.B * p.H * p.W * p.C);
        l.act(p.dy, p.dy_rep, (long long)p.K * p.N);
        gradient(l, p.out, p.out_rep, p.out_split, p.splits, ((long long)p.R * p.S * p.C + (p.has_bias ? 1 : 0)) * p.N, p.sgd_w, p.sgd_buf);
    } else if (has(name, "conv_first")) {
        const FirstConvParams& p = *(FirstConvParams*)args[0];
        l.order = p.order; l.n = (int)grid.y; l.es = 2;
        l.data(p.x, p.n_samples, p.B, (long long)p.H * p.W * p.C);
        l.act(p.out, p.out_rep, (long long)p.M * p.N);
        l.act(p.dy, p.dy_rep, (long long)p.M * p.N);
        if (p.gout) gradient(l, p.gout, p.gout_rep, p.gout_split, p.splits, (long long)(p.K + (p.bias ? 1 : 0)) * p.N, nullptr, nullptr);
    } else if (has(name, "wgrad_kernel") || has(name, "wgrad_taps_kernel") || has(name, "wgrad_images_kernel")) {
        const FastWgradParams& p = *(FastWgradParams*)args[0];
        l.order = p.order; l.n = p.n_active; l.es = 2;
        l.act(p.x, p.x_rep, (long long)p.K * p.C);
        l.act(p.dy, p.dy_rep, (long long)p.K * p.N);
        gradient(l, p.out, p.out_rep, p.out_split, p.splits, (long long)p.M * p.N, p.sgd_w, p.sgd_buf);
    } else if (has(name, "weight_copy_kernel") || has(name, "weight_prep_kernel")) {
        const bool general = has(name, "weight_copy");
        const WeightCopies& all = *(WeightCopies*)args[0];
        const WeightPrepParams& q = *(WeightPrepParams*)args[0];
        l.n = (int)(general ? grid.y : grid.z);
        for (int k = 0; k < (general ? all.count : 1); ++k) {
            const WeightCopyParams& c = all.layer[k];
            l.order = general ? c.order : q.order;
            const auto units = general && c.fragments ? weight_fragment_units : weight_copy_units;
            const long long nf = general ? units(c.bf16, c.N, c.taps, c.C) : (long long)q.C * q.N * q.taps;
            const long long nb = general ? units(c.bf16, c.C, c.taps, c.N) : nf;
            for (int g = 0; g < l.n; ++g) {
                const long long at = l.order[g] * (general ? c.wcopy_rep : q.wbf_rep);
                use(name, kCopy, (general ? c.wf : q.wf) + at, nf * 2);
                if (general ? c.wb : q.wb) use(name, kCopy, (general ? c.wb : q.wb) + at, nb * 2);
            }
        }
    } else if (has(name, "splitk_reduce")) {
        l.n = (int)grid.y;
        const long long stride = *(long long*)args[1];
        l.slots(kSplit, *(const float**)args[0], stride * *(int*)args[2], stride * *(int*)args[2]);
    } else if (has(name, "dense_rows_fwd")) {
        const DenseRowsParams& p = *(DenseRowsParams*)args[0];
        l.order = p.order; l.n = (int)grid.z; l.es = p.bf16 ? 2 : 4;
        if (p.cursor) l.data(p.x, p.n_samples, p.rows, p.K); else l.act(p.x, p.x_rep, (long long)p.rows * p.K);
        l.act(p.out, p.out_rep, (long long)p.rows * p.N);
        l.tensor(kParam, p.w, p.w_rep, (long long)(p.K + (p.has_bias ? 1 : 0)) * p.N * 4);
    } else if (has(name, "dense_pair")) {
        const DensePairParams& p = *(DensePairParams*)args[0];
        l.order = p.order; l.n = std::max(p.n_end, p.n_begin); l.es = p.bf16 ? 2 : 4;
        l.data(p.x, p.n_samples, p.batch, p.K);
        l.act(p.hidden, p.act_rep, (long long)p.batch * p.H);
        shares(l, p);
        l.tensor(kParam, p.w1, p.w_rep, (long long)(p.K + (p.has_bias1 ? 1 : 0)) * p.H * 4);
        l.tensor(kParam, p.w2, p.w_rep, (long long)(p.H + (p.has_bias2 ? 1 : 0)) * p.N * 4);
        l.tensor(kMom, p.m1, p.w_rep, (long long)(p.K + (p.has_bias1 ? 1 : 0)) * p.H * 4);
        l.tensor(kMom, p.m2, p.w_rep, (long long)(p.H + (p.has_bias2 ? 1 : 0)) * p.N * 4);
        use(name, kState, p.loss, 4 * l.n);
    } else if (has(name, "dense_small")) {
        const DenseSmallParams& p = *(DenseSmallParams*)args[0];
        l.order = p.order; l.n = (int)grid.y; l.es = p.bf16 ? 2 : 4;
        l.act(p.x, p.x_rep, (long long)p.rows * p.K);
        l.act(p.out, p.out_rep, (long long)p.rows * p.N);
        l.act(p.dy, p.dy_rep, (long long)p.rows * p.N);
        l.act(p.dx, p.dx_rep, (long long)p.rows * p.K);
        l.tensor(kParam, p.w, p.w_rep, (long long)(p.K + (p.has_bias ? 1 : 0)) * p.N * 4);
    } else if (has(name, "igemm")) {
        const GemmParams& p = *(GemmParams*)args[0];
        l.order = p.order; l.n = p.n_active > 0 ? p.n_active : (int)grid.z; l.es = has(name, "bf16") ? 2 : 4;
        const long long src = (long long)p.B * p.H * p.W * p.Cin, dst = (long long)p.B * p.Ho * p.Wo * p.Cout;
        if (p.cursor) l.data(p.a, p.n_samples, p.B, p.sample_sz); else l.act(p.a, p.a_rep, p.mode == kDgrad ? dst : src);
        if (p.mode == kWgrad) { l.act(p.dy, p.dy_rep, dst); gradient(l, p.out, p.out_rep, p.out_split, p.splits, (long long)p.M * p.N, nullptr, nullptr); }
        else l.act(p.out, p.out_rep, p.mode == kDgrad ? src : dst);
    } else if (has(name, "zero_kernel")) {
        const EwParams& p = *(EwParams*)args[0];
        l.order = p.order; l.n = (int)grid.y; l.es = p.bf16 ? 2 : 4;
        l.act(p.out, p.out_rep, p.count);
    } else if (has(name, "bn_")) batch_norm(l, *(BnParams*)args[0], (int)grid.y);
    else if (has(name, "softmax_ce")) {
        const LossParams& p = *(LossParams*)args[0];
        l.order = p.order; l.n = (int)grid.x; l.es = p.bf16 ? 2 : 4;
        l.act(p.logits, p.logits_rep, (long long)p.batch * p.n_classes);
        l.act(p.dlogits, p.dlogits_rep, (long long)p.batch * p.n_classes);
        for (int g = 0; g < l.n; ++g) use(name, kState, p.cursor + l.order[g], 8);
        use(name, kState, p.order, 4 * l.n);
        use(name, kState, p.loss, 4 * l.n);
    }
}

dim3 g_grid, g_block;
size_t g_shmem;
hipStream_t g_stream;

}  // namespace

extern "C" {

// ---- for the test ----
void check_reset(const unsigned long long* bufs, int n)
{
    g_bufs.clear(); g_report.clear(); g_trace.clear(); g_errors = 0; g_sums = {nullptr, 0, 0}; g_shares = {nullptr, 0};
    for (auto& m : g_used) m.clear();
    for (int i = 0; i < n; ++i) g_bufs.push_back({bufs[2 * i], bufs[2 * i + 1]});
}
const char* check_report() { return g_report.c_str(); }
const char* check_trace() { return g_trace.c_str(); }          // mangled kernel names, one a line, in launch order (conv_kernel: a line more where its rows are sorted)

// ---- the HIP runtime ----
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s)
{
    g_grid = grid; g_block = block; g_shmem = shmem; g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s)
{
    *grid = g_grid; *block = g_block; *shmem = g_shmem; *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t)
{
    const std::string& name = g_names[f];
    g_trace += name + "\n";
    look(name, grid, args);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(dst, src, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { std::memset(p, 0, sizeof(*p)); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char s[1 << 16]; *p = s; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)1; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }

}

// the copies' layout, as conv_general.hip defines it
long long hadfl::weight_copy_units(int bf16, int rows, int taps, int channels)
{
    const int per = bf16 ? 64 : 32, bytes = bf16 ? 128 : 192;
    return (long long)rows * taps * ((channels + per - 1) / per) * (bytes / 2);
}
long long hadfl::weight_fragment_units(int bf16, int rows, int taps, int channels) { return weight_copy_units(bf16, (rows + 31) / 32 * 32, taps, channels); }
