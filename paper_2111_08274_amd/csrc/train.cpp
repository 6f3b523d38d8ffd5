// Host-side schedule of hadfl_local_steps: a fixed launch sequence per sub-step s = 1..E_max, each launch grouped
// over the replicas that still have steps left (a prefix of the replicas ordered by step count, kept in device
// memory).  There is no host loop over replicas and no host read-back inside a cycle.
#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "train.h"
#include "kernels.h"
#include "train_kernels.h"

namespace hadfl {

class TrainEngine {
public:
    hadfl_config cfg;
    NetPlan plan;
    TrainBuffers buf;
    std::vector<int32_t> steps;
    int e_max = 0;
    std::vector<int> n_active;            // n_active[s] = replicas with E_k > s
    // per-tensor activation / gradient offsets (floats) inside one replica's block of `work`
    std::vector<int64_t> act_off, grad_off;
    int64_t rep_block = 0;                // floats of activations + gradients per replica
    std::vector<int64_t> saved_off;       // per layer (BN): offset of saved mean/istd inside the replica block
    int64_t shared_off = 0;               // start of the region shared by all layers (split-K partials, BN partials)
    int64_t shared_floats = 0;
    int64_t bn_off = 0, bn_floats = 0;    // per-chunk partial sums of the batch-norm reductions (their own region: weight
                                          // gradients may run beside them on the side stream)
    std::vector<int> splits;              // per layer: split-K factor of the weight gradient
    std::vector<std::vector<WgradPlan>> wgrad_plans;   // lean and general layers: the plan for 1, 2, ... active replicas instead
    std::vector<int> bn_chunks;           // per layer
    std::vector<char> grad_written;       // scratch for the backward pass
    // ReLU fusion: a ReLU that is the only consumer of a conv / dense / BN / add output is folded into that layer's
    // store (the layer writes the ReLU's output tensor; the ReLU layer itself issues nothing).  Its backward is folded
    // into whoever writes the gradient of that tensor: those kernels zero the gradient where the stored output is not
    // positive, so the tensor's gradient buffer holds the gradient before the ReLU.
    std::vector<int> out_tensor;          // per layer: tensor the layer writes (its own, or the fused ReLU's)
    std::vector<char> skip;               // per layer: fused away
    std::vector<char> fused_relu;         // per layer: applies max(., 0) in its store
    std::vector<char> masked;             // per tensor: gradient writers must apply the (value > 0) mask
    std::vector<int> unread;              // tensors that no layer reads, the network's output apart: their gradient is zero
    // Pool fusion: a 2x2 max-pool that is the only consumer of a batch-norm layer's (ReLU'd) output is folded into the
    // BN kernels: forward writes the pooled tensor as well, backward forms the full-resolution gradient on the fly from
    // the pooled gradient.  The pool layer itself issues nothing.
    std::vector<int> pool_of;             // per layer: index of the folded pool layer, or -1
    // Sum fusion: the addition of two tensors behind a batch norm that is only read there runs in that BN's forward store (the
    // second of two such BNs: the other operand exists by then).  Its backward pass copies the gradient to both operands,
    // but for those with no ReLU mask and no other reader: their gradient IS the sum's, and shares its buffer.
    std::vector<double> beside;           // per layer: flops of the data gradients of this layer and those below, one replica
    std::vector<int> add_into;            // per layer (BN): the ADD layer folded into its forward store, or -1
    std::vector<char> add_done;           // per layer (ADD): forward folded away
    // An operand that does need a copy, but whose next gradient comes from a convolution run from patches (the shortcut of a residual block
    // without a convolution in it: the block's first convolution), gets none: that convolution's data gradient adds the sum's
    // gradient from where it lies.
    std::vector<char> late_add;           // per layer (ADD): bit 0, 1: operand 0, 1 is one of these
    std::vector<int> pending_grad;        // per tensor, scratch for the backward pass: the tensor whose gradient is still to be added, or -1
    // Statistics fusion: a lean or general convolution whose output feeds a batch norm only leaves the per-channel
    // sums of its output in the BN partial region, and that BN's forward skips its own sums pass.
    std::vector<int> stat_for;            // per layer: the BN layer fed by this convolution's statistics, or -1
    std::vector<int> stat_from;           // per layer (BN): the convolution that supplies them, or -1
    std::vector<int> stat_rows;           // per layer (BN): rows per statistics entry of the latest forward launch
    // The same in the backward pass: the convolution whose data gradient completes the gradient of a batch norm's output leaves, from
    // its epilogue, the per-channel sums that batch norm's backward pass needs, and the BN skips its own sums pass.  In bf16 a lean
    // convolution that is the only consumer of the output (after its fused ReLU and folded pool) forms them from that output,
    // which it reads as its mask; else one run from patches, from the batch norm's input (bstat_input): the same sums as the pass forms,
    // for a read of that input in place of one of it, one of the gradient and a launch.  A ResNet-18 on 16 replicas, fp32, alone
    // on the chip: sums passes 2.76 -> 0.85 ms a cycle, the data gradients that form them 0.55 ms longer.
    std::vector<int> bstat_for;           // per layer (conv): the BN layer its data gradient serves, or -1
    std::vector<char> bstat_input;        // per layer (conv): sums with the BN's input
    std::vector<int> bstat_rows;          // per layer (BN): rows per entry of the latest data-gradient launch (0: none)
    std::vector<int64_t> bstat_rep;       // per layer (BN): floats per replica slot of those entries
    // bf16 configuration: regular convolution layers keep two bf16 weight matrices (forward / data-gradient order)
    std::vector<char> fast;               // per layer: the lean bf16 kernels apply (those of forward and data gradient unless `general`)
    std::vector<char> general, general_w; // per layer: the kernels of conv_general.hip apply (forward and data gradient; weight
                                          // gradient)
    std::vector<char> patch;              // per general layer: forward and data gradient run in conv_general_patch.hip
    std::vector<int64_t> wf_off, wb_off;  // per layer: offsets (2-byte units) inside one replica's block of weight copies, or -1
    int64_t wbf_rep = 0;                  // bf16 elements per replica
    int64_t wbf_off = 0;                  // start of the bf16 weight region inside `work` (floats)
    // Option HADFL_OPT_TILE_HINT: 1 makes the convolution kernels take their largest tiles wherever the layer shape allows,
    // whatever the launch size (lets small problems exercise them); 2 keeps the lean weight gradients in wgrad_kernel.
    int tile_hint = 0;
    // Weight gradients (and their split-K reduction / fused update) depend only on dY and the stored activations, not on
    // the data-gradient chain, so they run on a second stream beside it; joined before the update kernel.
    // Option HADFL_OPT_SIDE_STREAM = 0 turns this off.
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    bool use_side = true;
    // Layers whose weight-gradient kernel applies the update itself (lean kernel, no split): their slices of the
    // parameter rows, ascending; the update kernel runs over the segments in between.
    std::vector<char> fused_update;       // per layer
    std::vector<char> prepped;            // per layer: bf16 copies for the coming sub-step are already written
    std::vector<std::pair<int64_t, int64_t>> update_segments;   // [first, first + count) floats
    // Position tables of the regular convolution layers (see FastConvParams::perm): per layer HW sorted positions
    // followed by HW tap masks, all layers back to back in `tables`; copied to `work` at tab_off by the first run.
    std::vector<int64_t> tab_idx;         // per layer: start inside `tables`, or -1
    std::vector<int32_t> tables;
    int64_t tab_off = 0;                  // start of the table region inside `work` (floats)
    bool tables_uploaded = false;
};

namespace {

int ilog2_exact(int v) { int s = 0; while ((1 << s) < v) ++s; return (1 << s) == v ? s : -1; }

struct Layout {
    std::vector<int64_t> act_off, grad_off, saved_off;
    std::vector<int> splits, bn_chunks;
    std::vector<std::vector<WgradPlan>> wgrad_plans;
    int64_t rep_block = 0, shared_floats = 0, bn_floats = 0;
    std::vector<char> fast, general, general_w, patch;
    std::vector<int64_t> wf_off, wb_off;       // in 2-byte units inside one replica's block of weight copies
    int64_t wbf_rep = 0;
    std::vector<int64_t> tab_idx;
    int64_t tab_ints = 0;
};

bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

int64_t up64(int64_t v) { return (v + 63) / 64 * 64; }

// Measured on 32 replicas of the VGG-16 shape: forward and data gradient gain up to 8 x 8 images, the weight gradient up
// to 4 x 4; beyond that the scattered rows of a position-major tile cost more than the skipped taps save.
constexpr int kMaxTablePositions = 64, kMaxTablePositionsWgrad = 16;

// Stride-1 "same" convolutions with 64-multiple channels, not on the data set
bool regular_layer(const NetPlan& plan, const Layer& l)
{
    return l.type == HADFL_OP_CONV && l.in0 != 0 && l.stride == 1 && 2 * l.pad == l.k - 1 && l.k * l.k <= 32 &&
           plan.tensors[l.in0].c % 64 == 0 && l.cout % 64 == 0;
}

// bf16 configuration: the lean kernels take the regular convolutions on power-of-two images
bool lean_layer(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    return cfg.bf16 && regular_layer(plan, l) && is_pow2(plan.tensors[l.in0].h) && is_pow2(plan.tensors[l.in0].w);
}

// The kernels of conv_general.hip take the other convolution and dense layers whose channels come in 16-byte groups, and in
// fp32 the convolutions on the data set, gathered value by value (in bf16 those have kernels of their own).  Not narrow
// classifiers, which have their own kernels too.  Offsets inside one replica's tensor are 32-bit byte offsets.
// An fp32 network with convolutions and no batch norm amplifies the order of its sums: with the CNN workload's learning rate
// one rounding of the initial weights moves the weights after two cycles by 2e-6 to 7e-5, and a run of it is reproducible
// only in one order.  The layers of such networks that are not regular, the CNN workload's among them, keep the kernels whose
// sums run along K in one chain (gemm.hip, dense_small_fwd).  Regular layers never had one order (their tiles were
// walked in kernels of their own) and take the general kernels: a VGG of 64 to 512 channels without batch norm on 1 / 4 / 16
// replicas, batch 64, 1.06 / 2.41 / 7.36 ms a step against 3.02 / 5.11 / 15.5 in gemm.hip.
bool one_chain_net(const hadfl_config& cfg, const NetPlan& plan)
{
    bool conv = false, norm = false;
    for (const Layer& l : plan.layers) { conv = conv || l.type == HADFL_OP_CONV; norm = norm || l.type == HADFL_OP_BN; }
    return !cfg.bf16 && conv && !norm;
}

bool gather_layer(const hadfl_config& cfg, const Layer& l) { return !cfg.bf16 && l.type == HADFL_OP_CONV && l.in0 == 0; }

bool general_layer(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    if ((l.type != HADFL_OP_CONV && l.type != HADFL_OP_DENSE) || lean_layer(cfg, plan, l)) return false;
    if (one_chain_net(cfg, plan) && !regular_layer(plan, l)) return false;
    const TensorShape a = plan.tensors[l.in0], r = plan.tensors[l.out];
    const bool conv = l.type == HADFL_OP_CONV;
    const int64_t cin = conv ? a.c : a.numel(), taps = conv ? l.k * l.k : 1, unit = cfg.bf16 ? 8 : 4;
    const bool gather = gather_layer(cfg, l);
    // Eight channels in and out fill an eighth of a slab of bf16; with more than nine taps that outweighs what the faster weight
    // gradient gives (five 5 x 5 layers on 28 x 28 images, batch 32, 16 replicas: 1.07 ms a step, gemm_bf16.hip 0.93).
    if (cfg.bf16 && conv && cin <= 8 && l.cout <= 8 && taps > 9) return false;
    if (l.cout % unit != 0 || (!gather && (cin % unit != 0 || taps > 32))) return false;
    if (conv ? l.in0 == 0 && !gather : (l.cout <= 16 || (l.in0 == 0 && cin % 16 != 0))) return false;
    if (l.w_off % 4 != 0 || (l.bias && l.b_off != l.w_off + l.w_count)) return false;
    const int64_t limit = int64_t(1) << 31, B = cfg.batch;
    return B * a.numel() * 4 < limit && B * r.numel() * 4 < limit &&
           weight_copy_units(cfg.bf16, l.cout, (int)taps, (int)cin) * 2 < limit && weight_copy_units(cfg.bf16, (int)cin, (int)taps, l.cout) * 2 < limit;
}

// The classifier (a dense layer with at most 16 outputs, not on the data set) has its own kernels
bool small_dense_layer(const Layer& l)
{
    return l.type == HADFL_OP_DENSE && l.cout <= 16 && l.in0 != 0 && (!l.bias || l.b_off == l.w_off + l.w_count);
}

// Its backward pass in one launch walks the samples in four chains per 64 features: 10 outputs on 512 features, 4 replicas,
// 15 / 22 / 37 / 67 / 127 us at 64 / 128 / 256 / 512 / 1024 samples, where data gradient, weight gradient and its reduction
// take 37 / 41 / 43 / 47 / 48 us as launches of their own: beyond 256 samples they are the shorter way.
bool dense_one_pass_bwd(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    return small_dense_layer(l) && !one_chain_net(cfg, plan) && cfg.batch <= 256;
}

// Forward straight from the master weights: classifiers and the dense layers on the data set, whose copies no data gradient
// would use.  Classifiers on long rows have a workgroup per row instead (see the kernels).
bool dense_rows_layer(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    if (!dense_rows_supported(cfg.batch, plan.tensors[l.in0].numel())) return false;
    if (one_chain_net(cfg, plan) || (l.in0 != 0 && plan.tensors[l.in0].numel() >= 2048)) return false;
    return l.type == HADFL_OP_DENSE && (l.cout <= 16 || l.in0 == 0) && (!l.bias || l.b_off == l.w_off + l.w_count);
}

// A layer on the data set leaves that kernel, which shares no operand between workgroups, where the generic kernel's 128 x 128
// tiles fill the chip one and a half times.  2048 outputs, 256 samples on 8 / 12 / 16 replicas (256 / 384 / 512 tiles), generic
// and this, us: 784 features fp32 143 177 186 and 114 155 200, bf16 189 232 234 and 132 190 250; 100 features bf16, a step
// or none per wave, 42 51 52 and 42 61 77: there the line is at one round.
bool dense_rows_pays(const hadfl_config& cfg, const NetPlan& plan, const Layer& l, int n)
{
    const int64_t tiles = (int64_t)((cfg.batch + 127) / 128) * ((l.cout + 127) / 128) * n;
    return l.in0 != 0 || tiles <= (cfg.bf16 && plan.tensors[0].numel() < 512 ? 256 : 384);
}

// The network is a dense layer on the data set with a ReLU and a classifier behind it, of a size for dense_pair_kernel in a call of this many
// steps.  Four steps a call, us a step layer by layer and there, batch 8 / 32 / 64 / 128:
//   784 features, 128 hidden units:   1 replica 25 28 32 41 and 17 19 26 41,   4: 27 30 33 44 and 16 17 24 39,   16: 30 34 39 50 and 16 18 24 40,
//                                     64: 45 50 66 91 and 37 42 57 86,   128: 72 80 106 157 and 71 80 110 192
//   1024 features, 256 hidden units:  4: 30 34 39 49 and 19 22 32 52,   16: 44 48 55 74 and 23 27 38 61,   32: 51 58 73 100 and 47 54 74 120,
//                                     64: 83 94 118 182 and 89 104 146 267
//   128 features, 256 hidden units:   32: 26 29 38 53 and 20 22 31 51,   64: 32 35 46 67 and 36 41 75 133
// A compute unit holds one workgroup of sixteen hidden units: up to 256 this is the shorter way, but for batches above 64 on few replicas
// in calls of one step, which have no beginning to share a launch with (one replica, batch 128 43 and 45).  Beyond 256 the second round of
// workgroups costs as much as the first, and the line is at 6.5 million multiply-adds of a replica's hidden layer (layer by layer over
// this: below it, two steps a call and more, 0.91 to 1.46, half of them above 1.2; above it 0.73 to 1.15) and at small weights for calls of one step (1024 x 256, 32
// replicas 53 59 74 101 and 55 63 85 131).  From 512 on the layers' own kernels fill the chip: 1024 workgroups 0.50 to 1.06, 2048 0.39 to 0.93.
// More than 256 hidden units stay with them too (512, 128 features, 16 replicas 27 30 40 56 and 23 25 37 62; others not measured).  Rows of
// fewer than 128 features leave waves without a block; they stay with the single layers' kernels, though this one would be the faster for
// them too (32 features, 64 hidden units, 4 replicas: 20 22 28 38 and 9 10 13 20), so that networks of a few features still run those.
bool dense_pair_net(const hadfl_config& cfg, const NetPlan& plan, int steps)
{
    if (plan.layers.size() != 3) return false;
    const Layer &a = plan.layers[0], &r = plan.layers[1], &b = plan.layers[2];
    if (a.type != HADFL_OP_DENSE || a.in0 != 0 || r.type != HADFL_OP_RELU || r.in0 != a.out || b.type != HADFL_OP_DENSE || b.in0 != r.out) return false;
    if (b.cout != cfg.n_classes || (a.bias && a.b_off != a.w_off + a.w_count) || (b.bias && b.b_off != b.w_off + b.w_count)) return false;
    const int64_t K = plan.tensors[0].numel(), groups = (int64_t)(a.cout / 16) * cfg.n_replicas;
    if (K < 128 || K > 1024 || a.cout > 256 || (cfg.batch > 64 && cfg.n_replicas < 8)) return false;
    if (groups > 256 && (groups > 512 || cfg.batch * a.w_count > 6500000 || (steps == 1 && a.w_count > 131072))) return false;
    return dense_pair_supported(cfg.batch, (int)K, a.cout, b.cout);
}

// Directions of a general layer that run there.  A convolution on the data set is gathered value by value, which pays where the
// generic kernel (gemm.hip) would gather too.  That one reads its source in 16-byte pieces when the channels come in sixteens
// (forward) or fours (weight gradient), and is then the faster one, but for footprints that are one tile of 32 rows.
// Images of 32 x 32, batch 128, 8 replicas, generic over gathered time: forward, 3 x 3 filters, 16 outputs, 1 / 3 / 8 / 16 / 64
// channels 1.1 1.6 1.6 0.85 0.52; weight gradient, 96 outputs, 3 x 3 and 5 x 5, 3 channels 1.4 0.9, 4 channels 0.7 0.6, 8
// channels 0.8 0.9; 1 x 1, 4 / 16 / 32 channels 1.3 1.3 1.3.
bool general_forward(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    return general_layer(cfg, plan, l) && !(gather_layer(cfg, l) && plan.tensors[0].c % 16 == 0);
}
bool general_wgrad(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    return general_layer(cfg, plan, l) && !(gather_layer(cfg, l) && plan.tensors[0].c % 4 == 0 && l.k * l.k * plan.tensors[0].c > 32);
}

// Lean and general layers whose forward pass and data gradient run from patches (conv_general_patch.hip)
bool patch_layer(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    if (l.type != HADFL_OP_CONV || l.in0 == 0 || l.stride != 1 || 2 * l.pad != l.k - 1) return false;
    const TensorShape a = plan.tensors[l.in0];
    const bool fits = cfg.batch * (int64_t)a.h * a.w * std::max(a.c, l.cout) * 4 < int64_t(1) << 31 && (int64_t)l.k * l.k * a.c * l.cout * 2 < int64_t(1) << 31 && l.w_off % 4 == 0;
    return (lean_layer(cfg, plan, l) ? fits : general_layer(cfg, plan, l)) && conv_patch_supported(cfg.bf16, a.h, a.w, a.c, l.cout, l.k);
}

// Plan of a general layer's weight gradient with n active replicas
WgradPlan general_wgrad_plan(const hadfl_config& cfg, const NetPlan& plan, const Layer& l, int n)
{
    const TensorShape a = plan.tensors[l.in0], r = plan.tensors[l.out];
    const bool conv = l.type == HADFL_OP_CONV;
    const WgradPlan pixels = wgrad_general_plan((int)(conv ? l.k * l.k * a.c : a.numel()), l.cout, (int)(cfg.batch * (conv ? r.h * r.w : 1)), n, gather_layer(cfg, l));
    if (cfg.bf16 || !conv || l.in0 == 0 || l.k != 3 || l.stride != 1 || l.pad != 1 || !wgrad_positions_supported(cfg.batch, a.h, a.w, a.c, l.cout)) return pixels;
    // The estimate for the kernel that walks pixels is low for launches of few workgroups (64 channels, 32 x 32 images, batch 64, one
    // replica: 42 us, measured with the reduction 67, the other 46).  With this margin the choice is the faster one or within 1 us of
    // it on layers of 64 to 512 channels and 1 to 16 replicas.
    const WgradPlan positions = wgrad_positions_plan(cfg.batch, a.h, a.w, a.c, l.cout, n);
    return positions.time <= 1.25f * pixels.time + 1.0f ? positions : pixels;
}

// What the plan of a lean layer's follows from
FastWgradParams lean_wgrad_shape(const hadfl_config& cfg, const NetPlan& plan, const Layer& l)
{
    const TensorShape a = plan.tensors[l.in0];
    FastWgradParams f{};
    f.B = cfg.batch; f.H = a.h; f.W = a.w; f.C = a.c; f.N = l.cout; f.R = f.S = l.k; f.pad = l.pad;
    f.K = cfg.batch * a.h * a.w; f.has_bias = l.bias; f.M = l.k * l.k * a.c + (l.bias ? 1 : 0);
    return f;
}
// floats per replica of the statistics entries a convolution's epilogue leaves for `rows` outputs of c channels: one entry per
// tile, which has at least 128 rows in the lean kernels and 32 in the general ones
int64_t stat_floats(int64_t rows, int c, bool lean) { const int64_t tile = lean ? 128 : 32; return (rows + tile - 1) / tile * 2 * c; }

bool same_shape(const NetPlan& plan, const Layer& l, const Layer& m)
{
    const auto same = [&](int t, int u) { const TensorShape a = plan.tensors[t], b = plan.tensors[u]; return a.h == b.h && a.w == b.w && a.c == b.c; };
    return l.type == m.type && l.k == m.k && l.stride == m.stride && l.pad == m.pad && l.cout == m.cout && l.bias == m.bias &&
           (l.in0 == 0) == (m.in0 == 0) && same(l.in0, m.in0) && same(l.out, m.out);
}

Layout make_layout(const hadfl_config& cfg, const NetPlan& plan)
{
    Layout L;
    const int T = (int)plan.tensors.size();
    const int64_t B = cfg.batch;
    L.act_off.assign(T, -1); L.grad_off.assign(T, -1);
    int64_t off = 0;
    for (int t = 1; t < T; ++t) { L.act_off[t] = off; off += up64(B * plan.tensors[t].numel()); }
    for (int t = 1; t < T; ++t) { L.grad_off[t] = off; off += up64(B * plan.tensors[t].numel()); }
    L.saved_off.assign(plan.layers.size(), -1);
    L.splits.assign(plan.layers.size(), 1); L.wgrad_plans.resize(plan.layers.size());
    L.bn_chunks.assign(plan.layers.size(), 1);
    int64_t shared = 0, bn_shared = 0;
    for (size_t i = 0; i < plan.layers.size(); ++i) {
        const Layer& l = plan.layers[i];
        const TensorShape a = plan.tensors[l.in0], r = plan.tensors[l.out];
        if (l.type == HADFL_OP_BN) {
            L.saved_off[i] = off; off += up64(2 * (int64_t)a.c);
            const int64_t rows = B * a.h * a.w;
            int chunks = (int)std::min<int64_t>(128, std::max<int64_t>(1, rows / 128));
            L.bn_chunks[i] = chunks;
            bn_shared = std::max<int64_t>(bn_shared, (int64_t)cfg.n_replicas * chunks * 2 * a.c);
        } else if (l.type == HADFL_OP_CONV || l.type == HADFL_OP_DENSE) {
            // weight gradient: contraction over K = B*Ho*Wo rows; split it until the launch has enough workgroups
            const int64_t K = B * r.h * r.w;
            const int64_t M = (l.type == HADFL_OP_CONV ? (int64_t)l.k * l.k * a.c : a.numel()) + (l.bias ? 1 : 0);
            const int64_t tiles = ((M + 127) / 128) * ((l.cout + 127) / 128);
            int64_t want = (2048 + tiles * cfg.n_replicas - 1) / (tiles * cfg.n_replicas);
            int64_t maxs = std::max<int64_t>(1, K / 128);
            int s = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(want, maxs), 256));
            if (lean_layer(cfg, plan, l) || general_wgrad(cfg, plan, l)) {      // chosen per launch
                s = 1;
                size_t same = 0;                      // an earlier layer of the same shape has the same plans
                while (same < i && !(!L.wgrad_plans[same].empty() && same_shape(plan, plan.layers[same], l))) ++same;
                if (same < i) L.wgrad_plans[i] = L.wgrad_plans[same];
                else for (int n = 1; n <= cfg.n_replicas; ++n) {
                    L.wgrad_plans[i].push_back(lean_layer(cfg, plan, l) ? wgrad_fast_plan(lean_wgrad_shape(cfg, plan, l), n) : general_wgrad_plan(cfg, plan, l, n));
                    const int sn = L.wgrad_plans[i].back().splits;
                    if (sn > 1) shared = std::max<int64_t>(shared, (int64_t)n * sn * up64(M * l.cout));
                }
            }
            L.splits[i] = s;
            if (s > 1) shared = std::max<int64_t>(shared, (int64_t)cfg.n_replicas * s * up64(M * l.cout));
        }
    }
    L.rep_block = up64(off);
    L.shared_floats = up64(shared);
    L.fast.assign(plan.layers.size(), 0); L.general.assign(plan.layers.size(), 0); L.general_w.assign(plan.layers.size(), 0);
    L.patch.assign(plan.layers.size(), 0);
    L.wf_off.assign(plan.layers.size(), -1); L.wb_off.assign(plan.layers.size(), -1);
    {
        int64_t woff = 0;
        for (size_t i = 0; i < plan.layers.size(); ++i) {
            const Layer& l = plan.layers[i];
            L.general_w[i] = general_wgrad(cfg, plan, l);
            L.fast[i] = lean_layer(cfg, plan, l);
            L.patch[i] = patch_layer(cfg, plan, l);
            if (L.fast[i] && !L.patch[i]) {
                L.wf_off[i] = woff; woff += up64(l.w_count);
                L.wb_off[i] = woff; woff += up64(l.w_count);
            } else if (L.patch[i] || general_forward(cfg, plan, l)) {
                const TensorShape a = plan.tensors[l.in0];
                const int cin = (int)(l.type == HADFL_OP_CONV ? a.c : a.numel()), taps = l.type == HADFL_OP_CONV ? l.k * l.k : 1;
                L.general[i] = 1;
                if (dense_rows_layer(cfg, plan, l)) continue;
                if (gather_layer(cfg, l)) {                            // all taps and channels in one contraction, no data gradient
                    L.wf_off[i] = woff; woff += up64(weight_copy_units(0, l.cout, 1, taps * cin));
                    continue;
                }
                const auto units = L.patch[i] ? weight_fragment_units : weight_copy_units;
                L.wf_off[i] = woff; woff += up64(units(cfg.bf16, l.cout, taps, cin));
                L.wb_off[i] = woff; woff += up64(units(cfg.bf16, cin, taps, l.cout));
            }
        }
        L.wbf_rep = woff;
    }
    // a lean or general convolution in front of a batch norm leaves statistics entries of its output, and a lean one or one from
    // patches behind a batch norm leaves entries of that batch norm's gradient, the size of its own input
    for (size_t k = 0; k < plan.layers.size(); ++k) {
        const Layer& l = plan.layers[k];
        const TensorShape a = plan.tensors[l.in0];
        const bool behind = l.type == HADFL_OP_BN && l.in0 > 0 && (L.fast[l.in0 - 1] || L.general[l.in0 - 1]);
        if (!behind && !L.fast[k] && !L.patch[k]) continue;
        const bool lean = !L.general[behind ? l.in0 - 1 : (int)k];
        bn_shared = std::max<int64_t>(bn_shared, cfg.n_replicas * stat_floats(B * a.h * a.w, a.c, lean));
    }
    L.bn_floats = up64(bn_shared);
    // position tables: worth it for small images (many border pixels), and the weight gradient needs slabs of 32
    // contraction indices to hold a single position
    L.tab_idx.assign(plan.layers.size(), -1);
    for (size_t i = 0; i < plan.layers.size(); ++i) {
        if ((!L.fast[i] && !L.general[i]) || cfg.batch % 32 != 0) continue;
        const Layer& l = plan.layers[i];
        const TensorShape a = plan.tensors[l.in0];
        if (l.type != HADFL_OP_CONV || l.in0 == 0 || l.k == 1 || l.stride != 1 || 2 * l.pad != l.k - 1 || a.h * a.w > kMaxTablePositions) continue;
        L.tab_idx[i] = L.tab_ints; L.tab_ints += 2 * (int64_t)a.h * a.w;
    }
    return L;
}

}  // namespace

int64_t train_work_floats(const hadfl_config& cfg, const NetPlan& plan)
{
    if (cfg.net == HADFL_NET_NONE) return 0;
    const Layout L = make_layout(cfg, plan);
    return L.rep_block * cfg.n_replicas + L.shared_floats + L.bn_floats + up64(L.wbf_rep * cfg.n_replicas / 2 + 64) + up64(L.tab_ints);
}

hadfl_status train_create(const hadfl_config& cfg, const NetPlan& plan, const TrainBuffers& buf,
                          const std::vector<int32_t>& steps, const std::vector<int32_t>& order,
                          TrainEngine** out, std::string& err)
{
    (void)order;
    TrainEngine* e = new TrainEngine();
    e->cfg = cfg; e->plan = plan; e->buf = buf; e->steps = steps;
    e->e_max = *std::max_element(steps.begin(), steps.end());
    e->n_active.assign(e->e_max, 0);
    for (int s = 0; s < e->e_max; ++s)
        for (int32_t v : steps) e->n_active[s] += v > s ? 1 : 0;
    const Layout L = make_layout(cfg, plan);
    e->act_off = L.act_off; e->grad_off = L.grad_off; e->saved_off = L.saved_off;
    e->splits = L.splits; e->wgrad_plans = L.wgrad_plans; e->bn_chunks = L.bn_chunks;
    e->rep_block = L.rep_block;
    e->shared_off = L.rep_block * cfg.n_replicas;
    e->shared_floats = L.shared_floats;
    e->fast = L.fast; e->general = L.general; e->general_w = L.general_w; e->patch = L.patch; e->wf_off = L.wf_off; e->wb_off = L.wb_off; e->wbf_rep = L.wbf_rep;
    e->bn_off = e->shared_off + L.shared_floats;
    e->bn_floats = L.bn_floats;
    e->wbf_off = e->bn_off + L.bn_floats;
    {
        e->fused_update.assign(plan.layers.size(), 0);
        int64_t pos = 0;
        // (the padding between and behind the layers has neither gradient nor value: a piece of nothing else needs no update)
        auto segment = [&](int64_t first, int64_t end) {
            for (const Layer& l : plan.layers)
                if (l.w_count > 0 && l.w_off < end && l.w_off + l.w_count > first) { e->update_segments.push_back({first, end - first}); return; }
        };
        for (size_t i = 0; i < plan.layers.size(); ++i) {
            const Layer& l = plan.layers[i];
            if (l.type != HADFL_OP_CONV && l.type != HADFL_OP_DENSE) continue;
            // in the weight-gradient epilogue (lean and general kernels, K not split), or in the split-K reduction of a layer
            // whose fp32 weights nothing reads between its weight gradient and the update: the data gradients of the lean
            // and general layers read the copies, a layer on the data set has no data gradient
            const bool own_kernel = e->fast[i] || e->general_w[i];
            const bool in_reduce = e->splits[i] > 1 && l.in0 == 0;
            const bool small = dense_one_pass_bwd(cfg, plan, l);      // its backward kernel applies the update, element by element
            if (!own_kernel && !in_reduce && !small) continue;
            int64_t cnt = l.w_count + (l.bias ? l.cout : 0);      // bias sits directly behind the weights
            if (small) cnt = (cnt + 3) / 4 * 4;                   // (padding behind the slice: nothing there is ever updated)
            if (l.w_off % 4 != 0 || cnt % 4 != 0 || l.w_off < pos || (l.bias && l.b_off != l.w_off + l.w_count)) continue;
            e->fused_update[i] = 1;
            segment(pos, l.w_off);
            pos = l.w_off + cnt;
        }
        segment(pos, plan.train_end);
    }
    e->tab_off = e->wbf_off + up64(L.wbf_rep * cfg.n_replicas / 2 + 64);
    e->tab_idx = L.tab_idx;
    e->tables.assign((size_t)L.tab_ints, 0);
    for (size_t i = 0; i < plan.layers.size(); ++i) {
        if (L.tab_idx[i] < 0) continue;
        const Layer& l = plan.layers[i];
        const TensorShape a = plan.tensors[l.in0];
        const int hw = a.h * a.w;
        std::vector<uint32_t> mask(hw, 0);
        for (int pos = 0; pos < hw; ++pos)
            for (int t = 0; t < l.k * l.k; ++t) {
                const int yy = pos / a.w + t / l.k - l.pad, xx = pos % a.w + t % l.k - l.pad;
                if (yy >= 0 && yy < a.h && xx >= 0 && xx < a.w) mask[pos] |= 1u << t;
            }
        std::vector<int32_t> perm(hw);
        for (int pos = 0; pos < hw; ++pos) perm[pos] = pos;
        std::stable_sort(perm.begin(), perm.end(), [&](int x, int y) { return mask[x] < mask[y]; });
        for (int ps = 0; ps < hw; ++ps) {
            e->tables[L.tab_idx[i] + ps] = perm[ps];
            e->tables[L.tab_idx[i] + hw + ps] = (int32_t)mask[perm[ps]];
        }
    }
    {
        const int nl = (int)plan.layers.size(), T = (int)plan.tensors.size();
        e->out_tensor.resize(nl); e->skip.assign(nl, 0); e->fused_relu.assign(nl, 0); e->masked.assign(T, 0);
        std::vector<int> consumers(T, 0);
        for (const Layer& l : plan.layers) { consumers[l.in0]++; if (l.type == HADFL_OP_ADD) consumers[l.in1]++; }
        for (int i = 0; i < nl; ++i) e->out_tensor[i] = plan.layers[i].out;
        for (int t = 1; t < T - 1; ++t) if (!consumers[t]) e->unread.push_back(t);
        for (int j = 0; j < nl; ++j) {
            const Layer& r = plan.layers[j];
            if (r.type != HADFL_OP_RELU || r.in0 < 1 || consumers[r.in0] != 1 || r.out == T - 1) continue;
            const int i = r.in0 - 1;                       // layer i writes tensor i + 1
            const int pt = plan.layers[i].type;
            if (pt != HADFL_OP_CONV && pt != HADFL_OP_DENSE && pt != HADFL_OP_BN && pt != HADFL_OP_ADD) continue;
            e->out_tensor[i] = r.out; e->fused_relu[i] = 1; e->skip[j] = 1; e->masked[r.out] = 1;
        }
        e->stat_for.assign(nl, -1); e->stat_from.assign(nl, -1); e->stat_rows.assign(nl, 0);
        for (int k = 0; k < nl; ++k) {
            const Layer& b = plan.layers[k];
            if (b.type != HADFL_OP_BN || b.in0 < 1 || consumers[b.in0] != 1) continue;
            const int i = b.in0 - 1;                        // layer i writes tensor i + 1
            if ((!e->fast[i] && !e->general[i]) || plan.layers[i].type != HADFL_OP_CONV || e->out_tensor[i] != b.in0) continue;
            e->stat_for[i] = k; e->stat_from[k] = i;
        }
        e->pool_of.assign(nl, -1);
        const int vec = cfg.bf16 ? 8 : 4;
        for (int j = 0; j < nl; ++j) {
            const Layer& q = plan.layers[j];
            if (q.type != HADFL_OP_MAXPOOL || q.in0 < 1 || consumers[q.in0] != 1) continue;
            int i = -1;                                    // the BN layer that writes the pool's input
            for (int k = 0; k < nl; ++k)
                if (!e->skip[k] && e->out_tensor[k] == q.in0 && plan.layers[k].type == HADFL_OP_BN) i = k;
            if (i < 0) continue;
            const TensorShape t = plan.tensors[q.in0];
            if (t.c % vec != 0 || t.h % 2 != 0 || t.w % 2 != 0) continue;
            e->pool_of[i] = j; e->skip[j] = 1;
        }
        e->add_into.assign(nl, -1); e->add_done.assign(nl, 0);
        for (int j = nl; j-- > 0;) {
            const Layer& q = plan.layers[j];
            if (q.type != HADFL_OP_ADD || q.in0 == q.in1) continue;
            for (int side = 0; side < 2; ++side) {
                const int t = side ? q.in1 : q.in0, other = side ? q.in0 : q.in1;
                if (t < 1 || consumers[t] != 1) continue;
                if (!e->masked[t]) e->grad_off[t] = e->grad_off[e->out_tensor[j]];
                const int i = t - 1;
                if (plan.layers[i].type == HADFL_OP_BN && !e->fused_relu[i] && e->pool_of[i] < 0 && other < t && plan.tensors[t].c % vec == 0) {
                    e->add_into[i] = j; e->add_done[j] = 1;
                }
            }
        }
        e->late_add.assign(nl, 0);
        for (int j = 0; j < nl; ++j) {
            const Layer& q = plan.layers[j];
            if (q.type != HADFL_OP_ADD || q.in0 == q.in1) continue;
            for (int side = 0; side < 2; ++side) {
                const int t = side ? q.in1 : q.in0;
                if (t < 1 || e->grad_off[t] == e->grad_off[e->out_tensor[j]]) continue;
                int i = j - 1;                             // the reader whose gradient of t follows
                while (i >= 0 && plan.layers[i].in0 != t && !(plan.layers[i].type == HADFL_OP_ADD && plan.layers[i].in1 == t)) --i;
                if (i >= 0 && plan.layers[i].type == HADFL_OP_CONV && e->patch[i]) e->late_add[j] |= 1 << side;
            }
        }
        e->bstat_for.assign(nl, -1); e->bstat_rows.assign(nl, 0); e->bstat_rep.assign(nl, 0);
        if (cfg.bf16)
            for (int k = 0; k < nl; ++k) {
                if (plan.layers[k].type != HADFL_OP_BN || e->skip[k]) continue;
                // the tensor the rest of the net sees as this BN's output
                const int t_out = e->pool_of[k] >= 0 ? plan.layers[e->pool_of[k]].out : e->out_tensor[k];
                if (consumers[t_out] != 1) continue;
                for (int j = 0; j < nl; ++j)
                    if (plan.layers[j].type == HADFL_OP_CONV && plan.layers[j].in0 == t_out && (e->fast[j] || e->patch[j])) e->bstat_for[j] = k;
            }
        e->bstat_input.assign(nl, 0);
        for (int k = nl; k-- > 0;) {                       // (of several batch norms with one gradient the first of the backward pass)
            const Layer& b = plan.layers[k];
            if (b.type != HADFL_OP_BN || e->pool_of[k] >= 0) continue;
            int t = e->out_tensor[k];                      // the tensor whose gradient this batch norm takes: its own, or the sum's behind it
            for (int j = k + 1; j < nl; ++j) {
                const Layer& q = plan.layers[j];
                if (q.type == HADFL_OP_ADD && q.in0 != q.in1 && (q.in0 == b.out || q.in1 == b.out) && e->grad_off[b.out] == e->grad_off[e->out_tensor[j]]) t = e->out_tensor[j];
            }
            int i = 0;                                     // its first reader, the last to add to the gradient
            while (i < nl && plan.layers[i].in0 != t && !(plan.layers[i].type == HADFL_OP_ADD && plan.layers[i].in1 == t)) ++i;
            if (i == nl || plan.layers[i].type != HADFL_OP_CONV || !e->patch[i] || e->bstat_for[i] >= 0) continue;
            e->bstat_for[i] = k; e->bstat_input[i] = 1;
        }
    }
    e->beside.assign(plan.layers.size(), 0.0);
    for (size_t i = 0; i < plan.layers.size(); ++i) {
        const Layer& l = plan.layers[i];
        const TensorShape a = plan.tensors[l.in0], o = plan.tensors[l.out];
        double flops = 0.0;
        if (l.in0 != 0 && l.type == HADFL_OP_CONV) flops = 2.0 * cfg.batch * o.h * o.w * l.k * l.k * a.c * (double)l.cout;
        if (l.in0 != 0 && l.type == HADFL_OP_DENSE) flops = 2.0 * cfg.batch * (double)a.numel() * l.cout;
        e->beside[i] = (i ? e->beside[i - 1] : 0.0) + flops;
    }
    *out = e;
    return HADFL_OK;
}

void train_set_steps(TrainEngine* e, const std::vector<int32_t>& steps)
{
    e->steps = steps;
    e->e_max = steps.empty() ? 0 : *std::max_element(steps.begin(), steps.end());
    e->n_active.assign(e->e_max, 0);
    for (int s = 0; s < e->e_max; ++s)
        for (int32_t v : steps) e->n_active[s] += v > s ? 1 : 0;
}

void train_set_lr(TrainEngine* e, float lr) { e->cfg.lr = lr; }

void train_set_side_stream(TrainEngine* e, bool on) { e->use_side = on; }
void train_set_tile_hint(TrainEngine* e, int hint) { e->tile_hint = hint; }
bool train_has_momentum(const TrainEngine* e) { return e->buf.mom != nullptr; }

void train_destroy(TrainEngine* e)
{
    if (!e) return;
    if (e->side) { (void)hipStreamSynchronize(e->side); (void)hipStreamDestroy(e->side); }
    if (e->ev_fork) (void)hipEventDestroy(e->ev_fork);
    if (e->ev_join) (void)hipEventDestroy(e->ev_join);
    delete e;
}

namespace {

constexpr double kMinBesideFlops = 4e8;

struct Runner {
    TrainEngine& e;
    hipStream_t s;
    Profiler* prof;
    int na = 0;
    int step = 0;                         // steps of this call before the present one
    int cur_layer = -1;
    hipError_t rc = hipSuccess;
    const char* failed = nullptr;

    const float* act(int t) const { return t == 0 ? e.buf.x : e.buf.work + e.act_off[t]; }
    float* actw(int t) const { return e.buf.work + e.act_off[t]; }
    float* grad(int t) const { return e.buf.work + e.grad_off[t]; }
    hipStream_t main_stream = nullptr;
    bool forked = false;                  // a flag, not the handle: the caller's stream may be the null stream
    bool side_busy = false;               // the side stream has work of this sub-step
    // The launches that follow, a layer's weight gradient, go to the side stream, ordered after everything enqueued on the main
    // stream so far.  `beside`: flops of the data gradients that are still to come on the main stream, which is what the side stream's
    // work can lie beside; where they take less time than the events (some 20 us a sub-step) the weight gradients stay on the
    // main stream as long as nothing of this sub-step is on the side stream.  Behind the first that is there everything
    // follows in order, for the scratch of the split sums and the updated weights are the side stream's until the join.
    // Earlier the line was at 2e8 flops of the one weight gradient.  That / this, us a cycle: residual net of 64 to 128 channels on 5 replicas
    // 1327 / 1270, of 40 to 80 on 2 772 / 720; convolution net of 32 and 64 channels, batch 16, on 2 (302 Mflop beside) 329 / 296 and on 8
    // 379 / 372; perceptron of 784 x 128, batch 256, whose wide layer has nothing beside it, on 4 157 / 129 and on 16 199 / 153.
    // Lines at 2e8 / 4e8: a residual net of 24 to 48 channels on 8 (304) 653 / 636 (earlier 629), that convolution net on 2 326 / 296.
    void fork(double beside)
    {
        if (!e.use_side || !e.side || rc != hipSuccess) return;
        if (!side_busy && beside < kMinBesideFlops) return;
        side_busy = true;
        rc = hipEventRecord(e.ev_fork, s);
        if (rc == hipSuccess) rc = hipStreamWaitEvent(e.side, e.ev_fork, 0);
        if (rc != hipSuccess) { failed = "fork"; return; }
        main_stream = s; s = e.side; forked = true;
    }
    void unfork() { if (forked) { s = main_stream; forked = false; } }
    // the main stream waits for everything enqueued on the side stream
    void join()
    {
        if (!side_busy || rc != hipSuccess) return;
        side_busy = false;
        rc = hipEventRecord(e.ev_join, e.side);
        if (rc == hipSuccess) rc = hipStreamWaitEvent(s, e.ev_join, 0);
        if (rc != hipSuccess) failed = "join";
    }
    float* shared() const { return e.buf.work + e.shared_off; }
    // The region of the batch-norm partial sums, for one launch's entries of `rep` floats per replica, and what it holds for a
    // later launch: the forward sums of batch norm `owner`, or (kBackward + owner) those of its backward pass.  Other layers
    // may run between the convolution that leaves them and the batch norm, and take the region for sums of their own; the
    // batch norm then forms its sums itself.
    static constexpr int kBackward = 1 << 30;
    int sums_of = -1;
    float* bn_shared(int64_t rep, int owner)
    {
        sums_of = owner;
        if (na * rep > e.bn_floats && rc == hipSuccess) { rc = hipErrorInvalidValue; failed = "batch-norm sums beyond their region"; }
        return e.buf.work + e.bn_off;
    }
    __bf16* wbf() const { return reinterpret_cast<__bf16*>(e.buf.work + e.wbf_off); }
    const int* perm(size_t i) const { return e.tab_idx[i] < 0 ? nullptr : reinterpret_cast<const int*>(e.buf.work + e.tab_off) + e.tab_idx[i]; }
    const unsigned* posmask(size_t i) const
    {
        const TensorShape a = e.plan.tensors[e.plan.layers[i].in0];
        return e.tab_idx[i] < 0 ? nullptr : reinterpret_cast<const unsigned*>(e.buf.work + e.tab_off) + e.tab_idx[i] + a.h * a.w;
    }

    // K-contiguous copies of layer i's filters for the lean kernels (forward layout and flipped/transposed for the data
    // gradient; bf16, or split floats in the fp32 configuration), refreshed from the fp32 master for the first n replicas in step
    // order.  The general layers' are gathered, and written by one launch in write_copies.
    WeightCopies copies{};
    double copies_bytes = 0;
    int copies_layer = -1;                // the first of them
    void write_copies(int n)
    {
        if (copies.count == 0) return;
        const int keep_na = na, keep_layer = cur_layer;
        na = n; cur_layer = copies_layer;
        run("weight_prep", 0, copies_bytes, [&] { return launch_weight_copies(copies, na, s); });
        copies.count = 0; copies_bytes = 0;
        na = keep_na; cur_layer = keep_layer;
    }
    void prep_layer(size_t i, int n)
    {
        const int keep_na = na, keep_layer = cur_layer;
        na = n; cur_layer = (int)i;
        const Layer& l = e.plan.layers[i];
        if (e.general[i]) {
            if (copies.count == kWeightCopies) write_copies(n);
            if (copies.count == 0) copies_layer = (int)i;
            WeightCopyParams& w = copies.layer[copies.count++];
            w.w = e.buf.replicas + l.w_off; w.w_rep = e.plan.row_stride;
            w.wf = wbf() + e.wf_off[i]; w.wb = e.wb_off[i] >= 0 ? wbf() + e.wb_off[i] : nullptr; w.wcopy_rep = e.wbf_rep;
            w.C = layer_channels(l); w.N = l.cout; w.taps = l.type == HADFL_OP_CONV ? l.k * l.k : 1; w.bf16 = e.cfg.bf16; w.order = e.buf.order;
            if (gather_layer(e.cfg, l)) { w.C *= w.taps; w.taps = 1; }
            w.fragments = e.patch[i];
            copies_bytes += (e.cfg.bf16 ? 8.0 : 16.0) * l.w_count;
        } else {
            WeightPrepParams w{};
            w.w = e.buf.replicas + l.w_off; w.w_rep = e.plan.row_stride;
            w.wf = wbf() + e.wf_off[i]; w.wb = wbf() + e.wb_off[i]; w.wbf_rep = e.wbf_rep;
            w.C = e.plan.tensors[l.in0].c; w.N = l.cout; w.taps = l.k * l.k; w.order = e.buf.order;
            run("weight_prep", 0, 8.0 * l.w_count, [&] { return launch_weight_prep(w, na, s); });
        }
        na = keep_na; cur_layer = keep_layer;
    }
    int layer_channels(const Layer& l) const
    {
        const TensorShape a = e.plan.tensors[l.in0];
        return (int)(l.type == HADFL_OP_CONV ? a.c : a.numel());
    }
    // what forward and data gradient of a general layer have in common
    GeneralConvParams general_base(size_t i, const GemmParams& g) const
    {
        GeneralConvParams f{};
        f.bf16 = e.cfg.bf16; f.B = g.B; f.R = g.R; f.S = g.S; f.wmat_rep = e.wbf_rep; f.out_rep = e.rep_block; f.a_rep = e.rep_block;
        f.sstride = f.ostride = f.wst = f.classes = 1;
        f.order = e.buf.order; f.perm = perm(i); f.posmask = posmask(i); f.tile_hint = e.tile_hint;
        return f;
    }
    void prepare_weights()
    {
        for (size_t i = 0; i < e.plan.layers.size(); ++i) {
            if (e.wf_off[i] < 0) continue;
            if (e.prepped[i]) { e.prepped[i] = 0; continue; }      // written during the previous sub-step's backward pass
            prep_layer(i, na);
        }
        write_copies(na);
    }
    // A layer whose update is fused into its weight-gradient kernel has its final weights of this sub-step as soon as
    // that kernel ends, so the copies for the next sub-step are written right behind it on the same stream, off the
    // forward pass's critical path.  Not before this sub-step's data gradient of the layer has read the old copy:
    // the copy of layer i is therefore issued after the next fork, which follows that data gradient on the main stream.
    int na_next = 0;
    int pending_prep = -1;
    void flush_pending_prep()
    {
        if (pending_prep < 0) return;
        prep_layer((size_t)pending_prep, na_next);
        write_copies(na_next);
        e.prepped[pending_prep] = 1;
        pending_prep = -1;
    }

    // flops / bytes: algorithmic work of the launch for all active replicas (reported by the profiler)
    template <typename F> void run(const char* name, double flops, double bytes, F&& f)
    {
        if (rc != hipSuccess) return;
        if (prof) {
            if (prof->detail) {
                char tag[64];
                std::snprintf(tag, sizeof(tag), "%s:L%d:n%d", name, cur_layer, na);
                prof->begin(tag, s, flops * na, bytes * na);
            } else {
                prof->begin(name, s, flops * na, bytes * na);
            }
        }
        rc = f();
        if (prof) prof->end(s);
        if (rc != hipSuccess) failed = name;
    }

    // fp32 problems of the generic kernels that conv_chain.hip takes
    static bool chain(const GemmParams& p)
    {
        if (p.mode == kWgrad || p.stride != 1 || p.R != p.S || 2 * p.pad != p.R - 1 || p.Ho != p.H || p.Wo != p.W || p.H * p.W == 1) return false;
        if (p.cursor) return p.mode == kFwd && conv_chain_first_supported(p.B, p.H, p.W, p.Cin, p.Cout, p.R);
        return p.mode == kFwd ? conv_chain_supported(p.B, p.H, p.W, p.Cin, p.Cout, p.R) : conv_chain_supported(p.B, p.H, p.W, p.Cout, p.Cin, p.R);
    }
    hipError_t gemm(const GemmParams& p) const { if (!e.cfg.bf16 && chain(p)) return launch_conv_chain(p, na, s); return e.cfg.bf16 ? launch_gemm_bf16(p, na, s) : launch_gemm(p, na, s); }
    static double gemm_flops(const GemmParams& p) { return 2.0 * p.B * p.Ho * p.Wo * p.R * p.S * (double)p.Cin * p.Cout; }
    // activations are 2 bytes in the bf16 configuration, weights and their gradients 4
    double asz() const { return e.cfg.bf16 ? 0.5 : 1.0; }
    double gemm_bytes(const GemmParams& p) const
    {
        return 4.0 * (asz() * ((double)p.B * p.H * p.W * p.Cin + (double)p.B * p.Ho * p.Wo * p.Cout) + (double)p.R * p.S * p.Cin * p.Cout);
    }

    GemmParams gemm_base(const Layer& l) const
    {
        const TensorShape a = e.plan.tensors[l.in0], r = e.plan.tensors[l.out];
        GemmParams p{};
        p.B = e.cfg.batch;
        if (l.type == HADFL_OP_CONV) {
            p.H = a.h; p.W = a.w; p.Cin = a.c; p.Ho = r.h; p.Wo = r.w; p.Cout = l.cout;
            p.R = p.S = l.k; p.stride = l.stride; p.pad = l.pad;
        } else {
            p.H = p.W = p.Ho = p.Wo = 1; p.Cin = (int)a.numel(); p.Cout = l.cout;
            p.R = p.S = 1; p.stride = 1; p.pad = 0;
        }
        p.splits = 1; p.kchunk = 1 << 30;
        p.hw_shift = ilog2_exact(p.Ho * p.Wo); p.w_shift = ilog2_exact(p.Wo);
        if (p.hw_shift < 0 || p.w_shift < 0) p.hw_shift = p.w_shift = -1;
        p.w = e.buf.replicas + l.w_off; p.w_rep = e.plan.row_stride;
        p.has_bias = l.bias;
        p.order = e.buf.order;
        p.n_samples = e.cfg.n_samples; p.batch = e.cfg.batch; p.sample_sz = e.plan.tensors[0].numel();
        return p;
    }

    // All steps of a network of two dense layers, the end of each with the beginning of the next
    void dense_pair_steps()
    {
        const Layer &a = e.plan.layers[0], &b = e.plan.layers[2];
        float* const shares[2] = {grad(a.out), grad(e.plan.layers[1].out)};      // taken in turn: the room of gradients that these launches never write
        DensePairParams d{};
        d.x = e.buf.x; d.y = e.buf.y; d.cursor = e.buf.cursor; d.n_samples = e.cfg.n_samples; d.batch = e.cfg.batch;
        d.K = (int)e.plan.tensors[0].numel(); d.H = a.cout; d.N = b.cout; d.has_bias1 = a.bias; d.has_bias2 = b.bias;
        d.w1 = e.buf.replicas + a.w_off; d.w2 = e.buf.replicas + b.w_off; d.w_rep = e.plan.row_stride;
        d.m1 = e.buf.mom ? e.buf.mom + a.w_off : nullptr; d.m2 = e.buf.mom ? e.buf.mom + b.w_off : nullptr;
        d.lr = e.cfg.lr; d.momentum = e.cfg.momentum;
        d.hidden = actw(e.out_tensor[0]); d.act_rep = e.rep_block;
        d.loss = e.buf.loss; d.bf16 = e.cfg.bf16; d.order = e.buf.order;
        const double macs = (double)d.batch * ((double)d.K * d.H + (double)d.H * d.N), wbytes = 4.0 * (d.K + d.N) * d.H;
        cur_layer = 0;
        for (int s0 = 0; s0 <= e.e_max && e.e_max > 0; ++s0) {
            d.ahead = s0;
            d.share_in = shares[(s0 + 1) & 1]; d.share_out = shares[s0 & 1];
            d.n_end = s0 > 0 ? e.n_active[s0 - 1] : 0; d.n_begin = s0 < e.e_max ? e.n_active[s0] : 0;
            na = std::max(d.n_end, d.n_begin);
            const double ends = (double)d.n_end / na, begins = (double)d.n_begin / na;      // (work is given per replica)
            run("dense_step", 2.0 * (macs * begins + (macs + (double)d.batch * d.H * d.N) * ends),
                (4.0 * d.batch * d.K + wbytes) * begins + (4.0 * d.batch * d.K + (d.m1 ? 4.0 : 2.0) * wbytes) * ends, [&] { return launch_dense_pair(d, s); });
        }
    }

    void forward_layer(size_t i)
    {
        cur_layer = (int)i;
        if (e.skip[i]) return;
        const Layer& l = e.plan.layers[i];
        const TensorShape a = e.plan.tensors[l.in0], r = e.plan.tensors[l.out];
        const int64_t B = e.cfg.batch;
        const int ot = e.out_tensor[i];
        EwParams q{};
        q.order = e.buf.order; q.B = (int)B; q.H = a.h; q.W = a.w; q.C = a.c; q.bf16 = e.cfg.bf16;
        q.in = act(l.in0); q.in_rep = e.rep_block;
        q.out = actw(ot); q.out_rep = e.rep_block;
        q.relu = e.fused_relu[i];
        q.count = B * r.numel();
        switch (l.type) {
        case HADFL_OP_CONV:
        case HADFL_OP_DENSE: {
            GemmParams p = gemm_base(l);
            p.mode = kFwd;
            p.M = (int)(B * p.Ho * p.Wo); p.N = p.Cout; p.K = p.R * p.S * p.Cin;
            p.a = act(l.in0); p.a_rep = e.rep_block;
            p.cursor = l.in0 == 0 ? e.buf.cursor : nullptr; p.ahead = step;
            p.a_f32 = l.in0 == 0;
            p.out = actw(ot); p.out_rep = e.rep_block;
            p.relu = e.fused_relu[i];
            {
                FirstConvParams fc;
                if (first_conv(i, fc)) {
                    fc.out = actw(ot); fc.out_rep = e.rep_block; fc.relu = p.relu;
                    run("conv_fwd", gemm_flops(p), gemm_bytes(p), [&] { return launch_conv_first_fwd(fc, na, s); });
                    break;
                }
            }
            const bool rows_layer = dense_rows_layer(e.cfg, e.plan, l);
            if (rows_layer && dense_rows_pays(e.cfg, e.plan, l, na)) {
                DenseRowsParams d{};
                d.x = act(l.in0); d.x_rep = e.rep_block; d.cursor = p.cursor; d.ahead = p.ahead; d.n_samples = p.n_samples; d.batch = p.batch;
                d.w = p.w; d.w_rep = p.w_rep; d.out = actw(ot); d.out_rep = e.rep_block;
                d.rows = (int)B; d.K = p.Cin; d.N = l.cout; d.has_bias = l.bias; d.relu = p.relu; d.bf16 = e.cfg.bf16; d.order = e.buf.order;
                run("dense_fwd", gemm_flops(p), gemm_bytes(p), [&] { return launch_dense_rows_fwd(d, na, s); });
                break;
            }
            if (e.fast[i] && !e.general[i]) {
                FastConvParams f{};
                f.B = p.B; f.H = p.H; f.W = p.W; f.C = p.Cin; f.N = p.Cout; f.R = p.R; f.S = p.S; f.pad = p.pad;
                f.M = p.M; f.K = p.K;
                f.a = act(l.in0); f.a_rep = e.rep_block;
                f.wmat = wbf() + e.wf_off[i]; f.wmat_rep = e.wbf_rep;
                f.out = actw(ot); f.out_rep = e.rep_block;
                f.bias = l.bias ? e.buf.replicas + l.b_off : nullptr; f.bias_rep = e.plan.row_stride;
                f.relu = p.relu; f.order = e.buf.order; f.tile_hint = e.tile_hint;
                f.perm = perm(i); f.posmask = posmask(i);
                int* srows = nullptr;
                if (e.stat_for[i] >= 0) {
                    f.stat_rep = stat_floats(p.M, p.Cout, true); f.stat = bn_shared(f.stat_rep, e.stat_for[i]);
                    srows = &e.stat_rows[e.stat_for[i]];
                }
                run("conv_fwd", gemm_flops(p), gemm_bytes(p), [&] { return launch_conv_fast(f, 0, na, s, srows); });
                break;
            }
            if (e.general[i] && !rows_layer) {
                GeneralConvParams f = general_base(i, p);
                f.H = p.H; f.W = p.W; f.C = p.Cin; f.Ho = p.Ho; f.Wo = p.Wo; f.N = p.Cout; f.pad = p.pad; f.sstride = p.stride;
                f.a = act(l.in0); f.cursor = p.cursor; f.ahead = p.ahead; f.n_samples = p.n_samples; f.batch = p.batch; f.sample_sz = p.sample_sz;
                f.wmat = wbf() + e.wf_off[i];
                f.out = actw(ot);
                f.bias = l.bias && !bias_left_out(i) ? e.buf.replicas + l.b_off : nullptr; f.bias_rep = e.plan.row_stride;
                f.relu = p.relu;
                int* srows = nullptr;
                if (e.stat_for[i] >= 0) {
                    f.stat_rep = stat_floats(p.M, p.Cout, false); f.stat = bn_shared(f.stat_rep, e.stat_for[i]);
                    srows = &e.stat_rows[e.stat_for[i]];
                }
                run(l.type == HADFL_OP_CONV ? "conv_fwd" : "dense_fwd", gemm_flops(p), gemm_bytes(p), [&] { return e.patch[i] ? launch_conv_general_patch(f, 0, na, s, srows) : launch_conv_general(f, 0, na, s, srows); });
                break;
            }
            if (small_dense_layer(l) && !p.relu) {
                DenseSmallParams d = dense_small(l, p);
                d.out = actw(ot); d.out_rep = e.rep_block;
                run("dense_small_fwd", gemm_flops(p), gemm_bytes(p), [&] { return launch_dense_small_fwd(d, na, s); });
                break;
            }
            run(l.type == HADFL_OP_CONV ? "conv_fwd" : "dense_fwd", gemm_flops(p), gemm_bytes(p), [&] { return gemm(p); });
            break; }
        case HADFL_OP_RELU: run("relu_fwd", 0, asz() * (8.0 * q.count), [&] { return launch_relu_fwd(q, na, s); }); break;
        case HADFL_OP_MAXPOOL: run("maxpool_fwd", 0, asz() * (4.0 * (B * a.numel() + q.count)), [&] { return launch_maxpool_fwd(q, na, s); }); break;
        case HADFL_OP_ADD:
            if (e.add_done[i]) break;
            q.in2 = act(l.in1); q.in2_rep = e.rep_block;
            run("add_fwd", 0, asz() * (12.0 * q.count), [&] { return launch_add_fwd(q, na, s); });
            break;
        case HADFL_OP_GAP: run("gap_fwd", 0, asz() * (4.0 * (B * a.numel() + q.count)), [&] { return launch_gap_fwd(q, na, s); }); break;
        case HADFL_OP_BN: {
            const bool sums_done = e.stat_from[i] >= 0 && e.stat_rows[i] > 0 && sums_of == (int)i;
            BnParams b = bn_params(i);
            b.y = actw(ot); b.relu = e.fused_relu[i];
            if (sums_done) {                                 // the convolution in front left the sums
                b.stats_done = 1; b.stat_entries = (b.rows + e.stat_rows[i] - 1) / e.stat_rows[i];
                b.partial_rep = stat_floats(b.rows, b.C, !e.general[e.stat_from[i]]);
                const Layer& conv = e.plan.layers[e.stat_from[i]];
                b.stat_shift = conv.bias && !bias_left_out(e.stat_from[i]) ? e.buf.replicas + conv.b_off : nullptr; b.stat_shift_rep = e.plan.row_stride;
            }
            if (e.stat_from[i] >= 0 && bias_left_out(e.stat_from[i])) {
                b.left_out = e.buf.replicas + e.plan.layers[e.stat_from[i]].b_off; b.left_out_rep = e.plan.row_stride;
            }
            if (e.pool_of[i] >= 0) {
                b.pool = 1; b.H = a.h; b.W = a.w;
                b.pool_out = actw(e.plan.layers[e.pool_of[i]].out); b.pool_out_rep = e.rep_block;
            }
            const int j = e.add_into[i];
            if (j >= 0) {
                const Layer& sum = e.plan.layers[j];
                b.add = act(sum.in0 == l.out ? sum.in1 : sum.in0); b.add_rep = e.rep_block; b.add_relu = e.fused_relu[j];
                b.y = actw(e.out_tensor[j]);
            }
            run("bn_fwd", 0, asz() * ((j >= 0 ? 12.0 : 8.0) * B * a.numel()), [&] { return launch_bn_fwd(b, na, s); });
            break; }
        }
    }

    // An fp32 convolution whose output only a batch norm reads stores it without its bias (in bf16 the stored values are those of
    // the network as written, rounded).
    bool bias_left_out(size_t i) const { return !e.cfg.bf16 && e.general[i] && e.stat_for[i] >= 0 && e.plan.layers[i].bias; }

    DenseSmallParams dense_small(const Layer& l, const GemmParams& g) const
    {
        DenseSmallParams d{};
        d.x = act(l.in0); d.x_rep = e.rep_block; d.w = e.buf.replicas + l.w_off; d.w_rep = e.plan.row_stride;
        d.rows = g.B; d.K = g.Cin; d.N = l.cout; d.has_bias = l.bias; d.order = e.buf.order; d.bf16 = e.cfg.bf16;
        return d;
    }

    // bf16 configuration: the first convolution (data set in) has its own kernels when its footprint fits one MFMA
    bool first_conv(size_t i, FirstConvParams& f) const
    {
        const Layer& l = e.plan.layers[i];
        if (!e.cfg.bf16 || l.type != HADFL_OP_CONV || l.in0 != 0 || l.stride != 1) return false;
        if (l.bias && l.b_off != l.w_off + l.w_count) return false;
        const TensorShape a = e.plan.tensors[0], r = e.plan.tensors[l.out];
        if (r.h != a.h || r.w != a.w) return false;
        f = FirstConvParams{};
        f.x = e.buf.x; f.cursor = e.buf.cursor; f.ahead = step; f.n_samples = e.cfg.n_samples;
        f.B = e.cfg.batch; f.H = a.h; f.W = a.w; f.C = a.c; f.N = l.cout; f.R = f.S = l.k; f.pad = l.pad;
        f.K = l.k * l.k * a.c; f.M = e.cfg.batch * a.h * a.w;
        f.w = e.buf.replicas + l.w_off; f.w_rep = e.plan.row_stride;
        f.bias = l.bias ? e.buf.replicas + l.b_off : nullptr;
        f.order = e.buf.order;
        return conv_first_supported(f);
    }

    BnParams bn_params(size_t i)
    {
        const Layer& l = e.plan.layers[i];
        const TensorShape a = e.plan.tensors[l.in0];
        BnParams b{};
        b.x = act(l.in0); b.x_rep = e.rep_block;
        b.y = actw(l.out); b.y_rep = e.rep_block;
        b.params = e.buf.replicas; b.grads = e.buf.grad; b.row_stride = e.plan.row_stride;
        b.w_off = l.w_off; b.stat_off = l.stat_off;
        b.saved = e.buf.work + e.saved_off[i]; b.saved_rep = e.rep_block;
        b.rows = (int)((int64_t)e.cfg.batch * a.h * a.w); b.C = a.c;
        b.chunks = e.bn_chunks[i];
        b.chunk_rows = (b.rows + b.chunks - 1) / b.chunks;
        b.partial_rep = (long long)b.chunks * 2 * a.c; b.partial = bn_shared(b.partial_rep, -1);
        b.order = e.buf.order; b.bf16 = e.cfg.bf16;
        return b;
    }

    LossParams criterion() const
    {
        const int T = (int)e.plan.tensors.size();
        LossParams lp{};
        lp.logits = act(T - 1); lp.logits_rep = e.rep_block;
        lp.dlogits = grad(T - 1); lp.dlogits_rep = e.rep_block;
        lp.y = e.buf.y; lp.cursor = e.buf.cursor; lp.ahead = step; lp.n_samples = e.cfg.n_samples; lp.batch = e.cfg.batch;
        lp.n_classes = e.cfg.n_classes; lp.loss = e.buf.loss; lp.order = e.buf.order; lp.bf16 = e.cfg.bf16;
        return lp;
    }
    // The last layer is a classifier whose backward kernel forms the gradient of the loss itself
    bool forms_criterion(size_t i) const
    {
        const Layer& l = e.plan.layers[i];
        return i + 1 == e.plan.layers.size() && e.fused_update[i] && dense_one_pass_bwd(e.cfg, e.plan, l) && e.out_tensor[i] == (int)e.plan.tensors.size() - 1 &&
               l.cout == e.cfg.n_classes;
    }

    // Data gradient d of layer i, which is the whole gradient of a batch norm's output: it leaves that batch norm's sums.  Returns
    // where the rows per entry go.
    template <typename P> int* gradient_sums(P& f, size_t i, const GemmParams& d, bool lean)
    {
        const int k = e.bstat_for[i];
        if constexpr (std::is_same<P, GeneralConvParams>::value)
            if (e.bstat_input[i]) {
                BnParams b{};
                b.rows = d.M; b.C = d.N; b.bf16 = e.cfg.bf16;
                if (bn_backward_in_one_launch(b, na)) return nullptr;
                f.stat_rep = stat_floats(d.M, d.N, lean); f.stat = bn_shared(f.stat_rep, kBackward + k);
                f.stat_y = act(e.plan.layers[k].in0); f.stat_y_rep = e.rep_block;
                f.stat_mean = e.buf.work + e.saved_off[k]; f.stat_mean_rep = e.rep_block;
                e.bstat_rep[k] = f.stat_rep;
                return &e.bstat_rows[k];
            }
        f.stat_rep = stat_floats(d.M, d.N, lean); f.stat = bn_shared(f.stat_rep, kBackward + k);
        f.stat_y = act(e.plan.layers[i].in0); f.stat_y_rep = e.rep_block; f.stat_relu = e.fused_relu[k];
        e.bstat_rep[k] = f.stat_rep;
        return &e.bstat_rows[k];
    }

    // d(out) is complete; produce d(in0) (and d(in1)), and the parameter gradients of the layer
    void backward_layer(size_t i)
    {
        cur_layer = (int)i;
        if (e.skip[i]) return;
        const Layer& l = e.plan.layers[i];
        const TensorShape a = e.plan.tensors[l.in0], r = e.plan.tensors[l.out];
        const int64_t B = e.cfg.batch;
        const bool need_din = l.in0 != 0;
        const int acc0 = need_din ? (e.grad_written[l.in0] ? 1 : 0) : 0;
        const int ot = e.out_tensor[i];          // d(loss)/d(this layer's pre-ReLU output) lives in grad(ot)
        const float* mask0 = (need_din && e.masked[l.in0]) ? act(l.in0) : nullptr;
        EwParams q{};
        q.order = e.buf.order; q.B = (int)B; q.H = a.h; q.W = a.w; q.C = a.c; q.bf16 = e.cfg.bf16;
        q.accumulate = acc0;
        q.mask = mask0; q.mask_rep = e.rep_block;
        if (need_din) { q.out = grad(l.in0); q.out_rep = e.rep_block; }
        switch (l.type) {
        case HADFL_OP_CONV:
        case HADFL_OP_DENSE: {
            // weight (and bias) gradient
            GemmParams p = gemm_base(l);
            if (e.fused_update[i] && dense_one_pass_bwd(e.cfg, e.plan, l)) {
                DenseSmallParams d = dense_small(l, p);
                d.dy = grad(ot); d.dy_rep = e.rep_block; d.dx = grad(l.in0); d.dx_rep = e.rep_block;
                d.mask = mask0; d.mask_rep = e.rep_block; d.accumulate = acc0;
                d.buf = e.buf.mom ? e.buf.mom + l.w_off : nullptr; d.lr = e.cfg.lr; d.momentum = e.cfg.momentum;
                if (forms_criterion(i)) d.criterion = criterion();
                run("dense_small_bwd", 2.0 * gemm_flops(p), 2.0 * gemm_bytes(p), [&] { return launch_dense_small_bwd(d, na, s); });
                break;
            }
            p.mode = kWgrad;
            p.M = p.R * p.S * p.Cin + (l.bias ? 1 : 0); p.N = p.Cout; p.K = (int)(B * p.Ho * p.Wo);
            p.a = act(l.in0); p.a_rep = e.rep_block;
            p.cursor = l.in0 == 0 ? e.buf.cursor : nullptr; p.ahead = step;
            p.a_f32 = l.in0 == 0;
            p.dy = grad(ot); p.dy_rep = e.rep_block;
            const WgradPlan wgrad = e.wgrad_plans[i].empty() ? WgradPlan{e.splits[i], 0} : e.wgrad_plans[i][na - 1];
            p.splits = wgrad.splits;
            const int64_t mn = (int64_t)p.M * p.N;
            if (p.splits > 1) {
                const int unit = e.fast[i] ? 64 : e.general_w[i] ? 32 : 16;      // slab length of the kernel that will run
                const int slabs = (p.K + unit - 1) / unit;
                p.kchunk = ((slabs + p.splits - 1) / p.splits) * unit;
                p.out_split = (mn + 63) / 64 * 64;
                p.out = shared(); p.out_rep = p.out_split * p.splits;
            } else {
                p.out = e.buf.grad + l.w_off; p.out_rep = e.plan.row_stride;
            }
            fork(na * e.beside[i]);
            flush_pending_prep();
            FirstConvParams fc;
            if (first_conv(i, fc)) {
                fc.dy = grad(ot); fc.dy_rep = e.rep_block;
                fc.gout = p.out; fc.gout_rep = p.out_rep; fc.gout_split = p.out_split; fc.splits = p.splits; fc.kchunk = p.kchunk;
                run("conv_wgrad", gemm_flops(p), gemm_bytes(p), [&] { return launch_conv_first_wgrad(fc, na, s); });
            } else
            if (e.fast[i]) {
                FastWgradParams f = lean_wgrad_shape(e.cfg, e.plan, l);
                f.kchunk = p.kchunk; f.splits = p.splits; f.w_shift = p.w_shift;
                f.x = act(l.in0); f.x_rep = e.rep_block; f.dy = grad(ot); f.dy_rep = e.rep_block;
                f.out = p.out; f.out_rep = p.out_rep; f.out_split = p.out_split; f.order = e.buf.order;
                if (p.H * p.W <= kMaxTablePositionsWgrad && p.B % 64 == 0) { f.perm = perm(i); f.posmask = posmask(i); }
                f.tile_hint = e.tile_hint;
                if (e.fused_update[i]) {
                    f.sgd_w = e.buf.replicas + l.w_off; f.sgd_buf = e.buf.mom ? e.buf.mom + l.w_off : nullptr;
                    f.lr = e.cfg.lr; f.momentum = e.cfg.momentum;
                }
                run("conv_wgrad", gemm_flops(p), gemm_bytes(p), [&] { return launch_wgrad_fast(f, na, s); });
                if (e.fused_update[i] && na_next > 0) pending_prep = (int)i;
            } else
            if (e.general_w[i]) {
                GeneralWgradParams f{};
                f.bf16 = e.cfg.bf16;
                f.B = p.B; f.H = p.H; f.W = p.W; f.C = p.Cin; f.Ho = p.Ho; f.Wo = p.Wo; f.N = p.Cout; f.R = p.R; f.S = p.S; f.pad = p.pad;
                f.stride = p.stride; f.K = p.K; f.kchunk = p.kchunk; f.splits = p.splits; f.small_tiles = wgrad.small_tiles; f.has_bias = l.bias;
                f.x = act(l.in0); f.x_rep = e.rep_block; f.dy = grad(ot); f.dy_rep = e.rep_block;
                f.cursor = p.cursor; f.ahead = p.ahead; f.n_samples = p.n_samples; f.batch = p.batch; f.sample_sz = p.sample_sz; f.gather = gather_layer(e.cfg, l);
                f.out = p.out; f.out_rep = p.out_rep; f.out_split = p.out_split; f.order = e.buf.order;
                if (p.H * p.W <= kMaxTablePositionsWgrad) { f.perm = perm(i); f.posmask = posmask(i); }
                if (e.fused_update[i]) {
                    f.sgd_w = e.buf.replicas + l.w_off; f.sgd_buf = e.buf.mom ? e.buf.mom + l.w_off : nullptr;
                    f.lr = e.cfg.lr; f.momentum = e.cfg.momentum;
                }
                run(l.type == HADFL_OP_CONV ? "conv_wgrad" : "dense_wgrad", gemm_flops(p), gemm_bytes(p), [&] { return wgrad.positions ? launch_wgrad_positions(f, na, s) : launch_wgrad_general(f, na, s); });
                if (e.fused_update[i] && na_next > 0 && e.wf_off[i] >= 0) pending_prep = (int)i;
            } else
                run(l.type == HADFL_OP_CONV ? "conv_wgrad" : "dense_wgrad", gemm_flops(p), gemm_bytes(p), [&] { return gemm(p); });
            if (p.splits > 1 && e.fused_update[i])
                run("splitk_reduce", 0, 4.0 * mn * (p.splits + 4), [&] {
                    return launch_splitk_reduce_update(shared(), p.out_split, p.splits, e.buf.replicas + l.w_off,
                                                       e.buf.mom ? e.buf.mom + l.w_off : nullptr, e.plan.row_stride, mn, e.cfg.lr,
                                                       e.cfg.momentum, one_chain_net(e.cfg, e.plan), e.buf.order, na, s); });
            else if (p.splits > 1)
                run("splitk_reduce", 0, 4.0 * mn * (p.splits + 1), [&] { return launch_splitk_reduce(shared(), p.out_split, p.splits, e.buf.grad + l.w_off,
                                                                       e.plan.row_stride, mn, e.buf.order, na, s); });
            unfork();
            if (need_din) {
                GemmParams d = gemm_base(l);
                d.mode = kDgrad;
                d.M = (int)(B * d.H * d.W); d.N = d.Cin; d.K = d.R * d.S * d.Cout;
                d.a = grad(ot); d.a_rep = e.rep_block;
                d.out = grad(l.in0); d.out_rep = e.rep_block;
                d.accumulate = acc0;
                d.mask = mask0; d.mask_rep = e.rep_block;
                if (e.fast[i] && !e.general[i]) {
                    FastConvParams f{};
                    f.B = d.B; f.H = d.H; f.W = d.W; f.C = d.Cout; f.N = d.Cin; f.R = d.R; f.S = d.S; f.pad = d.R - 1 - d.pad;
                    f.M = d.M; f.K = d.K;
                    f.a = grad(ot); f.a_rep = e.rep_block;
                    f.wmat = wbf() + e.wb_off[i]; f.wmat_rep = e.wbf_rep;
                    f.out = grad(l.in0); f.out_rep = e.rep_block;
                    f.mask = mask0; f.mask_rep = e.rep_block; f.accumulate = acc0; f.order = e.buf.order; f.tile_hint = e.tile_hint;
                    f.perm = perm(i); f.posmask = posmask(i);
                    int* brows = nullptr;
                    if (e.bstat_for[i] >= 0 && !acc0) brows = gradient_sums(f, i, d, true);
                    run("conv_dgrad", gemm_flops(d), gemm_bytes(d), [&] { return launch_conv_fast(f, 1, na, s, brows); });
                } else if (e.general[i]) {
                    GeneralConvParams f = general_base(i, d);
                    f.H = d.Ho; f.W = d.Wo; f.C = d.Cout; f.Ho = d.H; f.Wo = d.W; f.N = d.Cin; f.pad = d.R - 1 - d.pad;
                    f.ostride = f.wst = d.stride; f.classes = d.stride * d.stride;
                    f.a = grad(ot);
                    f.wmat = wbf() + e.wb_off[i];
                    f.out = grad(l.in0);
                    f.mask = mask0; f.mask_rep = e.rep_block; f.accumulate = acc0;
                    int& pending = e.pending_grad[l.in0];
                    if (pending >= 0) { f.addend = grad(pending); f.addend_rep = e.rep_block; pending = -1; }
                    int* brows = nullptr;
                    if (e.bstat_for[i] >= 0 && (!acc0 || e.bstat_input[i])) brows = gradient_sums(f, i, d, false);
                    run(l.type == HADFL_OP_CONV ? "conv_dgrad" : "dense_dgrad", gemm_flops(d), gemm_bytes(d), [&] { return e.patch[i] ? launch_conv_general_patch(f, 1, na, s, brows) : launch_conv_general(f, 1, na, s); });
                } else
                run(l.type == HADFL_OP_CONV ? "conv_dgrad" : "dense_dgrad", gemm_flops(d), gemm_bytes(d), [&] { return gemm(d); });
            }
            break; }
        case HADFL_OP_RELU:
            q.in = act(l.in0); q.in_rep = e.rep_block; q.in2 = grad(l.out); q.in2_rep = e.rep_block;
            q.count = B * a.numel();
            run("relu_bwd", 0, asz() * (12.0 * q.count), [&] { return launch_relu_bwd(q, na, s); });
            break;
        case HADFL_OP_MAXPOOL:
            q.in = act(l.in0); q.in_rep = e.rep_block; q.in2 = grad(l.out); q.in2_rep = e.rep_block;
            q.count = B * r.numel();
            run("maxpool_bwd", 0, asz() * (4.0 * (2 * B * a.numel() + q.count)), [&] { return launch_maxpool_bwd(q, na, s); });
            break;
        case HADFL_OP_ADD: {
            q.in = grad(ot); q.in_rep = e.rep_block; q.count = B * a.numel();
            const int64_t own = e.grad_off[ot];                // operands that share this buffer need no copy
            const bool late0 = !acc0 && (e.late_add[i] & 1), late1 = !e.grad_written[l.in1] && (e.late_add[i] & 2);
            if (late0) e.pending_grad[l.in0] = ot;
            else if (e.grad_off[l.in0] != own) run("add_bwd", 0, asz() * (8.0 * q.count), [&] { return launch_pass_grad(q, na, s); });
            EwParams q2 = q;
            if (l.in1 == l.in0) q2.accumulate = 1; else q2.accumulate = e.grad_written[l.in1] ? 1 : 0;
            q2.out = grad(l.in1);
            q2.mask = e.masked[l.in1] ? act(l.in1) : nullptr;
            if (late1) e.pending_grad[l.in1] = ot;
            else if (e.grad_off[l.in1] != own) run("add_bwd", 0, asz() * (8.0 * q.count), [&] { return launch_pass_grad(q2, na, s); });
            e.grad_written[l.in1] = 1;
            break; }
        case HADFL_OP_GAP:
            q.in = grad(l.out); q.in_rep = e.rep_block; q.count = B * a.numel();
            run("gap_bwd", 0, asz() * (4.0 * (q.count + B * a.c)), [&] { return launch_gap_bwd(q, na, s); });
            break;
        case HADFL_OP_BN: {
            const bool sums_done = e.bstat_rows[i] > 0 && sums_of == kBackward + (int)i;
            BnParams b = bn_params(i);
            b.dy = grad(ot); b.dy_rep = e.rep_block;
            b.y = grad(l.in0); b.y_rep = e.rep_block;
            b.accumulate = acc0;
            b.mask = mask0; b.mask_rep = e.rep_block;
            if (e.pool_of[i] >= 0) {
                b.pool = 1; b.H = a.h; b.W = a.w; b.relu = e.fused_relu[i];
                b.pool_g = grad(e.plan.layers[e.pool_of[i]].out); b.pool_g_rep = e.rep_block;
            }
            if (sums_done) {                                 // the data gradient of the layer above left the sums
                const int64_t rows_out = e.pool_of[i] >= 0 ? b.rows / 4 : b.rows;
                const int by = (int)(std::find(e.bstat_for.begin(), e.bstat_for.end(), (int)i) - e.bstat_for.begin());
                b.bwd_stats_done = e.bstat_input[by] ? 2 : 1; b.stat_entries = (int)((rows_out + e.bstat_rows[i] - 1) / e.bstat_rows[i]);
                b.partial_rep = e.bstat_rep[i];
            }
            e.bstat_rows[i] = 0;
            run("bn_bwd", 0, asz() * (12.0 * B * a.numel()), [&] { return launch_bn_bwd(b, na, s); });
            break; }
        }
        if (need_din) e.grad_written[l.in0] = 1;
    }
};

}  // namespace

hadfl_status train_run(TrainEngine* e, hipStream_t s, Profiler* prof, std::string& err)
{
    Runner r{*e, s, (prof && prof->on) ? prof : nullptr};
    const int N = e->cfg.n_replicas;
    if (!e->tables_uploaded && !e->tables.empty()) {
        const hipError_t rc = hipMemcpyAsync(e->buf.work + e->tab_off, e->tables.data(), e->tables.size() * sizeof(int32_t), hipMemcpyHostToDevice, s);
        if (rc != hipSuccess) { err = std::string("copy position tables: ") + hipGetErrorString(rc); return HADFL_EDEVICE; }
        e->tables_uploaded = true;
    }
    if (e->use_side && !e->side) {
        if (hipStreamCreateWithFlags(&e->side, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&e->ev_fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&e->ev_join, hipEventDisableTiming) != hipSuccess) {
            err = "side stream"; return HADFL_EDEVICE;
        }
    }
    const int T = (int)e->plan.tensors.size();
    e->prepped.assign(e->plan.layers.size(), 0);       // the weights may have changed since the last call (aggregation)
    if (dense_pair_net(e->cfg, e->plan, e->e_max)) r.dense_pair_steps();
    else for (int step = 0; step < e->e_max && r.rc == hipSuccess; ++step) {
        r.na = e->n_active[step]; r.step = step;
        r.prepare_weights();
        for (size_t i = 0; i < e->plan.layers.size(); ++i) r.forward_layer(i);
        if (!r.forms_criterion(e->plan.layers.size() - 1)) {
            const LossParams lp = r.criterion();
            r.run("softmax_ce", 0, r.asz() * 8.0 * e->cfg.batch * e->cfg.n_classes, [&] { return launch_softmax_ce(lp, r.na, s); });
        }
        e->grad_written.assign(T, 0);
        e->grad_written[T - 1] = 1;
        e->pending_grad.assign(T, -1);
        r.na_next = step + 1 < e->e_max ? e->n_active[step + 1] : 0;
        for (int t : e->unread) {
            EwParams z{};
            z.out = r.grad(t); z.out_rep = e->rep_block; z.count = e->cfg.batch * e->plan.tensors[t].numel(); z.bf16 = e->cfg.bf16; z.order = e->buf.order;
            r.run("zero_grad", 0, r.asz() * 4.0 * z.count, [&] { return launch_zero(z, r.na, s); });
        }
        for (size_t i = e->plan.layers.size(); i-- > 0;) r.backward_layer(i);
        if (r.pending_prep >= 0) { r.fork(0.0); r.flush_pending_prep(); r.unfork(); }
        r.join();
        SgdParams sp{};
        sp.w = e->buf.replicas; sp.g = e->buf.grad; sp.buf = e->buf.mom; sp.row_stride = e->plan.row_stride;
        sp.lr = e->cfg.lr; sp.momentum = e->cfg.momentum;
        sp.order = e->buf.order;
        r.cur_layer = 0;
        // the pieces of the row no weight-gradient kernel has updated already, several per launch
        const size_t nseg = e->update_segments.size();
        for (size_t k0 = 0; k0 < nseg; k0 += kMaxSgdSegments) {
            const size_t k1 = std::min(nseg, k0 + kMaxSgdSegments);
            double floats = 0.0;
            sp.n_seg = (int)(k1 - k0);
            for (size_t k = k0; k < k1; ++k) {
                sp.first[k - k0] = e->update_segments[k].first; sp.count[k - k0] = e->update_segments[k].second;
                floats += (double)e->update_segments[k].second;
            }
            r.run("sgd", 0, (e->buf.mom ? 20.0 : 12.0) * floats, [&] { return launch_sgd(sp, r.na, s); });
        }
    }
    // Every step read its batch at the cursor and the steps before it in this call; the cursors and versions advance once, here.
    r.run("advance", 0, 24.0 * N / std::max(r.na, 1), [&] { return launch_advance(e->buf.steps, e->buf.versions, e->buf.cursor, N, s); });
    if (r.rc != hipSuccess) {
        err = std::string("kernel launch failed in ") + (r.failed ? r.failed : "?") + ": " + hipGetErrorString(r.rc);
        return HADFL_EDEVICE;
    }
    return HADFL_OK;
}

}  // namespace hadfl
