// Kernel launchers of the local-training path (paper Sec. 2.1: forward, backward, update), all grouped over
// replicas: grid z (or y) indexes a slot g of the active prefix, and order[g] is the replica it works on.
#pragma once
#include "hadfl_internal.h"

namespace hadfl {

enum GemmMode { kFwd = 0, kDgrad = 1, kWgrad = 2 };

// One grouped implicit-GEMM launch C[M x N] = A[M x K] * B[K x N] per active replica.
//  kFwd   : M = B*Ho*Wo, N = Cout,   K = R*S*Cin   A = im2col(X),        B = W[(r,s,ci)][co]
//  kDgrad : M = B*H*W,   N = Cin,    K = R*S*Cout  A = col(dY),          B = W^T per tap
//  kWgrad : M = R*S*Cin (+1 bias row), N = Cout, K = B*Ho*Wo  A = im2col(X)^T, B = dY   (split over K)
// A dense layer is the 1x1 case with H = W = 1 and Cin = flattened input size.
struct GemmParams {
    int mode;
    int B, H, W, Cin, Ho, Wo, Cout, R, S, stride, pad;
    int M, N, K;
    int tiles_m, tiles_n;
    int grid_y, n_active;         // set by the fp32 launcher: splits (or dgrad pixel classes) and active replicas
    int kchunk, splits;
    int hw_shift, w_shift;        // log2 of Ho*Wo and Wo (kWgrad) when powers of two, else -1
    // activation-side source: X (fwd, wgrad) or dY (dgrad)
    const float* a; long long a_rep;
    const long long* cursor; int n_samples, batch; long long sample_sz;   // a is the data set when cursor != null
    long long ahead;              // steps of this call so far: the cursor counts them at its end
    const float* w; long long w_rep;              // weights of this layer inside the replica rows
    const float* dy; long long dy_rep;            // kWgrad: dY
    float* out; long long out_rep, out_split;     // kWgrad with splits > 1: partial sums [g][split][M*N]
    int has_bias, relu, accumulate;
    // kDgrad: when set, the written gradient is zeroed where mask <= 0 (mask = the ReLU output stored in the tensor
    // whose gradient is being produced, so the result is the gradient before that fused ReLU)
    const float* mask; long long mask_rep;
    int a_f32;                    // bf16 kernel only: the activation-side source is the fp32 data set
    const int* order;
};
hipError_t launch_gemm(const GemmParams& p, int n_active, hipStream_t s);
// kFwd and kDgrad of stride-1 "same" convolutions, the same bits (conv_chain.hip): C source channels, N outputs, k x k filters; `first`: on
// the data set
bool conv_chain_supported(int B, int H, int W, int C, int N, int k);
bool conv_chain_first_supported(int B, int H, int W, int C, int N, int k);
hipError_t launch_conv_chain(const GemmParams& p, int n_active, hipStream_t s);
// Same problems with bf16 activations / activation gradients (pointers still typed float*: they are byte bases whose
// offsets and strides are counted in 4-byte units), fp32 weights rounded to bf16 on the fly, fp32 weight gradients.
hipError_t launch_gemm_bf16(const GemmParams& p, int n_active, hipStream_t s);
// out[rep][i] = sum_s partial[g][s][i], s ascending
hipError_t launch_splitk_reduce(const float* partial, long long split_stride, int splits, float* out, long long out_rep,
                                long long count, const int* order, int n_active, hipStream_t s);
// The same sum applied as the update of the layer's parameters (w, buf: first parameter of the layer in replica row 0;
// buf may be null).  Needs count, split_stride and row_stride multiples of 4 and 16-byte aligned pointers.  one_chain: the
// splits are added one after another, s ascending, whatever the launch size.
hipError_t launch_splitk_reduce_update(const float* partial, long long split_stride, int splits, float* w, float* buf,
                                       long long row_stride, long long count, float lr, float momentum, int one_chain, const int* order,
                                       int n_active, hipStream_t s);

// ---- lean bf16 kernels for regular stride-1 "same" convolutions (conv_bf16_fast.hip) ----
struct FastConvParams {      // out[m][n] = sum_k act[pixel(m) + tap(k)][c(k)] * wmat[n][k]; M = B*H*W, K = R*S*C
    int B, H, W, C, N, R, S, pad, M, K;
    const void* a; long long a_rep;            // bf16 activations (forward) or output gradient (data gradient)
    const __bf16* wmat; long long wmat_rep;    // bf16 [N][K], per-replica stride in elements
    void* out; long long out_rep;              // bf16 [M][N]
    const float* bias; long long bias_rep;     // forward: fp32 bias inside the replica rows, or null
    int relu;
    const void* mask; long long mask_rep; int accumulate;   // data gradient
    const int* order;
    int tile_hint;                             // 1: take the 256 x 256 tiles whenever the shape allows (N % 256 == 0); 2: as 0
    // optional position table (both null or both set): GEMM row ps * B + b is image b at pixel perm[ps]; posmask[ps] has
    // bit r * S + s set when tap (r, s) of that pixel lies inside the image
    const int* perm; const unsigned* posmask;
    int n_active;                              // set by the launcher
    // forward only, optional: per-channel sums of the stored outputs for the batch norm that follows.  Entry e of slot g
    // covers GEMM rows [e * R, (e + 1) * R), R = the chosen kernel's rows per tile (reported by the launcher):
    // stat[g * stat_rep + e * 2 * N + n] = sum of out[m][n], [.. + N + n] = sum of out[m][n]^2 (values as rounded to bf16)
    float* stat; long long stat_rep;
    // data gradient only, with stat set: the tensor whose gradient is being written is the output y of a batch norm
    // (after its fused ReLU and, if the pool is folded into it, after the pool), and the same entries receive what that
    // batch norm's backward pass needs instead:  [..+ n] = sum of g,  [.. + N + n] = sum of g * y,  g the stored gradient
    // (zero where stat_relu is set and y <= 0).  With xhat = (y - beta) / gamma wherever the gradient passes, these give
    // d(beta) = sum g and d(gamma) = (sum g*y - beta * sum g) / gamma without another pass over the tensors.
    const void* stat_y; long long stat_y_rep; int stat_relu;
};
// epi 0: forward (+bias, ReLU); epi 1: data gradient (mask, accumulate).  Needs C % 64 == 0 and N % 64 == 0.
// stat_rows (may be null): receives the rows per statistics entry of the kernel that was launched (128 or 256).
hipError_t launch_conv_fast(const FastConvParams& p, int epi, int n_active, hipStream_t s, int* stat_rows = nullptr);

struct FastWgradParams {     // dW[(tap, ci) | bias row][co] over pixels; needs C % 8 == 0, N % 64 == 0, H, W powers of two
    int B, H, W, C, N, R, S, pad, M, K, kchunk, splits, w_shift, has_bias;
    const void* x; long long x_rep;
    const void* dy; long long dy_rep;
    float* out; long long out_rep, out_split;
    const int* order;
    const int* perm; const unsigned* posmask;   // optional position table as in FastConvParams; needs B % 64 == 0, kchunk % 64 == 0
    int tile_hint;                              // 1: 256-row tiles in wgrad_kernel whenever N % 128 == 0; 2: wgrad_kernel for any image
    // splits == 1 only: when sgd_w is set the epilogue applies the update (buf = momentum*buf + g; w -= lr*buf) to the
    // layer's slice of the parameter rows (same per-replica stride as `out`) instead of storing the gradient
    float* sgd_w; float* sgd_buf; float lr, momentum;
    int n_active;                               // set by the launcher
};
hipError_t launch_wgrad_fast(const FastWgradParams& p, int n_active, hipStream_t s);
// split-K factor; general kernels: 64 x 64 tiles, wgrad_positions.hip; estimated cost with the reduction in us
struct WgradPlan { int splits, small_tiles, positions = 0; float time = 0.f; };
WgradPlan wgrad_fast_plan(const FastWgradParams& shape, int n_active);        // (from the fields above x)

// ---- bf16 configuration, first convolution (fp32 data set in, few channels): conv_first_bf16.hip ----
struct FirstConvParams {     // K = R*S*C footprint values per pixel (K + bias row <= 32), N = 32 or 64 output channels, stride 1
    const float* x; const long long* cursor; long long ahead; int n_samples;     // data set [replica][n_samples][H][W][C] and batch cursors (see GemmParams)
    int B, H, W, C, N, R, S, pad, K, M;                          // M = B*H*W pixels of a batch
    const float* w; long long w_rep;                             // fp32 weights [K][N] inside the replica rows (stride w_rep)
    const float* bias;                                           // inside the same rows, or null
    void* out; long long out_rep; int relu;                      // forward: bf16 [M][N]
    const void* dy; long long dy_rep;                            // weight gradient: bf16 [M][N]
    float* gout; long long gout_rep, gout_split; int splits, kchunk;   // rows 0..K-1 weights, row K bias; split over pixels
    const int* order;
};
bool conv_first_supported(const FirstConvParams& p);
hipError_t launch_conv_first_fwd(const FirstConvParams& p, int n_active, hipStream_t s);
hipError_t launch_conv_first_wgrad(const FirstConvParams& p, int n_active, hipStream_t s);

struct WeightPrepParams {    // fp32 W[tap][C][N] -> bf16 Wf[N][tap*C + ci] and Wb[C][(taps-1-tap)*N + co]
    const float* w; long long w_rep;
    __bf16* wf; __bf16* wb; long long wbf_rep;
    int C, N, taps;
    const int* order;
};
hipError_t launch_weight_prep(const WeightPrepParams& p, int n_active, hipStream_t s);

// ---- convolutions and dense layers of any geometry (conv_general.hip): fp32 on split floats, and the bf16 layers that are not lean ----
struct GeneralConvParams {     // out[pixel][n] = sum over taps and channels of a[source pixel][c] * wmat[n][tap][c]
    int bf16;                                  // element type of the tensors (pointers are typed float*, strides count 4 bytes)
    int B, H, W, C;                            // source: X (forward) or dY (data gradient)
    int Ho, Wo, N;                             // output image and channels
    int R, S, pad;                             // filter in the copy's (forward or flipped) order
    int sstride;                               // source pixels per output pixel: the stride (forward), 1 (data gradient)
    int ostride, wst, classes;                 // data gradient: stride, stride, stride^2; forward 1, 1, 1
    const float* a; long long a_rep;
    // forward of an fp32 convolution on the data set (a) when cursor != null: any C, the copy is [N][1][R*S*C]
    const long long* cursor; int n_samples, batch; long long sample_sz, ahead;
    const __bf16* wmat; long long wmat_rep;    // weight copy, per-replica stride in 2-byte units
    float* out; long long out_rep;
    const float* bias; long long bias_rep;     // forward: bias inside the replica rows, or null
    int relu;
    const float* mask; long long mask_rep; int accumulate;   // data gradient
    // with accumulate, conv_general_patch.hip: what is added to, if not what `out` holds; not masked yet
    const float* addend; long long addend_rep;
    const int* order;
    const int* perm; const unsigned* posmask;  // optional position table as in FastConvParams (stride 1)
    float* stat; long long stat_rep;           // forward, optional: statistics entries as in FastConvParams
    int tile_hint;                             // 1: the largest tiles whatever the launch size; 2: as 0
    int tiles_m, n_active;                     // set by the launcher
    int halo; unsigned inv_hw, inv_w;          // the same (conv_general_patch.hip): pixels of border before and behind a tile, 2^32 / HW, 2^32 / W
    const float* stat_y; long long stat_y_rep; int stat_relu;      // bf16 data gradient with stat set (conv_general_patch.hip): as in FastConvParams
    // data gradient with stat set (conv_general_patch.hip): stat_y is the INPUT of the batch norm whose output gradient this is and stat_mean
    // its channels' means; the second sum is that of g * (stat_y - mean)
    const float* stat_mean; long long stat_mean_rep;
};
// epi 0: forward (+bias, ReLU); epi 1: data gradient (mask, accumulate).  Needs C % 4 == 0 (bf16: 8), N % 4 == 0, R * S <= 32,
// tensors of less than 4 GiB per replica.  stat_rows (may be null): rows per statistics entry of the kernel that was launched.
hipError_t launch_conv_general(const GeneralConvParams& p, int epi, int n_active, hipStream_t s, int* stat_rows = nullptr);
// The same for stride-1 "same" convolutions (conv_general_patch.hip) that conv_patch_supported accepts: k x k filters, C channels of the
// source and N of the result in either direction.  The copy is in fragments.
bool conv_patch_supported(int bf16, int H, int W, int C, int N, int k);
hipError_t launch_conv_general_patch(const GeneralConvParams& p, int epi, int n_active, hipStream_t s, int* stat_rows = nullptr);
struct GeneralWgradParams {    // dW[(tap, ci)][co] over pixels, then (has_bias) the bias gradient as row R*S*C
    int bf16;                                  // element type of x and dy
    int B, H, W, C, Ho, Wo, N, R, S, pad, stride;
    int gather;                                // fp32 convolution on the data set: any C
    int K, kchunk, splits, has_bias;           // K = B*Ho*Wo; kchunk a multiple of 32 when splits > 1
    int small_tiles;                           // of the plan the splits are from
    const float* x; long long x_rep;
    const long long* cursor; int n_samples, batch; long long sample_sz, ahead;   // x is the (fp32) data set when cursor != null
    const float* dy; long long dy_rep;
    float* out; long long out_rep, out_split;
    const int* order;
    const int* perm; const unsigned* posmask;  // optional position table as in FastWgradParams; stride 1, B % 32 == 0
    float* sgd_w; float* sgd_buf; float lr, momentum;    // as in FastWgradParams
    int n_active;                              // set by the launcher
};
// Needs C and N multiples of 4 (bf16: 8), tensors of less than 4 GiB per replica.
hipError_t launch_wgrad_general(const GeneralWgradParams& p, int n_active, hipStream_t s);
WgradPlan wgrad_general_plan(int rows, int N, int K, int n_active, int gather);   // for rows = R*S*C weights
// The same for fp32 3 x 3 stride-1 "same" convolutions (wgrad_positions.hip); kchunk, small_tiles and the position table are not read.
bool wgrad_positions_supported(int B, int H, int W, int C, int N);
WgradPlan wgrad_positions_plan(int B, int H, int W, int C, int N, int n_active);
hipError_t launch_wgrad_positions(const GeneralWgradParams& p, int n_active, hipStream_t s);
long long weight_copy_units(int bf16, int rows, int taps, int channels);   // 2-byte units of a copy [rows][taps][channels]
long long weight_fragment_units(int bf16, int rows, int taps, int channels);   // the same in fragments
struct WeightCopyParams {    // fp32 W[tap][C][N] -> copies Wf[N][tap][C] and (unless null) Wb[C][taps-1-tap][N]
    const float* w; long long w_rep;
    __bf16* wf; __bf16* wb; long long wcopy_rep;
    int C, N, taps, bf16;
    int fragments;                             // in the order of conv_general_patch.hip
    const int* order;
};
constexpr int kWeightCopies = 32;
struct WeightCopies {        // layers whose copies one launch writes
    WeightCopyParams layer[kWeightCopies];
    int first[kWeightCopies];                  // a layer's first workgroup
    int count;
};
hipError_t launch_weight_copies(WeightCopies& p, int n_active, hipStream_t s);

struct LossParams {
    const float* logits; long long logits_rep;
    float* dlogits; long long dlogits_rep;
    const int* y; const long long* cursor; long long ahead; int n_samples, batch, n_classes;
    float* loss;
    int bf16;
    const int* order;
};
struct DenseRowsParams {      // out[m][n] = sum_k x[m][k] w[k][n] + bias[n]
    const float* x; long long x_rep;
    const long long* cursor; int n_samples, batch; long long ahead;    // x is the (fp32) data set when cursor != null
    const float* w; long long w_rep;     // weights [K][N] followed by bias [N]
    float* out; long long out_rep;
    int rows, K, N, has_bias, relu, bf16;
    const int* order;
};
bool dense_rows_supported(int rows, long long K);
hipError_t launch_dense_rows_fwd(const DenseRowsParams& p, int n_active, hipStream_t s);

struct DenseSmallParams {     // dense layer with N <= 16 outputs.  Forward: out[m][n] = sum_k x[m][k] w[k][n] + bias[n].  Backward:
    // dx[m][k] (+)= sum_n dy[m][n] w[k][n], zero where mask <= 0; then w and buf (the momentum of these parameters, or
    // null; same stride) take the update of w's gradient sum_m x[m][k] dy[m][n]
    const float* x; long long x_rep;
    float* w; long long w_rep;           // weights [K][N] followed by bias [N]
    float* out; long long out_rep;       // forward
    int rows, K, N, has_bias;
    int bf16;
    const int* order;
    const float* dy; long long dy_rep;
    float* dx; long long dx_rep;
    const float* mask; long long mask_rep; int accumulate;
    float* buf; float lr, momentum;
    // backward, optional (at most 256 rows): dy is the gradient of the softmax cross-entropy of this layer's output, formed here; the
    // mean loss of every replica goes to loss
    LossParams criterion;                 // (none: criterion.loss null)
};
hipError_t launch_dense_small_fwd(const DenseSmallParams& p, int n_active, hipStream_t s);
hipError_t launch_dense_small_bwd(const DenseSmallParams& p, int n_active, hipStream_t s);

// A network of two dense layers, H hidden units with a ReLU and N classes: the end of a local step of the first n_end replicas in
// step order and the beginning of the next of the first n_begin, in one launch.
struct DensePairParams {
    const float* x; const int* y; const long long* cursor; int ahead;    // ahead: steps of the call before the one that begins
    int n_samples, batch, K, H, N;
    int has_bias1, has_bias2;
    float* w1; float* w2; long long w_rep;   // weights [K][H] followed by bias [H]; [H][N] followed by bias [N]
    float* m1; float* m2;                    // momentum of the same, or null; same stride
    float lr, momentum;
    float* hidden; long long act_rep;        // hidden units [batch][H]
    const float* share_in; float* share_out;             // shares of the logits of the step that ends and of the one that begins, floats [H / 16][batch][16]; two buffers
    float* loss;
    int n_end, n_begin;
    int bf16;
    const int* order;
};
bool dense_pair_supported(int batch, int K, int H, int N);
hipError_t launch_dense_pair(const DensePairParams& p, hipStream_t s);

struct EwParams {     // element-wise / pooling kernels
    const float* in; long long in_rep;
    const float* in2; long long in2_rep;
    float* out; long long out_rep;
    long long count;              // elements per replica of `out`
    int B, H, W, C;               // input geometry where needed
    int accumulate;
    int relu;                     // forward kernels: apply max(., 0) to the result
    const float* mask; long long mask_rep;   // backward kernels: zero the written gradient where mask <= 0
    int bf16;                     // tensors are bf16 (strides still in 4-byte units)
    const int* order;
};
hipError_t launch_relu_fwd(const EwParams& p, int n_active, hipStream_t s);
// out(din) (+)= in2(dout) where in(x) > 0
hipError_t launch_relu_bwd(const EwParams& p, int n_active, hipStream_t s);
hipError_t launch_maxpool_fwd(const EwParams& p, int n_active, hipStream_t s);
// in = pool input x, in2 = dout (pooled shape), out = din (input shape)
hipError_t launch_maxpool_bwd(const EwParams& p, int n_active, hipStream_t s);
hipError_t launch_add_fwd(const EwParams& p, int n_active, hipStream_t s);
// out(din) (+)= in(dout)
hipError_t launch_pass_grad(const EwParams& p, int n_active, hipStream_t s);
hipError_t launch_zero(const EwParams& p, int n_active, hipStream_t s);       // out = 0
hipError_t launch_gap_fwd(const EwParams& p, int n_active, hipStream_t s);
hipError_t launch_gap_bwd(const EwParams& p, int n_active, hipStream_t s);

struct BnParams {
    const float* x; long long x_rep;       // [rows][C]
    float* y; long long y_rep;             // forward output / backward dx
    const float* dy; long long dy_rep;
    float* params; long long row_stride;   // replica rows; gamma at w_off, beta at w_off + C, running stats at stat_off
    float* grads;                          // gradient rows (same layout)
    long long w_off, stat_off;
    float* saved; long long saved_rep;     // [2][C]: mean, 1/sqrt(var+eps)
    float* partial; long long partial_rep; // [chunks][2][C]
    int rows, C, chunks, chunk_rows;
    int cvb;                               // set by the launcher: channel vectors per workgroup (vector kernels)
    int accumulate;
    int relu;                              // forward: y = max(bn(x), 0)
    const float* mask; long long mask_rep; // backward: zero dx where mask <= 0
    int bf16;
    const int* order;
    // a 2x2 / stride-2 max-pool folded into the layer (vector kernels only; H, W even): forward writes the pooled
    // output only; backward takes the gradient of the pooled output instead of dy and forms each window's outputs
    // again from x
    int pool, H, W;
    // forward: the producing convolution already left per-entry sums of d = x - x0 and d^2 in `partial`
    // ([stat_entries][2][C]) and the sums pass is skipped; the shift x0 of channel c is that convolution's bias
    // stat_shift[c] (zero without one): what the outputs are centred on when the bias is large beside their spread
    int stats_done, stat_entries;
    const float* stat_shift; long long stat_shift_rep;
    // forward: a bias that the producing convolution left out of x, since a normalised value does not depend on it; the running
    // mean is that of x with it (a bias large beside the spread of x would cost x the low bits of its sums)
    const float* left_out; long long left_out_rep;
    // backward: the data-gradient kernel of the layer above already left per-entry sums of g and g * y in `partial`
    // ([stat_entries][2][C], see FastConvParams::stat_y); the sums pass is skipped and d(gamma) is formed from them
    int bwd_stats_done;                    // 1; 2: sums of g and g * (x - mean)
    // forward, optional (vector kernels, no pool): y = max(bn(x) + add, 0) or without the ReLU, bn(x) rounded to the stored
    // type first as if it were stored: the layer that adds a second tensor to this one's output, folded in
    const float* add; long long add_rep; int add_relu;
    float* pool_out; long long pool_out_rep;
    const float* pool_g; long long pool_g_rep;
};
hipError_t launch_bn_fwd(const BnParams& p, int n_active, hipStream_t s);
hipError_t launch_bn_bwd(const BnParams& p, int n_active, hipStream_t s);
bool bn_backward_in_one_launch(const BnParams& p, int n_active);       // sums that a data gradient left would make it two

hipError_t launch_softmax_ce(const LossParams& p, int n_active, hipStream_t s);

constexpr int kMaxSgdSegments = 16;
struct SgdParams {
    float* w; const float* g; float* buf; long long row_stride;
    float lr, momentum;
    // the launch covers n_seg pieces of each row: floats [first[k], first[k] + count[k]), all multiples of 4
    int n_seg; long long first[kMaxSgdSegments], count[kMaxSgdSegments];
    const int* order;
};
hipError_t launch_sgd(const SgdParams& p, int n_active, hipStream_t s);
// versions[k] = steps[k], cursor[k] += steps[k]
hipError_t launch_advance(const int* steps, int* versions, long long* cursor, int n, hipStream_t s);

}  // namespace hadfl
