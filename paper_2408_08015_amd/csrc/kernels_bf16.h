// Host-side launchers of the bf16-operand / fp32-accumulate kernels (NHWC images and
// [rows][features] token matrices).  All matrix products run on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16) from LDS-staged tiles.  None of the launchers allocates.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace ast {

typedef unsigned short bf16_t;

// ---- weight copies (refreshed by the optimizer step from the fp32 master weights)
// conv: master [Cout][Cin][k][k] -> fwd operand [Cout][tap][Cin] and input-gradient operand [Cin][tap'][Cout] with tap' the
// point-reflected tap; or in the layout of the kernel that reads it (CONV_*): halo [Cin/64][tap][Cout][64] /
// [Cout/64][tap'][Cin][64], resident the fragments [Cout/32][Cin/16][tap][64 lanes][8] / [Cin/32][Cout/16][tap'][64][8] (padded
// with zeros, conv_res_pack_elems).
enum : int { CONV_GENERAL = 0, CONV_HALO = 1, CONV_RESIDENT = 2 };
void conv_weight_shadow_bf16(hipStream_t st, const float* w, bf16_t* sh_fwd, bf16_t* sh_dgrad, int Cout,
                             int Cin, int k, int kernel_fwd, int kernel_dgrad);
// linear: master [Cout][Cin] -> copy [Cout][Cin] and transpose [Cin][Cout]
void linear_weight_shadow_bf16(hipStream_t st, const float* w, bf16_t* sh, bf16_t* sh_t, int Cout, int Cin,
                               bool tiled, bool tiled_t);
// ... and for all dense layers of a stage in one launch: the table lives in device memory, block_task maps a
// block to its matrix, a matrix takes linear_shadow_blocks() consecutive blocks from block0.
struct LinShadowTask {
  const float* w;
  bf16_t* sh;
  bf16_t* sht;
  int Cout, Cin, tiled, tiled_t;
  unsigned block0;
};
unsigned linear_shadow_blocks(int Cout, int Cin);
void linear_weight_shadow_all_bf16(hipStream_t st, const LinShadowTask* tasks_dev, const unsigned short* block_task_dev,
                                   int nblocks);

// ---- dense 'same' convolution, stride 1, NHWC, k in {1,3}
// taps (of these and of conv_bf16_wgrad): the partials of the kernel with all taps in a wavefront, conv_bf16_wgrad_taps() of them
// as asked for at create; 0: another kernel runs.
int conv_bf16_wgrad_taps(int N, int H, int W, int Cin, int Cout, int k, int most);
size_t conv_bf16_ws_bytes(int N, int H, int W, int Cin, int Cout, int k, int taps);
// y = act(conv(x) + bias)
void conv_bf16_fwd(hipStream_t st, const bf16_t* x, const bf16_t* sh_fwd, const float* bias, bf16_t* y,
                   int N, int H, int W, int Cin, int Cout, int k, int act, int kernel);
// dx = conv^T(g); with `relu_out` ([N][H][W][Cin], may be NULL: the output of a ReLU that feeds this
// conv) dx is zeroed where relu_out <= 0: that ReLU's backward, folded into the epilogue.
void conv_bf16_dgrad(hipStream_t st, const bf16_t* g, const bf16_t* sh_dgrad, bf16_t* dx, const bf16_t* relu_out,
                     int N, int H, int W, int Cin, int Cout, int k, int kernel);
// The same 3x3 product with the input tile and its halo staged in LDS once per 64-channel slice
// (conv_bf16_halo.hip), or once for all channels (conv_bf16_res.hip).  conv_bf16_kernel(N, H, W, Cin, Cout, k): the kernel
// (CONV_*) for this shape, which expects its layout of the weight copy; the input gradient asks with Cin and Cout
// exchanged.  Asked once, at create (it needs a device: the halo kernel's LDS size has to be granted).
// conv3x3_halo_bf16: act is 0 or ReLU; the output is zeroed where mask <= 0 (mask may be NULL).
int conv_bf16_kernel(int N, int H, int W, int Cin, int Cout, int k);
bool conv_res_supported(int N, int H, int W, int Cin, int Cout);
size_t conv_res_pack_elems(int Cin, int Cout);
hipError_t conv_res_allow();  // before the first launch on a device
void conv_res_bf16(hipStream_t st, const bf16_t* x, const bf16_t* w, const float* bias, const bf16_t* mask, bf16_t* y, int N,
                   int H, int W, int Cin, int Cout, int act);
bool conv3x3_halo_supported(int N, int H, int W, int Cin, int Cout);
void conv3x3_halo_bf16(hipStream_t st, const bf16_t* x, const bf16_t* w, const float* bias, const bf16_t* mask,
                       bf16_t* y, int N, int H, int W, int Cin, int Cout, int act);
// Weight gradient with both operands read transposed from LDS (conv_bf16_wgrad.hip): partials
// part[split][tap][Cout][Cin], conv_wgrad_tr_splits() of them (a function of the shape alone), and,
// with bias_part, the splits' column sums of dy [split][Cout] (the bias gradient's partials).
// conv_bf16_wgrad uses it where conv_wgrad_tr_supported() (needs a device: LDS size granted).
int conv_wgrad_tr_splits(long P, int Cin, int Cout, int taps);
bool conv_wgrad_tr_supported(int N, int H, int W, int Cin, int Cout, int k);
void conv_wgrad_tr_bf16(hipStream_t st, const bf16_t* dy, const bf16_t* x, float* part, float* bias_part, int N, int H,
                        int W, int Cin, int Cout, int k);
// ... with all nine taps of a 32 x 32 tile in one wavefront (conv_bf16_wgrad_taps.hip): the same partials, `splits` =
// conv_wgrad_taps_splits(.., most) of them, at most `most`.
int conv_wgrad_taps_splits(int N, int H, int W, int Cin, int Cout, int most);
hipError_t conv_wgrad_taps_allow();  // before the first launch on a device
bool conv_wgrad_taps_supported(int N, int H, int W, int Cin, int Cout);
void conv_wgrad_taps_bf16(hipStream_t st, const bf16_t* dy, const bf16_t* x, float* part, float* bias_part, int N, int H, int W,
                          int Cin, int Cout, int splits);
// Grouped weight gradients of linear layers: the same kernel, one launch for many products.  A product is formed in one share of
// its rows and added straight into its gradient, or in several, whose partials part[share][Cout][Cin], bias_part[share][Cout]
// are left to the caller.  The caller builds one descriptor per product on the host (wgrad_group_task returns the product's
// block count) and a list of blocks, product << 16 | block of the product, and copies both to the device once.
size_t wgrad_group_task_bytes();
bool wgrad_group_supported(size_t rows, int Cin, int Cout);
int wgrad_group_shares(size_t rows, int splits);  // the shares that a wish for `splits` makes
int wgrad_group_task(void* task_out, const bf16_t* dy, const bf16_t* x, float* GW, float* Gb, size_t rows, int Cin, int Cout,
                     int shares, float* part, float* bias_part);
void wgrad_group_launch(hipStream_t st, const void* tasks_dev, const unsigned* blocks_dev, int nblocks);
// The shares of every product of a group, at most `most`, so that its blocks fill the chip evenly (each product: rows, Cin, Cout).
struct WgradProduct { size_t rows; int cin, cout, splits; };
constexpr int kWgradMostShares = 12;
void wgrad_group_split(WgradProduct* products, size_t n, int most);
// Rearranges n blocks from `first` on in a launch's list so that neighbours run on one XCD.
void wgrad_group_order(unsigned* blocks, size_t first, size_t n);
// Scratch layout of a weight-gradient call: `splits` partial copies of the weight gradient at
// ws[0, ...), `bias_parts` partial bias gradients ([bias_parts][Cout]) from float offset bias_off.
struct WgradParts { int splits; size_t bias_off; int bias_parts; };
WgradParts conv_bf16_wgrad_parts(int N, int H, int W, int Cin, int Cout, int k, int taps);
// GW[Cout][Cin][k][k] += conv weight gradient, Gb[Cout] += sum of g (if has_bias).  With
// `defer` only the partials are written and the caller reduces them (reduce_tasks_f32).
void conv_bf16_wgrad(hipStream_t st, const bf16_t* g, const bf16_t* x, float* GW, float* Gb, bool has_bias,
                     bool defer, void* ws, int N, int H, int W, int Cin, int Cout, int k, int taps);

// ---- linear on [R][Cin] rows
// Whether the product of [R][K] rows with an [N][K] weight matrix runs in the direct-to-LDS kernel,
// which reads its weights from the tiled copy [K/64][N][64] (linear_weight_shadow_bf16: `tiled` for
// the forward copy with K = Cin, N = Cout; `tiled_t` for the transposed one with K = Cout, N = Cin).
bool linear_dl_supported(size_t R, int K, int N);
void linear_dl_bf16(hipStream_t st, const bf16_t* a, const bf16_t* b, const float* bias, bf16_t* c, bf16_t* pre,
                    const bf16_t* add, const bf16_t* gmul, size_t R, int K, int N, int act);
size_t linear_bf16_ws_bytes(size_t R, int Cin, int Cout, int splits = 1);
// ... of a product of the grouped launch in `splits` shares
WgradParts linear_bf16_group_parts(size_t R, int Cin, int Cout, int splits);
// y = act(x W^T + b) (+ add); with act == GELU the pre-activation goes to `pre` as well
// `add` (may be NULL): residual input [R][Cout] added to the rounded output.
void linear_bf16_fwd(hipStream_t st, const bf16_t* x, const bf16_t* sh, const float* bias, bf16_t* y,
                     bf16_t* pre, const bf16_t* add, size_t R, int Cin, int Cout, int act);
// dx = g W; with `gelu_pre` ([R][Cin], may be NULL) dx is further multiplied by GELU'(gelu_pre):
// the backward of a GELU in front of this layer, folded into the epilogue; with `add` ([R][Cin],
// may be NULL) the gradient arriving over a residual connection is added.  At most one of the two.
void linear_bf16_dgrad(hipStream_t st, const bf16_t* g, const bf16_t* sh_t, bf16_t* dx, const bf16_t* gelu_pre,
                       const bf16_t* add, size_t R, int Cin, int Cout);
WgradParts linear_bf16_wgrad_parts(size_t R, int Cin, int Cout);
void linear_bf16_wgrad(hipStream_t st, const bf16_t* g, const bf16_t* x, float* GW, float* Gb, bool has_bias,
                       bool defer, void* ws, size_t R, int Cin, int Cout);

// ---- elementwise on bf16
// g' = g * act'(.) : ReLU masks by the OUTPUT y (> 0), GELU uses the stashed pre-activation.
void act_bwd_bf16(hipStream_t st, const bf16_t* g, const bf16_t* ref, bf16_t* out, size_t n, int act);
void act_fwd_bf16(hipStream_t st, const bf16_t* x, bf16_t* y, size_t n, int act);
void add_bf16(hipStream_t st, const bf16_t* a, const bf16_t* b, bf16_t* y, size_t n);
void maxpool_fwd_bf16(hipStream_t st, const bf16_t* x, bf16_t* y, int N, int H, int W, int C);
void maxpool_bwd_bf16(hipStream_t st, const bf16_t* g, const bf16_t* x, bf16_t* dx, int N, int H, int W,
                      int C, bool relu_mask);

// ---- LayerNorm over the last dimension of [R][D]
size_t layernorm_bf16_ws_bytes(size_t R, int D);
void layernorm_fwd_bf16(hipStream_t st, const bf16_t* x, const float* gamma, const float* beta,
                        bf16_t* y, float* stat /*[2][R]*/, size_t R, int D, float eps);
// Backward in two launches: dx (+ add, the gradient arriving over a residual connection around
// the LayerNorm; may be NULL) and per-block partials of dgamma / dbeta into ws; then
// Ggamma / Gbeta += the partials (may run on another stream once the first launch is done).
void layernorm_bwd_bf16(hipStream_t st, const bf16_t* g, const bf16_t* x, const float* stat,
                        const float* gamma, const bf16_t* add, bf16_t* dx, void* ws, size_t R, int D);
void layernorm_bwd_params_bf16(hipStream_t st, const void* ws, float* Ggamma, float* Gbeta, size_t R, int D);
int layernorm_bwd_parts(size_t R);  // number of [2][D] partial rows the backward kernel writes

// ---- self-attention core on packed qkv [B][S][3D] (head size 64, S % 32 == 0, S <= 256):
// o [B][S][D], lse [B][H][S]
size_t mha_bf16_ws_bytes(int B, int S, int D, int heads);
void attention_fwd_bf16(hipStream_t st, const bf16_t* qkv, bf16_t* o, float* lse, int B, int S, int D,
                        int heads);
// `dsum` is scratch of mha_bf16_ws_bytes() bytes
void attention_bwd_bf16(hipStream_t st, const bf16_t* qkv, const bf16_t* o, const bf16_t* d_o,
                        const float* lse, bf16_t* dqkv, float* dsum, int B, int S, int D, int heads);

// bf16 <-> fp32 conversion of flat buffers
void f32_to_bf16(hipStream_t st, const float* src, bf16_t* dst, size_t n);

}  // namespace ast
