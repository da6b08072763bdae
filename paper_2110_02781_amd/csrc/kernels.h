// Host-side launch interface of the HIP kernels.  All functions enqueue work on
// `st` and return immediately; none allocates.  `dt` selects the storage type
// of activations / activation gradients / working weights (0 = float,
// 1 = bfloat16); statistics, weight gradients and accumulators are fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace ftp {

// Optional per-launch timing (diagnostics for benchmarks): when tracing is on, a
// KScope brackets one kernel launch with two HIP events on the launch stream and
// records the kernel family, the bytes the launch must move at least (each operand
// once) and its floating-point operations.
struct KScope {
  KScope(hipStream_t st, const char* name, double alg_bytes, double flops, long d0 = -1, long d1 = -1, long d2 = -1);
  ~KScope();
  void route(const char* name);      // which kernel of the family took it (a literal)
  int slot;
  hipStream_t st;
};

// A launcher that finds its own launch plan outside what its kernel was written for skips the launch and says so here;
// the stage call that enqueued it returns an error (launch_plan_failure_take returns the text once, or nullptr).
void launch_plan_failed(const char* what);
const char* launch_plan_failure_take();

struct HView {  // same layout as the device-side View
  const void* z;
  const float* scale;
  const float* shift;
  int act;
};

// BatchNorm statistics that have been reduced to partial[P][2][C] but not finalised yet
struct BnPending {
  const float* partial;
  int P;
  size_t M;
  const float* gamma;
  const float* beta;
  float *mean, *invstd, *scale, *shift, *run_mean, *run_var;
};

// a BatchNorm backward still to be done: gradient dA of the activated output `out`
struct BnBwdIn {
  const void* dA;
  HView out;
  const float *gamma, *mean, *invstd;
  float *g_gamma, *g_beta;
};

// n / d as a multiplication, for n * d < 2^32 (a 32-bit division is some 25 instructions, a 64-bit one more than 100)
struct FastDiv {
  uint32_t d, mul;
  static FastDiv of(int d) { return FastDiv{(uint32_t)d, d > 1 ? (uint32_t)((0x100000000ull + (uint32_t)d - 1) / (uint32_t)d) : 0u}; }
#ifdef __HIPCC__
  __device__ __forceinline__ uint32_t div(uint32_t n) const { return d == 1 ? n : __umulhi(n, mul); }
#endif
};

struct ConvGeom {
  int N, Hin, Win, Cin, Hout, Wout, Cout, kh, kw, stride, ph, pw;
};

// Launch shape for kernels that walk a [M][C] tensor by rows, 8 channels per thread.
struct RowTile {
  int W;                  // column groups handled by one block
  int R;                  // rows handled per block iteration
  int nslab;              // grid.y
  size_t rows_per_block;
  int P;                  // grid.x = number of row chunks = number of partials
};
RowTile make_rowtile(size_t M, int C, int max_partials);
enum { kMaxPartials = 512 };
// row-streaming BatchNorm reductions: more, shorter blocks (occupancy); each block covers >= kBnMinRows rows so
// the partials stay small next to the tensor
enum { kBnPartials = 512, kBnMinRows = 32 };

// ---- BatchNorm ---------------------------------------------------------------
// partial[P][2][C] <- per-chunk sums of z and z*z
void bn_stats(int dt, hipStream_t st, const void* z, size_t M, int C, float* partial, int* P_out);
// mean/invstd/scale/shift (each [C]) from the partials; updates running stats
void bn_finalize(hipStream_t st, const float* partial, int P, size_t M, int C, const float* gamma,
                 const float* beta, float* mean, float* invstd, float* scale, float* shift,
                 float* run_mean, float* run_var, float eps, float momentum);
// partial[P][2][C] <- sums of dY and dY*z with dY = dA * act'(scale*z+shift)
void bn_bwd_reduce(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C,
                   const float* scale, const float* shift, int act, float* partial, int* P_out);
// g_gamma += dgamma, g_beta += dbeta; coef[3][C] for dz = k1*dY + k2*z + k3
void bn_bwd_finalize(hipStream_t st, const float* partial, int P, size_t M, int C, const float* gamma,
                     const float* mean, const float* invstd, float* g_gamma, float* g_beta, float* coef);
// dz (may alias dA) = k1*dA*act'(y) + k2*z + k3
void bn_bwd_apply(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C,
                  const float* scale, const float* shift, int act, const float* coef, void* dz);
// the three steps above in one launch for short tensors (bn_bwd_small_ok); dz must not alias dA
int bn_bwd_small_ok(size_t M, int C);
void bn_bwd_small(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C, const float* scale,
                  const float* shift, int act, const float* gamma, const float* mean, const float* invstd,
                  float* g_gamma, float* g_beta, void* dz);
// the last two steps in one launch (bn_finish_ok): from P partial sums, no coef; sums: partial, P, M, gamma, mean, invstd
int bn_finish_ok(size_t M, int C, int P);
int bn_left_sums_ok(size_t M, int C, int P);
void bn_bwd_finish_apply(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C, const float* scale, const float* shift, int act,
                         const BnPending& sums, float* g_gamma, float* g_beta, void* dz);
// the same for forward (bn_finish_ok): finishes the pending statistics of z and writes act(scale*z+shift) (+ res)
void bn_finish_apply(int dt, hipStream_t st, const BnPending& pend, const void* z, size_t M, int C, int act, float eps, float momentum,
                     const void* res, void* out);
// out = act(scale*z+shift) (+ res)
void bn_apply(int dt, hipStream_t st, HView in, size_t M, int C, const void* res, void* out);

// finalize the pending statistics of z and write act(scale*z+shift) (+ res), one launch, short tensors
int bn_finalize_apply_small_ok(size_t M, int C);
void bn_finalize_apply_small(int dt, hipStream_t st, const BnPending& pend, const void* z, size_t M, int C, int act, float eps,
                             float momentum, const void* res, void* out);

// ---- pooling, loss, optimiser ---------------------------------------------------
// pend.partial != nullptr: the BatchNorm of the input is still partial sums; finished here
// open != nullptr (in is a view): also, for each image, how many positions of a channel the activation passes and the sum of the raw values there,
// open[N][2][C]: all that the backward sums of that BatchNorm need of the tensor
void gap_fwd(int dt, hipStream_t st, HView in, const BnPending& pend, float eps, float momentum, int N, int HW, int C, void* out,
             float* open = nullptr);
// sums != nullptr: also the partial sums [*P_out][2][C] that bn_bwd_reduce would compute for that BatchNorm + activation
void gap_bwd(int dt, hipStream_t st, const void* dOut, int N, int HW, int C, void* dIn, const float* open = nullptr, float* sums = nullptr,
             int* P_out = nullptr);
// dlogits[B][classes] = (softmax - onehot)/B, mean loss into *loss; row_loss: B floats of scratch, rounded up to a multiple of 8.  arrived: kCeCounters zeros, zeros again afterwards,
// for one call at a time; without them what softmax_ce_arrives takes a launch more
int softmax_ce_arrives(int B, int classes);
enum { kCeRows = 8, kCeGroups = 32, kCeLine = 16, kCeCounters = (kCeGroups + 1) * kCeLine };     // rows of a block, groups of blocks
void softmax_ce(int dt, hipStream_t st, const void* logits, const int32_t* labels, int B, int classes,
                float* row_loss, void* dlogits, float* loss, unsigned* arrived);
// g_bias[j] += sum_b d[b][j]
void bias_grad(int dt, hipStream_t st, const void* d, int B, int Nout, float* g_bias);
// the whole backward of a fully connected layer d[B][N] -> in[B][K] in one launch: g_w += d^T in, g_b += column sums of d,
// and unless dIn is nullptr dIn = d W.  HW >= 1: the layer stands behind an average over HW positions and dIn [B][HW][K] is
// that one's input gradient, and with sums != nullptr the layer also leaves them as gap_bwd does.  fc_bwd_ok: few enough rows that the tiles' walks over them stay short.
int fc_bwd_ok(int B, int N, int K);
int fc_bwd_gap_ok(int B, int HW, int K);
void fc_bwd(int dt, hipStream_t st, const void* d, HView in, const void* w, int B, int N, int K, float* g_w, float* g_b, void* dIn, int HW,
            const float* open = nullptr, float* sums = nullptr, int* P_out = nullptr);
// g += wd*w; v = mu*v+g; w -= lr*v; g = 0; optional working copy w_lp (bfloat16)
void sgd_update(hipStream_t st, float* w, float* g, float* v, void* w_lp, size_t n, float lr, float mu,
                float wd);
// weight aggregation: w = mean of up to 8 stashed versions (fp32, summed in order), optional bfloat16 copy
struct AggSources { const float* p[8]; };
void aggregate_weights(hipStream_t st, float* w, void* w_lp, const AggSources& src, int n, size_t count);
void fill_zero(hipStream_t st, void* p, size_t bytes);
void calibration_copy(hipStream_t st, const void* src, void* dst, size_t bytes);
void f32_to_storage(int dt, hipStream_t st, const float* src, void* dst, size_t n);

// ---- generic small dense convolution (stem 3x3, conv1d) ---------------------------
int conv_direct_supported(const ConvGeom& g);
void conv_direct_fwd(int dt, hipStream_t st, HView in, const void* w, const ConvGeom& g, void* z);
// many pixels, few taps: im2col + GEMM with the BatchNorm statistics in its epilogue (conv_direct_gemm_ok);
// im2col: conv_direct_im2col_elems(g) elements, wpad: conv_direct_gemm_wpad_elems(g) elements of scratch
int conv_direct_gemm_ok(const ConvGeom& g);
size_t conv_direct_gemm_wpad_elems(const ConvGeom& g);
void conv_direct_fwd_gemm(int dt, hipStream_t st, HView in, const void* w, const ConvGeom& g, void* im2col, void* wpad, void* z,
                          float* stats, int* P_out);
void conv_direct_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* dIn);
// stride-1 data gradient as im2col(dz) x flipped weights on the GEMM (conv_direct_dgrad_gemm_ok); scratch sizes in elements
int conv_direct_dgrad_gemm_ok(const ConvGeom& g);
size_t conv_direct_dgrad_gemm_im2col_elems(const ConvGeom& g);
size_t conv_direct_dgrad_gemm_w_elems(const ConvGeom& g);
void conv_direct_dgrad_gemm(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* im2col, void* wscratch,
                            void* dIn);
// g_w[Cout][kh][kw][Cin] += dW; im2col: scratch of conv_direct_im2col_elems(g) activation elements
size_t conv_direct_wgrad_ws(const ConvGeom& g);  // floats of workspace needed
size_t conv_direct_im2col_elems(const ConvGeom& g);
// patches_ready: im2col already holds this layer's patch matrix (left there by conv_direct_fwd_gemm on the same input)
void conv_direct_wgrad(int dt, hipStream_t st, const void* dz, HView in, const ConvGeom& g, void* im2col, float* ws,
                       float* g_w, bool patches_ready = false);
// g[(j % C) * stride_c + (j / C) * stride_q] += sum_p ws[p * QC + j]; columns j % C >= valid_c skipped (-1: none)
void reduce_partials(hipStream_t st, const float* ws, int P, size_t QC, int C, size_t stride_q, size_t stride_c,
                     float* g, int valid_c = -1);
// the same for several tensors in one launch (P >= 1 each)
struct ReduceJob { const float* ws; float* g; int P, QC, C, stride_q, stride_c, valid_c; };
void reduce_group(hipStream_t st, const ReduceJob* jobs, int n);

// ---- 1 x kw convolutions, stride 1, same length, at most 64 channels (conv1d_ok): implicit GEMMs, no scratch but ws ----
int conv1d_ok(const ConvGeom& g);
int conv1d_small_ok(const ConvGeom& g);     // few rows
int conv1d_bwd_sums_ok(int dt, const ConvGeom& g);      // conv1d_bwd_small with sums pays
// of the layers that are conv1d_ok: whether they run here or through patch matrices.  first: no data gradient is wanted, alone: the
// stage's only convolution, forks: the stage runs weight gradients on a second stream
int conv1d_pays(int dt, const ConvGeom& g, bool first, bool alone, bool forks);
// pend.partial != nullptr (few rows, or conv1d_finish_ok for its P): the BatchNorm of the input is still partial sums, not those in `stats`; finished here
int conv1d_finish_ok(const ConvGeom& g, int P);
void conv1d_fwd(int dt, hipStream_t st, HView in, const BnPending& pend, float eps, float momentum, const void* w, const ConvGeom& g, void* z,
                float* stats, int* P_out);
// sums != nullptr (prev is a view): also the partial sums bn_bwd_reduce would compute for the BatchNorm + activation `prev`
void conv1d_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* dIn, HView prev, float* sums, int* P_out);
size_t conv1d_wgrad_ws(const ConvGeom& g);
// partial sums, if any, are left in ws and appended to `left`
void conv1d_wgrad(int dt, hipStream_t st, const void* dz, HView in, const ConvGeom& g, float* ws, float* g_w, std::vector<ReduceJob>* left);
// few rows (conv1d_small_ok): weight and data gradient (dIn != nullptr) in one launch.  sums != nullptr (conv1d_bwd_sums_ok): the BatchNorm backward of the layer's own
// output `own` is still to be done, from those sums; dz is not looked at.  left != nullptr (`in` is a view): also the partial sums
// bn_bwd_reduce would compute for the BatchNorm + activation `in`, [*P_out][2][Cin]
void conv1d_bwd_small(int dt, hipStream_t st, const void* dz, const void* w, HView in, const ConvGeom& g, float* g_w, void* dIn,
                      const BnPending* sums = nullptr, const BnBwdIn* own = nullptr, float* left = nullptr, int* P_out = nullptr);

// ---- depthwise 3x3 ----------------------------------------------------------------
// stats != nullptr (only if dw_fwd_stats_ok): the kernel also writes the BatchNorm partial sums [*P_out][2][C] of z
int dw_fwd_stats_ok(int dt, const ConvGeom& g);
void dw_fwd(int dt, hipStream_t st, HView in, const void* w, const ConvGeom& g, void* z, float* stats = nullptr,
            int* P_out = nullptr);
// convolution + BatchNorm statistics + finalize in one launch for short tensors (dw_fwd_bn_small_ok)
int dw_fwd_bn_small_ok(const ConvGeom& g);
// pend.partial != nullptr: the BatchNorm of the input is still partial sums (pw_fwd's epilogue); the kernel
// finishes it for the channels it owns (writes the per-channel vectors and the running statistics)
void dw_fwd_bn_small(int dt, hipStream_t st, HView in, const BnPending& pend, const void* w, const ConvGeom& g, const float* gamma,
                     const float* beta, float* mean, float* invstd, float* scale, float* shift, float* run_mean,
                     float* run_var, float eps, float momentum, void* z);
// depthwise dgrad + wgrad + the BatchNorm backward of the layer in front, one launch, short tensors
// (dw_bwd_small_ok): dz_prev = gradient of the raw output of the convolution that feeds `in`
int dw_bwd_small_ok(const ConvGeom& g);
// after the BatchNorm backward of the depthwise layer's own output
// (bo: gradient of the activated output, the output view, its BatchNorm vectors and gradient slots)
void dw_bwd_small(int dt, hipStream_t st, const BnBwdIn& bo, const void* w, HView in, const ConvGeom& g,
                  const float* gamma, const float* mean, const float* invstd, float* g_w, float* g_gamma, float* g_beta,
                  void* dz_prev);
// The whole backward of a layer in one pass (dIn == nullptr: without the data gradient): from the gradient dA of its activated output own (whose BatchNorm backward it does on the way, from
// coef or, sums_in != nullptr, from up to 256 partial sums; dIn must not be dA) or, own == nullptr, from dz = dA.  Leaves the weight gradient's
// partial sums gw_part[P][9][C] (dw_bwd_ws floats) and, sums != nullptr (in is a view), those of the BatchNorm + activation in front [P][2][C]
int dw_bwd_partials(int dt, const ConvGeom& g);      // P
size_t dw_bwd_ws(int dt, const ConvGeom& g);
void dw_bwd(int dt, hipStream_t st, const void* dA, const HView* own, const BnPending* sums_in, const float* coef, float* g_gamma, float* g_beta, const void* w,
            const ConvGeom& g, void* dIn, HView in, float* sums, float* gw_part);

// ---- pointwise / fully connected GEMMs (MFMA) ---------------------------------------
// Z[M][N] = A'[M][K] * W[N][K]^T (+ bias[N]); when stats != nullptr also writes the per-column
// partial sums stats[P][2][N] of the stored Z and Z*Z (same layout as bn_stats), P into *P_out
void pw_fwd(int dt, hipStream_t st, HView a, const void* w, const float* bias, size_t M, int K, int N,
            void* z, float* stats, int* P_out);
// Short layers whose operand is formed on the way in (pw_pro_ok: R = reduction extent).  Forward: x is a raw output whose BatchNorm is
// still partial sums; A = act(scale * x + shift) (+ x_add), also written to x_out.
int pw_pro_ok(int dt, size_t M, int R, int ncols);
void pw_fwd_pro(int dt, hipStream_t st, const BnPending& pend, HView x, const void* x_add, void* x_out, float eps, float momentum, const void* w,
                size_t M, int K, int N, void* z, float* stats, int* P_out);
// dA[M][K] = dZ[M][N] * W[N][K] (+ res[M][K]).  sums != nullptr (only if pw_dgrad_sums_ok): also the partial sums [*P_out][2][K] that
// bn_bwd_reduce would compute for the BatchNorm of the view `of` (of.scale == nullptr: without activation, of.z its raw output), dA being the gradient of its output
int pw_dgrad_sums_ok(int dt, size_t M, int K, int N, HView of);
void pw_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const void* res, size_t M, int K,
              int N, void* dA, HView of = HView{}, float* sums = nullptr, int* P_out = nullptr);
// the consumer of such sums (pw_pro_ok): BatchNorm backward of bn (no activation), dz written, then dA = dz * W
void pw_dgrad_pro(int dt, hipStream_t st, const BnPending& sums, const BnBwdIn& bn, void* dz, const void* w, size_t M, int K, int N, void* dA);
// g_w[N][K] += dZ[M][N]^T * A'[M][K]
size_t pw_wgrad_ws(size_t M, int K, int N);
// K_out >= 0: g_w is [N][K_out] and the last K - K_out columns of A are zero padding
void pw_wgrad(int dt, hipStream_t st, const void* dz, HView a, size_t M, int K, int N, float* ws,
              float* g_w, int K_out = -1);

// Weight gradients of several pointwise layers together (K and N multiples of 8); short ones are added to g_w at once, the
// others leave partial sums in their ws (pw_wgrad_group_ws floats of its own) and append what is left to sum
struct PwWgradJob { const void* dz; HView a; size_t M; int K, N; float* ws; float* g_w; };
// share: how many layers such a group holds when it is complete, those the transposing kernel takes and the others (the same numbers
// in both calls)
struct PwShare { int tr, other; };
size_t pw_wgrad_group_ws(int dt, size_t M, int K, int N, PwShare share);
void pw_wgrad_group(int dt, hipStream_t st, const PwWgradJob* jobs, int n, PwShare share, std::vector<ReduceJob>* left);

// Narrow-to-wide pointwise layer (K inputs, N >= 2K outputs, bfloat16, input stored activated), whole backward behind
// the BatchNorm reductions in one pass: dz = k1*dA*act'(out) + k2*z + k3 formed per row tile on chip,
// dIn = dz * W (+ res), g_w += dz^T * A.  coef: [3][N] from bn_bwd_finalize.  ws: pw_bwd_fused_ws(M, K, N) floats.
// The kernel's partial weight gradients are summed on st_sum; if that is not st, ev_sum orders the sum behind the kernel.
// left != nullptr: they are not summed here, the sum is appended there.
int pw_bwd_fused_ok(int dt, size_t M, int K, int N, HView a);
size_t pw_bwd_fused_ws(size_t M, int K, int N);
void pw_bwd_fused(hipStream_t st, const void* dA, HView out, const float* coef, const void* w, const void* a_in,
                  const void* res, size_t M, int K, int N, float* ws, float* g_w, void* dIn, hipStream_t st_sum,
                  hipEvent_t ev_sum, std::vector<ReduceJob>* left = nullptr, const void* z_in = nullptr, float* sums = nullptr);
// z_in: also the backward sums of the BatchNorm without activation whose raw output z_in is ([pw_bwd_fused_sums][2][K], which is not 0)
int pw_bwd_fused_sums(size_t M, int K, int N);


// Pointwise layers on double-buffered LDS tiles: forward (A' * W^T, BatchNorm partial sums as pw_fwd leaves them) and data gradient (dZ * W (+ res)).
// Which layers, in either type: deep_plan in k_gemm_deep.hip.  pw_fwd and pw_dgrad dispatch to them.  R = reduction extent, NC = output columns.
// They return the tile for the trace.
int pw_deep_ok(int dt, size_t M, int R, int NC, bool dgrad);
const char* pw_fwd_deep(int dt, hipStream_t st, HView a, const void* w, size_t M, int K, int N, void* z, float* stats, int* P_out);
const char* pw_dgrad_deep(int dt, hipStream_t st, const void* dz, const void* w, const void* res, size_t M, int K, int N, void* dA, HView of, float* sums, int* P_out);
int pw_deep_sums_ok(int dt, size_t M, int R, int NC);
// the weight gradient for bfloat16 layers with more than 2048 rows: operands staged untransposed, transposed on the
// way out of LDS (pw_wgrad dispatches to it; ws: pw_wgrad_tr_ws floats)
int pw_wgrad_tr_ok(int dt, size_t M, int K, int N);
size_t pw_wgrad_tr_ws(size_t M, int K, int N, int share = 1);
void pw_wgrad_tr(hipStream_t st, const void* dz, HView a, size_t M, int K, int N, float* ws, float* g_w, int K_out);
void pw_wgrad_tr_group(hipStream_t st, const PwWgradJob* jobs, int n, int share, std::vector<ReduceJob>* left);   // skips what is not pw_wgrad_tr_ok

// wgrad (g_w +=) then dgrad (dA =) of one layer on one stream; one launch for short problems
void pw_bwd(int dt, hipStream_t st, const void* dz, const void* w, const void* res, HView a, size_t M, int K, int N,
            float* ws, float* g_w, void* dA);

}  // namespace ftp
