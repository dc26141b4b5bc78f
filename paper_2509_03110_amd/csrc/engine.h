// Internal declarations shared by the host engine and the kernel launchers.
// Nothing here is part of the public boundary (include/lsam.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/lsam.h"
#include "b32s.h"
#include "langevin.h"

namespace lsam {

constexpr int kMaxK = LSAM_MAX_REPLICAS;

// Small per-replica tables handed to kernels by value.
struct ReplicaScalars {
  float v[kMaxK];
};
struct DueList {
  int32_t n;
  int32_t idx[kMaxK];
};

// Message that lsam_last_error() returns on the calling thread (copied).
void set_last_error(const char* msg);

// One coordinate of the sampler step (Algorithm 2, asynchronous sampling step, driven by
// momentum SGD): G = g + lam (x - y); v <- mu v + G; x <- x - lr (G + mu v) [Nesterov] or
// x - lr v [heavy ball], plus the Langevin term xi (0 without noise); S <- S + x.  The one
// definition both the streaming kernel and the fused GEMM epilogue use, so that they round alike.
__device__ __forceinline__ void sampler_step(float g, float y, float lam, float lr, float mu,
                                             int nesterov, float xi, float& x, float& v, float& S) {
  const float G = g + lam * (x - y);
  const float vn = mu * v + G;
  const float xn = (nesterov ? x - lr * (G + mu * vn) : x - lr * vn) + xi;
  v = vn;
  x = xn;
  S += xn;
}

// One coordinate of the ascent step x~ = x + scale g, scale = rho / (||g|| + gamma) (Formulation,
// first-order solution of the inner maximisation); shared by the streaming kernel and the
// GEMM epilogue for the same reason.
__device__ __forceinline__ float ascent_point(float x, float scale, float g) {
  return __builtin_fmaf(scale, g, x);
}

// Parameters that the next kernels read back: streamed past the caches when all replicas
// together are far larger than they are (K d floats; measured at 3.2 GB: +5-9 % for the two
// kernels with streaming stores), left in them when they fit (at 67 MB the following forward
// GEMMs and the next descent find them there: -2 % per step).
constexpr int64_t kCacheResidentBytes = 96ll << 20;

// ---- streaming kernels (update path) ---------------------------------------------------

// Sum of squares, pass 1: per (replica, block) partial sums in double.
// g: [K] rows of `n` floats with row stride `g_stride` (any n, stride and 4-byte alignment);
// partials: [K, nblk] doubles.  `restart`: as in launch_norm_finish, which then gets none.
void launch_sumsq_partials(const float* g, int64_t g_stride, int64_t n, int K, double* partials,
                           int nblk, hipStream_t s, int32_t* restart = nullptr);
// How many partial sums a row of n values is cut into: pieces of 4096 values, up to
// kProloguePartials of them, while that leaves a piece at most 16384 values (four rounds of four
// loads per lane), otherwise pieces of 16384 and more, at most kMaxPartials.
// Pieces of 65536 left most of the chip idle in short rows: 18 us for 4 x 270410 values.
constexpr int kProloguePartials = 128;
constexpr int kMaxPartials = 1024;
int sumsq_blocks(int64_t n);
// Pass 2: norms[k] = sqrt(sum_{b<nblk} partials[k * partials_stride + b]); scale[k] = rho / (norm + gamma).
// If loss_rows != nullptr also reduces loss_rows [K,B] to loss_out[k] = mean (both passes of
// the tree are fixed-order, so the result is run-to-run deterministic).
// `restart` (may be null): the per-replica marks described at launch_center; this kernel, which
// runs once per step before anything touches the iterate sums, counts every mark down by one.
void launch_norm_finish(const double* partials, int nblk, int64_t partials_stride, int K, float rho, float gamma,
                        float* norms, float* scale, const float* loss_rows, int B,
                        float* loss_out, hipStream_t s, int32_t* restart = nullptr);
// x~ = x + scale[k] * g.  Writes fp32 (xt_f32), or, if xt_bf16 is non-null, the bf16 operand
// copy of the weight matrices in the blocked layout described by `map` (replica stride
// `shadow_stride` elements).
// `sums` (fp32, may be null): the norm is still in at most kProloguePartials partial sums per replica, and
// this launch does launch_norm_finish's work, whose arguments it holds, as well.
struct NormSums {
  const double* partials; int n; int64_t pstride;
  float rho, gamma;
  float* norms; float* scale;
  const float* loss_rows; int B; float* loss_out;
  int32_t* restart;
};
void launch_perturb(const float* x, const float* g, int64_t g_stride, const float* scale,
                    float* xt_f32, uint16_t* xt_bf16, const ShadowMap* map, int64_t shadow_stride,
                    int64_t stride, int64_t n, int K, hipStream_t s, const NormSums* sums = nullptr);
// Descent + coupling for all K replicas, y read once per index:
//   G = g + lam[k] (x - y); v = mu v + G; x -= lr (G + mu v) [nesterov] | lr v; S += x.
// Also refreshes the bf16 operand copy of the weight matrices if `shadow` is non-null, and adds
// the Langevin noise described by `noise` (null: none) to the new x.  A replica whose mark in
// `restart` (may be null) is 1 starts its sum afresh: S = x, without reading S.
void launch_descent(float* x, const float* g, int64_t g_stride, float* v, float* S,
                    const float* y, uint16_t* shadow, const ShadowMap* map, int64_t shadow_stride,
                    int64_t stride, int64_t n, int K, const ReplicaScalars& lam, float lr, float mu,
                    int nesterov, const NoiseMap* noise, hipStream_t s, const int32_t* restart = nullptr);
// A step on gradients that are both at hand, in two launches: the norm of g1, then one pass for x~ =
// x + scale g1 (xt null: not wanted) and the descent on g2.  A third adds the norm's partial sums up
// where the descent does not.  n, the strides of g1 and g2 and their 4-byte alignment are the caller's;
// x, v, S, xt, y as in launch_descent, xt over none of the others.  nblk: sumsq_blocks(n).
struct AscentPass {
  const float* g1 = nullptr; int64_t g1_stride = 0;
  float* xt = nullptr;
  double* partials = nullptr; int nblk = 0;
  float rho = 0.f, gamma = 0.f;
  float* norms = nullptr; float* scale = nullptr;
  bool finish_in_descent() const { return xt != nullptr && nblk <= kProloguePartials; }
};
void launch_raw_norm(int64_t n, int K, hipStream_t s, int32_t* restart, const AscentPass& up);
void launch_raw_descent(float* x, const float* g2, int64_t g_stride, float* v, float* S, const float* y,
                        int64_t stride, int64_t n, int K, const ReplicaScalars& lam, float lr, float mu,
                        int nesterov, const NoiseMap* noise, hipStream_t s, const int32_t* restart, const AscentPass& up);
// dst[c * dst_stride + i] = (1/K) sum_k src[k * src_stride + i] for c < copies, i < n; the K
// terms are added in replica order.  dst may be src (each index is read in full before it is
// written).
void launch_grad_mean(const float* src, int64_t src_stride, float* dst, int64_t dst_stride,
                      int64_t n, int K, int copies, hipStream_t s);
// Center update over the due replicas (Algorithm 2, synchronous optimization step).  The sums of
// the due replicas start again from zero afterwards.  Without `restart` the kernel writes the
// zeros.  With it (K words of device memory, zero at first) it writes none: it sets the mark of
// every due replica to 2, which means "this sum reads as zero, its memory is stale"; the next
// step's launch_norm_finish makes that a 1, which tells that step's sampler kernels to start the
// sum from x alone instead of reading it, and the step after makes it 0 again.  All of it is
// data on the device, so a captured step replays correctly.  Saves writing and reading back
// 4 bytes per parameter of every replica served.
void launch_center(float* S, float* y, float* gprev, int64_t stride, int64_t n,
                   const DueList& due, float inv_m, float beta, float lr_center, int has_prev,
                   hipStream_t s, int32_t* restart = nullptr);
// dst[k, :] = src[:] for k < K (fp32).
void launch_broadcast(const float* src, float* dst, int64_t stride, int64_t n, int K, hipStream_t s);
// Rebuilds the bf16 operand copy of K replicas from their fp32 parameters.
void launch_shadow_refresh(const float* x, uint16_t* shadow, const ShadowMap& map, int64_t stride,
                           int64_t shadow_stride, int64_t n, int K, hipStream_t s);
// Row-major bf16 [K][rows][cols] -> blocked layout, one matrix per replica (dst pre-zeroed
// padding is left untouched).
void launch_rowmajor_to_b32s(const uint16_t* src, uint16_t* dst, int rows, int cols, int K,
                             hipStream_t s);
void launch_fill_zero(void* p, size_t bytes, hipStream_t s);
// Row-padded copy: dst[r, 0:cols] = src[r, 0:cols], rows of `elem` bytes-sized elements.
void launch_pad_rows(const void* src, void* dst, int64_t rows, int cols, int ld_dst, int elem,
                     hipStream_t s);

// ---- model kernels ------------------------------------------------------------------------

enum GemmEpilogue { EPI_BIAS = 0, EPI_BIAS_RELU = 1, EPI_MASK = 2, EPI_PLAIN = 3 };

// A product whose split contraction is not added up yet: n > 1 pieces [rows of all replicas][ld], `stride`
// floats apart, to which bias and ReLU have still to be applied; n = 1: the product is complete.
struct SplitResult {
  const float* p; int64_t stride; int ld, n;
  const float* bias; int64_t strideBias;
};

// C[k][m, n] = sum_kk A(k; m, kk) * B(k; n, kk), batched over replicas k.
// An operand is "k-major" when kk is its contiguous index (row pitch ld along m resp. n),
// otherwise "m-major" (kk selects the row, m resp. n is contiguous).
struct GemmDesc {
  const void* A; int64_t strideA; int ldA; int a_kmajor;
  const void* B; int64_t strideB; int ldB; int b_kmajor;
  void* C; int64_t strideC; int ldC;
  int M, N, Kd, batch;
  int in_bf16;        // operands bf16 (else fp32)
  int out_bf16;       // output bf16 (else fp32)
  int epilogue;       // GemmEpilogue
  const float* bias; int64_t strideBias;          // EPI_BIAS*: bias[n]
  const float* bias_dir; const float* bias_scale; // if set: bias[n] + bias_scale[k] * bias_dir[n]
  const void* mask; int64_t strideMask; int ldMask; // EPI_MASK: keep where mask[m,n] > 0 (operand dtype)
  const uint8_t* keep;                              // launch_splitk_reduce: the mask as bits (ConvGemmDesc)
  float* splitk_ws; size_t splitk_bytes;            // scratch for split-K partial sums (may be null)
  // bf16 tensors in the blocked layout (b32s.h): column blocks of the stored A, B, bf16 C, mask;
  // strideA/B/C/Mask then count elements of one replica's stored matrix and ld* are unused
  int b32s; int cbA, cbB, cbC, cbMask;
  // If set (fp32 results only): every workgroup that writes results also writes the sum of
  // their squares, in double, to sumsq[k * sumsq_stride + slot], slot = 0 .. slots-1 inside a
  // replica; `slots` comes back through launch_gemm.  Fixed summation order.
  double* sumsq; int64_t sumsq_stride;
  // fp32 only.  unfold = 1: A is not stored as [M][Kd]; it is the unfolded image of a 3x3
  // convolution (stride 1, zero rim 1) read straight from the image A points to, [M pixels]
  // [unfold_C] with M a multiple of unfold_H * unfold_W, Kd = 9 * unfold_C, both operands
  // k-major.  unfold = 2: the same for B as an m-major operand: B points to the image
  // [Kd pixels][unfold_C], N = 9 * unfold_C, both operands m-major.  unfold_C must be a
  // multiple of 32; ldA resp. ldB is then ignored apart from the alignment checks.
  int unfold, unfold_C, unfold_H, unfold_W;
  // fp32 operands only: round both operands to bfloat16 on their way into the matrix unit
  // (v_mfma_f32_32x32x16_bf16, fp32 accumulate); memory traffic and results stay fp32.
  int bf16_math;
  // If set (bf16 operands, fp32 result, EPI_PLAIN): the result, a weight gradient at the
  // perturbed point, is not stored.  The epilogue takes the sampler step on it instead
  // (Algorithm 2, asynchronous sampling step, with Nesterov or heavy-ball momentum), element
  // (m, n) of replica k living at offset k * strideC + m * ldC + n of x, v and S and at
  // m * ldC + n of y:  G = C + lam[k] (x - y);  v = mu v + G;  x -= lr (G + mu v)  [or lr v];
  // S += x;  and bf16(x) goes to the blocked operand copy `shadow` (replica stride
  // shadow_stride elements, cbShadow column blocks).  C is ignored.
  const struct SamplerFusion* fuse;
  // If set (same kind of launch, a weight gradient of the first pass recomputed once its norm
  // is known): the result is not stored either; the epilogue writes the operand copy of the
  // perturbed weights, bf16(x + scale[k] * C), x addressed like the result.
  const struct AscentFusion* ascend;
  // If set (same kind of launch, `sumsq` given): only the sums of squares are written.
  int sumsq_only;
  const float* add; int64_t strideAdd; int ldAdd;   // launch_splitk_reduce only: ConvGemmDesc::add
  // If set (fp32 operands, EPI_BIAS_RELU): a split contraction is left in pieces, described here.
  SplitResult* parts;
};
struct AscentFusion {
  const float* x; const float* scale;
  uint16_t* shadow; int64_t shadow_stride; int cbShadow;
};
struct SamplerFusion {
  float* x; float* v; float* S; const float* y;
  uint16_t* shadow; int64_t shadow_stride; int cbShadow;
  ReplicaScalars lam;
  float lr, mu;
  int nesterov;
  const int32_t* restart;     // marks of launch_center (may be null)
};
// 0 ok, <0 unsupported shape; *sumsq_slots (if non-null) = slots written per replica
int launch_gemm(const GemmDesc& d, hipStream_t s, int* sumsq_slots = nullptr);
// Upper bound of the slots any launch of an [M, N] result can use.
int gemm_sumsq_capacity(int M, int N);
size_t gemm_splitk_bytes(const GemmDesc& d);          // scratch this GEMM would like (0: none)
// bf16 fast path (direct-to-LDS ring); returns 1 when the shape is left to the generic kernel.
int launch_gemm_bf16(const GemmDesc& d, int tile_override, hipStream_t s, int* sumsq_slots);

// A dense layer for the launches that take several at once (n <= LSAM_MAX_LAYERS): dz [B][out] and act
// [B][in] of K replicas, replicas one stored size apart; bf16 in the blocked layout, or fp32 with rows
// padded to 8 values (launch_dense_gradients).
struct DenseLayer {
  const void* dz; const void* act;
  int out, in, ldw;
  int64_t w_off, b_off;       // of W_l and b_l inside a replica's parameters
  int64_t shadow_off;         // of its operand copy inside a replica's
};
// Squared norms of the weight gradients dZ^T A, which are not stored, as partial sums: returns the
// slots written per replica, or -1.
int launch_gram_norms(const DenseLayer* layers, int n, int K, int B, double* sumsq, int64_t sumsq_stride, hipStream_t s);
int gram_slots(int n, int K, int B);
// The products dZ^T A of all layers with the step `f`, or else the ascent `a`, in their epilogues
// (GemmDesc::fuse, ::ascend; pointers to the whole vectors, replicas `stride` apart), for a state that
// stays in the caches.  0, or -1.
int launch_fused_group(const DenseLayer* layers, int n, int K, int B, int64_t stride, const SamplerFusion* f,
                       const AscentFusion* a, hipStream_t s);
// fp32 (bf16_math: operands of the products rounded): the weight and bias gradients of n layers and (may be null) of the narrow head, into g.  Returns the
// sum-of-squares slots written per replica (at most gemm_sumsq_capacity of every product, one per 64 biases,
// head_sumsq_slots), or -1.
// The products that dense_gradients_alone marks are left out, not so their biases: those take a launch_gemm each.
void dense_gradients_alone(const DenseLayer* layers, int n, int K, int B, int bf16_math, bool* alone);
int launch_dense_gradients(const DenseLayer* layers, int n, const DenseLayer* head, int K, int B, float* g, int64_t strideG,
                           double* sumsq, int64_t sumsq_stride, int bf16_math, hipStream_t s);
// Column sums of every layer's dz into g; slots as launch_bias_grad's.  `step` (may be null): the biases
// take their sampler step as well (pointers to the whole vectors, like g).
int launch_bias_grads_blocked(const DenseLayer* layers, int n, int K, int B, float* g, int64_t strideG, double* sumsq,
                              int64_t sumsq_stride, const SamplerFusion* step, hipStream_t s);

// Adds the `splits` partial results of a split contraction ([M][ldP] per replica, split_stride
// floats apart) in a fixed order and finishes them as `d` says (C, epilogue, bias, mask, sumsq;
// its operands are ignored).  Returns the sum-of-squares slots written per replica.
int launch_splitk_reduce(const GemmDesc& d, const float* partial, int splits, int64_t split_stride, int ldP, hipStream_t s);

// The same for several products at once: partial sums of weight gradients that nothing waits for before the pass's end
// (EPI_PLAIN; each in workspace of its own) are listed and added up in one launch.
struct ReduceList {
  static constexpr int kMax = 40;
  struct Job {
    const float* partial; int64_t split_stride;
    float* C; int64_t strideC;
    int M, N, ldC, ldP, splits;
    int first, slot;          // first of its workgroups; of its sum-of-squares slots
  };
  Job job[kMax];
  int n = 0, blocks = 0;
  double* sumsq = nullptr; int64_t sumsq_stride = 0;    // slots of replica k at sumsq + k sumsq_stride (null: none wanted)
};
int launch_reduce_list(const ReduceList& list, int K, hipStream_t s);

// ---- convolution products on plane tensors (kernels_conv_gemm.hip) ------------------------
// A plane tensor holds every fp32 value as np bfloat16 values, `plane` elements apart: np = 1 the
// rounded value, np = 3 an exact split.
struct PlaneImage {
  const uint16_t* p; int64_t stride, plane;      // replica and plane strides (elements, multiples of 8)
  int C, oH, oW, sH, sW, st;                     // images [sH][sW][C], C % 8 == 0; output pixels [oH][oW]
  int nu, nv, du0, dv0;                          // tap (a, c) of nu x nv reads pixel (st i + du0 + a, st j + dv0 + c)
};
// wgrad = 0: C[m, n] = sum over (tap, c) of image(pixel m, tap, c) * other[n][(tap, c)], M output
//   pixels, Kd = taps * C, other [N][ld] with zeros from Kd to the next multiple of 32.
// wgrad = 1: C[m, (tap, c)] = sum over output pixels k of other[k][m] * image(k, tap, c), other
//   [Kd][M] (ld = M), N = taps * C.
// Epilogues as in GemmDesc (bias, mask: fp32).
struct ConvGemmDesc {
  int np, wgrad;
  PlaneImage image;
  const uint16_t* other; int64_t other_stride, other_plane; int ld;
  float* C; int64_t strideC; int ldC;
  int M, N, Kd, batch;
  int epilogue;
  const float* bias; int64_t strideBias;
  const float* mask; int64_t strideMask; int ldMask;
  // In place of mask if set: the same as bits, a byte to four columns (value (m, n) is kept if bit n % 4 of byte
  // (m ldMask + n) / 4 is set; strideMask still counts values).
  const uint8_t* keep;
  float* splitk_ws; size_t splitk_bytes;
  double* sumsq; int64_t sumsq_stride;
  // If set: [M][ldAdd] of every replica, added to the results behind the bias and in front of ReLU or mask (with
  // out_step 2 its pixels are those of even row and column, [oH][oW]).  Not for weight gradients.
  const float* add = nullptr; int64_t strideAdd = 0; int ldAdd = 0;
  // 2: the input gradient of a stride-2 convolution.  The image is the output gradient [oH][oW], C and
  // the mask are images of [2 oH][2 oW].  An input pixel meets the taps of its row's and its
  // column's parity only: four classes of pixels, each a convolution of 1, 2, 2 or 4 taps whose filters
  // follow each other in `other` (see FilterBank); M counts one class's pixels, Kd all nine taps.
  int out_step = 1;
  // Column sums of the results C (dense, ldC = N) as a normalisation wants them, by chunks of rows, where the launch can take
  // them (a contraction cut over workgroups cannot; `made` says).  1: statistics, as launch_bn_stats leaves them in its scratch;
  // 2: as launch_bn_backward_partials does, the results being dY, with Z and its statistics.
  int sums = 0;
  // If set (weight gradients): partial sums are listed there instead of added up, the sum-of-squares slots from list_slot on.
  ReduceList* list = nullptr; int list_slot = 0;
  float* sum_part = nullptr; const float* sum_z = nullptr; const float* sum_stats = nullptr;
};
// Chunks of `rows` rows each (the last one fewer), or none (chunks 0).
struct ChunkSums {
  int chunks = 0, rows = 0;
};
int launch_conv_gemm(const ConvGemmDesc& d, hipStream_t s, int* sumsq_slots = nullptr, ChunkSums* made = nullptr);   // 0, or -1: not served
int conv_gemm_sum_chunks(int64_t rows);       // room for the chunks of any launch that writes `rows` rows a replica
size_t conv_gemm_splitk_bytes(const ConvGemmDesc& d);
// Planes of n consecutive floats (n % 4 == 0).
int launch_split_planes(const float* src, uint16_t* dst, int np, int64_t plane, int64_t n, hipStream_t s);
// One filter bank [rows][cols] (row pitch ldw) at `src` of every replica's parameters as the plane
// products read it, `dst` elements into every plane.  taps = 0: [K][rows][ldp], zeros from cols on
// (cols, ldw, ldp multiples of 4); taps = 1 or 9: mirrored and transposed, `cols` counting one tap's
// columns: [K][cols][ldp], value (c, tap * rows + o) = W[o][(taps - 1 - tap) * cols + c], zeros beyond.
// With stride 2 the nine taps come class by class instead, as the input pixels of even / odd row and
// column read them: (1,1) | (1,2) (1,0) | (2,1) (0,1) | (2,2) (2,0) (0,2) (0,0).
struct FilterBank {
  int64_t src, dst;
  int32_t rows, cols, ldw, ldp, taps;
  int32_t first;            // first workgroup that serves the bank
  int32_t stride;
};
int filter_bank_blocks(const FilterBank& f);
// All n banks of the table (device memory) for K replicas; blocks: workgroups of all of them.
int launch_filters(const float* params, int64_t strideParams, const FilterBank* banks, int n, int blocks, uint16_t* dst,
                   int np, int64_t plane, int K, hipStream_t s);

// Softmax cross-entropy, forward and backward.  logits [K,B,ld] fp32; labels [K,B];
// dz = (softmax - onehot)/B: fp32 [K,B,ld_dz] row-major with zeros in the padded columns, or
// (dz_bf16) bf16 in the blocked layout, ld_dz then being one replica's stored size in elements;
// loss_rows [K,B] = lse - logit[label] (may be null).
void launch_softmax_ce(const float* logits, int ld, const int32_t* labels, void* dz, int64_t ld_dz,
                       int dz_bf16, float* loss_rows, int K, int B, int C, hipStream_t s);
// db[k][n] = sum_b dz[k][b][n], dz fp32 of row pitch ld.
// If sumsq is non-null, workgroup j of replica k also writes the sum of squares of its 64
// results to sumsq[k * sumsq_stride + j]; returns the number of such slots per replica.
int launch_bias_grad(const float* dz, int64_t ld, float* db, int64_t strideDb, int K, int B, int N, double* sumsq,
                     int64_t sumsq_stride, hipStream_t s);
// dgamma and dbeta (at gam_off and bet_off of each replica's gradient) from the chunk sums that
// launch_bn_backward_partials left; returns the sum-of-squares slots written per replica.
int launch_norm_param_grads(const float* part, float* grad, int64_t strideGrad, int64_t gam_off, int64_t bet_off,
                            int K, int chunks, int C, double* sumsq, int64_t sumsq_stride, hipStream_t s);

// Narrow classifier head in fp32 (head_fits: few classes, an input row that fits LDS, a
// moderate batch): forward of the last layer, loss, dZ and the masked dX in one kernel (A: the
// layer's input [K,B,ld], a ReLU output, ld = `in` rounded up to 8; W, bias: the layer's
// parameters inside each replica, replica stride strideW, row pitch ld; dz [K,B,ld_dz] gets
// the padded dZ; dA [K,B,ld], if non-null, dZ W where A > 0; returns <0 if the launch could
// not be set up); its weight and bias gradient is launch_dense_gradients' (head_sumsq_slots(in) partial sums).
// `parts` (may be null): A is still in pieces, and is completed and written by the head's kernel.
bool head_fits(int B, int C, int in);
int head_sumsq_slots(int in);
int launch_head_forward_backward(float* A, const SplitResult* parts, const float* W, const float* bias, int64_t strideW,
                                 const int32_t* labels, float* dz, int ld_dz, float* loss_rows,
                                 float* dA, int K, int B, int C, int in, hipStream_t s);

// 3x3 convolution support (fp32, tensors [K][B][H][W][C], C contiguous).  All return 0, or -1
// when the shape does not fit the kernel (pitches and channel counts that are not multiples
// of 4 where stated).
// col[k][(b,i,j)][(u,v,c)] = X[k][b][i+u-1][j+v-1][c], zero outside the image and in the
// padding columns 9C..ld-1 (ld % 4 == 0; any C): np = 0 as floats, otherwise as np bfloat16 planes
// `plane` elements apart.
// `stride` 1 or 2: the image is [stride H][stride W][C] and col row (b,i,j) holds the window
// around pixel (stride i, stride j); H x W is the convolution's output.
int launch_unfold3x3(const float* X, int64_t strideX, void* col, int np, int64_t plane, int ld, int K,
                     int B, int H, int W, int C, int stride, hipStream_t s);
// dX[k][b][i][j][c] = sum_{u,v} dcol[k][(b,i-u+1,j-v+1)][(u,v,c)], taps added in (u,v) order,
// set to zero where mask (same shape as dX, may be null) is not positive.  C % 4 == 0.
int launch_fold3x3(const float* dcol, int64_t strideCol, int ld, float* dX, const float* mask,
                   int64_t strideX, int K, int B, int H, int W, int C, int stride, hipStream_t s);
// A first convolution layer with C = 1..3 input channels and a multiple of 8 output channels up to 256
// (first_conv_fits) has kernels of its own that gather the image straight into the MFMA
// operands.  Forward: out[k][p][o] = b[o] + conv, rectified if `relu`, parameters taken from
// params + k * strideParams at w_off (row pitch ldw) and b_off.  Weight gradient: dW and db
// into grad + k * strideParams at the same offsets, through `partial`
// ([K][first_conv_chunks(rows, Cout, K)][Cout][32] floats of scratch), plus, if sumsq is non-null, the
// sums of their squares in sumsq[k * sumsq_stride + slot]; returns the slots written per
// replica (Cout / 2), or -1.  `round`: both operands of every product are rounded to bfloat16
// first.  `skip_bias`: the weight-gradient kernels leave db alone (with rounded operands they
// would sum rounded values, the caller then takes the column sums of dout instead; below a
// batch normalisation the bias gradient is zero).
bool first_conv_fits(int C, int Cout, int64_t rows, int K, int round);
int first_conv_chunks(int64_t rows, int Cout, int K);
// `sums` (may be null): the statistics of the results by chunks of rows, as ConvGemmDesc's sums = 1.  `norm` (z null: dout is
// the gradient of the convolution's output): dout is dY of the normalisation behind it, and its gradient is formed from these.
struct FirstNorm {
  const float* z = nullptr; const float* stats = nullptr; const float* params = nullptr; const float* grad = nullptr;
  long long gam_off = 0, bet_off = 0;
};
int launch_first_conv_forward(const float* X, const float* params, int64_t strideParams, int64_t w_off,
                              int64_t b_off, int ldw, float* out, int relu, int round, int K,
                              int64_t rows, int H, int W, int C, int Cout, float* sums, ChunkSums* made, hipStream_t s);
int launch_first_conv_wgrad(const float* X, const float* dout, const FirstNorm& norm, float* partial, float* grad,
                            int64_t strideParams, int64_t w_off, int64_t b_off, int ldw, int round,
                            int skip_bias, int K, int64_t rows, int H, int W, int C, int Cout,
                            double* sumsq, int64_t sumsq_stride, hipStream_t s);
// Where a kernel also writes its fp32 result as plane tensors (np = 0: it does not), and, if `keep` is set, which
// values are positive: bit r of a byte for value r of four, the mask of the gradient that comes back.
struct PlaneOut {
  uint16_t* p = nullptr; int np = 0; int64_t plane = 0;
  uint8_t* keep = nullptr;
};

// Training-mode batch normalisation of K matrices Z [rows][C] (C % 4 == 0, C <= 1024), per
// replica and column over the rows.  Forward (launch_bn_stats, then launch_bn_apply or the same joined with the pool that
// follows): stats[k][0][c] = mean, stats[k][1][c] =
// 1/sqrt(biased variance + eps); out = relu(gamma Xh + beta), Xh = (Z - mean) stats[1], gamma
// and beta read from params + k * strideParams at gam_off / bet_off.  `scratch`: 2 * K *
// bn_chunks(rows, C, K) * C floats.  Backward: launch_bn_backward_partials leaves chunk sums
// part[k][chunk][0..C) = sum dY Xh and [C..2C) = sum dY (returns the chunk count; launch_norm_param_grads
// over them gives dgamma and dbeta); launch_bn_backward_apply then writes
// dZ = gamma stats[1] (dY - dbeta/rows - Xh dgamma/rows) [+ add] to `dZ`, which may be dY itself or Z
// (or null: planes only), dgamma and dbeta read from grad + k * strideParams at the same offsets.  -1: shape not supported.

// Where that pass finds dY: floats g [K][rows][C], or (HW > 0) the gradient g [image][ld] of a global average over HW
// positions; set to zero where `keep` (bits of a word; may be null) is clear.
struct GradSource {
  const float* g; const uint8_t* keep;
  int HW, ld;
};

// Shortcut of a residual block (He et al., CIFAR variant, parameter-free): the block input
// src [K][B][step H][step W][Cs] (replica stride `stride` floats) enters the block output
// [B][H][W][C] as src[b][step i][step j][c] for c < Cs and 0 for the channels beyond.  Cs % 4 == 0.
// A projection shortcut instead (that paper's 1x1 convolution with batch normalisation): `pz`
// [K][rows][C] is the 1x1 convolution's output, `pstats` its statistics (launch_bn_stats), and
// gamma_p, beta_p sit at pgam_off, pbet_off of each replica's parameters; pz null: no projection.
struct ShortcutDesc {
  const float* src; int64_t stride;
  int H, W, Cs, step;
  const float* pz = nullptr; const float* pstats = nullptr;
  int64_t pgam_off = 0, pbet_off = 0;
};
// stats[k] = (mean, 1/sqrt(var + eps)) per channel of Z [K][rows][C].  `have`: the
// chunks of the scratch that the product that wrote Z has left there; none: they are taken from Z.
int launch_bn_stats(const float* Z, float* scratch, const ChunkSums& have, float* stats, int K, int64_t rows, int C, float eps,
                    hipStream_t s);
// dst[i] += src[i] for i < n (n % 4 == 0; both 16-byte aligned, not overlapping).
int launch_add_into(float* dst, const float* src, int64_t n, hipStream_t s);
// dst[img][i][j][c] = src[img][2 i][2 j][c] for `images` images [2H][2W][C] (C % 4 == 0).
int launch_subsample2(const float* src, float* dst, int64_t images, int H, int W, int C, hipStream_t s);
int bn_chunks(int64_t rows, int C, int K);
// `shortcut` (may be null): added to the normalised output before the ReLU.  `out` may be null: planes (and bits) only.
int launch_bn_apply(const float* Z, const float* stats, const float* params, int64_t strideParams, int64_t gam_off, int64_t bet_off,
                    float* out, int K, int64_t rows, int C, const ShortcutDesc* shortcut, const PlaneOut& planes, hipStream_t s);
// Followed by the 2x2 max-pool of [H][W] images (`images` a replica): P (may be null) and the planes are the pooled image's;
// for the backward pass zmax (Z at each window's first maximum), arg (which one, two bits a channel, a byte a word) and
// planes.keep.
int launch_bn_pool(const float* Z, const float* stats, const float* params, int64_t strideParams, int64_t gam_off, int64_t bet_off,
                   float* P, float* zmax, uint8_t* arg, int K, int64_t images, int H, int W, int C, const PlaneOut& planes,
                   hipStream_t s);
// Followed by global average pooling as launch_avgpool does it; keep: the image's bits.
int launch_bn_avgpool(const float* Z, const float* stats, const float* params, int64_t strideParams, int64_t gam_off,
                      int64_t bet_off, float* P, int K, int64_t images, int HW, int C, int ldp, const ShortcutDesc* shortcut,
                      uint8_t* keep, hipStream_t s);
// dIn (shape of d.src) += the gradient dY [K][rows][C] of the block output, through the shortcut,
// kept only where mask (shape of dIn, the ReLU output the block read; may be null) is positive.
int launch_shortcut_backward(const float* dY, float* dIn, const float* mask, const ShortcutDesc& d, int K,
                             int64_t rows, int C, hipStream_t s);
// Global average pooling over `images` images [HW][C] into rows of pitch ldp, and its backward
// pass fused with the ReLU mask of the image (as floats or, in its place, as bits; both null: no mask).
int launch_avgpool(const float* A, float* P, int64_t images, int HW, int C, int ldp, hipStream_t s);
int launch_avgpool_backward(const float* dP, const float* mask, const uint8_t* keep, float* dA, int64_t images, int HW, int C,
                            int ldp, hipStream_t s);
int launch_bn_backward_partials(const float* Z, const GradSource& dY, const float* stats, float* part, int K,
                                int64_t rows, int C, hipStream_t s);
void launch_bn_backward_apply(const float* Z, const GradSource& dY, float* dZ, const float* stats,
                              const float* params, const float* grad, int64_t strideParams,
                              int64_t gam_off, int64_t bet_off, int K, int64_t rows, int C, const float* add,
                              const PlaneOut& planes, hipStream_t s);
// The latter behind launch_bn_pool, from the pooled image's gradient dP (the former takes zmax and dP with their bits).
void launch_bn_pool_backward(const float* Z, const float* dP, const uint8_t* arg, const uint8_t* keep, float* dZ, const float* stats,
                             const float* params, const float* grad, int64_t strideParams, int64_t gam_off, int64_t bet_off, int K,
                             int64_t images, int H, int W, int C, const PlaneOut& planes, hipStream_t s);
// Wt[k][c][(u,v,o)] = W[k][o][(2-u,2-v,c)] for K filter banks W [Cout][3][3][Cin] (row pitch ldw,
// replica stride strideW); Wt is dense, [K][Cin][9 Cout].  Cout must be a multiple of 32.
void launch_flip_filters(const float* W, int64_t strideW, int ldw, float* Wt, int K, int Cout, int Cin,
                         hipStream_t s);
// Column sums of K contiguous [rows][N] matrices, first stage: partial[k][chunk][n] = sum of
// the rows of chunk `chunk` (colsum_chunks(rows, N, K) chunks of equal height, the last one ragged);
// returns the chunk count, -1 if N is not a multiple of 4 in 4..1024.  launch_bias_grad over
// the partials finishes the sum.  keep: bits, as in GradSource.
int colsum_chunks(int64_t rows, int N, int K);
int launch_colsum_partials(const float* A, const uint8_t* keep, int64_t rows, int N, int K, float* partial, hipStream_t s);
// 2x2/stride-2 max-pool over `images` contiguous [H][W][C] images A, ReLU outputs (P may be null: planes only), and the
// backward pass of ReLU-then-pool: dA (may be null) and its planes = dP at the first maximum of each window if it is positive,
// else 0; arg and planes.keep of the forward pass say where (see launch_bn_pool).  C % 4 == 0, H and W even.
int launch_maxpool2(const float* A, float* P, uint8_t* arg, int64_t images, int H, int W, int C, const PlaneOut& planes, hipStream_t s);
int launch_maxpool2_backward(const float* dP, const uint8_t* arg, const uint8_t* keep, float* dA, int64_t images, int H,
                             int W, int C, const PlaneOut& planes, hipStream_t s);

// Measured ceilings: device copy (GB/s, read + written) between the halves of `scratch`, and
// MFMA-only loops (TFLOP/s, bf16 32x32x16 and fp32 32x32x2).  Blocks until done; 0 or -1.
int probe_peaks(void* scratch, size_t bytes, hipStream_t s, double* copy_gbs, double* bf16_tflops,
                double* f32_tflops);

}  // namespace lsam
