// Host engine behind include/lsam.h: configuration checks, workspace carve-up, the integer
// communication schedule, and the kernel sequence of one LSAM step / one center update.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "engine.h"

namespace lsam {
namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return fail(LSAM_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

inline int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// ---- communication schedule (integers only) -------------------------------------------------
// Period generator: s_{j+1} = A s_j + C mod 2^64, draw_j = (s_{j+1} >> 33) mod range + min.
// Replica i is due when its local count reaches its period: the trigger of Algorithm 2's
// synchronous optimization step (total local iterations reaching a multiple of n tau), taken
// per replica so that periods may differ; with equal periods every replica is due at the same
// tick and the two coincide.
class Schedule {
 public:
  void init(const lsam_config& c) {
    K_ = c.K;
    lo_ = c.tau_min;
    hi_ = c.tau_max;
    redraw_ = c.sched_mode == LSAM_SCHED_REDRAW;
    state_ = c.sched_seed;
    explicit_ = c.tau != nullptr;
    tau_.resize(K_);
    count_.assign(K_, 0);
    t_y_ = 0;
    for (int i = 0; i < K_; ++i) tau_[i] = explicit_ ? c.tau[i] : draw();
  }
  int32_t draw() {
    state_ = state_ * 6364136223846793005ULL + 1442695040888963407ULL;
    const uint64_t range = (uint64_t)(hi_ - lo_ + 1);
    return (int32_t)((state_ >> 33) % range) + lo_;
  }
  void tick() {
    for (int i = 0; i < K_; ++i) ++count_[i];
  }
  DueList due() const {
    DueList d;
    d.n = 0;
    for (int i = 0; i < K_; ++i)
      if (count_[i] >= tau_[i]) d.idx[d.n++] = i;
    return d;
  }
  int64_t samples(const DueList& d) const {
    int64_t m = 0;
    for (int j = 0; j < d.n; ++j) m += count_[d.idx[j]];
    return m;
  }
  void served(const DueList& d) {
    for (int j = 0; j < d.n; ++j) {
      count_[d.idx[j]] = 0;
      if (redraw_ && !explicit_) tau_[d.idx[j]] = draw();
    }
    ++t_y_;
  }
  const std::vector<int32_t>& tau() const { return tau_; }
  const std::vector<int32_t>& count() const { return count_; }
  int64_t t_y() const { return t_y_; }
  uint64_t generator_state() const { return state_; }
  // Overwrites counts, periods in force, the generator state and the sync count (resume).
  bool restore(const int64_t* count, const int64_t* tau, uint64_t state, int64_t t_y) {
    if (t_y < 0) return false;
    for (int i = 0; i < K_; ++i)
      if (count[i] < 0 || count[i] > INT32_MAX || tau[i] < 1 || tau[i] > INT32_MAX) return false;
    for (int i = 0; i < K_; ++i) {
      count_[i] = (int32_t)count[i];
      tau_[i] = (int32_t)tau[i];
    }
    state_ = state;
    t_y_ = t_y;
    return true;
  }

 private:
  int K_ = 0, lo_ = 1, hi_ = 1;
  bool redraw_ = false, explicit_ = false;
  uint64_t state_ = 0;
  std::vector<int32_t> tau_, count_;
  int64_t t_y_ = 0;
};

// ---- layout -----------------------------------------------------------------------------------
struct Layer {
  int in, out;          // true extents
  int ldw;              // row pitch of W in the padded layout (floats)
  int64_t w_off, b_off; // offsets inside one replica of the padded layout (floats)
  int64_t w_flat, b_flat; // offsets inside the public flat layout
  bool bn = false;        // batch-normalised convolution: gamma and beta follow the bias
  int64_t gam_off = 0, bet_off = 0, gam_flat = 0, bet_flat = 0;
  // projection shortcut closed by this convolution: W_p [out][proj_in] (row pitch proj_in, a
  // multiple of 8), b_p, gamma_p, beta_p follow the layer's own parameters
  bool proj = false;
  int proj_in = 0;
  int64_t pw_off = 0, pb_off = 0, pgam_off = 0, pbet_off = 0;
};

// One parameter group as the copies between the flat and the padded layout and the noise
// generator see it: `rows` rows of `cols` values, row pitch `ld` in the padded layout.
struct Piece {
  int64_t off, flat;
  int rows, cols, ld;
  int code;               // 8 * layer + {0 W, 1 b, 2 gamma, 3 beta, 4..7 the projection's four}
};

// One 3x3 convolution layer: image [H][W][Cin] -> [H][W][Cout] (-> [H/2][W/2][Cout] if pooled).
struct ConvLayer {
  int H, W, Cin, Cout, pool;   // H x W: the convolution's output image (before the pool)
  int stride;          // 1 or 2: the layer reads an image of [stride H][stride W][Cin]
  bool skip;           // closes a residual block: the input of the layer below is added before the ReLU
  int skip_C, skip_step;   // channels of that block input; 2 if the block halved the image, else 1
  bool proj;           // that shortcut is a projection (1x1 convolution + batch normalisation)
  size_t psub, pz, pstats; // gradient of its input pixels [K][rows][skip_C], its convolution
                           // output [K][rows][Cout] (later: that output's gradient), its statistics
  int64_t rows;        // B H W: rows of the unfolded image and of the layer's output
  int ldc;             // pitch of the unfolded image, 9 Cin rounded up to 8
  // Which products serve the layer.  `fast`: the bf16 matrix units on plane tensors
  // (kernels_conv_gemm.hip); otherwise the fp32-storage GEMM (small layers and, in fp32 arithmetic, channel
  // counts that are no multiples of 8; plane_products_pay).
  // Both can read an unfolded image straight from the image: `direct_in` for the layer's input
  // (forward and dW), `direct_dx` for its output gradient (dX, with the mirrored filters, `wt` for
  // the fp32-storage GEMM).  Otherwise the unfolded image (`col`, planes if fast) resp. its gradient
  // (the shared `dcol`) is stored.
  // `first`: layer 0 with 1..3 input channels runs its forward pass and its weight gradient
  // in kernels of their own (no unfolded image at all).
  bool fast, direct_in, direct_dx, first;
  // `keep`: bits of the layer's positive outputs (behind its pool), where they are written by the normalisation or the pool and
  // all that asks for the sign reads them.  `floats`: something reads the outputs themselves in front of the pool, `pooled_floats`
  // behind it (a product on plane tensors does not).
  bool has_keep, floats, pooled_floats;
  // Normalisation and what follows it in one kernel: the 2x2 pool, or the global average, whose gradient is then never
  // written for every position either (unless a shortcut hands it on).
  bool bn_pool, bn_gap;
  size_t keep, arg, zmax;  // pools: which value of a window is its first maximum; with bn_pool that value's Z
  size_t first_partial;   // scratch of the first layer's weight gradient
  bool bn;                // batch-normalised: `z` keeps the convolution's output, `stats` the
  size_t z, stats;        // per-channel mean and 1/sqrt(var + eps) of each replica
  size_t col, out, pooled, dout, dpooled, wt;   // workspace offsets ([K] contiguous replicas each)
  // plane tensors (kernels_conv_gemm.hip): the image this layer reads, kept from the forward pass
  // for the weight gradient; `plane_elems` elements per plane (all replicas).  Present if the layer
  // itself (fast and direct_in) or the fast projection of the block it opens reads it.
  bool planes;
  bool planes_above;   // they are written by the kernel that writes the image (normalisation or pool of the layer below)
  size_t xp;
  int64_t plane_elems;
  // filters as the plane products read them, elements into a plane of lo.wp: forward and dX, the
  // same of the projection
  int64_t wf, wx, pwf, pwx;
  // partial sums of its weight gradient and of its projection's, which wait for the end of the pass (0 bytes: there are none, or
  // they are added up at once and lie where all others do)
  size_t wpart, wpart_bytes, pwpart, pwpart_bytes;
  int in_H, in_W;      // that image
};

struct Layout {
  int K = 0, L = 0, B = 0;
  int n_conv = 0;              // layers 0..n_conv-1 are convolutions
  bool preact = false;         // residual blocks sum un-normalised convolution outputs (wide residual networks)
  std::vector<ConvLayer> conv;
  size_t dcol = 0;             // gradient of an unfolded image (largest layer that needs one)
  int np = 0;                  // planes per plane tensor: 1 with bf16 products, 3 (exact split) without
  size_t wp = 0, dzp = 0;      // planes of all filters, and of one layer's output gradient (reused layer by layer)
  int64_t wp_elems = 0, dzp_elems = 0;   // per plane
  std::vector<FilterBank> banks;         // the filters in wp; their device copy and the workgroups they take
  size_t banks_at = 0;
  int bank_blocks = 0;
  size_t restart = 0;         // K marks: which iterate sums read as zero / start afresh (launch_center)
  int gap_hw = 0;              // > 0: global average pooling over that many positions feeds the dense layers
  size_t gap_out = 0, gap_grad = 0;   // [K][B][ld] pooled vector and its gradient
  size_t colsum = 0;           // first-stage column sums of the bias gradients and normalisations
  size_t pcolsum = 0;          // the same of a projection's normalisation, which are made before the block's own are used
  bool bf16 = false, raw = false;
  bool bf16_math = false;      // convolutional model with bf16 matrix products on fp32 tensors
  int64_t d = 0, d_pad = 0;
  std::vector<Layer> layers;
  std::vector<Piece> pieces; // every parameter group, in the order of the flat layout
  size_t noise_segs = 0;     // device copy of the noise generator's table (Langevin sampler only)
  std::vector<int> ld;       // activation pitches ld[0..L]
  bool need_a0 = false;
  int nblk = 1;
  // byte offsets into the workspace
  size_t gmean = 0;   // raw-vector mode, data-parallel baseline: the averaged gradient [d_pad]
  size_t x = 0, g = 0, v = 0, S = 0, xt = 0, y = 0, gprev = 0, partials = 0, norms = 0, scale = 0,
         loss_rows = 0, loss = 0, logits = 0, a0 = 0, splitk = 0, splitk_bytes = 0, total = 0;
  std::vector<size_t> act, dz;  // act[l] for l = 1..L-1, dz[l] for l = 1..L (index l)
  // bf16 mode: every bf16 tensor is stored in the blocked layout (b32s.h)
  std::vector<int64_t> shadow_off;   // offset of W_l's operand copy inside a replica's copy
  int64_t shadow_stride = 0;         // elements of one replica's operand copy
  ShadowMap map{};
  size_t es() const { return bf16 ? 2 : 4; }
  // elements of one replica's stored [B][dims] activation-like matrix
  int64_t act_elems(int width, int pitch) const {
    return bf16 ? b32s_size(B, width) : (int64_t)B * pitch;
  }
};

int check_config(const lsam_config* c) {
  if (!c) return fail(LSAM_EINVAL, "config is NULL");
  if (c->K < 1 || c->K > LSAM_MAX_REPLICAS)
    return fail(LSAM_EINVAL, "K=%d outside 1..%d", c->K, LSAM_MAX_REPLICAS);
  if (c->n_layers < 0 || c->n_layers > LSAM_MAX_LAYERS)
    return fail(LSAM_EINVAL, "n_layers=%d outside 0..%d", c->n_layers, LSAM_MAX_LAYERS);
  if (c->n_layers == 0) {
    if (c->d_raw < 1) return fail(LSAM_EINVAL, "raw-vector mode needs d_raw >= 1");
  } else {
    if (!c->dims) return fail(LSAM_EINVAL, "dims is NULL");
    for (int l = 0; l <= c->n_layers; ++l)
      if (c->dims[l] < 1) return fail(LSAM_EINVAL, "dims[%d]=%d must be >= 1", l, c->dims[l]);
    if (c->batch < 1) return fail(LSAM_EINVAL, "batch must be >= 1");
    if ((int64_t)c->K * c->batch > (1 << 24)) return fail(LSAM_EINVAL, "K*batch too large");
    if (c->gemm_dtype != LSAM_GEMM_FP32 && c->gemm_dtype != LSAM_GEMM_BF16)
      return fail(LSAM_EINVAL, "gemm_dtype must be 0 (fp32) or 1 (bf16)");
    if (c->n_conv < 0 || c->n_conv >= c->n_layers)
      return fail(LSAM_EINVAL, "n_conv=%d must leave at least one dense layer of %d", c->n_conv,
                  c->n_layers);
    if (c->n_conv == 0 && c->bn_mask) return fail(LSAM_EINVAL, "bn_mask needs convolution layers");
    if (c->n_conv == 0 && (c->stride_mask || c->skip_mask || c->proj_mask || c->global_avg_pool || c->preact))
      return fail(LSAM_EINVAL, "stride_mask, skip_mask, proj_mask, global_avg_pool and preact need convolution layers");
    if (c->n_conv > 0) {
      if (c->img_h < 1 || c->img_w < 1) return fail(LSAM_EINVAL, "img_h, img_w must be >= 1");
      if (c->bn_mask >> c->n_conv) return fail(LSAM_EINVAL, "bn_mask names a layer that is no convolution");
      if (c->bn_mask && !(c->bn_eps > 0.f)) return fail(LSAM_EINVAL, "bn_eps must be > 0");
      if ((c->stride_mask >> c->n_conv) || (c->skip_mask >> c->n_conv) || (c->pool_mask >> c->n_conv))
        return fail(LSAM_EINVAL, "stride_mask, skip_mask or pool_mask names a layer that is no convolution");
      if (c->proj_mask & ~c->skip_mask)
        return fail(LSAM_EINVAL, "proj_mask names a layer that closes no residual block");
      if (c->global_avg_pool != 0 && c->global_avg_pool != 1)
        return fail(LSAM_EINVAL, "global_avg_pool must be 0 or 1");
      if (c->preact != 0 && c->preact != 1) return fail(LSAM_EINVAL, "preact must be 0 or 1");
      if (c->preact && c->bn_mask != ((1ull << c->n_conv) - 1))
        return fail(LSAM_EINVAL, "pre-activation blocks need every convolution batch-normalised");
      int64_t h = c->img_h, w = c->img_w;
      int64_t in_h[LSAM_MAX_LAYERS + 1], in_w[LSAM_MAX_LAYERS + 1];   // image each convolution reads
      for (int l = 0; l < c->n_conv; ++l) {
        in_h[l] = h; in_w[l] = w;
        if (c->dims[l + 1] % 8)
          return fail(LSAM_EINVAL, "dims[%d]=%d: convolution outputs must be multiples of 8", l + 1,
                      c->dims[l + 1]);
        if ((c->stride_mask >> l) & 1u) {
          if (h % 2 || w % 2)
            return fail(LSAM_EINVAL, "convolution %d: stride 2 needs even image sides (%lldx%lld)", l,
                        (long long)h, (long long)w);
          h /= 2;
          w /= 2;
        }
        if ((c->skip_mask >> l) & 1u) {
          if (l < 2) return fail(LSAM_EINVAL, "convolution %d: a residual block needs two convolutions below its closing one", l);
          if (!((c->bn_mask >> l) & 1u))
            return fail(LSAM_EINVAL, "convolution %d: the closing convolution of a residual block must be batch-normalised", l);
          if (((c->pool_mask >> (l - 1)) & 1u) || ((c->pool_mask >> (l - 2)) & 1u))
            return fail(LSAM_EINVAL, "convolution %d: no pool may sit inside a residual block or in front of it", l);
          const int64_t sh = in_h[l - 1], sw = in_w[l - 1];
          const bool proj = ((c->proj_mask >> l) & 1u) != 0;
          // (a pre-activation block without projection adds two sums of the same shape)
          if (!((sh == h && sw == w) || (sh == 2 * h && sw == 2 * w)) ||
              (!proj && c->dims[l - 1] > c->dims[l + 1]) || c->dims[l - 1] % (proj ? 8 : 4) ||
              (c->preact && !proj && (sh != h || sw != w || c->dims[l - 1] != c->dims[l + 1])))
            return fail(LSAM_EINVAL, "convolution %d: the block input (%lldx%lldx%d) does not fit the block output (%lldx%lldx%d)",
                        l, (long long)sh, (long long)sw, c->dims[l - 1], (long long)h, (long long)w, c->dims[l + 1]);
        }
        // one replica's unfolded image is a GEMM operand addressed with 32-bit byte offsets
        const int64_t widest = std::max<int64_t>(round_up(9 * (int64_t)c->dims[l], 8), c->dims[l + 1]);
        if ((int64_t)c->batch * h * w * widest * 4 >= 0x7FFFFFF0LL)
          return fail(LSAM_EINVAL, "convolution %d: batch * image * channels too large", l);
        if ((c->pool_mask >> l) & 1u) {
          if (h % 2 || w % 2)
            return fail(LSAM_EINVAL, "convolution %d: pooling needs even image sides (%lldx%lld)", l,
                        (long long)h, (long long)w);
          h /= 2;
          w /= 2;
        }
      }
      if (!c->global_avg_pool && h * w * c->dims[c->n_conv] > (1 << 24))
        return fail(LSAM_EINVAL, "flattened image too wide for the dense layers");
    }
  }
  if (!(c->rho >= 0.f) || !(c->gamma >= 0.f)) return fail(LSAM_EINVAL, "rho, gamma must be >= 0");
  if (!(c->lr > 0.f) && c->lambda_abs < 0.f)
    return fail(LSAM_EINVAL, "lr must be > 0 when lambda is derived as lambda0/(lr*tau)");
  if (!(c->lr >= 0.f)) return fail(LSAM_EINVAL, "lr must be >= 0");
  if (!(c->momentum >= 0.f && c->momentum < 1.f))
    return fail(LSAM_EINVAL, "momentum must be in [0,1)");
  if (!std::isfinite(c->beta) || !std::isfinite(c->lr_center) || !std::isfinite(c->lambda0))
    return fail(LSAM_EINVAL, "beta, lr_center, lambda0 must be finite");
  if (c->tau) {
    for (int i = 0; i < c->K; ++i)
      if (c->tau[i] < 1) return fail(LSAM_EINVAL, "tau[%d]=%d must be >= 1", i, c->tau[i]);
  } else {
    if (c->tau_min < 1 || c->tau_max < c->tau_min)
      return fail(LSAM_EINVAL, "need 1 <= tau_min <= tau_max");
  }
  if (c->sched_mode != LSAM_SCHED_FIXED && c->sched_mode != LSAM_SCHED_REDRAW)
    return fail(LSAM_EINVAL, "sched_mode must be 0 or 1");
  if (c->algorithm != LSAM_ALG_LSAM && c->algorithm != LSAM_ALG_DATA_PARALLEL)
    return fail(LSAM_EINVAL, "algorithm must be LSAM_ALG_LSAM or LSAM_ALG_DATA_PARALLEL");
  if (!(c->noise_scale >= 0.f) || !std::isfinite(c->noise_scale))
    return fail(LSAM_EINVAL, "noise_scale must be finite and >= 0");
  return LSAM_OK;
}

size_t take(size_t& cursor, size_t bytes) {
  const size_t at = cursor;
  cursor = (size_t)round_up((int64_t)(cursor + bytes), 2048);   // whole 2 KiB blocks of the bf16 layout
  return at;
}

// Whether the plane products serve a convolution (rows: output pixels per replica).  They take a
// launch a pass for all filters, and planes of every image and gradient, and pay from about 1e8
// multiply-adds over all replicas, 3e8 with more than 32 channels (fewer, larger workgroups).
// Time of a step of three equal layers, as a fraction of the fp32-storage GEMM's: 32 channels 0.98
// at 9e6, 0.90 at 1.5e8, 0.74 at 2.4e9; 16 channels 0.93 at 2e7, 0.60 at 6e8; 64 channels 1.13 at
// 7.5e7, 0.98 at 6e8; 128 channels 0.87 at 1.2e9 (fp32 arithmetic; with bf16 products 1.0, 0.94, 0.78;
// 0.92, 0.59; 1.02, 0.90; 0.91).  One plane leaves little to gain on few, small images: 256 channels on
// 2048 pixels 0.95 in fp32, 1.07 with bf16 products, which therefore want 4096.  Channel counts that are no
// multiples of 32 have a stored unfolded image to save: from 2e7, and above 32 channels 1e8 on at least
// 4096 pixels (two equal layers, fp32 / bf16 products: 16 channels at 9e6 0.94 to 1.03 / 0.95, at 2e7 0.95 /
// 0.91; 24 at 2e7 0.95, 4e8 0.72, 2.7e9 0.40 / 0.42; 40 at 1.2e8 0.97, 2.4e8 0.84 / 0.90; 72 at 1.9e8 0.99, 3e9
// 0.50; 152 at 2.3e10 0.46; but 104 channels at 1e8 on 1024 pixels 1.16).  On fewer pixels the
// conversions weigh more (the second of two layers, fp32), unless the layer narrows to a quarter: below 5120 from 1.5e8,
// and 2.5e8 where it widens (4096 pixels: 64 to 56 channels at 1.3e8 1.04, 80 to 80 at 2.4e8 1.01, 112 to 40 at 1.7e8
// 0.98, 184 to 24 at 1.6e8 0.91, 176 to 16 at 1.3e8 0.87; 56 to 112 at 2.3e8 1.03, 40 to 184 at 2.7e8 0.96), with bf16 products
// below 6144 from 1.15e8 (48 at 1.1e8 beside a projection 1.03, 56 at 1.2e8 0.95 to 0.98, 152 to 16 at 1e8 0.94).
// In fp32 a layer of many times its input's channels, no multiple of 16, whose dX the ring computes for 8 or
// 16 columns of its tiles' 32, stays there, from 16 channels on 32768 pixels and more (6.6e4 pixels: 8 to 88 channels 0.99,
// to 104 1.06, to 184 1.26, 16 to 168 0.99, to 184 1.03, to 248 1.07; in whole 16s, by patches, 8 to 128 0.81, 16 to 128 0.77;
// 16800 pixels: 8 to 184 1.08, 16 to 184 0.91, to 248 0.93).
// A layer on the data (`dx`: whether there is an input gradient to compute) saves its own image only, and in a single
// layer of 8 or 16 channels that pays from 10240 pixels, of 24 from 8192 (fp32 / bf16 products: 16 to 24 channels on 7424
// 1.05 / 1.00, on 9216 1.01 / 1.00, on 16384 0.92; 8 to 128 on 11520 0.97; 24 to 24 on 7424 1.01 / 0.98, on 9216 0.96 / 0.95).
// The loader takes the data of a multiple of 32 channels without a stored image; planes still win with bf16 products or up
// to 16 channels of output, and beyond those in fp32 on more pixels (32 to 16 on 7168 1.02 / 0.98, on 12544 0.96 / 0.95;
// 96 to 8 on 16400 0.78 / 0.91; 128 to 16 on 7168 0.93 / 1.03, on 13312 0.85 / 0.97; 32 to 40 on 13312 1.06 / 0.98, on 16400
// 0.98 / 0.97; 64 to 48 on 9800 1.06 / 1.02; 32 to 72 on 7168 1.06 / 1.00, on 9800 0.98 / 0.99).
// Counts that are no multiples of 8 are taken with a stored unfolded image, nine times the image either way: with one
// plane that pays from 3e8.
bool plane_products_pay(int np, int K, int64_t rows, int Cin, int Cout, bool dx) {
  const double macs = (double)K * (double)rows * 9.0 * Cin * Cout;
  if (np == 1 && K * rows < 4096) return false;
  if (Cin % 8 || Cout % 8) return np == 1 && macs >= 3e8;
  // In fp32 arithmetic 24 channels beside a multiple of 32 stay with the fp32-storage GEMM.  Planes would be faster (6.6e4
  // pixels, as a fraction of its time: 24 to 32 channels 0.78, 32 to 24 0.66, 128 to 24 0.48), but lsam_layer_info has always
  // named these layers as the GEMM's, and its answers are held to that.
  if (np == 3 && std::min(Cin, Cout) == 24 && std::max(Cin, Cout) % 32 == 0) return false;
  if (np == 3 && dx && Cout % 16 && Cout > 11 * Cin && (Cin < 16 || K * rows >= 32768)) return false;
  bool stored = Cin % 32 || Cout % 32;       // on the fp32-storage GEMM
  if (!dx && Cin % 32 == 0) {
    int enough = std::max(Cin, Cout) > 32 ? 0 : np == 1 && Cout <= 16 ? 5632 : 9216;
    if (np == 3 && Cout > 16) enough = Cout < 64 ? 14336 : 9216;
    stored = stored && K * rows >= enough;
  }
  if (!dx && Cin < 32 && K * rows < (Cin > 16 ? 8192 : 10240) && macs < 3e8) return false;
  if (std::max(Cin, Cout) <= 32) return macs >= (stored ? 2e7 : 1e8);
  if (!stored || K * rows < 4096) return macs >= 3e8;
  if (Cin >= 4 * Cout) return macs >= 1e8;
  if (np == 1) return macs >= (K * rows < 6144 ? 1.15e8 : 1e8);
  return macs >= (K * rows >= 5120 ? 1e8 : Cout > Cin ? 2.5e8 : 1.5e8);
}

// Whether convolution l opens a residual block whose shortcut hands a gradient down to the block's input, and whether the
// product that writes that gradient adds it (both halve the image in the same step).
bool opens_block(const Layout& lo, int l) {
  return l + 1 < lo.n_conv && lo.conv[l + 1].skip && (lo.conv[l + 1].proj || !lo.preact);
}
bool shortcut_joins_product(const Layout& lo, int l) {
  const ConvLayer& cv = lo.conv[l];
  return l > 0 && opens_block(lo, l) && cv.fast && cv.direct_dx && !lo.conv[l - 1].pool && lo.conv[l + 1].H == cv.H &&
         lo.conv[l + 1].W == cv.W && lo.conv[l + 1].skip_step == cv.stride;
}

// Whether a last layer's normalisation is joined with the global average behind it.  A workgroup then walks the HW positions of one
// image, 64 channels and 16 positions at a time, where the normalisation alone has a thread a word: few images leave the chip
// idle, the sooner where a shortcut is another load to wait for.  A step apart / joined, `images` those of all replicas:
//   8x8 positions, no shortcut: 4 images of 64 channels 199 / 196 us, 512 282 / 270
//   8x8, a shortcut: 48 of 16 channels 320 / 323, 48 of 256 696 / 697, 100 of 256 1072 / 1062
//   16x16, no shortcut: 48 of 64 257 / 260, 16 of 256 413 / 412, 100 of 64 274 / 270, 192 of 64 310 / 296
//   16x16, a shortcut: 100 of 64 402 / 415, 192 of 64 460 / 466, 512 of 64 738 / 724
//   28x32, a shortcut: 10 of 8 604 / 687
//   32x32, no shortcut: 48 of 64 365 / 379, 100 of 64 417 / 410, 192 of 64 645 / 542
//   32x32, a shortcut: 16 of 16 317 / 413, 192 of 64 1012 / 1070
bool joined_average_pays(int64_t images, int HW, int C, bool shortcut) {
  if (HW <= (shortcut ? 16 : 64)) return true;
  return shortcut ? HW <= 256 && images * C >= 20480 : images * C >= 6144;
}

void build_layout(const lsam_config& c, Layout& lo) {
  lo.K = c.K;
  lo.L = c.n_layers;
  lo.raw = c.n_layers == 0;
  lo.B = lo.raw ? 0 : c.batch;
  lo.bf16 = !lo.raw && c.gemm_dtype == LSAM_GEMM_BF16 && c.n_conv == 0;
  lo.bf16_math = !lo.raw && c.gemm_dtype == LSAM_GEMM_BF16 && c.n_conv > 0;
  lo.np = lo.bf16_math ? 1 : 3;
  int64_t off = 0, flat = 0;
  if (lo.raw) {
    lo.d = c.d_raw;
    lo.d_pad = round_up(c.d_raw, 64);
  } else {
    lo.n_conv = c.n_conv;
    lo.preact = c.n_conv > 0 && c.preact != 0;
    // width[l]: columns of the matrix layer l reads (l < L), of the logits (l = L)
    std::vector<int> width(lo.L + 1);
    {
      int h = c.img_h, w = c.img_w;
      for (int l = 0; l <= lo.L; ++l) {
        width[l] = c.dims[l];
        if (l < lo.n_conv) {
          ConvLayer cv{};
          cv.stride = ((c.stride_mask >> l) & 1u) ? 2 : 1;
          h /= cv.stride; w /= cv.stride;
          cv.H = h; cv.W = w; cv.Cin = c.dims[l]; cv.Cout = c.dims[l + 1];
          cv.pool = (int)((c.pool_mask >> l) & 1u);
          cv.skip = ((c.skip_mask >> l) & 1u) != 0;
          if (cv.skip) {
            // the block input is what convolution l-1 read: [stride_{l-1} H_{l-1}] rows of C_{l-1} channels
            const ConvLayer& first = lo.conv[l - 1];
            cv.skip_C = first.Cin;
            cv.skip_step = first.stride * first.H / h;
            cv.proj = ((c.proj_mask >> l) & 1u) != 0;
          }
          cv.rows = (int64_t)c.batch * h * w;
          cv.ldc = (int)round_up(9 * (int64_t)cv.Cin, 8);
          lo.conv.push_back(cv);
          width[l] = 9 * cv.Cin;
          if (cv.pool) { h /= 2; w /= 2; }
        } else if (lo.n_conv > 0 && l == lo.n_conv) {
          width[l] = c.global_avg_pool ? c.dims[l] : h * w * c.dims[l];
          lo.gap_hw = c.global_avg_pool ? h * w : 0;
        }
      }
    }
    lo.ld.resize(lo.L + 1);
    for (int l = 0; l <= lo.L; ++l) lo.ld[l] = (int)round_up(width[l], 8);
    lo.need_a0 = lo.n_conv == 0 && (c.dims[0] % 8) != 0;
    for (int l = 0; l < lo.L; ++l) {
      Layer s;
      s.in = width[l];
      s.out = c.dims[l + 1];
      s.ldw = lo.ld[l];
      s.w_off = off;
      off = round_up(off + (int64_t)s.out * s.ldw, 64);
      s.b_off = off;
      off = round_up(off + s.out, 64);
      s.w_flat = flat;
      flat += (int64_t)s.out * s.in;
      s.b_flat = flat;
      flat += s.out;
      if (l < lo.n_conv && ((c.bn_mask >> l) & 1u)) {
        s.bn = true;
        s.gam_off = off;
        off = round_up(off + s.out, 64);
        s.bet_off = off;
        off = round_up(off + s.out, 64);
        s.gam_flat = flat;
        s.bet_flat = flat + s.out;
        flat += 2 * (int64_t)s.out;
      }
      lo.pieces.push_back(Piece{s.w_off, s.w_flat, s.out, s.in, s.ldw, 8 * l});
      lo.pieces.push_back(Piece{s.b_off, s.b_flat, 1, s.out, (int)round_up(s.out, 4), 8 * l + 1});
      if (s.bn) {
        lo.pieces.push_back(Piece{s.gam_off, s.gam_flat, 1, s.out, (int)round_up(s.out, 4), 8 * l + 2});
        lo.pieces.push_back(Piece{s.bet_off, s.bet_flat, 1, s.out, (int)round_up(s.out, 4), 8 * l + 3});
      }
      if (l < lo.n_conv && lo.conv[l].proj) {
        s.proj = true;
        s.proj_in = lo.conv[l].skip_C;
        s.pw_off = off;
        off = round_up(off + (int64_t)s.out * s.proj_in, 64);
        int64_t* slot[3] = {&s.pb_off, &s.pgam_off, &s.pbet_off};
        lo.pieces.push_back(Piece{s.pw_off, flat, s.out, s.proj_in, s.proj_in, 8 * l + 4});
        flat += (int64_t)s.out * s.proj_in;
        for (int q = 0; q < (lo.preact ? 1 : 3); ++q) {
          *slot[q] = off;
          lo.pieces.push_back(Piece{off, flat, 1, s.out, (int)round_up(s.out, 4), 8 * l + 5 + q});
          off = round_up(off + s.out, 64);
          flat += s.out;
        }
      }
      lo.layers.push_back(s);
    }
    lo.d = flat;
    lo.d_pad = off;
    if (lo.bf16) {
      lo.need_a0 = true;     // the input is always re-stored in the blocked layout
      lo.map.n = lo.L;
      int64_t so = 0;
      for (int l = 0; l < lo.L; ++l) {
        const Layer& ly = lo.layers[l];
        lo.shadow_off.push_back(so);
        lo.map.ldw[l] = ly.ldw;
        lo.map.cblocks[l] = b32s_blocks(ly.in);
        lo.map.begin[l] = ly.w_off;
        lo.map.end[l] = ly.w_off + (int64_t)ly.out * ly.ldw;
        lo.map.shadow[l] = so;
        so += b32s_size(ly.out, ly.in);
      }
      lo.shadow_stride = so;
    }
  }
  if (lo.raw) {
    lo.nblk = sumsq_blocks(lo.d);
  } else {
    // the first backward pass leaves one partial sum of squares per workgroup that wrote a
    // piece of the gradient: room for the most any tile choice can produce
    int64_t cap = 0;
    for (const Layer& ly : lo.layers)
      cap += std::max(gemm_sumsq_capacity(ly.out, ly.in),
                      std::max(head_sumsq_slots(ly.in), ly.out / 2)) +   // ly.out / 2: first-layer kernels
             (ly.out + 63) / 64 + (ly.bn ? 2 * ((ly.out + 63) / 64) : 0) +
             (ly.proj ? gemm_sumsq_capacity(ly.out, ly.proj_in) + 2 * ((ly.out + 63) / 64) : 0);
    lo.nblk = (int)cap;
  }

  size_t cur = 0;
  const size_t vec = (size_t)lo.K * lo.d_pad * 4;
  lo.x = take(cur, vec);
  lo.v = take(cur, vec);
  lo.S = take(cur, vec);
  lo.g = lo.raw ? 0 : take(cur, vec);
  lo.xt = take(cur, lo.bf16 ? (size_t)lo.K * lo.shadow_stride * 2 : vec);
  lo.y = take(cur, (size_t)lo.d_pad * 4);
  lo.gprev = take(cur, (size_t)lo.d_pad * 4);
  if (lo.raw && c.algorithm == LSAM_ALG_DATA_PARALLEL) lo.gmean = take(cur, (size_t)lo.d_pad * 4);
  lo.partials = take(cur, (size_t)lo.K * lo.nblk * 8);
  lo.restart = take(cur, (size_t)lo.K * 4);
  lo.norms = take(cur, (size_t)lo.K * 4);
  lo.scale = take(cur, (size_t)lo.K * 4);
  lo.loss = take(cur, (size_t)lo.K * 4);
  if (!lo.raw) {
    const size_t rows = (size_t)lo.K * lo.B;
    lo.loss_rows = take(cur, rows * 4);
    lo.act.assign(lo.L + 1, 0);
    lo.dz.assign(lo.L + 1, 0);
    auto wd = [&](int l) { return l < lo.L ? lo.layers[l].in : lo.layers[lo.L - 1].out; };
    auto act_bytes = [&](int l) { return (size_t)lo.K * lo.act_elems(wd(l), lo.ld[l]) * lo.es(); };
    size_t dcol_bytes = 0;
    for (int l = 0; l < lo.n_conv; ++l) {
      ConvLayer& cv = lo.conv[l];
      cv.bn = lo.layers[l].bn;
      const bool small = cv.rows < (1 << 24);      // (first-layer kernels: pixel indices exact in fp32)
      cv.fast = plane_products_pay(lo.np, lo.K, cv.rows, cv.Cin, cv.Cout, l > 0);
      // unfolding by address: whole taps or parts of one tap make up a 32-deep k-step; the
      // fp32-storage GEMM knows stride 1 and parts of taps only
      auto fits = [&](int C) { return C % (cv.fast ? 8 : 32) == 0; };
      cv.direct_in = small && fits(cv.Cin) && (cv.fast || cv.stride == 1);
      // (stride 2: since the product in classes leaves the sums below it and the layer below no floats, it wins against
      // one with a stored gradient and its fold unless three planes meet many columns that fill the 64-wide
      // tiles badly.  Steps of one such layer between two others, 4 replicas of 64 images of 32 x 32, stored / classes: 40
      // channels 1242 / 1163 us, 72 2462 / 2433, 80 2686 / 2601, 104 3968 / 3868, 160 6674 / 6630; 136 6221 / 6287, 152 7031 / 7120)
      // Where the classes' tiles do not fill the chip twice over their longest contraction, four taps of all outputs, is what takes
      // long: 72 to 320 channels on 1792 pixels, 112 tiles, 2.1 % more, to 160 on 3072, 192 tiles, 3 % less; 112 to 224 with 112
      // tiles 0.3 % more, with 192 2.3 % less, to 448 with 64 6 % more, 192 0.4 %; 160 to 320 with 96 2.9 % more, 168 1.4 % less;
      // 224 to 448 with 80 6 % more, 384 1.2 %.  (Columns that fill their tiles have always been taken in classes.)
      const int columns = (cv.Cin + 63) / 64 * 64;
      const bool classes_pay = lo.np == 1 || cv.Cin <= 32 || columns * 8 <= cv.Cin * 9 ||
                               ((cv.Cin <= 128 || columns * 5 <= cv.Cin * 6) &&
                                lo.K * ((cv.rows + 127) / 128) * (columns / 64) * 4 * 390 >= (int64_t)cv.Cout * cv.Cout);
      cv.direct_dx = small && l > 0 && fits(cv.Cout) && (cv.stride == 1 || (cv.fast && classes_pay));
      cv.first = l == 0 && cv.stride == 1 && first_conv_fits(cv.Cin, cv.Cout, cv.rows, lo.K, lo.bf16_math);
    }
    for (int l = 0; l < lo.n_conv; ++l) {
      ConvLayer& cv = lo.conv[l];
      const ConvLayer* next = l + 1 < lo.n_conv ? &lo.conv[l + 1] : nullptr;
      const ConvLayer* closing = l + 2 < lo.n_conv && lo.conv[l + 2].skip ? &lo.conv[l + 2] : nullptr;
      const bool post_sum = cv.skip && !lo.preact;
      cv.bn_pool = cv.bn && cv.pool && !post_sum;
      cv.bn_gap = cv.bn && !cv.pool && !next && lo.gap_hw > 0 &&
                  joined_average_pays((int64_t)lo.K * lo.B, lo.gap_hw, cv.Cout, post_sum);
      cv.has_keep = cv.pool || (cv.bn &&
                    (next ? next->fast && next->direct_dx && (!opens_block(lo, l + 1) || shortcut_joins_product(lo, l + 1))
                          : lo.gap_hw > 0));
      cv.pooled_floats = cv.pool && (!next || !next->fast || !next->direct_in);
      if (cv.pool || !next) cv.floats = !cv.bn_pool && !cv.bn_gap;
      else cv.floats = !cv.has_keep || !next->fast || !next->direct_in || (closing && (closing->proj ? !closing->fast : !lo.preact));
    }
    for (int l = 0; l < lo.n_conv; ++l) {
      ConvLayer& cv = lo.conv[l];
      const size_t full = (size_t)lo.K * cv.rows * cv.Cout * 4;
      if (cv.first)
        cv.first_partial = take(cur, (size_t)lo.K * first_conv_chunks(cv.rows, cv.Cout, lo.K) * cv.Cout * 32 * 4);
      else if (!cv.direct_in) cv.col = take(cur, (size_t)lo.K * cv.rows * cv.ldc * (cv.fast ? 2 * lo.np : 4));
      if (cv.direct_dx && !cv.fast) cv.wt = take(cur, (size_t)lo.K * cv.Cin * 9 * cv.Cout * 4);
      cv.in_H = cv.H * cv.stride; cv.in_W = cv.W * cv.stride;
      cv.planes = (cv.fast && cv.direct_in && !cv.first) || (l + 1 < lo.n_conv && lo.conv[l + 1].proj &&
                  plane_products_pay(lo.np, lo.K, lo.conv[l + 1].rows, lo.conv[l + 1].Cin, lo.conv[l + 1].Cout, true));
      cv.planes_above = cv.planes && l > 0 && (lo.conv[l - 1].pool || lo.conv[l - 1].bn);
      if (cv.planes) {
        cv.plane_elems = (int64_t)lo.K * lo.B * cv.in_H * cv.in_W * cv.Cin;
        cv.xp = take(cur, (size_t)cv.plane_elems * 2 * lo.np);
      }
      if (cv.fast) {
        const Layer& ly = lo.layers[l];
        auto bank = [&](int64_t src, int rows, int cols, int ldw, int taps) {
          FilterBank f{src, lo.wp_elems, rows, cols, ldw, 0, taps, lo.bank_blocks, cv.stride};
          f.ldp = (int)round_up(taps ? taps * rows : cols, 32);
          lo.wp_elems += (int64_t)lo.K * (taps ? cols : rows) * f.ldp;
          lo.bank_blocks += filter_bank_blocks(f);
          lo.banks.push_back(f);
          return f.dst;
        };
        // (a stored unfolded image has the filters' row pitch, zeros in the padding of both)
        if (!cv.first) cv.wf = bank(ly.w_off, cv.Cout, cv.direct_in ? ly.in : ly.ldw, ly.ldw, 0);
        if (l > 0) cv.wx = cv.direct_dx ? bank(ly.w_off, cv.Cout, cv.Cin, ly.ldw, 9) : bank(ly.w_off, cv.Cout, cv.ldc, ly.ldw, 1);
        if (cv.proj) {
          cv.pwf = bank(ly.pw_off, cv.Cout, ly.proj_in, ly.proj_in, 0);
          cv.pwx = bank(ly.pw_off, cv.Cout, ly.proj_in, ly.proj_in, 1);
        }
        lo.dzp_elems = std::max(lo.dzp_elems, (int64_t)lo.K * cv.rows * cv.Cout);
      }
      if (cv.floats) cv.out = take(cur, full);
      if (cv.has_keep) cv.keep = take(cur, full / (cv.pool ? 64 : 16));
      if (cv.pool) cv.arg = take(cur, full / 64);
      if (cv.bn_pool) cv.zmax = take(cur, full / 4);
      cv.dout = take(cur, full);
      if (cv.bn) {
        cv.z = take(cur, full);
        cv.stats = take(cur, (size_t)lo.K * 2 * cv.Cout * 4);
      }
      if (cv.pool) {
        if (cv.pooled_floats) cv.pooled = take(cur, full / 4);
        cv.dpooled = take(cur, full / 4);
      }
      if (cv.proj) {
        cv.psub = take(cur, (size_t)lo.K * cv.rows * cv.skip_C * 4);
        cv.pz = take(cur, full);
        if (!lo.preact) cv.pstats = take(cur, (size_t)lo.K * 2 * cv.Cout * 4);
      }
      if (l > 0 && !cv.direct_dx) dcol_bytes = std::max(dcol_bytes, (size_t)lo.K * cv.rows * cv.ldc * 4);
    }
    if (dcol_bytes) lo.dcol = take(cur, dcol_bytes);
    if (lo.wp_elems) {
      lo.wp = take(cur, (size_t)lo.wp_elems * 2 * lo.np);
      lo.banks_at = take(cur, lo.banks.size() * sizeof(FilterBank));
    }
    if (lo.dzp_elems) lo.dzp = take(cur, (size_t)lo.dzp_elems * 2 * lo.np);
    if (lo.n_conv > 0) {
      size_t most = 0;
      for (const ConvLayer& cv : lo.conv) {
        const int chunks = std::max(colsum_chunks(cv.rows, cv.Cout, lo.K), cv.pool ? colsum_chunks(cv.rows / 4, cv.Cout, lo.K) : 0);
        most = std::max(most, (size_t)lo.K * chunks * cv.Cout * 4);
      }
      size_t proj = 0;
      for (const ConvLayer& cv : lo.conv) {
        if (!cv.bn) continue;
        const int chunks = std::max(bn_chunks(cv.rows, cv.Cout, lo.K), cv.pool ? bn_chunks(cv.rows / 4, cv.Cout, lo.K) : 0);
        const size_t sums = (size_t)lo.K * std::max(chunks, conv_gemm_sum_chunks(cv.rows)) * 2 * cv.Cout * 4;
        most = std::max(most, sums);
        if (cv.proj && !lo.preact) proj = std::max(proj, sums);
      }
      lo.colsum = take(cur, most);
      if (proj) lo.pcolsum = take(cur, proj);
    }
    // the dense layers start at n_conv; their input and its gradient are the last
    // convolution's (pooled) output and that buffer's gradient
    if (lo.n_conv > 0) {
      const ConvLayer& cv = lo.conv[lo.n_conv - 1];
      lo.act[lo.n_conv] = cv.pool ? cv.pooled : cv.out;
      lo.dz[lo.n_conv] = cv.pool ? cv.dpooled : cv.dout;
      if (lo.gap_hw) {
        lo.gap_out = take(cur, rows * lo.ld[lo.n_conv] * 4);
        lo.gap_grad = take(cur, rows * lo.ld[lo.n_conv] * 4);
        lo.act[lo.n_conv] = lo.gap_out;
        lo.dz[lo.n_conv] = lo.gap_grad;
      }
    }
    for (int l = lo.n_conv + 1; l < lo.L; ++l) lo.act[l] = take(cur, act_bytes(l));
    for (int l = lo.n_conv + 1; l <= lo.L; ++l) lo.dz[l] = take(cur, act_bytes(l));
    lo.logits = take(cur, rows * lo.ld[lo.L] * 4);
    if (lo.need_a0) lo.a0 = take(cur, act_bytes(0));
    // scratch for split-K partial sums: the largest request among this model's GEMMs
    size_t need = 0;
    for (int l = 0; l < lo.L; ++l) {
      const Layer& ly = lo.layers[l];
      if (lo.bf16) break;      // split-K serves the fp32 kernel only
      GemmDesc d{};
      d.batch = lo.K; d.in_bf16 = lo.bf16; d.bf16_math = lo.bf16_math;
      const ConvLayer* cv = l < lo.n_conv ? &lo.conv[l] : nullptr;
      const int rows = cv ? (int)cv->rows : lo.B;
      if (!cv || !cv->fast) {
        d.M = rows; d.N = ly.out; d.Kd = ly.in; d.a_kmajor = 1; d.b_kmajor = 1;     // forward
        d.unfold = cv && cv->direct_in ? 1 : 0;
        need = std::max(need, gemm_splitk_bytes(d));
        d.M = rows; d.N = ly.in; d.Kd = ly.out; d.a_kmajor = 1; d.b_kmajor = 0;     // dX
        d.unfold = 0;
        if (cv && cv->direct_dx) { d.N = cv->Cin; d.Kd = 9 * cv->Cout; d.b_kmajor = 1; d.unfold = 1; }
        if (l > 0) need = std::max(need, gemm_splitk_bytes(d));
        d.M = ly.out; d.N = ly.in; d.Kd = rows; d.a_kmajor = 0; d.b_kmajor = 0;     // dW
        d.unfold = cv && cv->direct_in ? 2 : 0;
        need = std::max(need, gemm_splitk_bytes(d));
        if (ly.proj) {       // the projection's three products
          d.unfold = 0;
          d.M = rows; d.N = ly.out; d.Kd = ly.proj_in; d.a_kmajor = 1; d.b_kmajor = 1;
          need = std::max(need, gemm_splitk_bytes(d));
          d.M = rows; d.N = ly.proj_in; d.Kd = ly.out; d.a_kmajor = 1; d.b_kmajor = 0;
          need = std::max(need, gemm_splitk_bytes(d));
          d.M = ly.out; d.N = ly.proj_in; d.Kd = rows; d.a_kmajor = 0; d.b_kmajor = 0;
          need = std::max(need, gemm_splitk_bytes(d));
        }
        continue;
      }
      auto planes = [&](int wgrad, int C, int stride, int side, int M, int N, int Kd) {
        ConvGemmDesc q{};
        q.np = lo.np; q.wgrad = wgrad; q.batch = lo.K;
        q.image = PlaneImage{nullptr, 0, 0, C, cv->H, cv->W, cv->H * stride, cv->W * stride, stride, side, side, 0, 0};
        q.M = M; q.N = N; q.Kd = Kd;
        const size_t bytes = conv_gemm_splitk_bytes(q);
        if (!wgrad) need = std::max(need, bytes);
        return bytes;
      };
      ConvLayer& own = lo.conv[l];
      if (cv->direct_in) {
        planes(0, cv->Cin, cv->stride, 3, rows, ly.out, ly.in);
        own.wpart_bytes = planes(1, cv->Cin, cv->stride, 3, ly.out, ly.in, rows);
      } else if (!cv->first) {
        planes(0, cv->ldc, 1, 1, rows, ly.out, cv->ldc);
        own.wpart_bytes = planes(1, cv->ldc, 1, 1, ly.out, cv->ldc, rows);
      }
      if (cv->direct_dx && cv->stride == 1) planes(0, cv->Cout, 1, 3, rows, cv->Cin, 9 * cv->Cout);
      else if (cv->direct_dx) {}          // one launch per class of pixels, never split
      else if (l > 0) planes(0, cv->Cout, 1, 1, rows, cv->ldc, cv->Cout);
      if (ly.proj) {           // the projection's three products
        planes(0, ly.proj_in, cv->skip_step, 1, rows, ly.out, ly.proj_in);
        planes(0, ly.out, 1, 1, rows, ly.proj_in, ly.out);
        own.pwpart_bytes = planes(1, ly.proj_in, cv->skip_step, 1, ly.out, ly.proj_in, rows);
      }
    }
    // Of the weight gradients that leave partial sums, as many as the pass's list holds get a place of their own, in the order
    // of conv_backward.  Sums past 20 MiB (16 where there are workgroups enough to add them up alone, 512) are not worth a place: added
    // up at once, from memory that the product before has used as well, they are read from the caches.  A step with all
    // listed / as the rule has it: 112 channels with 28 MiB a layer, two replicas of 40 images of 28 x 20, bf16, 929 / 896 us, 152
    // and 304 channels with 19 MiB, two of 18 of 12 x 20, 1354 / 1321, 304 channels with 25 MiB, four of 8 of 16 x 20, 2232 / 2182; listed
    // and at once 64 channels with 18 MiB and 144 workgroups (a residual net of 16 to 64 channels) 5318 / 5348, 144 channels with
    // 6 MiB 445 / 453.
    int listed = 0;
    auto place = [&](size_t& at, size_t& bytes, int64_t results) {
      if (!bytes) return;
      if (listed < ReduceList::kMax && bytes <= (size_t)(lo.K * results >= (512 << 10) ? 16 : 20) << 20) {
        at = take(cur, bytes);
        ++listed;
      } else {
        need = std::max(need, bytes);
        bytes = 0;
      }
    };
    for (int l = lo.n_conv - 1; l >= 0; --l) {
      place(lo.conv[l].pwpart, lo.conv[l].pwpart_bytes, (int64_t)lo.layers[l].out * lo.layers[l].proj_in);
      place(lo.conv[l].wpart, lo.conv[l].wpart_bytes, (int64_t)lo.layers[l].out * lo.layers[l].in);
    }
    lo.splitk_bytes = need;
    if (need) lo.splitk = take(cur, need);
    if (c.noise_scale > 0.f) lo.noise_segs = take(cur, lo.pieces.size() * sizeof(NoiseSeg));
  }
  lo.total = cur;
}

// ---- per-kernel timing ---------------------------------------------------------------------------
enum KernelClass {
  KC_GEMM_FWD = 0, KC_GEMM_DX, KC_GEMM_DW, KC_SOFTMAX_CE, KC_BIAS_GRAD, KC_SUMSQ, KC_NORM_FINISH,
  KC_PERTURB, KC_DESCENT, KC_CENTER, KC_MISC, KC_HEAD, KC_UNFOLD, KC_POOL, KC_CONV_FIRST, KC_BATCHNORM,
  KC_GEMM_DW_STEP, KC_GEMM_DW_NORM, KC_GEMM_DW_ASCEND, KC_COUNT
};
const char* const kClassNames[KC_COUNT] = {
    "gemm_fwd", "gemm_dx", "gemm_dw", "softmax_ce", "bias_grad", "sumsq_partials", "norm_finish",
    "perturb", "descent", "center", "misc", "head", "unfold_fold", "pool", "conv_first", "batchnorm",
    "gemm_dw_step", "gemm_dw_norm", "gemm_dw_ascend"};

struct TimedLaunch {
  int cls;
  hipEvent_t a, b;
};

}  // namespace
}  // namespace lsam

namespace lsam {
void set_last_error(const char* msg) { g_err = msg ? msg : ""; }
}  // namespace lsam

using namespace lsam;

struct lsam_ctx {
  lsam_config cfg;
  std::vector<int32_t> dims, tau_explicit;
  Layout lo;
  Schedule sched;
  char* ws = nullptr;
  hipStream_t stream = nullptr;
  float lr = 0.f, rho = 0.f;
  int norm_slots = 0;   // partial sums of squares left by the last first-pass backward
  uint32_t t_step = 0;  // sampler steps taken (counter word of the Langevin noise)
  void* stage = nullptr;   // pinned host staging buffer for the read-out / restore calls (lazy)
  NoiseMap noise{};     // where the Langevin noise goes; used when cfg.noise_scale > 0
  bool fuse_step = true;   // take the sampler step inside the second pass's dW epilogues where possible
  // timing
  bool timing = false;
  std::vector<TimedLaunch> pending;
  std::vector<hipEvent_t> free_events;
  int64_t t_count[KC_COUNT] = {0};
  double t_ms[KC_COUNT] = {0};

  template <typename T> T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
};

namespace {

struct LaunchTimer {
  lsam_ctx* c;
  TimedLaunch t;
  bool on;
  LaunchTimer(lsam_ctx* ctx, int cls) : c(ctx), on(ctx->timing) {
    if (!on) return;
    t.cls = cls;
    t.a = grab();
    t.b = grab();
    if (t.a == nullptr || t.b == nullptr) { on = false; return; }
    (void)hipEventRecord(t.a, c->stream);
  }
  ~LaunchTimer() {
    if (!on) return;
    (void)hipEventRecord(t.b, c->stream);
    c->pending.push_back(t);
  }
  hipEvent_t grab() {
    if (!c->free_events.empty()) {
      hipEvent_t e = c->free_events.back();
      c->free_events.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};

int drain_timing(lsam_ctx* c) {
  if (c->pending.empty()) return LSAM_OK;
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (auto& t : c->pending) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.a, t.b) == hipSuccess) {
      c->t_ms[t.cls] += ms;
      c->t_count[t.cls] += 1;
    }
    c->free_events.push_back(t.a);
    c->free_events.push_back(t.b);
  }
  c->pending.clear();
  return LSAM_OK;
}

int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LSAM_EHIP, "launch of %s failed: %s", what, hipGetErrorString(e));
  return LSAM_OK;
}

float coupling(const lsam_ctx* c, int i) {
  if (c->cfg.algorithm == LSAM_ALG_DATA_PARALLEL) return 0.f;
  if (c->cfg.lambda_abs >= 0.f) return c->cfg.lambda_abs;
  return (float)((double)c->cfg.lambda0 / ((double)c->lr * (double)c->sched.tau()[i]));
}

// Split-K scratch shared by all GEMMs of a step.
void split(const lsam_ctx* c, GemmDesc& d) {
  d.splitk_ws = c->lo.splitk_bytes ? c->at<float>(c->lo.splitk) : nullptr;
  d.splitk_bytes = c->lo.splitk_bytes;
  d.bf16_math = c->lo.bf16_math;     // every GEMM of a step shares the arithmetic mode, too
}

// ---- plane products (kernels_conv_gemm.hip) ----
// The image layer `cv` reads as the operand of its 3x3 convolution ...
PlaneImage layer_image(const lsam_ctx* c, const ConvLayer& cv) {
  return PlaneImage{c->at<uint16_t>(cv.xp), cv.plane_elems / c->lo.K, cv.plane_elems, cv.Cin, cv.H, cv.W, cv.in_H, cv.in_W,
                    cv.stride, 3, 3, -1, -1};
}
// ... or, where the unfolded image is stored, that image under a single tap;
PlaneImage stored_image(const lsam_ctx* c, const ConvLayer& cv) {
  return PlaneImage{c->at<uint16_t>(cv.col), cv.rows * cv.ldc, (int64_t)c->lo.K * cv.rows * cv.ldc, cv.ldc, cv.H, cv.W,
                    cv.H, cv.W, 1, 1, 1, 0, 0};
}
// ... and, as the input of the block that convolution `top` (one above) closes, of its projection:
// every skip_step-th pixel.
PlaneImage projection_image(const lsam_ctx* c, const ConvLayer& below, const ConvLayer& top) {
  return PlaneImage{c->at<uint16_t>(below.xp), below.plane_elems / c->lo.K, below.plane_elems, below.Cin, top.H, top.W,
                    below.in_H, below.in_W, top.skip_step, 1, 1, 0, 0};
}
// A layer's output gradient (the planes in dzp) as a stride-1 image under `taps` = 3 x 3 or 1 x 1 taps.
PlaneImage gradient_image(const lsam_ctx* c, const ConvLayer& cv, int side) {
  return PlaneImage{c->at<uint16_t>(c->lo.dzp), cv.rows * cv.Cout, c->lo.dzp_elems, cv.Cout, cv.H, cv.W, cv.H, cv.W, 1,
                    side, side, side == 3 ? -1 : 0, side == 3 ? -1 : 0};
}
// `filters`: where in wp the launch's filters lie (unused for a weight gradient).
ConvGemmDesc plane_desc(const lsam_ctx* c, const PlaneImage& im, int wgrad, int64_t filters, int M, int N, int Kd) {
  const Layout& lo = c->lo;
  ConvGemmDesc d{};
  d.np = lo.np; d.wgrad = wgrad; d.image = im;
  d.M = M; d.N = N; d.Kd = Kd; d.batch = lo.K;
  d.epilogue = EPI_PLAIN;
  d.splitk_ws = lo.splitk_bytes ? c->at<float>(lo.splitk) : nullptr;
  d.splitk_bytes = lo.splitk_bytes;
  if (wgrad) {     // contraction with the output gradient in dzp
    d.other = c->at<uint16_t>(lo.dzp);
    d.other_stride = (int64_t)Kd * M; d.other_plane = lo.dzp_elems; d.ld = M;
  } else {         // filters in wp, rows padded to whole k-steps
    d.other = c->at<uint16_t>(lo.wp) + filters;
    d.ld = (int)round_up(Kd, 32);
    d.other_stride = (int64_t)N * d.ld; d.other_plane = lo.wp_elems;
  }
  return d;
}
int split_gradient(const lsam_ctx* c, const float* dz, const ConvLayer& cv) {
  const Layout& lo = c->lo;
  return launch_split_planes(dz, c->at<uint16_t>(lo.dzp), lo.np, lo.dzp_elems, (int64_t)lo.K * cv.rows * cv.Cout, c->stream);
}

// The planes of convolution l's input, for the kernel that writes that image.
PlaneOut input_planes(const lsam_ctx* c, int l) {
  const Layout& lo = c->lo;
  PlaneOut o;
  if (l < lo.n_conv && lo.conv[l].planes_above) {
    const ConvLayer& cv = lo.conv[l];
    o.p = c->at<uint16_t>(cv.xp); o.np = lo.np; o.plane = cv.plane_elems;
  }
  return o;
}

// Forward pass of the convolution layers: unfold, GEMM with bias + ReLU, pool.  `params`: x or
// the perturbed copy (fp32).  The result is the dense layers' input, lo.act[n_conv].
int conv_forward(lsam_ctx* c, const float* X, const float* params) {
  const Layout& lo = c->lo;
  hipStream_t s = c->stream;
  const float* in = X;
  float* scratch = c->at<float>(lo.colsum);
  float* pscratch = c->at<float>(lo.pcolsum);
  if (!lo.banks.empty()) {
    LaunchTimer t(c, KC_MISC);
    if (launch_filters(params, lo.d_pad, c->at<FilterBank>(lo.banks_at), (int)lo.banks.size(), lo.bank_blocks,
                       c->at<uint16_t>(lo.wp), lo.np, lo.wp_elems, lo.K, s) != 0)
      return fail(LSAM_EINVAL, "planes of the filters rejected");
  }
  for (int l = 0; l < lo.n_conv; ++l) {
    const ConvLayer& cv = lo.conv[l];
    const Layer& ly = lo.layers[l];
    ChunkSums have, phave;        // statistics that the products leave in the scratch
    if (cv.planes && !cv.planes_above) {
      LaunchTimer t(c, KC_UNFOLD);
      if (launch_split_planes(in, c->at<uint16_t>(cv.xp), lo.np, cv.plane_elems, cv.plane_elems, s) != 0)
        return fail(LSAM_EINVAL, "planes of the input of convolution %d rejected", l);
    }
    if (cv.first) {
      LaunchTimer t(c, KC_CONV_FIRST);
      if (launch_first_conv_forward(in, params, lo.d_pad, ly.w_off, ly.b_off, ly.ldw,
                                    c->at<float>(cv.bn ? cv.z : cv.out), cv.bn ? 0 : 1,
                                    lo.bf16_math ? 1 : 0, lo.K, cv.rows, cv.H, cv.W, cv.Cin, cv.Cout,
                                    cv.bn ? scratch : nullptr, &have, s) != 0)
        return fail(LSAM_EINVAL, "first convolution rejected");
    } else if (!cv.direct_in) {
      LaunchTimer t(c, KC_UNFOLD);
      if (launch_unfold3x3(in, cv.rows * cv.stride * cv.stride * cv.Cin, c->at<char>(cv.col), cv.fast ? lo.np : 0,
                           (int64_t)lo.K * cv.rows * cv.ldc, cv.ldc, lo.K, lo.B, cv.H, cv.W, cv.Cin, cv.stride, s) != 0)
        return fail(LSAM_EINVAL, "unfold of convolution %d rejected", l);
    }
    if (cv.proj && cv.fast) {
      // projection shortcut: the block input's pixels (every second one if the block halved
      // the image) through a 1x1 convolution
      LaunchTimer t(c, KC_GEMM_FWD);
      ConvGemmDesc d = plane_desc(c, projection_image(c, lo.conv[l - 1], cv), 0, cv.pwf, (int)cv.rows, cv.Cout, ly.proj_in);
      d.C = c->at<float>(cv.pz); d.strideC = cv.rows * cv.Cout; d.ldC = cv.Cout;
      d.epilogue = EPI_BIAS;
      d.bias = params + ly.pb_off; d.strideBias = lo.d_pad;
      if (!lo.preact) { d.sums = 1; d.sum_part = pscratch; }
      if (launch_conv_gemm(d, s, nullptr, &phave) != 0)
        return fail(LSAM_EINVAL, "projection of convolution %d rejected", l);
    }
    if (!cv.first && cv.fast) {
      // filters of ldw columns: 9 C_in, and zeros up to the unfolded image's pitch where that is stored
      LaunchTimer t(c, KC_GEMM_FWD);
      const int cols = cv.direct_in ? ly.in : ly.ldw;
      ConvGemmDesc d = plane_desc(c, cv.direct_in ? layer_image(c, cv) : stored_image(c, cv), 0, cv.wf, (int)cv.rows, cv.Cout, cols);
      d.C = c->at<float>(cv.bn ? cv.z : cv.out); d.strideC = cv.rows * cv.Cout; d.ldC = cv.Cout;
      d.epilogue = cv.bn ? EPI_BIAS : EPI_BIAS_RELU;
      d.bias = params + ly.b_off; d.strideBias = lo.d_pad;
      if (cv.skip && lo.preact) {
        // a pre-activation block's sum: the bare projection, or the sum two convolutions below
        d.add = c->at<float>(cv.proj ? cv.pz : lo.conv[l - 2].z); d.strideAdd = cv.rows * cv.Cout; d.ldAdd = cv.Cout;
      }
      if (cv.bn) { d.sums = 1; d.sum_part = scratch; }
      if (launch_conv_gemm(d, s, nullptr, &have) != 0)
        return fail(LSAM_EINVAL, "forward product of convolution %d rejected", l);
    } else if (!cv.first) {
      GemmDesc d{};
      d.A = c->at<float>(cv.col); d.strideA = cv.rows * cv.ldc; d.ldA = cv.ldc; d.a_kmajor = 1;
      if (cv.direct_in) {
        d.A = in; d.strideA = cv.rows * cv.Cin; d.ldA = cv.Cin;
        d.unfold = 1; d.unfold_C = cv.Cin; d.unfold_H = cv.H; d.unfold_W = cv.W;
      }
      d.B = params + ly.w_off; d.strideB = lo.d_pad; d.ldB = ly.ldw; d.b_kmajor = 1;
      d.C = c->at<float>(cv.bn ? cv.z : cv.out); d.strideC = cv.rows * cv.Cout; d.ldC = cv.Cout;
      d.M = (int)cv.rows; d.N = cv.Cout; d.Kd = ly.in; d.batch = lo.K;
      d.epilogue = cv.bn ? EPI_BIAS : EPI_BIAS_RELU;
      d.bias = params + ly.b_off; d.strideBias = lo.d_pad;
      split(c, d);
      LaunchTimer t(c, KC_GEMM_FWD);
      if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "forward GEMM of convolution %d rejected", l);
    }
    if (cv.proj) {
      if (!cv.fast) {
        const ConvLayer& src = lo.conv[l - 2];
        const float* sub = c->at<float>(src.out);
        if (cv.skip_step == 2) {
          LaunchTimer t(c, KC_UNFOLD);
          if (launch_subsample2(sub, c->at<float>(cv.psub), (int64_t)lo.K * lo.B, cv.H, cv.W, cv.skip_C, s) != 0)
            return fail(LSAM_EINVAL, "projection of convolution %d: gather rejected", l);
          sub = c->at<float>(cv.psub);
        }
        GemmDesc d{};
        d.A = sub; d.strideA = cv.rows * cv.skip_C; d.ldA = cv.skip_C; d.a_kmajor = 1;
        d.B = params + ly.pw_off; d.strideB = lo.d_pad; d.ldB = ly.proj_in; d.b_kmajor = 1;
        d.C = c->at<float>(cv.pz); d.strideC = cv.rows * cv.Cout; d.ldC = cv.Cout;
        d.M = (int)cv.rows; d.N = cv.Cout; d.Kd = ly.proj_in; d.batch = lo.K;
        d.epilogue = EPI_BIAS;
        d.bias = params + ly.pb_off; d.strideBias = lo.d_pad;
        split(c, d);
        {
          LaunchTimer t(c, KC_GEMM_FWD);
          if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "projection of convolution %d rejected", l);
        }
      }
      if (lo.preact && cv.fast) {
        // (the sum is taken where the convolution's product is written)
      } else if (lo.preact) {
        // the bare projection joins the convolution's output in front of the normalisation
        LaunchTimer t(c, KC_POOL);
        if (launch_add_into(c->at<float>(cv.z), c->at<float>(cv.pz), (int64_t)lo.K * cv.rows * cv.Cout, s) != 0)
          return fail(LSAM_EINVAL, "projection of convolution %d: sum rejected", l);
      } else {
        LaunchTimer t(c, KC_BATCHNORM);
        if (launch_bn_stats(c->at<float>(cv.pz), pscratch, phave, c->at<float>(cv.pstats), lo.K,
                            cv.rows, cv.Cout, c->cfg.bn_eps, s) != 0)
          return fail(LSAM_EINVAL, "projection of convolution %d: statistics rejected", l);
      }
    } else if (cv.skip && lo.preact && !cv.fast) {
      // identity shortcut of a pre-activation block: the sum two convolutions below
      LaunchTimer t(c, KC_POOL);
      if (launch_add_into(c->at<float>(cv.z), c->at<float>(lo.conv[l - 2].z), (int64_t)lo.K * cv.rows * cv.Cout,
                          s) != 0)
        return fail(LSAM_EINVAL, "shortcut of convolution %d: sum rejected", l);
    }
    if (cv.bn) {
      LaunchTimer t(c, KC_BATCHNORM);
      ShortcutDesc sc{};
      const bool post_sum = cv.skip && !lo.preact;     // the shortcut joins behind the normalisation
      if (post_sum && cv.proj) {
        sc.pz = c->at<float>(cv.pz); sc.pstats = c->at<float>(cv.pstats);
        sc.pgam_off = ly.pgam_off; sc.pbet_off = ly.pbet_off;
      } else if (post_sum) {
        // the block input: what convolution l-1 read, i.e. the ReLU output of convolution l-2
        sc.src = c->at<float>(lo.conv[l - 2].out);
        sc.stride = lo.conv[l - 2].rows * cv.skip_C;
        sc.H = cv.H; sc.W = cv.W; sc.Cs = cv.skip_C; sc.step = cv.skip_step;
      }
      const float* z = c->at<float>(cv.z);
      const float* stats = c->at<float>(cv.stats);
      PlaneOut o = cv.pool && !cv.bn_pool ? PlaneOut{} : input_planes(c, l + 1);
      if (cv.has_keep && (!cv.pool || cv.bn_pool)) o.keep = c->at<uint8_t>(cv.keep);
      int rc = launch_bn_stats(z, scratch, have, c->at<float>(cv.stats), lo.K, cv.rows, cv.Cout, c->cfg.bn_eps, s);
      if (rc == 0 && cv.bn_pool)
        rc = launch_bn_pool(z, stats, params, lo.d_pad, ly.gam_off, ly.bet_off, cv.pooled_floats ? c->at<float>(cv.pooled) : nullptr,
                            c->at<float>(cv.zmax), c->at<uint8_t>(cv.arg), lo.K, lo.B, cv.H, cv.W, cv.Cout, o, s);
      else if (rc == 0 && cv.bn_gap)
        rc = launch_bn_avgpool(z, stats, params, lo.d_pad, ly.gam_off, ly.bet_off, c->at<float>(lo.gap_out), lo.K, lo.B, lo.gap_hw,
                               cv.Cout, lo.ld[lo.n_conv], post_sum ? &sc : nullptr, o.keep, s);
      else if (rc == 0)
        rc = launch_bn_apply(z, stats, params, lo.d_pad, ly.gam_off, ly.bet_off, cv.floats ? c->at<float>(cv.out) : nullptr, lo.K,
                             cv.rows, cv.Cout, post_sum ? &sc : nullptr, o, s);
      if (rc != 0) return fail(LSAM_EINVAL, "batch normalisation of convolution %d rejected", l);
    }
    in = cv.floats ? c->at<float>(cv.out) : nullptr;
    if (cv.pool) {
      if (!cv.bn_pool) {
        LaunchTimer t(c, KC_POOL);
        PlaneOut o = input_planes(c, l + 1);
        o.keep = c->at<uint8_t>(cv.keep);
        if (launch_maxpool2(in, cv.pooled_floats ? c->at<float>(cv.pooled) : nullptr, c->at<uint8_t>(cv.arg), (int64_t)lo.K * lo.B,
                            cv.H, cv.W, cv.Cout, o, s) != 0)
          return fail(LSAM_EINVAL, "pool of convolution %d rejected", l);
      }
      in = cv.pooled_floats ? c->at<float>(cv.pooled) : nullptr;
    }
  }
  if (lo.gap_hw && !lo.conv[lo.n_conv - 1].bn_gap) {
    LaunchTimer t(c, KC_POOL);
    const ConvLayer& cv = lo.conv[lo.n_conv - 1];
    if (launch_avgpool(in, c->at<float>(lo.gap_out), (int64_t)lo.K * lo.B, lo.gap_hw, cv.Cout,
                       lo.ld[lo.n_conv], s) != 0)
      return fail(LSAM_EINVAL, "global average pooling rejected");
  }
  return LSAM_OK;
}

// Backward pass of the convolution layers.  On entry lo.dz[n_conv] holds the gradient of the
// dense layers' input (already zero where that input is zero).  Appends the layers' partial
// sums of squares at ssq[*slots...] when ssq is non-null.
int conv_backward(lsam_ctx* c, const float* X, const float* params, double* ssq, int* slots) {
  const Layout& lo = c->lo;
  hipStream_t s = c->stream;
  float* g = c->at<float>(lo.g);
  // The gradient of a normalised last image's average is the same for every position; it is written for each only where a
  // shortcut hands it on.
  const ConvLayer& last = lo.conv[lo.n_conv - 1];
  const bool from_average = last.bn_gap && !(last.skip && !last.proj && !lo.preact);
  if (lo.gap_hw && !from_average) {
    // the pooled vector's gradient goes back to every position, through the ReLU the image came
    // from unless a pool sits in between (whose backward pass applies that mask)
    LaunchTimer t(c, KC_POOL);
    if (launch_avgpool_backward(c->at<float>(lo.gap_grad), last.pool || last.has_keep ? nullptr : c->at<float>(last.out),
                                last.has_keep && !last.pool ? c->at<uint8_t>(last.keep) : nullptr,
                                c->at<float>(last.pool ? last.dpooled : last.dout), (int64_t)lo.K * lo.B, lo.gap_hw, last.Cout,
                                lo.ld[lo.n_conv], s) != 0)
      return fail(LSAM_EINVAL, "global average pooling (backward) rejected");
  }
  ReduceList list;            // weight gradients whose partial sums wait for the end of the pass
  list.sumsq = ssq; list.sumsq_stride = lo.nblk;
  const auto wait_for_end = [&](ConvGemmDesc& d, size_t at, size_t bytes) {
    d.splitk_ws = c->at<float>(at); d.splitk_bytes = bytes;
    d.list = &list; d.list_slot = *slots;
  };
  ChunkSums have;             // sums of the layer's gradient and normalised values, left by the product that wrote the gradient
  for (int l = lo.n_conv - 1; l >= 0; --l) {
    const ConvLayer& cv = lo.conv[l];
    const Layer& ly = lo.layers[l];
    float* dout = c->at<float>(cv.dout);
    // room for every partial sum of squares this layer's kernels may write, checked up front
    if (ssq && *slots + std::max(gemm_sumsq_capacity(ly.out, ly.in), ly.out / 2) + (ly.out + 63) / 64 +
                       (ly.bn ? 2 * ((ly.out + 63) / 64) : 0) +
                       (ly.proj ? gemm_sumsq_capacity(ly.out, ly.proj_in) + 2 * ((ly.out + 63) / 64) : 0) > lo.nblk)
      return fail(LSAM_ESTATE, "gradient-norm partials would overrun their buffer at convolution %d", l);
    // A block's closing convolution keeps dY: it is also the gradient of the shortcut, added
    // to the block input's gradient further down.  Its dZ goes where Z was (Z is not needed again).
    float* dz = (cv.bn && cv.skip && !lo.preact) ? c->at<float>(cv.z) : dout;
    // In a pre-activation network this convolution's sum may be the identity shortcut of the block
    // above: that block's sum hands its gradient (complete since its own backward pass) down unchanged
    const float* handed = lo.preact && l + 2 < lo.n_conv && lo.conv[l + 2].skip && !lo.conv[l + 2].proj
                              ? c->at<float>(lo.conv[l + 2].dout) : nullptr;
    PlaneOut po;                 // fast layers: dZ as planes, for dW and dX
    if (cv.fast && !cv.first) {
      po.p = c->at<uint16_t>(lo.dzp); po.np = lo.np; po.plane = lo.dzp_elems;
    }
    const uint8_t* keep = cv.has_keep ? c->at<uint8_t>(cv.keep) : nullptr;
    const float* dpooled = cv.pool ? c->at<float>(cv.dpooled) : nullptr;
    GradSource dy{dout, nullptr, 0, 0};     // the gradient behind the ReLU
    if (from_average && l == lo.n_conv - 1) dy = GradSource{c->at<float>(lo.gap_grad), keep, lo.gap_hw, lo.ld[lo.n_conv]};
    if (cv.pool && !cv.bn_pool) {
      // (without a normalisation that is dZ: as floats for a first layer's gradients and the fp32-storage GEMM only)
      LaunchTimer t(c, KC_POOL);
      if (launch_maxpool2_backward(dpooled, c->at<uint8_t>(cv.arg), keep, !cv.bn && po.p ? nullptr : dout, (int64_t)lo.K * lo.B, cv.H,
                                   cv.W, cv.Cout, cv.bn ? PlaneOut{} : po, s) != 0)
        return fail(LSAM_EINVAL, "pool backward of convolution %d rejected", l);
    }
    auto own_gradient = [&]() {
      // nothing reads the floats of a fast layer's dZ but the convolution its sum is handed down to
      const bool floats = !po.p || (lo.preact && cv.skip && !cv.proj);
      if (cv.bn_pool)
        launch_bn_pool_backward(c->at<float>(cv.z), dpooled, c->at<uint8_t>(cv.arg), keep, floats ? dz : nullptr,
                                c->at<float>(cv.stats), params, g, lo.d_pad, ly.gam_off, ly.bet_off, lo.K, lo.B, cv.H, cv.W, cv.Cout,
                                po, s);
      else
        launch_bn_backward_apply(c->at<float>(cv.z), dy, floats ? dz : nullptr, c->at<float>(cv.stats), params, g,
                                 lo.d_pad, ly.gam_off, ly.bet_off, lo.K, cv.rows, cv.Cout, cv.fast ? handed : nullptr, po, s);
    };
    FirstNorm first_norm;
    // The projection of a post-activation block goes first: its planes take the same place
    const bool own_last = cv.proj && !lo.preact;
    if (cv.bn) {
      // dout holds the gradient behind the ReLU; turn it into the gradient of the convolution's
      // output and leave dgamma, dbeta in g
      LaunchTimer t(c, KC_BATCHNORM);
      float* part = c->at<float>(lo.colsum);
      const int chunks = have.chunks ? have.chunks
                         : cv.bn_pool  ? launch_bn_backward_partials(c->at<float>(cv.zmax), GradSource{dpooled, keep, 0, 0},
                                                                   c->at<float>(cv.stats), part, lo.K, cv.rows / 4, cv.Cout, s)
                                       : launch_bn_backward_partials(c->at<float>(cv.z), dy, c->at<float>(cv.stats), part, lo.K,
                                                                     cv.rows, cv.Cout, s);
      if (chunks < 0) return fail(LSAM_EINVAL, "batch normalisation of convolution %d rejected", l);
      {
        const int used = launch_norm_param_grads(part, g, lo.d_pad, ly.gam_off, ly.bet_off, lo.K, chunks, cv.Cout,
                                                 ssq ? ssq + *slots : nullptr, lo.nblk, s);
        if (ssq) *slots += used;
      }
      // (a first layer's weight gradient forms its dZ itself, unless that is a shortcut's as well)
      if (cv.first && !cv.bn_pool && dy.HW == 0 && !handed)
        first_norm = FirstNorm{c->at<float>(cv.z), c->at<float>(cv.stats), params, g, ly.gam_off, ly.bet_off};
      else if (!own_last) own_gradient();
      if (cv.proj && !lo.preact) {
        // the same gradient dY enters the projection's normalisation: dgamma_p, dbeta_p, then
        // the gradient of the 1x1 convolution's output, which takes that output's place
        float* pz = c->at<float>(cv.pz);
        const int pchunks = launch_bn_backward_partials(pz, dy, c->at<float>(cv.pstats), part, lo.K,
                                                        cv.rows, cv.Cout, s);
        if (pchunks < 0) return fail(LSAM_EINVAL, "projection of convolution %d: normalisation rejected", l);
        const int used = launch_norm_param_grads(part, g, lo.d_pad, ly.pgam_off, ly.pbet_off, lo.K, pchunks, cv.Cout,
                                                 ssq ? ssq + *slots : nullptr, lo.nblk, s);
        if (ssq) *slots += used;
        launch_bn_backward_apply(pz, dy, po.p ? nullptr : pz, c->at<float>(cv.pstats), params, g, lo.d_pad, ly.pgam_off,
                                 ly.pbet_off, lo.K, cv.rows, cv.Cout, nullptr, po, s);
      }
    }
    if (handed && !cv.fast) {
      LaunchTimer t(c, KC_POOL);
      if (launch_add_into(dz, handed, (int64_t)lo.K * cv.rows * cv.Cout, s) != 0)
        return fail(LSAM_EINVAL, "shortcut into convolution %d: sum rejected", l);
    }
    if (cv.proj) {
      // dW_p = dZ_p^T S and dS = dZ_p W_p; dS replaces the gathered pixels and reaches the block
      // input's gradient once the block's opening convolution has written that gradient.  In a
      // pre-activation block the projection's output gradient is the sum's own.
      const float* dzp = lo.preact ? dz : c->at<float>(cv.pz);
      float* psub = c->at<float>(cv.psub);
      if (cv.fast) {
        {
          LaunchTimer t(c, KC_GEMM_DW);
          ConvGemmDesc d = plane_desc(c, projection_image(c, lo.conv[l - 1], cv), 1, 0, cv.Cout, ly.proj_in, (int)cv.rows);
          d.C = g + ly.pw_off; d.strideC = lo.d_pad; d.ldC = ly.proj_in;
          if (ssq) { d.sumsq = ssq + *slots; d.sumsq_stride = lo.nblk; }
          if (cv.pwpart_bytes) wait_for_end(d, cv.pwpart, cv.pwpart_bytes);
          int used = 0;
          if (launch_conv_gemm(d, s, &used) != 0) return fail(LSAM_EINVAL, "projection of convolution %d: dW rejected", l);
          if (ssq) *slots += used;
        }
        LaunchTimer t(c, KC_GEMM_DX);
        ConvGemmDesc d = plane_desc(c, gradient_image(c, cv, 1), 0, cv.pwx, (int)cv.rows, ly.proj_in, cv.Cout);
        d.C = psub; d.strideC = cv.rows * cv.skip_C; d.ldC = cv.skip_C;
        if (launch_conv_gemm(d, s) != 0)
          return fail(LSAM_EINVAL, "projection of convolution %d: dX rejected", l);
      } else {
        {
          GemmDesc d{};
          d.A = dzp; d.strideA = cv.rows * cv.Cout; d.ldA = cv.Cout; d.a_kmajor = 0;
          d.B = cv.skip_step == 2 ? psub : c->at<float>(lo.conv[l - 2].out);
          d.strideB = cv.rows * cv.skip_C; d.ldB = cv.skip_C; d.b_kmajor = 0;
          d.C = g + ly.pw_off; d.strideC = lo.d_pad; d.ldC = ly.proj_in;
          d.M = cv.Cout; d.N = ly.proj_in; d.Kd = (int)cv.rows; d.batch = lo.K;
          d.epilogue = EPI_PLAIN;
          split(c, d);
          if (ssq) { d.sumsq = ssq + *slots; d.sumsq_stride = lo.nblk; }
          int used = 0;
          LaunchTimer t(c, KC_GEMM_DW);
          if (launch_gemm(d, s, &used) != 0) return fail(LSAM_EINVAL, "projection of convolution %d: dW rejected", l);
          if (ssq) *slots += used;
        }
        GemmDesc d{};
        d.A = dzp; d.strideA = cv.rows * cv.Cout; d.ldA = cv.Cout; d.a_kmajor = 1;
        d.B = params + ly.pw_off; d.strideB = lo.d_pad; d.ldB = ly.proj_in; d.b_kmajor = 0;
        d.C = psub; d.strideC = cv.rows * cv.skip_C; d.ldC = cv.skip_C;
        d.M = (int)cv.rows; d.N = ly.proj_in; d.Kd = cv.Cout; d.batch = lo.K;
        d.epilogue = EPI_PLAIN;
        split(c, d);
        LaunchTimer t(c, KC_GEMM_DX);
        if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "projection of convolution %d: dX rejected", l);
      }
    }
    if (own_last) {
      LaunchTimer t(c, KC_BATCHNORM);
      own_gradient();
    } else if (po.p && !cv.bn && !cv.pool) {
      LaunchTimer t(c, KC_UNFOLD);
      if (split_gradient(c, dout, cv) != 0) return fail(LSAM_EINVAL, "planes of the gradient of convolution %d rejected", l);
    }
    dout = dz;
    if (cv.first) {
      LaunchTimer t(c, KC_CONV_FIRST);
      const int used = launch_first_conv_wgrad(X, dout, first_norm, c->at<float>(cv.first_partial), g, lo.d_pad,
                                               ly.w_off, ly.b_off, ly.ldw, lo.bf16_math ? 1 : 0,
                                               (lo.bf16_math || cv.bn) ? 1 : 0, lo.K,
                                               cv.rows, cv.H, cv.W, cv.Cin, cv.Cout,
                                               ssq ? ssq + *slots : nullptr, lo.nblk, s);
      if (used < 0) return fail(LSAM_EINVAL, "first convolution's weight gradient rejected");
      if (ssq) *slots += used;
      if (!lo.bf16_math) continue;    // otherwise the bias gradient is still to come, below
    }
    if (!cv.first && cv.fast) {
      LaunchTimer t(c, KC_GEMM_DW);
      ConvGemmDesc d = cv.direct_in ? plane_desc(c, layer_image(c, cv), 1, 0, cv.Cout, ly.in, (int)cv.rows)
                                    : plane_desc(c, stored_image(c, cv), 1, 0, cv.Cout, ly.ldw, (int)cv.rows);
      d.C = g + ly.w_off; d.strideC = lo.d_pad; d.ldC = ly.ldw;
      if (ssq) { d.sumsq = ssq + *slots; d.sumsq_stride = lo.nblk; }
      if (cv.wpart_bytes) wait_for_end(d, cv.wpart, cv.wpart_bytes);
      int used = 0;
      if (launch_conv_gemm(d, s, &used) != 0) return fail(LSAM_EINVAL, "dW product of convolution %d rejected", l);
      if (ssq) *slots += used;
    } else if (!cv.first) {
      GemmDesc d{};
      d.A = dout; d.strideA = cv.rows * cv.Cout; d.ldA = cv.Cout; d.a_kmajor = 0;
      d.B = c->at<float>(cv.col); d.strideB = cv.rows * cv.ldc; d.ldB = cv.ldc; d.b_kmajor = 0;
      if (cv.direct_in) {
        d.B = l == 0 ? X : c->at<float>(lo.conv[l - 1].pool ? lo.conv[l - 1].pooled : lo.conv[l - 1].out);
        d.strideB = cv.rows * cv.Cin; d.ldB = cv.Cin;
        d.unfold = 2; d.unfold_C = cv.Cin; d.unfold_H = cv.H; d.unfold_W = cv.W;
      }
      d.C = g + ly.w_off; d.strideC = lo.d_pad; d.ldC = ly.ldw;
      d.M = cv.Cout; d.N = ly.in; d.Kd = (int)cv.rows; d.batch = lo.K;
      d.epilogue = EPI_PLAIN;
      split(c, d);
      if (ssq) { d.sumsq = ssq + *slots; d.sumsq_stride = lo.nblk; }
      int used = 0;
      LaunchTimer t(c, KC_GEMM_DW);
      if (launch_gemm(d, s, &used) != 0) return fail(LSAM_EINVAL, "dW GEMM of convolution %d rejected", l);
      if (ssq) *slots += used;
    }
    // The bias of a normalised convolution has no influence on the loss: its gradient, the
    // column sums of dZ = gamma/sigma (dY - mean dY - Xh mean(dY Xh)), is zero because Xh sums
    // to zero.  It is left at the zero the gradient buffer starts from instead of being summed
    // up as rounding noise.
    if (!cv.bn) {
      // bias gradient: column sums of dout, in two fixed-order stages
      LaunchTimer t(c, KC_BIAS_GRAD);
      const int chunks = cv.pool ? launch_colsum_partials(dpooled, keep, cv.rows / 4, cv.Cout, lo.K, c->at<float>(lo.colsum), s)
                                 : launch_colsum_partials(dout, nullptr, cv.rows, cv.Cout, lo.K, c->at<float>(lo.colsum), s);
      if (chunks < 0) return fail(LSAM_EINVAL, "bias gradient of convolution %d rejected", l);
      const int used = launch_bias_grad(c->at<float>(lo.colsum), cv.Cout, g + ly.b_off, lo.d_pad,
                                        lo.K, chunks, cv.Cout, ssq ? ssq + *slots : nullptr, lo.nblk, s);
      if (ssq) *slots += used;
    }
    // If this convolution opened a residual block, the gradient of the block output (kept by the closing
    // convolution) also reaches the block input through the shortcut: where the product of this one
    // writes that gradient, or by a launch of its own
    const bool opens = opens_block(lo, l);
    bool shortcut_done = false;
    have = ChunkSums{};
    if (l > 0 && cv.direct_dx) {
      // dX as a convolution of the output gradient with the mirrored filters, written straight
      // into the gradient of the image this layer read.  The product on plane tensors masks it by the ReLU output it came
      // from, pooled or not: the column sums a normalisation takes with it are those of masked values.  The fp32-storage one
      // leaves a pooled image's mask to the pool's backward pass.
      const ConvLayer& below = lo.conv[l - 1];
      if (cv.fast) {
        LaunchTimer t(c, KC_GEMM_DX);
        // (stride 2: in four classes of pixels, the multiply-adds of a product with a stored gradient of
        // the unfolded image without that gradient, nine values written and read per pixel: a step of
        // 64 / 128-channel residual blocks with bf16 products 4.93 -> 4.72 ms, of 16 / 32 / 64 channels in
        // fp32 2.84 -> 2.76; 4 replicas of 128 images of 32 x 32)
        ConvGemmDesc d = plane_desc(c, gradient_image(c, cv, 3), 0, cv.wx, (int)cv.rows, cv.Cin, 9 * cv.Cout);
        d.out_step = cv.stride;
        const int64_t image = (int64_t)lo.B * cv.in_H * cv.in_W * cv.Cin;
        d.C = c->at<float>(below.pool ? below.dpooled : below.dout);
        d.strideC = image; d.ldC = cv.Cin;
        d.epilogue = EPI_MASK;
        if (below.has_keep) d.keep = c->at<uint8_t>(below.keep);
        else d.mask = c->at<float>(below.out);
        d.strideMask = image; d.ldMask = cv.Cin;
        if (shortcut_joins_product(lo, l)) {
          const ConvLayer& top = lo.conv[l + 1];
          d.ldAdd = top.proj ? top.skip_C : top.Cout;
          d.add = c->at<float>(top.proj ? top.psub : top.dout); d.strideAdd = top.rows * d.ldAdd;
          shortcut_done = true;
        }
        if (below.bn && (!below.pool || below.bn_pool) && (!opens || shortcut_done)) {      // the gradient is complete: its sums with it
          d.sums = 2; d.sum_part = c->at<float>(lo.colsum);
          d.sum_z = c->at<float>(below.bn_pool ? below.zmax : below.z); d.sum_stats = c->at<float>(below.stats);
        }
        if (launch_conv_gemm(d, s, nullptr, &have) != 0)
          return fail(LSAM_EINVAL, "dX product of convolution %d rejected", l);
      } else {
        float* wt = c->at<float>(cv.wt);
        {
          LaunchTimer t(c, KC_MISC);
          launch_flip_filters(params + ly.w_off, lo.d_pad, ly.ldw, wt, lo.K, cv.Cout, cv.Cin, s);
        }
        GemmDesc d{};
        d.A = dout; d.strideA = cv.rows * cv.Cout; d.ldA = cv.Cout; d.a_kmajor = 1;
        d.unfold = 1; d.unfold_C = cv.Cout; d.unfold_H = cv.H; d.unfold_W = cv.W;
        d.B = wt; d.strideB = (int64_t)cv.Cin * 9 * cv.Cout; d.ldB = 9 * cv.Cout; d.b_kmajor = 1;
        d.C = c->at<float>(below.pool ? below.dpooled : below.dout);
        d.strideC = cv.rows * cv.Cin; d.ldC = cv.Cin;
        d.M = (int)cv.rows; d.N = cv.Cin; d.Kd = 9 * cv.Cout; d.batch = lo.K;
        d.epilogue = below.pool ? EPI_PLAIN : EPI_MASK;
        if (!below.pool) {
          d.mask = c->at<float>(below.out); d.strideMask = cv.rows * cv.Cin; d.ldMask = cv.Cin;
        }
        split(c, d);
        LaunchTimer t(c, KC_GEMM_DX);
        if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "dX GEMM of convolution %d rejected", l);
      }
    } else if (l > 0) {
      const ConvLayer& below = lo.conv[l - 1];
      float* dcol = c->at<float>(lo.dcol);
      if (cv.fast) {
        LaunchTimer t(c, KC_GEMM_DX);
        ConvGemmDesc d = plane_desc(c, gradient_image(c, cv, 1), 0, cv.wx, (int)cv.rows, cv.ldc, cv.Cout);
        d.C = dcol; d.strideC = cv.rows * cv.ldc; d.ldC = cv.ldc;
        if (launch_conv_gemm(d, s) != 0)
          return fail(LSAM_EINVAL, "dX product of convolution %d rejected", l);
      } else {
        GemmDesc d{};
        d.A = dout; d.strideA = cv.rows * cv.Cout; d.ldA = cv.Cout; d.a_kmajor = 1;
        d.B = params + ly.w_off; d.strideB = lo.d_pad; d.ldB = ly.ldw; d.b_kmajor = 0;
        d.C = dcol; d.strideC = cv.rows * cv.ldc; d.ldC = cv.ldc;
        d.M = (int)cv.rows; d.N = ly.in; d.Kd = cv.Cout; d.batch = lo.K;
        d.epilogue = EPI_PLAIN;
        split(c, d);
        LaunchTimer t(c, KC_GEMM_DX);
        if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "dX GEMM of convolution %d rejected", l);
      }
      // the image this layer read is the layer below's pooled output (its gradient then still
      // has to pass that pool and ReLU) or its ReLU output (masked here)
      LaunchTimer t(c, KC_UNFOLD);
      if (launch_fold3x3(dcol, cv.rows * cv.ldc, cv.ldc,
                         c->at<float>(below.pool ? below.dpooled : below.dout),
                         below.pool ? nullptr : c->at<float>(below.out),
                         cv.rows * cv.stride * cv.stride * cv.Cin, lo.K, lo.B, cv.H, cv.W, cv.Cin,
                         cv.stride, s) != 0)
        return fail(LSAM_EINVAL, "fold of convolution %d rejected", l);
    }
    if (opens && !shortcut_done) {
      const ConvLayer& top = lo.conv[l + 1];
      const ConvLayer& below = lo.conv[l - 1];
      const ShortcutDesc sc{nullptr, below.rows * top.skip_C, top.H, top.W, top.skip_C, top.skip_step};
      LaunchTimer t(c, KC_POOL);
      if (launch_shortcut_backward(c->at<float>(top.proj ? top.psub : top.dout), c->at<float>(below.dout),
                                   c->at<float>(below.out), sc, lo.K, top.rows,
                                   top.proj ? top.skip_C : top.Cout, s) != 0)
        return fail(LSAM_EINVAL, "shortcut of the block closed by convolution %d rejected", l + 1);
    }
  }
  {
    LaunchTimer t(c, KC_GEMM_DW);
    if (launch_reduce_list(list, lo.K, s) != 0) return fail(LSAM_EINVAL, "sums of the weight gradients rejected");
  }
  return LSAM_OK;
}

// Whether the narrow-classifier-head kernels serve the last layer (fp32 dense arithmetic only).
bool head_is_fused(const Layout& lo) {
  return !lo.raw && !lo.bf16 && !lo.bf16_math &&
         head_fits(lo.B, lo.layers[lo.L - 1].out, lo.layers[lo.L - 1].in);
}

// Whether the norm of a layer's unsaved first-pass weight gradient comes from the Gram matrices
// of its factors, half of each (launch_gram_norms): B^2 (out + in) flops, when they take at most a
// quarter of those of the product itself.  (The line of when whole matrices were formed and stored, at half of
// the flops; lsam_layer_info reports the route, and its answers are held to it.)
bool gram_norm_pays(int B, int out, int in) {
  return 2 * (int64_t)B * (out + in) <= (int64_t)out * in;
}

// Whether the fused step and ascent of a bf16 dense model go through all layers in one launch, on 64x64 tiles: where
// the state stays in the caches, unless its products are work enough for 128x128 tiles and a launch each.  Those take
// a launch more a layer and pass and win from about 1e10 multiply-adds a layer (together / a launch each): one
// 3072-4096-1000 with 1024 rows 418 / 402 us, with 4096 1013 / 873; one 2048-2048-2048-2048-2048 with 2048 783 / 776, with
// 4096 1318 / 1195; four 3072-1024-1024-10 with 2048 685 / 669, with 4096 1183 / 1071; one 2500-4000-3000-900 with
// 1024 679 / 710, with 2048 1008 / 988.  A step on 128x128 tiles deals groups of 4 x 4 of them to the eight XCDs, so layers of
// fewer groups do not count: 16 512-512-512-512 with 2048 rows (one group) 772 / 1244.
bool fused_in_group(const Layout& lo) {
  if ((int64_t)lo.K * lo.d_pad * 4 > kCacheResidentBytes) return false;
  double work = 0.;
  for (const Layer& ly : lo.layers)
    if ((int64_t)((ly.out + 511) / 512) * ((ly.in + 511) / 512) >= 8) work += (double)lo.K * lo.B * ly.out * ly.in;
  return work < 1e10 * lo.L;
}

// The dense layers with the dZ and the inputs that the last pass left (A0: the first one's).
void dense_layers(const lsam_ctx* c, const void* A0, DenseLayer* out) {
  const Layout& lo = c->lo;
  for (int l = lo.n_conv; l < lo.L; ++l) {
    const Layer& ly = lo.layers[l];
    out[l] = DenseLayer{c->at<char>(lo.dz[l + 1]), l == lo.n_conv ? A0 : c->at<char>(lo.act[l]), ly.out, ly.in, ly.ldw,
                        ly.w_off, ly.b_off, lo.bf16 ? lo.shadow_off[l] : 0};
  }
}

// forward + backward of all replicas; weights taken from `wts` (fp32 or bf16 per mode).
// `second` selects the pass at the perturbed point: its biases are x_b + scale * g1_b, which in
// fp32 mode sit in the perturbed copy and in bf16 mode are formed in the GEMM epilogue from
// the fp32 master bias and the first-pass bias gradient (only matrix operands are rounded).
// With convolution layers (fp32) the dense layers are l0 = n_conv .. L-1 and read what the
// convolution stack produced.
int forward_backward(lsam_ctx* c, const void* X, const int32_t* labels, const void* wts,
                     bool second, bool fuse_norm, const SamplerFusion* fuse = nullptr,
                     bool norm_only = false) {
  const bool want_loss = !second;
  const Layout& lo = c->lo;
  const int K = lo.K, B = lo.B, L = lo.L, l0 = lo.n_conv;
  const int bf = lo.bf16 ? 1 : 0;
  hipStream_t s = c->stream;
  const float* params = static_cast<const float*>(wts);   // fp32 mode: x or the perturbed copy
  const void* A0 = X;
  if (l0 > 0) {
    int rc = conv_forward(c, static_cast<const float*>(X), params);
    if (rc != LSAM_OK) return rc;
    A0 = c->at<char>(lo.act[l0]);
  }
  // weight matrix l as a GEMM operand: fp32 rows inside the flat vector, or its blocked bf16 copy
  auto wptr = [&](int l) {
    return bf ? (const char*)wts + (size_t)lo.shadow_off[l] * 2
              : (const char*)wts + (size_t)lo.layers[l].w_off * 4;
  };
  const int64_t wstride = bf ? lo.shadow_stride : lo.d_pad;
  auto width = [&](int l) { return l < L ? lo.layers[l].in : lo.layers[L - 1].out; };
  auto astride = [&](int l) { return lo.act_elems(width(l), lo.ld[l]); };

  // A narrow fp32 classifier head is not run as GEMMs: two fused kernels cover its forward
  // pass, the loss, dZ, dX, dW and db.
  const bool head = head_is_fused(lo);
  SplitResult parts{nullptr, 0, 0, 1, nullptr, 0};     // of the product below the head
  for (int l = l0; l < (head ? L - 1 : L); ++l) {
    const Layer& ly = lo.layers[l];
    const bool last = l == L - 1;
    GemmDesc d{};
    d.b32s = bf;
    d.A = l == l0 ? A0 : c->at<char>(lo.act[l]);
    d.strideA = astride(l); d.ldA = lo.ld[l]; d.a_kmajor = 1; d.cbA = b32s_blocks(ly.in);
    d.B = wptr(l); d.strideB = wstride; d.ldB = ly.ldw; d.b_kmajor = 1; d.cbB = b32s_blocks(ly.in);
    d.C = last ? c->at<char>(lo.logits) : c->at<char>(lo.act[l + 1]);
    d.strideC = last ? (int64_t)B * lo.ld[l + 1] : astride(l + 1); d.ldC = lo.ld[l + 1];
    d.cbC = b32s_blocks(ly.out);
    d.M = B; d.N = ly.out; d.Kd = ly.in; d.batch = K;
    d.in_bf16 = bf; d.out_bf16 = bf && !last;
    d.epilogue = last ? EPI_BIAS : EPI_BIAS_RELU;
    d.bias = c->at<float>(lo.x) + ly.b_off; d.strideBias = lo.d_pad;
    if (second && !bf) d.bias = c->at<float>(lo.xt) + ly.b_off;
    if (second && bf) {
      d.bias_dir = c->at<float>(lo.g) + ly.b_off;
      d.bias_scale = c->at<float>(lo.scale);
    }
    split(c, d);
    if (head && l == L - 2) d.parts = &parts;
    LaunchTimer t(c, KC_GEMM_FWD);
    if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "forward GEMM of layer %d rejected", l);
  }
  // the gradient of the first dense layer's input is needed when convolutions sit below it
  const bool need_dA0 = l0 > 0;
  if (head) {
    const Layer& ly = lo.layers[L - 1];
    float* in_act = L - 1 == l0 ? static_cast<float*>(const_cast<void*>(A0)) : c->at<float>(lo.act[L - 1]);   // written only where `parts`
    LaunchTimer t(c, KC_HEAD);
    if (launch_head_forward_backward(in_act, &parts, params + ly.w_off, params + ly.b_off, lo.d_pad, labels,
                                     c->at<float>(lo.dz[L]), lo.ld[L],
                                     want_loss ? c->at<float>(lo.loss_rows) : nullptr,
                                     (L - 1 > l0 || need_dA0) ? c->at<float>(lo.dz[L - 1]) : nullptr,
                                     K, B, ly.out, ly.in, s) != 0)
      return fail(LSAM_EHIP, "classifier-head kernel could not be launched");
  } else {
    LaunchTimer t(c, KC_SOFTMAX_CE);
    launch_softmax_ce(c->at<float>(lo.logits), lo.ld[L], labels, c->at<char>(lo.dz[L]),
                      bf ? astride(L) : (int64_t)lo.ld[L], bf,
                      want_loss ? c->at<float>(lo.loss_rows) : nullptr, K, B, lo.layers[L - 1].out, s);
  }
  float* g = c->at<float>(lo.g);
  // first pass: the kernels that write the gradient also leave the partial sums of its squares
  double* ssq = fuse_norm ? c->at<double>(lo.partials) : nullptr;
  int slots = 0;
  int bias_slots = 0;
  for (int l = l0; l < L; ++l) bias_slots += (lo.layers[l].out + 63) / 64;
  DenseLayer dense[LSAM_MAX_LAYERS], gram[LSAM_MAX_LAYERS];
  int grams = 0;
  dense_layers(c, A0, dense);
  // fp32: all weight and bias gradients share a launch once the dZ are there
  const bool grouped = !bf;
  bool alone[LSAM_MAX_LAYERS] = {};
  if (grouped) dense_gradients_alone(dense + l0, (head ? L - 1 : L) - l0, K, B, lo.bf16_math, alone + l0);
  for (int l = L - 1; l >= l0; --l) {
    const Layer& ly = lo.layers[l];
    const char* dz = c->at<char>(lo.dz[l + 1]);
    const int ld_dz = lo.ld[l + 1];
    const void* act = l == l0 ? A0 : (const void*)c->at<char>(lo.act[l]);
    // the layer's kernels may write this many partial sums of squares: checked before they run
    if (ssq && slots + std::max(gemm_sumsq_capacity(ly.out, ly.in), head_sumsq_slots(ly.in)) +
                       (ly.out + 63) / 64 > lo.nblk)
      return fail(LSAM_ESTATE, "gradient-norm partials would overrun their buffer at layer %d", l);
    if (head && l == L - 1) continue;      // (its dX is done)
    auto weight_grad = [&]() -> int {
      GemmDesc d{};
      d.b32s = bf;
      d.A = dz; d.strideA = astride(l + 1); d.ldA = ld_dz; d.a_kmajor = 0; d.cbA = b32s_blocks(ly.out);
      d.B = act; d.strideB = astride(l); d.ldB = lo.ld[l]; d.b_kmajor = 0; d.cbB = b32s_blocks(ly.in);
      d.C = g + ly.w_off; d.strideC = lo.d_pad; d.ldC = ly.ldw;
      d.M = ly.out; d.N = ly.in; d.Kd = B; d.batch = K;
      d.in_bf16 = bf; d.out_bf16 = 0; d.epilogue = EPI_PLAIN;
      split(c, d);
      if (ssq) { d.sumsq = ssq + slots; d.sumsq_stride = lo.nblk; }
      d.sumsq_only = (ssq && norm_only) ? 1 : 0;   // the gradient itself is recomputed by ascend_pass
      // Of a gradient that is not stored only the norm is wanted, which the Gram matrices of its factors give
      if (d.sumsq_only && gram_norm_pays(B, ly.out, ly.in)) {
        gram[grams++] = dense[l];
        return LSAM_OK;
      }
      SamplerFusion f;
      if (fuse) {
        if (fused_in_group(lo)) return LSAM_OK;
        // this layer's share of the sampler step happens in the epilogue: W_l of x, v, S, y
        f = *fuse;
        f.x += ly.w_off; f.v += ly.w_off; f.S += ly.w_off; f.y += ly.w_off;
        f.shadow += lo.shadow_off[l];
        f.cbShadow = b32s_blocks(ly.in);
        d.fuse = &f;
      }
      int used = 0;
      LaunchTimer t(c, fuse ? KC_GEMM_DW_STEP : d.sumsq_only ? KC_GEMM_DW_NORM : KC_GEMM_DW);
      if (launch_gemm(d, s, &used) != 0) return fail(LSAM_EINVAL, "dW GEMM of layer %d rejected", l);
      if (ssq) slots += used;
      return LSAM_OK;
    };
    auto input_grad = [&]() -> int {
      GemmDesc d{};
      d.b32s = bf;
      d.A = dz; d.strideA = astride(l + 1); d.ldA = ld_dz; d.a_kmajor = 1; d.cbA = b32s_blocks(ly.out);
      d.B = wptr(l); d.strideB = wstride; d.ldB = ly.ldw; d.b_kmajor = 0; d.cbB = b32s_blocks(ly.in);
      d.C = c->at<char>(lo.dz[l]); d.strideC = astride(l); d.ldC = lo.ld[l]; d.cbC = b32s_blocks(ly.in);
      d.M = B; d.N = ly.in; d.Kd = ly.out; d.batch = K;
      d.in_bf16 = bf; d.out_bf16 = bf; d.epilogue = EPI_MASK;
      d.mask = act; d.strideMask = astride(l); d.ldMask = lo.ld[l]; d.cbMask = b32s_blocks(ly.in);
      split(c, d);
      LaunchTimer t(c, KC_GEMM_DX);
      if (launch_gemm(d, s) != 0) return fail(LSAM_EINVAL, "dX GEMM of layer %d rejected", l);
      return LSAM_OK;
    };
    const bool want_dx = l > l0 || need_dA0;
    int rc = LSAM_OK;
    // With the fused step the weight-gradient kernel overwrites the operand copy of W_l that
    // the input gradient still has to read, so that one goes first.
    if (fuse && want_dx && (rc = input_grad()) != LSAM_OK) return rc;
    if ((!grouped || alone[l]) && (rc = weight_grad()) != LSAM_OK) return rc;
    if (!fuse && want_dx && (rc = input_grad()) != LSAM_OK) return rc;
  }
  if (grouped) {
    int most = slots + bias_slots + (head ? head_sumsq_slots(lo.layers[L - 1].in) : 0);
    for (int l = l0; l < (head ? L - 1 : L); ++l)
      if (!alone[l]) most += gemm_sumsq_capacity(lo.layers[l].out, lo.layers[l].in);
    if (ssq && most > lo.nblk) return fail(LSAM_ESTATE, "gradient-norm partials would overrun their buffer at the dense layers");
    LaunchTimer t(c, KC_GEMM_DW);
    const int used = launch_dense_gradients(dense + l0, (head ? L - 1 : L) - l0, head ? dense + L - 1 : nullptr, K, B, g,
                                            lo.d_pad, ssq ? ssq + slots : nullptr, lo.nblk, lo.bf16_math, s);
    if (used < 0) return fail(LSAM_EINVAL, "weight gradients of the dense layers rejected");
    if (ssq) slots += used;
  }
  if (bf) {
    if (ssq && slots + (grams ? gram_slots(grams, K, B) : 0) + bias_slots > lo.nblk)
      return fail(LSAM_ESTATE, "gradient-norm partials would overrun their buffer at the Gram products");
    if (grams > 0) {
      LaunchTimer t(c, KC_GEMM_DW_NORM);
      const int used = launch_gram_norms(gram, grams, K, B, ssq + slots, lo.nblk, s);
      if (used < 0) return fail(LSAM_EINVAL, "Gram products rejected");
      slots += used;
    }
    if (fuse && fused_in_group(lo)) {
      LaunchTimer t(c, KC_GEMM_DW_STEP);
      if (launch_fused_group(dense, L, K, B, lo.d_pad, fuse, nullptr, s) != 0) return fail(LSAM_EINVAL, "step GEMMs rejected");
    }
    LaunchTimer t(c, KC_BIAS_GRAD);
    const int used = launch_bias_grads_blocked(dense, L, K, B, g, lo.d_pad, ssq ? ssq + slots : nullptr, lo.nblk, fuse, s);
    if (ssq) slots += used;
  }
  if (l0 > 0) {
    int rc = conv_backward(c, static_cast<const float*>(X), params, ssq, &slots);
    if (rc != LSAM_OK) return rc;
  }
  if (ssq) {
    if (slots > lo.nblk) return fail(LSAM_ESTATE, "gradient-norm partials overran their buffer");
    c->norm_slots = slots;
  }
  return check_launch("forward/backward");
}

// bf16 dense model with the fused step: the weight gradients of the first pass were only summed
// (their squares), not stored.  Now that the norm is known each is computed once more from the
// dZ_l and A_{l-1} the first pass left behind, and its epilogue writes the operand copy of the
// perturbed weights bf16(x + scale g1) directly: 6 bytes per parameter (x read, copy written)
// instead of the 14 of storing g1, reading it back with x and writing the copy, at the price of
// one more contraction per layer, which the matrix units have room for.  Biases need no copy:
// the second pass's GEMMs form x_b + scale g1_b from the stored bias gradient.
int ascend_pass(lsam_ctx* c, const void* A0) {
  const Layout& lo = c->lo;
  const int K = lo.K, B = lo.B, L = lo.L;
  if (fused_in_group(lo)) {
    DenseLayer dense[LSAM_MAX_LAYERS];
    dense_layers(c, A0, dense);
    const AscentFusion f{c->at<float>(lo.x), c->at<float>(lo.scale), c->at<uint16_t>(lo.xt), lo.shadow_stride, 0};
    LaunchTimer t(c, KC_GEMM_DW_ASCEND);
    if (launch_fused_group(dense, L, K, B, lo.d_pad, nullptr, &f, c->stream) != 0) return fail(LSAM_EINVAL, "ascent GEMMs rejected");
    return check_launch("ascent GEMMs");
  }
  auto width = [&](int l) { return l < L ? lo.layers[l].in : lo.layers[L - 1].out; };
  auto astride = [&](int l) { return lo.act_elems(width(l), lo.ld[l]); };
  for (int l = L - 1; l >= 0; --l) {
    const Layer& ly = lo.layers[l];
    GemmDesc d{};
    d.b32s = 1;
    d.A = c->at<char>(lo.dz[l + 1]); d.strideA = astride(l + 1); d.ldA = lo.ld[l + 1]; d.a_kmajor = 0;
    d.cbA = b32s_blocks(ly.out);
    d.B = l == 0 ? A0 : (const void*)c->at<char>(lo.act[l]); d.strideB = astride(l); d.ldB = lo.ld[l];
    d.b_kmajor = 0; d.cbB = b32s_blocks(ly.in);
    d.C = c->at<float>(lo.g) + ly.w_off; d.strideC = lo.d_pad; d.ldC = ly.ldw;
    d.M = ly.out; d.N = ly.in; d.Kd = B; d.batch = K;
    d.in_bf16 = 1; d.out_bf16 = 0; d.epilogue = EPI_PLAIN;
    AscentFusion f;
    f.x = c->at<float>(lo.x) + ly.w_off;
    f.scale = c->at<float>(lo.scale);
    f.shadow = c->at<uint16_t>(lo.xt) + lo.shadow_off[l];
    f.shadow_stride = lo.shadow_stride;
    f.cbShadow = b32s_blocks(ly.in);
    d.ascend = &f;
    LaunchTimer t(c, KC_GEMM_DW_ASCEND);
    if (launch_gemm(d, c->stream) != 0) return fail(LSAM_EINVAL, "ascent GEMM of layer %d rejected", l);
  }
  return check_launch("ascent GEMMs");
}

// Norm of g1 and the perturbed point.  `partials_ready`: the kernels that wrote g1 already
// left the partial sums of its squares.  With rho = 0 the perturbed point is x itself and is
// not written.
int update_tail_first(lsam_ctx* c, const float* g1, int64_t g_stride, int64_t n, float* loss,
                      bool partials_ready, bool perturb = true) {
  const Layout& lo = c->lo;
  hipStream_t s = c->stream;
  const int nparts = partials_ready ? c->norm_slots : std::min(lo.nblk, kMaxPartials);
  if (!partials_ready) {
    LaunchTimer t(c, KC_SUMSQ);
    launch_sumsq_partials(g1, g_stride, n, lo.K, c->at<double>(lo.partials), nparts, s);
  }
  const NormSums sums{c->at<double>(lo.partials), nparts, partials_ready ? lo.nblk : nparts, c->rho, c->cfg.gamma,
                      c->at<float>(lo.norms), c->at<float>(lo.scale), lo.raw ? nullptr : c->at<float>(lo.loss_rows), lo.B,
                      lo.raw ? nullptr : (loss ? loss : c->at<float>(lo.loss)), c->at<int32_t>(lo.restart)};
  const bool with_perturb = c->rho != 0.f && perturb;
  const bool joined = with_perturb && !lo.bf16 && nparts <= kProloguePartials;
  if (!joined) {
    LaunchTimer t(c, KC_NORM_FINISH);
    launch_norm_finish(sums.partials, nparts, sums.pstride, lo.K, sums.rho, sums.gamma, sums.norms, sums.scale,
                       sums.loss_rows, lo.B, sums.loss_out, s, sums.restart);
  }
  if (with_perturb) {
    LaunchTimer t(c, KC_PERTURB);
    launch_perturb(c->at<float>(lo.x), g1, g_stride, sums.scale, lo.bf16 ? nullptr : c->at<float>(lo.xt),
                   lo.bf16 ? c->at<uint16_t>(lo.xt) : nullptr, &lo.map, lo.shadow_stride, lo.d_pad, n, lo.K, s,
                   joined ? &sums : nullptr);
  }
  return check_launch("norm/perturb");
}

// Whether the sampler step of this configuration can ride in the epilogues of the second
// pass's weight-gradient GEMMs: bf16 dense model, Algorithm 2 (the data-parallel baseline needs
// the averaged gradient first), no Langevin noise.
bool can_fuse_step(const lsam_ctx* c) {
  return c->lo.bf16 && c->cfg.algorithm == LSAM_ALG_LSAM && !(c->cfg.noise_scale > 0.f) && c->fuse_step;
}

// `up`: the norm of g1 and the perturbed point are still to come as well (raw vectors).
int update_tail_second(lsam_ctx* c, const float* g2, int64_t g_stride, int64_t n, bool already_stepped = false,
                       const AscentPass* up = nullptr) {
  const Layout& lo = c->lo;
  if (already_stepped) {
    ++c->t_step;
    c->sched.tick();
    return check_launch("descent");
  }
  ReplicaScalars lam;
  for (int i = 0; i < lo.K; ++i) lam.v[i] = coupling(c, i);
  const NoiseMap* noise = nullptr;
  if (c->cfg.noise_scale > 0.f) {
    c->noise.step = c->t_step;
    c->noise.amp = (float)((double)c->cfg.noise_scale * std::sqrt(2.0 * (double)c->lr));
    noise = &c->noise;
  }
  if (up) {
    LaunchTimer t(c, KC_DESCENT);
    launch_raw_descent(c->at<float>(lo.x), g2, g_stride, c->at<float>(lo.v), c->at<float>(lo.S), c->at<float>(lo.y),
                       lo.d_pad, n, lo.K, lam, c->lr, c->cfg.momentum, c->cfg.nesterov, noise, c->stream,
                       c->at<int32_t>(lo.restart), *up);
  } else {
    LaunchTimer t(c, KC_DESCENT);
    launch_descent(c->at<float>(lo.x), g2, g_stride, c->at<float>(lo.v), c->at<float>(lo.S),
                   c->at<float>(lo.y), lo.bf16 ? c->at<uint16_t>(lo.xt) : nullptr, &lo.map,
                   lo.shadow_stride, lo.d_pad, n, lo.K, lam, c->lr, c->cfg.momentum, c->cfg.nesterov,
                   noise, c->stream, c->at<int32_t>(lo.restart));
  }
  ++c->t_step;
  c->sched.tick();
  return check_launch("descent");
}

// Host <-> device transfers go through a pinned staging buffer owned by the context, in
// pieces of at most kStageBytes, each followed by a stream synchronisation: pageable-memory
// copies are left to no one else's staging (a strided device-to-host copy into fresh pageable
// memory was seen to return with a few words not yet written when run under the profiler).
constexpr size_t kStageBytes = 64u << 20;

int ensure_stage(lsam_ctx* c) {
  if (c->stage) return LSAM_OK;
  HIP_TRY(hipHostMalloc(&c->stage, kStageBytes, hipHostMallocDefault));
  return LSAM_OK;
}

int to_host(lsam_ctx* c, void* dst, const void* src_dev, size_t bytes) {
  int rc = ensure_stage(c);
  if (rc != LSAM_OK) return rc;
  char* d = static_cast<char*>(dst);
  const char* s = static_cast<const char*>(src_dev);
  for (size_t off = 0; off < bytes; off += kStageBytes) {
    const size_t n = std::min(kStageBytes, bytes - off);
    HIP_TRY(hipMemcpyAsync(c->stage, s + off, n, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    memcpy(d + off, c->stage, n);
  }
  return LSAM_OK;
}

int to_device(lsam_ctx* c, void* dst_dev, const void* src, size_t bytes) {
  int rc = ensure_stage(c);
  if (rc != LSAM_OK) return rc;
  char* d = static_cast<char*>(dst_dev);
  const char* s = static_cast<const char*>(src);
  for (size_t off = 0; off < bytes; off += kStageBytes) {
    const size_t n = std::min(kStageBytes, bytes - off);
    memcpy(c->stage, s + off, n);
    HIP_TRY(hipMemcpyAsync(d + off, c->stage, n, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  return LSAM_OK;
}

// Copies between the public flat layout (host) and one padded replica vector (device): the
// rows of W_l lose or gain their padding on the host side of the staging buffer.
int copy_in(lsam_ctx* c, const float* src_flat, float* dst_dev) {
  const Layout& lo = c->lo;
  if (lo.raw) return to_device(c, dst_dev, src_flat, (size_t)lo.d * 4);
  int rc = ensure_stage(c);
  if (rc != LSAM_OK) return rc;
  float* stage = static_cast<float*>(c->stage);
  for (const Piece& p : lo.pieces) {
    if (p.rows == 1) {
      if ((rc = to_device(c, dst_dev + p.off, src_flat + p.flat, (size_t)p.cols * 4)) != LSAM_OK) return rc;
      continue;
    }
    const int64_t rows_per = std::max<int64_t>(1, (int64_t)(kStageBytes / 4) / p.ld);
    for (int64_t r0 = 0; r0 < p.rows; r0 += rows_per) {
      const int64_t nr = std::min<int64_t>(rows_per, p.rows - r0);
      for (int64_t r = 0; r < nr; ++r) {
        memcpy(stage + r * p.ld, src_flat + p.flat + (r0 + r) * p.cols, (size_t)p.cols * 4);
        if (p.ld > p.cols) memset(stage + r * p.ld + p.cols, 0, (size_t)(p.ld - p.cols) * 4);
      }
      HIP_TRY(hipMemcpyAsync(dst_dev + p.off + r0 * p.ld, stage, (size_t)nr * p.ld * 4,
                             hipMemcpyHostToDevice, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
    }
  }
  return LSAM_OK;
}

int copy_out(lsam_ctx* c, const float* src_dev, float* dst_flat) {
  const Layout& lo = c->lo;
  if (lo.raw) return to_host(c, dst_flat, src_dev, (size_t)lo.d * 4);
  int rc = ensure_stage(c);
  if (rc != LSAM_OK) return rc;
  const float* stage = static_cast<const float*>(c->stage);
  for (const Piece& p : lo.pieces) {
    if (p.rows == 1) {
      if ((rc = to_host(c, dst_flat + p.flat, src_dev + p.off, (size_t)p.cols * 4)) != LSAM_OK) return rc;
      continue;
    }
    const int64_t rows_per = std::max<int64_t>(1, (int64_t)(kStageBytes / 4) / p.ld);
    for (int64_t r0 = 0; r0 < p.rows; r0 += rows_per) {
      const int64_t nr = std::min<int64_t>(rows_per, p.rows - r0);
      HIP_TRY(hipMemcpyAsync(c->stage, src_dev + p.off + r0 * p.ld, (size_t)nr * p.ld * 4,
                             hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      for (int64_t r = 0; r < nr; ++r)
        memcpy(dst_flat + p.flat + (r0 + r) * p.cols, stage + r * p.ld, (size_t)p.cols * 4);
    }
  }
  return LSAM_OK;
}

}  // namespace

extern "C" {

const char* lsam_last_error(void) { return g_err.c_str(); }

int64_t lsam_num_params(const lsam_config* cfg) {
  if (check_config(cfg) != LSAM_OK) return -1;
  Layout lo;
  build_layout(*cfg, lo);
  return lo.d;
}

size_t lsam_workspace_bytes(const lsam_config* cfg) {
  if (check_config(cfg) != LSAM_OK) return 0;
  Layout lo;
  build_layout(*cfg, lo);
  return lo.total;
}

int lsam_schedule_replay(const lsam_config* cfg, int32_t n_ticks, int32_t* due_out,
                         int32_t* tau_out) {
  int rc = check_config(cfg);
  if (rc != LSAM_OK) return rc;
  if (n_ticks < 0 || (!due_out && !tau_out)) return fail(LSAM_EINVAL, "nothing to replay into");
  Schedule s;
  s.init(*cfg);
  for (int t = 0; t < n_ticks; ++t) {
    if (tau_out)
      for (int i = 0; i < cfg->K; ++i) tau_out[(int64_t)t * cfg->K + i] = s.tau()[i];
    s.tick();
    DueList d = s.due();
    if (due_out) {
      for (int i = 0; i < cfg->K; ++i) due_out[(int64_t)t * cfg->K + i] = 0;
      for (int j = 0; j < d.n; ++j) due_out[(int64_t)t * cfg->K + d.idx[j]] = 1;
    }
    if (d.n) s.served(d);
  }
  return LSAM_OK;
}

int lsam_init(const lsam_config* cfg, const float* init_params, int64_t n_init, void* workspace,
              size_t workspace_bytes, void* stream, lsam_ctx** out) {
  if (!out) return fail(LSAM_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_config(cfg);
  if (rc != LSAM_OK) return rc;
  if (!init_params) return fail(LSAM_EINVAL, "init_params is NULL");
  if (!workspace) return fail(LSAM_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(workspace) & 255)
    return fail(LSAM_EINVAL, "workspace must be 256-byte aligned");
  lsam_ctx* c = new (std::nothrow) lsam_ctx();
  if (!c) return fail(LSAM_ENOMEM, "host allocation failed");
  c->cfg = *cfg;
  if (cfg->n_layers > 0) {
    c->dims.assign(cfg->dims, cfg->dims + cfg->n_layers + 1);
    c->cfg.dims = c->dims.data();
  } else {
    c->cfg.dims = nullptr;
  }
  if (cfg->tau) {
    c->tau_explicit.assign(cfg->tau, cfg->tau + cfg->K);
    c->cfg.tau = c->tau_explicit.data();
  }
  build_layout(c->cfg, c->lo);
  const Layout& lo = c->lo;
  if (n_init != lo.d && n_init != (int64_t)(lo.K + 1) * lo.d) {
    delete c;
    return fail(LSAM_EINVAL, "n_init=%lld must be d=%lld or (K+1)*d", (long long)n_init,
                (long long)lo.d);
  }
  if (workspace_bytes < lo.total) {
    delete c;
    return fail(LSAM_ENOMEM, "workspace holds %zu bytes, %zu needed", workspace_bytes, lo.total);
  }
  c->ws = static_cast<char*>(workspace);
  c->stream = static_cast<hipStream_t>(stream);
  {
    NoiseMap& nm = c->noise;
    nm.key0 = (uint32_t)(c->cfg.noise_seed & 0xFFFFFFFFu);
    nm.key1 = (uint32_t)(c->cfg.noise_seed >> 32);
    nm.raw_n = lo.raw ? lo.d : 0;
    nm.n = 0;
    nm.seg = nullptr;
  }
  c->lr = cfg->lr;
  c->rho = cfg->rho;
  c->sched.init(c->cfg);

  auto bail = [&](int code) {
    if (c->stage) (void)hipHostFree(c->stage);
    delete c;
    return code;
  };
  launch_fill_zero(c->ws, lo.total, c->stream);
  if (check_launch("zero fill") != LSAM_OK) return bail(LSAM_EHIP);
  if (hipStreamSynchronize(c->stream) != hipSuccess)
    return bail(fail(LSAM_EHIP, "stream synchronize failed during init"));
  if (lo.noise_segs) {
    // the noise generator's table: one run per parameter group, in the layout's order
    std::vector<NoiseSeg> segs;
    for (const Piece& p : lo.pieces)
      segs.push_back(NoiseSeg{p.off, p.off + (p.rows == 1 ? (int64_t)p.cols : (int64_t)p.rows * p.ld), p.ld,
                              p.cols, p.code, 0});
    if ((rc = to_device(c, c->at<char>(lo.noise_segs), segs.data(), segs.size() * sizeof(NoiseSeg))) != LSAM_OK)
      return bail(rc);
    c->noise.seg = c->at<NoiseSeg>(lo.noise_segs);
    c->noise.n = (int)segs.size();
  }
  if (!lo.banks.empty() &&
      (rc = to_device(c, c->at<char>(lo.banks_at), lo.banks.data(), lo.banks.size() * sizeof(FilterBank))) != LSAM_OK)
    return bail(rc);
  float* x = c->at<float>(lo.x);
  float* y = c->at<float>(lo.y);
  if (n_init == lo.d) {
    if ((rc = copy_in(c, init_params, y)) != LSAM_OK) return bail(rc);
    launch_broadcast(y, x, lo.d_pad, lo.d_pad, lo.K, c->stream);
  } else {
    for (int i = 0; i < lo.K; ++i)
      if ((rc = copy_in(c, init_params + (int64_t)i * lo.d, x + (int64_t)i * lo.d_pad)) != LSAM_OK)
        return bail(rc);
    if ((rc = copy_in(c, init_params + (int64_t)lo.K * lo.d, y)) != LSAM_OK) return bail(rc);
  }
  if (lo.bf16)
    launch_shadow_refresh(x, c->at<uint16_t>(lo.xt), lo.map, lo.d_pad, lo.shadow_stride, lo.d_pad,
                          lo.K, c->stream);
  if (check_launch("parameter broadcast") != LSAM_OK) return bail(LSAM_EHIP);
  if (hipStreamSynchronize(c->stream) != hipSuccess)
    return bail(fail(LSAM_EHIP, "stream synchronize failed during init"));
  *out = c;
  return LSAM_OK;
}

int lsam_step(lsam_ctx* c, const void* X, const int32_t* labels, float* loss) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  if (c->lo.raw) return fail(LSAM_ESTATE, "lsam_step needs an MLP configuration");
  if (!X || !labels) return fail(LSAM_EINVAL, "X or labels is NULL");
  const Layout& lo = c->lo;
  const void* A0 = X;
  if (reinterpret_cast<uintptr_t>(X) & 15) return fail(LSAM_EINVAL, "X must be 16-byte aligned");
  if (lo.bf16) {
    LaunchTimer t(c, KC_MISC);     // the input joins the other bf16 tensors in the blocked layout
    launch_rowmajor_to_b32s(static_cast<const uint16_t*>(X), c->at<uint16_t>(lo.a0), lo.B,
                            lo.layers[0].in, lo.K, c->stream);
    A0 = c->at<char>(lo.a0);
  } else if (lo.need_a0) {
    LaunchTimer t(c, KC_MISC);
    launch_pad_rows(X, c->at<char>(lo.a0), (int64_t)lo.K * lo.B, lo.layers[0].in, lo.ld[0],
                    (int)lo.es(), c->stream);
    A0 = c->at<char>(lo.a0);
  }
  int rc;
  const bool dp = c->cfg.algorithm == LSAM_ALG_DATA_PARALLEL;
  float* g = c->at<float>(lo.g);
  // data-parallel baseline: every replica's gradient is replaced by the average over replicas
  auto average = [&]() {
    LaunchTimer t(c, KC_MISC);
    launch_grad_mean(g, lo.d_pad, g, lo.d_pad, lo.d_pad, lo.K, lo.K, c->stream);
  };
  const void* w1 = lo.bf16 ? (const void*)c->at<char>(lo.xt) : (const void*)c->at<char>(lo.x);
  // bf16 dense model, Algorithm 2, no noise: neither gradient of a weight matrix is stored.
  // First pass: sums of squares only; then the ascent GEMMs; second pass: the sampler step in
  // the weight-gradient epilogues.
  const bool fused = c->rho != 0.f && can_fuse_step(c);
  if ((rc = forward_backward(c, A0, labels, w1, false, !dp, nullptr, fused)) != LSAM_OK) return rc;
  if (dp) average();
  if ((rc = update_tail_first(c, g, lo.d_pad, lo.d_pad, loss, !dp, !fused)) != LSAM_OK) return rc;
  if (fused && (rc = ascend_pass(c, A0)) != LSAM_OK) return rc;
  bool stepped = false;
  if (c->rho != 0.f) {     // otherwise the perturbed point is x and g already is its gradient
    SamplerFusion f;
    if (fused) {
      f.x = c->at<float>(lo.x); f.v = c->at<float>(lo.v); f.S = c->at<float>(lo.S);
      f.restart = c->at<int32_t>(lo.restart);
      f.y = c->at<float>(lo.y);
      f.shadow = c->at<uint16_t>(lo.xt); f.shadow_stride = lo.shadow_stride; f.cbShadow = 0;
      for (int i = 0; i < lo.K; ++i) f.lam.v[i] = coupling(c, i);
      f.lr = c->lr; f.mu = c->cfg.momentum; f.nesterov = c->cfg.nesterov;
      stepped = true;
    }
    if ((rc = forward_backward(c, A0, labels, c->at<char>(lo.xt), true, false, stepped ? &f : nullptr)) != LSAM_OK)
      return rc;
    if (dp) average();
  }
  return update_tail_second(c, g, lo.d_pad, lo.d_pad, stepped);
}

int lsam_step_grads(lsam_ctx* c, const float* g1, const float* g2) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  if (!c->lo.raw) return fail(LSAM_ESTATE, "lsam_step_grads needs raw-vector mode");
  if (!g1 || !g2) return fail(LSAM_EINVAL, "g1 or g2 is NULL");
  if ((reinterpret_cast<uintptr_t>(g1) & 3) || (reinterpret_cast<uintptr_t>(g2) & 3))
    return fail(LSAM_EINVAL, "gradients must be 4-byte aligned");
  int rc;
  const Layout& lo = c->lo;
  if (c->cfg.algorithm == LSAM_ALG_DATA_PARALLEL) {
    // one averaged vector, read by every replica (row stride 0)
    float* m = c->at<float>(lo.gmean);
    {
      LaunchTimer t(c, KC_MISC);
      launch_grad_mean(g1, lo.d, m, 0, lo.d, lo.K, 1, c->stream);
    }
    if ((rc = update_tail_first(c, m, 0, lo.d, nullptr, false)) != LSAM_OK) return rc;
    {
      LaunchTimer t(c, KC_MISC);
      launch_grad_mean(g2, lo.d, m, 0, lo.d, lo.K, 1, c->stream);
    }
    return update_tail_second(c, m, 0, lo.d);
  }
  AscentPass up;
  up.g1 = g1; up.g1_stride = lo.d;
  up.partials = c->at<double>(lo.partials); up.nblk = lo.nblk;
  up.rho = c->rho; up.gamma = c->cfg.gamma;
  up.norms = c->at<float>(lo.norms); up.scale = c->at<float>(lo.scale);
  if (c->rho != 0.f) up.xt = c->at<float>(lo.xt);
  {
    LaunchTimer t(c, KC_SUMSQ);
    launch_raw_norm(lo.d, lo.K, c->stream, c->at<int32_t>(lo.restart), up);
  }
  return update_tail_second(c, g2, lo.d, lo.d, false, &up);
}

int lsam_sync(lsam_ctx* c) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  if (c->cfg.algorithm == LSAM_ALG_DATA_PARALLEL) return 0;   // no center in that baseline
  const Layout& lo = c->lo;
  const DueList due = c->sched.due();
  if (due.n == 0) return 0;
  const int64_t m = c->sched.samples(due);
  {
    LaunchTimer t(c, KC_CENTER);
    launch_center(c->at<float>(lo.S), c->at<float>(lo.y), c->at<float>(lo.gprev), lo.d_pad,
                  lo.raw ? lo.d : lo.d_pad, due, (float)(1.0 / (double)m), c->cfg.beta,
                  c->cfg.lr_center, c->sched.t_y() > 0 ? 1 : 0, c->stream, c->at<int32_t>(lo.restart));
  }
  int rc = check_launch("center update");
  if (rc != LSAM_OK) return rc;
  c->sched.served(due);
  return due.n;
}

int lsam_get_buffer(lsam_ctx* c, int32_t which, int32_t replica, float* dst, int64_t n) {
  if (!c || !dst) return fail(LSAM_EINVAL, "ctx or dst is NULL");
  const Layout& lo = c->lo;
  if (n != lo.d) return fail(LSAM_EINVAL, "n=%lld must equal d=%lld", (long long)n, (long long)lo.d);
  if (replica < -1 || replica >= lo.K) return fail(LSAM_EINVAL, "replica %d out of range", replica);
  HIP_TRY(hipStreamSynchronize(c->stream));
  const int64_t roff = (int64_t)(replica < 0 ? 0 : replica) * lo.d_pad;
  switch (which) {
    case LSAM_BUF_PARAMS:
      return copy_out(c, replica < 0 ? c->at<float>(lo.y) : c->at<float>(lo.x) + roff, dst);
    case LSAM_BUF_CENTER_DIR:
      return copy_out(c, c->at<float>(lo.gprev), dst);
    default: break;
  }
  if (replica < 0) return fail(LSAM_EINVAL, "replica -1 is valid for the parameters only");
  switch (which) {
    case LSAM_BUF_VELOCITY: return copy_out(c, c->at<float>(lo.v) + roff, dst);
    case LSAM_BUF_ITER_SUM: {
      // a sum the last center update served reads as zero; its memory is rewritten by the next step
      int32_t mark = 0;
      int rc = to_host(c, &mark, c->at<int32_t>(lo.restart) + replica, 4);
      if (rc != LSAM_OK) return rc;
      if (mark == 2) {
        memset(dst, 0, (size_t)n * 4);
        return LSAM_OK;
      }
      return copy_out(c, c->at<float>(lo.S) + roff, dst);
    }
    case LSAM_BUF_GRAD:
      if (lo.raw) return fail(LSAM_ESTATE, "raw-vector mode keeps no gradient buffer");
      return copy_out(c, c->at<float>(lo.g) + roff, dst);
    case LSAM_BUF_PERTURBED: {
      if (!lo.bf16) return copy_out(c, c->at<float>(lo.xt) + roff, dst);
      // bf16 operand copy of the weight matrices: fetch this replica's copy, widen and undo
      // the blocked layout on the host; biases are not part of the copy (the GEMMs read the
      // fp32 ones), they are reported from the master parameters
      std::vector<uint16_t> h((size_t)lo.shadow_stride);
      int rc0 = to_host(c, h.data(), c->at<uint16_t>(lo.xt) + (int64_t)replica * lo.shadow_stride,
                        (size_t)lo.shadow_stride * 2);
      if (rc0 != LSAM_OK) return rc0;
      int rc = copy_out(c, c->at<float>(lo.x) + roff, dst);
      if (rc != LSAM_OK) return rc;
      for (int l = 0; l < lo.L; ++l) {
        const Layer& ly = lo.layers[l];
        const int cb = b32s_blocks(ly.in);
        for (int r = 0; r < ly.out; ++r)
          for (int q = 0; q < ly.in; ++q) {
            const uint32_t u = (uint32_t)h[(size_t)(lo.shadow_off[l] + b32s_offset(r, q, cb))] << 16;
            float f;
            memcpy(&f, &u, 4);
            dst[ly.w_flat + (int64_t)r * ly.in + q] = f;
          }
      }
      return LSAM_OK;
    }
    default: return fail(LSAM_EINVAL, "unknown buffer id %d", which);
  }
}

int lsam_set_buffer(lsam_ctx* c, int32_t which, int32_t replica, const float* src, int64_t n) {
  if (!c || !src) return fail(LSAM_EINVAL, "ctx or src is NULL");
  const Layout& lo = c->lo;
  if (n != lo.d) return fail(LSAM_EINVAL, "n=%lld must equal d=%lld", (long long)n, (long long)lo.d);
  if (replica < -1 || replica >= lo.K) return fail(LSAM_EINVAL, "replica %d out of range", replica);
  HIP_TRY(hipStreamSynchronize(c->stream));
  const int64_t roff = (int64_t)(replica < 0 ? 0 : replica) * lo.d_pad;
  float* dst = nullptr;
  switch (which) {
    case LSAM_BUF_PARAMS: dst = replica < 0 ? c->at<float>(lo.y) : c->at<float>(lo.x) + roff; break;
    case LSAM_BUF_CENTER_DIR: dst = c->at<float>(lo.gprev); break;
    case LSAM_BUF_VELOCITY: dst = replica < 0 ? nullptr : c->at<float>(lo.v) + roff; break;
    case LSAM_BUF_ITER_SUM: dst = replica < 0 ? nullptr : c->at<float>(lo.S) + roff; break;
    default: return fail(LSAM_EINVAL, "buffer id %d cannot be set", which);
  }
  if (!dst) return fail(LSAM_EINVAL, "replica -1 is valid for the parameters only");
  int rc = copy_in(c, src, dst);
  if (rc != LSAM_OK) return rc;
  if (which == LSAM_BUF_ITER_SUM) {
    // the sum is what the caller wrote from now on, not "zero since the last center update"
    const int32_t none = 0;
    if ((rc = to_device(c, c->at<int32_t>(lo.restart) + replica, &none, 4)) != LSAM_OK) return rc;
  }
  if (which == LSAM_BUF_PARAMS && replica >= 0 && lo.bf16) {
    launch_shadow_refresh(dst, c->at<uint16_t>(lo.xt) + (int64_t)replica * lo.shadow_stride, lo.map,
                          lo.d_pad, lo.shadow_stride, lo.d_pad, 1, c->stream);
    if ((rc = check_launch("bf16 operand refresh")) != LSAM_OK) return rc;
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  return LSAM_OK;
}

int lsam_get_params(lsam_ctx* c, int32_t replica, float* dst, int64_t n) {
  return lsam_get_buffer(c, LSAM_BUF_PARAMS, replica, dst, n);
}

int lsam_get_norms(lsam_ctx* c, float* dst) {
  if (!c || !dst) return fail(LSAM_EINVAL, "ctx or dst is NULL");
  HIP_TRY(hipStreamSynchronize(c->stream));
  {
    int rc0 = to_host(c, dst, c->at<float>(c->lo.norms), (size_t)c->lo.K * 4);
    if (rc0 != LSAM_OK) return rc0;
  }
  return LSAM_OK;
}

int lsam_get_schedule(lsam_ctx* c, int32_t* tau_out, int32_t* count_out, int64_t* t_y_out) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  for (int i = 0; i < c->lo.K; ++i) {
    if (tau_out) tau_out[i] = c->sched.tau()[i];
    if (count_out) count_out[i] = c->sched.count()[i];
  }
  if (t_y_out) *t_y_out = c->sched.t_y();
  return LSAM_OK;
}

int lsam_layer_info(lsam_ctx* c, int32_t layer, int32_t* info, int32_t n) {
  if (!c || !info) return fail(LSAM_EINVAL, "ctx or info is NULL");
  const Layout& lo = c->lo;
  if (lo.raw) return fail(LSAM_ESTATE, "raw-vector mode has no layers");
  if (layer < 0 || layer >= lo.L) return fail(LSAM_EINVAL, "layer %d out of range 0..%d", layer, lo.L - 1);
  if (n < LSAM_LAYER_INFO_FIELDS) return fail(LSAM_EINVAL, "info needs %d entries", LSAM_LAYER_INFO_FIELDS);
  const Layer& ly = lo.layers[layer];
  int kind = LSAM_LAYER_DENSE, dx_stored = 0;
  int64_t rows = lo.B;
  if (layer < lo.n_conv) {
    const ConvLayer& cv = lo.conv[layer];
    kind = cv.first ? LSAM_LAYER_CONV_FIRST : cv.direct_in ? LSAM_LAYER_CONV_DIRECT : LSAM_LAYER_CONV_STORED;
    dx_stored = (layer > 0 && !cv.direct_dx) ? 1 : 0;
    rows = cv.rows;
  } else if (layer == lo.L - 1 && head_is_fused(lo)) {
    kind = LSAM_LAYER_HEAD;
  }
  const bool fused = c->rho != 0.f && can_fuse_step(c);
  info[0] = kind;
  info[1] = dx_stored;
  info[2] = fused ? (gram_norm_pays(lo.B, ly.out, ly.in) ? 2 : 1) : 0;
  info[3] = (int32_t)rows;
  info[4] = ly.in;
  info[5] = ly.out;
  info[6] = ly.proj ? ly.proj_in : 0;
  info[7] = ly.proj ? lo.conv[layer].skip_step : 0;
  if (n > LSAM_LAYER_INFO_FIELDS) info[8] = layer < lo.n_conv && lo.conv[layer].fast && !lo.conv[layer].first ? lo.np : 0;
  return LSAM_OK;
}

int lsam_set_fused_step(lsam_ctx* c, int32_t on) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  c->fuse_step = on != 0;
  return can_fuse_step(c) ? 1 : 0;
}

int lsam_note_replay(lsam_ctx* c) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  // a captured step carries the kernel arguments of the step it was captured from: the coupling
  // coefficients lambda0/(lr tau_i) and the noise counter are frozen in the graph
  if (c->cfg.noise_scale > 0.f)
    return fail(LSAM_ESTATE, "a replayed step would repeat its Langevin noise");
  if (c->cfg.sched_mode == LSAM_SCHED_REDRAW && !c->cfg.tau && c->cfg.lambda_abs < 0.f &&
      c->cfg.algorithm == LSAM_ALG_LSAM)
    return fail(LSAM_ESTATE, "redrawn periods change lambda_i, which a replayed step cannot follow");
  ++c->t_step;
  c->sched.tick();
  return LSAM_OK;
}

int lsam_get_counters(lsam_ctx* c, int64_t* state, int64_t n) {
  if (!c || !state) return fail(LSAM_EINVAL, "ctx or state is NULL");
  const int K = c->lo.K;
  if (n != 2 * (int64_t)K + 3) return fail(LSAM_EINVAL, "n=%lld must equal 2K+3=%d", (long long)n, 2 * K + 3);
  for (int i = 0; i < K; ++i) {
    state[i] = c->sched.count()[i];
    state[K + i] = c->sched.tau()[i];
  }
  state[2 * K] = (int64_t)c->sched.generator_state();
  state[2 * K + 1] = c->sched.t_y();
  state[2 * K + 2] = (int64_t)c->t_step;
  return LSAM_OK;
}

int lsam_set_counters(lsam_ctx* c, const int64_t* state, int64_t n) {
  if (!c || !state) return fail(LSAM_EINVAL, "ctx or state is NULL");
  const int K = c->lo.K;
  if (n != 2 * (int64_t)K + 3) return fail(LSAM_EINVAL, "n=%lld must equal 2K+3=%d", (long long)n, 2 * K + 3);
  if (state[2 * K + 2] < 0 || state[2 * K + 2] > (int64_t)UINT32_MAX)
    return fail(LSAM_EINVAL, "noise step %lld out of range", (long long)state[2 * K + 2]);
  if (!c->sched.restore(state, state + K, (uint64_t)state[2 * K], state[2 * K + 1]))
    return fail(LSAM_EINVAL, "counts must be >= 0, periods >= 1, the sync count >= 0");
  c->t_step = (uint32_t)state[2 * K + 2];
  return LSAM_OK;
}

int lsam_get_activation(lsam_ctx* c, int32_t layer, int32_t replica, float* dst, int64_t n) {
  if (!c || !dst) return fail(LSAM_EINVAL, "ctx or dst is NULL");
  const Layout& lo = c->lo;
  if (lo.raw || lo.n_conv > 0) return fail(LSAM_ESTATE, "activations can be read from a dense model only");
  if (layer < 1 || layer >= lo.L) return fail(LSAM_EINVAL, "layer %d is not a hidden layer (1..%d)", layer, lo.L - 1);
  if (replica < 0 || replica >= lo.K) return fail(LSAM_EINVAL, "replica %d out of range", replica);
  const int width = lo.layers[layer].in, B = lo.B;
  if (n != (int64_t)B * width)
    return fail(LSAM_EINVAL, "n=%lld must equal batch*width=%lld", (long long)n, (long long)B * width);
  HIP_TRY(hipStreamSynchronize(c->stream));
  const int64_t elems = lo.act_elems(width, lo.ld[layer]);
  if (!lo.bf16) {
    std::vector<float> h((size_t)elems);
    int rc = to_host(c, h.data(), c->at<float>(lo.act[layer]) + (int64_t)replica * elems, (size_t)elems * 4);
    if (rc != LSAM_OK) return rc;
    for (int b = 0; b < B; ++b)
      memcpy(dst + (int64_t)b * width, h.data() + (int64_t)b * lo.ld[layer], (size_t)width * 4);
    return LSAM_OK;
  }
  std::vector<uint16_t> h((size_t)elems);
  int rc = to_host(c, h.data(), c->at<uint16_t>(lo.act[layer]) + (int64_t)replica * elems, (size_t)elems * 2);
  if (rc != LSAM_OK) return rc;
  const int cb = b32s_blocks(width);
  for (int b = 0; b < B; ++b)
    for (int q = 0; q < width; ++q) {
      const uint32_t u = (uint32_t)h[(size_t)b32s_offset(b, q, cb)] << 16;
      memcpy(dst + (int64_t)b * width + q, &u, 4);
    }
  return LSAM_OK;
}

int lsam_set_scalars(lsam_ctx* c, float lr, float rho) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  if (!(rho >= 0.f) || !(lr >= 0.f)) return fail(LSAM_EINVAL, "lr and rho must be >= 0");
  if (!(lr > 0.f) && c->cfg.lambda_abs < 0.f)
    return fail(LSAM_EINVAL, "lr must be > 0 when lambda is derived as lambda0/(lr*tau)");
  c->lr = lr;
  c->rho = rho;
  return LSAM_OK;
}

int lsam_timing_enable(lsam_ctx* c, int32_t on) {
  if (!c) return fail(LSAM_EINVAL, "ctx is NULL");
  int rc = drain_timing(c);
  if (rc != LSAM_OK) return rc;
  c->timing = on != 0;
  if (!on) {
    for (int i = 0; i < KC_COUNT; ++i) { c->t_count[i] = 0; c->t_ms[i] = 0.0; }
  }
  return LSAM_OK;
}

int lsam_timing_read(lsam_ctx* c, int32_t cap, const char** names, int64_t* counts,
                     double* total_ms) {
  if (!c || !names || !counts || !total_ms) return fail(LSAM_EINVAL, "NULL argument");
  int rc = drain_timing(c);
  if (rc != LSAM_OK) return rc;
  int n = 0;
  for (int i = 0; i < KC_COUNT && n < cap; ++i) {
    names[n] = kClassNames[i];
    counts[n] = c->t_count[i];
    total_ms[n] = c->t_ms[i];
    ++n;
  }
  return n;
}

int lsam_probe_peaks(void* scratch, size_t scratch_bytes, void* stream, double* copy_gbytes_per_s,
                     double* mfma_bf16_tflops, double* mfma_fp32_tflops) {
  if (!scratch || !copy_gbytes_per_s || !mfma_bf16_tflops || !mfma_fp32_tflops)
    return fail(LSAM_EINVAL, "NULL argument");
  if (scratch_bytes < 32768 || (reinterpret_cast<uintptr_t>(scratch) & 15))
    return fail(LSAM_EINVAL, "scratch must be 16-byte aligned and hold at least 32 KiB");
  if (probe_peaks(scratch, scratch_bytes, static_cast<hipStream_t>(stream), copy_gbytes_per_s,
                  mfma_bf16_tflops, mfma_fp32_tflops) != 0)
    return fail(LSAM_EHIP, "peak probe failed: %s", hipGetErrorString(hipGetLastError()));
  return LSAM_OK;
}

void lsam_destroy(lsam_ctx* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  for (auto& t : c->pending) { (void)hipEventDestroy(t.a); (void)hipEventDestroy(t.b); }
  for (auto e : c->free_events) (void)hipEventDestroy(e);
  if (c->stage) (void)hipHostFree(c->stage);
  delete c;
}

}  // extern "C"
