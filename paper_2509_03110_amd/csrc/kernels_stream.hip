// Streaming kernels of the update path: gradient-norm reduction, ascent perturbation,
// descent + coupling, center update.  All are HBM-bandwidth bound: every array is touched
// once per kernel with 128-bit accesses, consecutive lanes on consecutive 16-byte words.
#include <type_traits>

#include "engine.h"

namespace lsam {
namespace {

constexpr int kThreads = 256;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// A row of a gradient that a caller hands in starts wherever its length puts it: four floats that are
// aligned as one (global memory takes 128-bit accesses at any multiple of 4 bytes).
typedef f32x4 f32x4_any __attribute__((aligned(4)));

__device__ __forceinline__ f32x4 ldv(const float* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
}
template <bool STREAM>
__device__ __forceinline__ f32x4 ld_any(const float* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p));
  else return *reinterpret_cast<const f32x4_any*>(p);
}
__device__ __forceinline__ void stv(float* p, f32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
}
template <bool STREAM>
__device__ __forceinline__ void st_param(float* p, f32x4 v) {
  if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p));
  else *reinterpret_cast<f32x4*>(p) = v;
}
// y / g'_prev are re-read by later kernels and other replicas: ordinary cached access.
__device__ __forceinline__ f32x4 ldc(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

__device__ __forceinline__ unsigned short bf16_bits(float f) {
  return __builtin_bit_cast(unsigned short, static_cast<__bf16>(f));
}
__device__ __forceinline__ void store_bf16(uint16_t* p, const f32x4& v) {
  u16x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = bf16_bits(v[i]);
  // Plain store: a wavefront's 64-byte pieces of neighbouring blocks merge in L2 before they
  // go out; the streaming hint measured no better once the copy became blocked.
  *reinterpret_cast<u16x4*>(p) = o;
}

enum Ascent { ASCENT_NONE = 0, ASCENT_SCALE, ASCENT_SUMS };   // see descent_kernel

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// One step further for a replica's mark (launch_center): 2 (sum just served) -> 1 (restart it in
// this step) -> 0.
__device__ __forceinline__ void count_mark(int32_t* mark) {
  const int32_t m = *mark;
  if (m > 0) *mark = m - 1;
}

// Sum over the block in a fixed order; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double part[kThreads / 64];
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) part[wave] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) r += part[w];
  }
  __syncthreads();
  return r;
}

// Mean of a replica's B losses; valid in thread 0.
__device__ __forceinline__ double mean_loss(const float* rows, int B) {
  double l = 0.0;
  for (int i = threadIdx.x; i < B; i += kThreads) l += (double)rows[i];
  return block_sum(l) / (double)B;
}

// ---- gradient norm, pass 1 ------------------------------------------------------------------
// HBM-bound: 4 bytes per value, four 16-byte loads in flight per lane.  nv whole words of four and
// `rem` values behind them; rows may start at any multiple of 4 bytes.
template <bool STREAM>
__global__ __launch_bounds__(kThreads) void sumsq_partials_kernel(
    const float* __restrict__ g, int64_t g_stride, int64_t nv, int rem, double* __restrict__ partials,
    int nblk, int32_t* __restrict__ restart) {
  const int k = blockIdx.y;
  if (restart != nullptr && blockIdx.x == 0 && threadIdx.x == 0) count_mark(restart + k);
  const int64_t chunk = (nv + nblk - 1) / nblk;
  const int64_t beg = (int64_t)blockIdx.x * chunk;
  const int64_t end = beg + chunk < nv ? beg + chunk : nv;
  const float* gk = g + (int64_t)k * g_stride;
  float a[4] = {0.f, 0.f, 0.f, 0.f};
  int64_t i = beg + threadIdx.x;
  for (; i + 3 * kThreads < end; i += 4 * kThreads) {
    f32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ld_any<STREAM>(gk + (i + j * kThreads) * 4);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[j] += v[j][e] * v[j][e];
  }
  for (; i < end; i += kThreads) {
    const f32x4 v0 = ld_any<STREAM>(gk + i * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) a[0] += v0[e] * v0[e];
  }
  if (blockIdx.x == 0 && (int)threadIdx.x < rem) {
    const float v0 = gk[nv * 4 + threadIdx.x];
    a[1] += v0 * v0;
  }
  double s = ((double)a[0] + (double)a[1]) + ((double)a[2] + (double)a[3]);
  s = block_sum(s);
  if (threadIdx.x == 0) partials[(int64_t)k * nblk + blockIdx.x] = s;
}

// ---- gradient norm, pass 2 (+ mean loss) ----------------------------------------------------
__global__ __launch_bounds__(kThreads) void norm_finish_kernel(
    const double* __restrict__ partials, int nblk, int64_t pstride, float rho, float gamma,
    float* __restrict__ norms, float* __restrict__ scale, const float* __restrict__ loss_rows,
    int B, float* __restrict__ loss_out, int32_t* __restrict__ restart) {
  const int k = blockIdx.x;
  if (restart != nullptr && threadIdx.x == 0) count_mark(restart + k);
  double s = 0.0;
  for (int i = threadIdx.x; i < nblk; i += kThreads) s += partials[(int64_t)k * pstride + i];
  s = block_sum(s);
  if (threadIdx.x == 0) {
    const double n = sqrt(s);
    norms[k] = (float)n;
    scale[k] = (float)((double)rho / (n + (double)gamma));
  }
  if (loss_rows != nullptr && loss_out != nullptr) {
    const double l = mean_loss(loss_rows + (int64_t)k * B, B);
    if (threadIdx.x == 0) loss_out[k] = (float)l;
  }
}

// ---- ascent perturbation ----------------------------------------------------------------------
// The norm from its partial sums and the scale rho / (norm + gamma), by every wavefront for itself: at most
// kProloguePartials sums.
__device__ __forceinline__ float scale_from_sums(const double* part, int n, float rho, float gamma, float& norm) {
  const int lane = threadIdx.x & 63;
  double s = lane < n ? part[lane] : 0.0;
  if (lane + 64 < n) s += part[lane + 64];
  s = __shfl(wave_sum(s), 0, 64);
  const double r = sqrt(s);
  norm = (float)r;
  return (float)((double)rho / (r + (double)gamma));
}

// SUMS: what norm_finish_kernel does (norm, scale, mean loss, marks) happens here, before the lanes' own
// values are touched, where the partial sums are few: a launch less (3 us of a step that takes 50).
template <bool STREAM, bool SUMS>
__global__ __launch_bounds__(kThreads) void perturb_kernel(
    const float* __restrict__ x, const float* __restrict__ g, int64_t g_stride,
    const float* __restrict__ scale, float* __restrict__ xt, int64_t stride, int64_t nv, int rem, NormSums fin) {
  const int k = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const float* xk = x + (int64_t)k * stride + i * 4;
  const float* gk = g + (int64_t)k * g_stride + i * 4;
  float* tk = xt + (int64_t)k * stride + i * 4;
  f32x4 xv = {}, gv = {};
  if (i < nv) {
    xv = ldv(xk);
    gv = ld_any<true>(gk);
  }
  float sc;
  if constexpr (SUMS) {
    float norm;
    sc = scale_from_sums(fin.partials + (int64_t)k * fin.pstride, fin.n, fin.rho, fin.gamma, norm);
    if (blockIdx.x == 0) {
      if (threadIdx.x == 0) {
        if (fin.restart != nullptr) count_mark(fin.restart + k);
        fin.norms[k] = norm;
        fin.scale[k] = sc;
      }
      if (fin.loss_rows != nullptr && fin.loss_out != nullptr) {
        const double l = mean_loss(fin.loss_rows + (int64_t)k * fin.B, fin.B);
        if (threadIdx.x == 0) fin.loss_out[k] = (float)l;
      }
    }
  } else {
    sc = scale[k];
  }
  if (i < nv) {
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = ascent_point(xv[e], sc, gv[e]);
    st_param<STREAM>(tk, o);
  } else if (i == nv) {
    for (int e = 0; e < rem; ++e) tk[e] = ascent_point(xk[e], sc, gk[e]);
  }
}

// For bf16 operands x~ exists only as the operand copy of the weight matrices (blocked layout);
// elements of no weight matrix (biases, padding) are not stored at all: the perturbed biases are
// formed in the GEMM epilogue from x, g1 and scale.  This kernel walks the weight matrices in tiles: a
// workgroup takes 8 rows x 128 columns of one matrix, a wavefront 8 rows x 32 columns, so that the
// wavefront's 256 results are 512 consecutive bytes of one block of the copy (the flat walk
// writes 64-byte pieces of 8 different blocks per wavefront and reached 67 % of HBM peak here
// against 80 % for the fp32 kernel) while x and g1 are still read in 512-byte row pieces.
struct TileMap {
  int32_t n;
  int32_t first[LSAM_MAX_LAYERS + 1];   // first workgroup of each matrix; [n] = total
  int32_t ctiles[LSAM_MAX_LAYERS];      // 128-column tiles per row of W_l
  int32_t rows[LSAM_MAX_LAYERS];
};

__global__ __launch_bounds__(kThreads) void perturb_tiled_kernel(
    const float* __restrict__ x, const float* __restrict__ g, int64_t g_stride,
    const float* __restrict__ scale, uint16_t* __restrict__ xt16, ShadowMap map, TileMap tiles,
    int64_t shadow_stride, int64_t stride) {
  const int k = blockIdx.y;
  int s = 0;
  while (s + 1 < tiles.n && (int)blockIdx.x >= tiles.first[s + 1]) ++s;
  const int t = blockIdx.x - tiles.first[s];
  const int rg = t / tiles.ctiles[s], ct = t - rg * tiles.ctiles[s];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = rg * 8 + (lane >> 3);
  const int c = ct * 128 + wave * 32 + (lane & 7) * 4;
  if (r >= tiles.rows[s] || c >= map.ldw[s]) return;
  const int64_t flat = map.begin[s] + (int64_t)r * map.ldw[s] + c;
  const float sc = scale[k];
  const auto xv = ldv(x + (int64_t)k * stride + flat);
  const auto gv = ldv(g + (int64_t)k * g_stride + flat);
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = ascent_point(xv[e], sc, gv[e]);
  store_bf16(xt16 + (int64_t)k * shadow_stride + map.shadow[s] + b32s_offset(r, c, map.cblocks[s]), o);
}

// ---- descent + coupling -------------------------------------------------------------------------
// One workgroup updates 256 vector words of one replica; consecutive workgroups take the same
// words of the K replicas in turn, so the K readers of a piece of y run close together and y
// comes from HBM once.  (Looping over the replicas inside one thread, which reads y exactly
// once, measured 8-12 % slower at K = 8 and 16; sending the K workgroups of a piece to the same
// XCD, so that y misses only one L2, measured 4-9 % slower: the other XCDs' misses are served
// by the memory-side cache, and the launch order here keeps each XCD on fewer DRAM pages.)
//
// ASCENT: both gradients are at hand (nothing is computed at the perturbed point in between), and
// x~ = x + scale g1 is written by the same pass, which reads x once: 36 instead of 12 + 28 bytes per
// value.  Ten streams that miss the caches run faster the fewer bytes are in flight: one workgroup of 256
// per compute unit (`room` keeps the others out), two words per lane, takes 4.76 ms for 8 x 10^8 values (6.05
// TB/s), one word per lane 5.22; two workgroups with one word per lane 4.90, three 4.97, eight 5.27; four
// words and as many workgroups as fit 5.35; a workgroup of 1024 4.91; the two kernels it replaces take 5.21.
// ASCENT_SUMS: the norm pass left at most kProloguePartials partial sums per replica, and
// every wavefront adds them up itself while its loads are under way, which saves the launch that
// would do it (4 us of a step that takes 14 at 4 x 270410 values; 42 with four launches, norms by
// 20 workgroups and single floats); the first workgroup of a replica writes norm and scale.
// The caches hold more of the joined pass's vectors, which is read by the next step's: one workgroup per compute unit
// and streaming stores pay from 128 MB a vector (steps of vectors of 105 MB, two / eight / sixteen replicas: 213 / 207 / 226
// us streamed, 202 / 186 / 179 as below; 130 MB 257 / 254 / 255 and 266 / 241 / 227; 150 MB 298 / 293 / 297 and 311 / 308 / 305).
// The center, kept in the caches for all replicas, counts for a third of a vector: one replica of 103 MB 218 and 224.
constexpr int64_t kAscentResidentBytes = 128ll << 20;
template <int ASCENT, bool STREAM> struct DescentShape {
  static constexpr bool wide = ASCENT != 0 && STREAM;
  static constexpr int words = wide ? 2 : 1;
};

template <int ASCENT, bool SHADOW, bool STREAM, typename NOISE>
__global__ __launch_bounds__(kThreads) void descent_kernel(
    float* __restrict__ x, const float* __restrict__ g, int64_t g_stride, float* __restrict__ v,
    float* __restrict__ S, const float* __restrict__ y, uint16_t* __restrict__ shadow,
    ShadowMap map, int64_t shadow_stride, int64_t stride, int64_t n, int K, ReplicaScalars lam,
    float lr, float mu, int nesterov, NOISE noise, const int32_t* __restrict__ restart, AscentPass up) {
  using Shape = DescentShape<ASCENT, STREAM>;
  constexpr int W = Shape::words;
  constexpr bool ascend = ASCENT != ASCENT_NONE;
  if constexpr (Shape::wide) {
    __shared__ unsigned char room[84 << 10];
    asm volatile("" ::"v"(room));      // allocated, never touched
  }
  const int k = (int)(blockIdx.x % (unsigned)K);
  const int64_t beg = (int64_t)(blockIdx.x / (unsigned)K) * (kThreads * W * 4);      // first value of the workgroup
  const int lane = threadIdx.x & 63;
  const unsigned at = ((threadIdx.x >> 6) * (64 * W) + lane) * 4;    // of the lane, relative to it
  float* xk = x + (int64_t)k * stride + beg;
  const float* gk = g + (int64_t)k * g_stride + beg;
  const float* hk = ascend ? up.g1 + (int64_t)k * up.g1_stride + beg : nullptr;
  float* vk = v + (int64_t)k * stride + beg;
  float* Sk = S + (int64_t)k * stride + beg;
  const float* yk = y + beg;
  float* tk = ascend ? up.xt + (int64_t)k * stride + beg : nullptr;
  const bool fresh = restart != nullptr && restart[k] == 1;      // the sum starts afresh: its memory is stale
  const bool whole = beg + kThreads * W * 4 <= n;
  f32x4 yv[W], xv[W], gv[W], vv[W], sv[W], hv[W];
  if (whole) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const unsigned o = at + w * 256;
      yv[w] = ldc(yk + o);
      xv[w] = ldv(xk + o);
      gv[w] = ld_any<true>(gk + o);
      vv[w] = ldv(vk + o);
      if constexpr (ascend) hv[w] = ld_any<true>(hk + o);
      sv[w] = f32x4{};
    }
    if (!fresh) {
#pragma unroll
      for (int w = 0; w < W; ++w) sv[w] = ldv(Sk + at + w * 256);
    }
  }
  float sc = 0.f;
  if constexpr (ASCENT == ASCENT_SUMS) {
    float norm;
    sc = scale_from_sums(up.partials + (int64_t)k * up.nblk, up.nblk, up.rho, up.gamma, norm);
    if (beg == 0 && threadIdx.x == 0) {
      up.norms[k] = norm;
      up.scale[k] = sc;
    }
  } else if constexpr (ASCENT == ASCENT_SCALE) {
    sc = up.scale[k];
  }
  const float lk = lam.v[k];
  if (whole) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const unsigned o = at + w * 256;
      f32x4 tv = {};
      float xi[4] = {0.f, 0.f, 0.f, 0.f};      // sigma sqrt(2 eta) xi of the Langevin sampler
      if constexpr (!std::is_same<NOISE, NoNoise>::value) langevin4(noise, k, beg + o, xi);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float xe = xv[w][e], ve = vv[w][e], se = sv[w][e];
        if constexpr (ascend) tv[e] = ascent_point(xe, sc, hv[w][e]);
        sampler_step(gv[w][e], yv[w][e], lk, lr, mu, nesterov, xi[e], xe, ve, se);
        vv[w][e] = ve;
        xv[w][e] = xe;
        sv[w][e] = se;
      }
      st_param<STREAM>(xk + o, xv[w]);
      stv(vk + o, vv[w]);
      stv(Sk + o, sv[w]);
      // (without this the compiler joins these stores with those of the last workgroup below and drops their hints)
      asm volatile("" ::: "memory");
      if constexpr (ascend) st_param<STREAM>(tk + o, tv);
      if constexpr (SHADOW) {
        const int64_t so = shadow_offset4(map, beg + o);
        if (so >= 0) store_bf16(shadow + (int64_t)k * shadow_stride + so, xv[w]);
      }
    }
    return;
  }
  // a replica's last workgroup, value by value
  for (int w = 0; w < W; ++w) {
    const unsigned o = at + w * 256;
    if (beg + o >= n) return;
    const int m = n - beg - o < 4 ? (int)(n - beg - o) : 4;
    float xi[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (!std::is_same<NOISE, NoNoise>::value) langevin4(noise, k, beg + o, xi);
    f32x4 nx = {};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e >= m) continue;
      float xe = xk[o + e], ve = vk[o + e], se = fresh ? 0.f : Sk[o + e];
      if constexpr (ascend) tk[o + e] = ascent_point(xe, sc, hk[o + e]);
      sampler_step(gk[o + e], yk[o + e], lk, lr, mu, nesterov, xi[e], xe, ve, se);
      xk[o + e] = nx[e] = xe;
      vk[o + e] = ve;
      Sk[o + e] = se;
    }
    if constexpr (SHADOW) {
      const int64_t so = shadow_offset4(map, beg + o);
      if (so >= 0) store_bf16(shadow + (int64_t)k * shadow_stride + so, nx);
    }
  }
}

// ---- average over replicas (synchronous data-parallel baseline) ---------------------------------
__global__ __launch_bounds__(kThreads) void grad_mean_kernel(
    const float* src, int64_t src_stride, float* dst, int64_t dst_stride, int64_t nv, int rem, int K,
    int copies) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const float inv = 1.f / (float)K;
  if (i < nv) {
    f32x4 acc = ld_any<true>(src + i * 4);
    for (int k = 1; k < K; ++k) acc += ld_any<true>(src + (int64_t)k * src_stride + i * 4);
    acc *= inv;
    for (int c = 0; c < copies; ++c) stv(dst + (int64_t)c * dst_stride + i * 4, acc);
  } else if (i == nv) {
    for (int64_t j = i * 4; j < i * 4 + rem; ++j) {
      float acc = src[j];
      for (int k = 1; k < K; ++k) acc += src[(int64_t)k * src_stride + j];
      for (int c = 0; c < copies; ++c) dst[(int64_t)c * dst_stride + j] = acc * inv;
    }
  }
}

// ---- center update ------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void center_kernel(
    float* __restrict__ S, float* __restrict__ y, float* __restrict__ gprev, int64_t stride,
    int64_t nv, DueList due, float inv_m, float beta, float lr_center, int has_prev,
    int32_t* __restrict__ restart) {
  // (no thread of this kernel reads a mark: a replica that is due has taken a step since it
  // was last served, and that step's norm kernel had counted its mark down to at most 1)
  if (restart != nullptr && blockIdx.x == 0 && (int)threadIdx.x < due.n) restart[due.idx[threadIdx.x]] = 2;
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= nv) return;
  f32x4 tot = {};
  for (int j = 0; j < due.n; ++j) {
    float* p = S + (int64_t)due.idx[j] * stride + i * 4;
    tot += ldv(p);
    if (restart == nullptr) stv(p, f32x4{});
  }
  f32x4 yv = ldc(y + i * 4);
  const f32x4 pv = ldc(gprev + i * 4);
  f32x4 gp;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float gpe = tot[e] * inv_m - yv[e];
    const float ge = has_prev ? gpe + beta * (gpe - pv[e]) : gpe;
    gp[e] = gpe;
    yv[e] = yv[e] + lr_center * ge;
  }
  *reinterpret_cast<f32x4*>(y + i * 4) = yv;
  *reinterpret_cast<f32x4*>(gprev + i * 4) = gp;
}

// ---- small utility kernels ------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void broadcast_kernel(
    const float* __restrict__ src, float* __restrict__ dst, int64_t stride, int64_t nv, int K) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= nv) return;
  const f32x4 sv = ldc(src + i * 4);
  for (int k = 0; k < K; ++k) stv(dst + (int64_t)k * stride + i * 4, sv);
}

// bf16 operand copy of the weight matrices of replica blockIdx.y from its fp32 parameters.
__global__ __launch_bounds__(kThreads) void shadow_refresh_kernel(
    const float* __restrict__ x, uint16_t* __restrict__ shadow, ShadowMap map, int64_t stride,
    int64_t shadow_stride, int64_t nv) {
  const int k = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= nv) return;
  const int64_t so = shadow_offset4(map, i * 4);
  if (so < 0) return;
  store_bf16(shadow + (int64_t)k * shadow_stride + so, ldc(x + (int64_t)k * stride + i * 4));
}

// Row-major bf16 matrix of replica blockIdx.y -> blocked layout; one thread per 8 elements.
__global__ __launch_bounds__(kThreads) void rowmajor_to_b32s_kernel(
    const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int rows, int cols, int cblocks,
    int64_t dst_stride) {
  const int k = blockIdx.y;
  const int units = (cols + 7) / 8;
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= (int64_t)rows * units) return;
  const int r = (int)(i / units), c = (int)(i % units) * 8;
  const uint16_t* sp = src + ((int64_t)k * rows + r) * cols + c;
  uint16_t* dp = dst + (int64_t)k * dst_stride + b32s_offset(r, c, cblocks);
  if (c + 8 <= cols && (cols % 8) == 0) {
    *reinterpret_cast<uint4*>(dp) = *reinterpret_cast<const uint4*>(sp);
  } else {
    for (int e = 0; e < 8 && c + e < cols; ++e) dp[e] = sp[e];
  }
}

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(uint4* __restrict__ p, int64_t n16) {
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (; i < n16; i += step) p[i] = make_uint4(0, 0, 0, 0);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void pad_rows_kernel(const T* __restrict__ s,
                                                           T* __restrict__ d, int64_t rows,
                                                           int cols, int ld) {
  const int64_t total = rows * cols;
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (; i < total; i += step) {
    const int64_t r = i / cols;
    const int c = (int)(i - r * cols);
    d[r * ld + c] = s[i];
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }
inline unsigned capped_blocks(int64_t n) {
  int64_t b = (n + kThreads - 1) / kThreads;
  return (unsigned)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

}  // namespace

int sumsq_blocks(int64_t n) {
  const int64_t small = (n + 4095) / 4096, large = (n + 16383) / 16384;
  if (large <= kProloguePartials) return (int)(small < 1 ? 1 : small < kProloguePartials ? small : kProloguePartials);
  return (int)(large < kMaxPartials ? large : kMaxPartials);
}

void launch_sumsq_partials(const float* g, int64_t g_stride, int64_t n, int K, double* partials,
                           int nblk, hipStream_t s, int32_t* restart) {
  dim3 grid(nblk, K);
  if ((int64_t)K * n * 4 > kCacheResidentBytes)
    sumsq_partials_kernel<true><<<grid, kThreads, 0, s>>>(g, g_stride, n / 4, (int)(n % 4), partials, nblk, restart);
  else
    sumsq_partials_kernel<false><<<grid, kThreads, 0, s>>>(g, g_stride, n / 4, (int)(n % 4), partials, nblk, restart);
}

void launch_norm_finish(const double* partials, int nblk, int64_t partials_stride, int K, float rho,
                        float gamma, float* norms, float* scale, const float* loss_rows, int B,
                        float* loss_out, hipStream_t s, int32_t* restart) {
  norm_finish_kernel<<<K, kThreads, 0, s>>>(partials, nblk, partials_stride, rho, gamma, norms,
                                            scale, loss_rows, B, loss_out, restart);
}

void launch_perturb(const float* x, const float* g, int64_t g_stride, const float* scale,
                    float* xt_f32, uint16_t* xt_bf16, const ShadowMap* map, int64_t shadow_stride,
                    int64_t stride, int64_t n, int K, hipStream_t s, const NormSums* sums) {
  if (xt_bf16) {
    // bf16 mode only exists for the MLP layouts, which are always vector-aligned
    TileMap tm{};
    tm.n = map->n;
    int total = 0;
    for (int l = 0; l < map->n; ++l) {
      tm.first[l] = total;
      tm.ctiles[l] = (map->ldw[l] + 127) / 128;
      tm.rows[l] = (int)((map->end[l] - map->begin[l]) / map->ldw[l]);
      total += tm.ctiles[l] * ((tm.rows[l] + 7) / 8);
    }
    tm.first[map->n] = total;
    dim3 grid(total, K);
    perturb_tiled_kernel<<<grid, kThreads, 0, s>>>(x, g, g_stride, scale, xt_bf16, *map, tm,
                                                   shadow_stride, stride);
  } else {
    dim3 grid(blocks_for((n + 3) / 4), K);
    auto go = [&](auto kernel, const NormSums& fin) {
      kernel<<<grid, kThreads, 0, s>>>(x, g, g_stride, scale, xt_f32, stride, n / 4, (int)(n % 4), fin);
    };
    const bool stream = (int64_t)K * n * 4 > kCacheResidentBytes;
    if (sums) stream ? go(perturb_kernel<true, true>, *sums) : go(perturb_kernel<false, true>, *sums);
    else stream ? go(perturb_kernel<true, false>, NormSums{}) : go(perturb_kernel<false, false>, NormSums{});
  }
}

template <int ASCENT, typename NOISE>
void launch_descent_with(float* x, const float* g, int64_t g_stride, float* v, float* S,
                         const float* y, uint16_t* shadow, const ShadowMap* map,
                         int64_t shadow_stride, int64_t stride, int64_t n, int K,
                         const ReplicaScalars& lam, float lr, float mu, int nesterov,
                         const NOISE& noise, hipStream_t s, const int32_t* restart, const AscentPass& up) {
  ShadowMap none{};
  auto go = [&](auto kernel, auto shape, uint16_t* copy, const ShadowMap& m, int64_t copy_stride) {
    using Shape = decltype(shape);
    const unsigned grid = blocks_for(((n + 3) / 4 + Shape::words - 1) / Shape::words) * (unsigned)K;
    kernel<<<grid, kThreads, 0, s>>>(x, g, g_stride, v, S, y, copy, m, copy_stride, stride, n, K, lam, lr,
                                           mu, nesterov, noise, restart, up);
  };
  if constexpr (ASCENT == ASCENT_NONE) {
    if (shadow) {
      go(descent_kernel<ASCENT, true, true, NOISE>, DescentShape<ASCENT, true>{}, shadow, *map, shadow_stride);
      return;
    }
  }
  if (ASCENT == ASCENT_NONE ? (int64_t)K * n * 4 > kCacheResidentBytes : (3 * (int64_t)K + 1) * n * 4 > 3 * kAscentResidentBytes)
    go(descent_kernel<ASCENT, false, true, NOISE>, DescentShape<ASCENT, true>{}, nullptr, none, 0);
  else
    go(descent_kernel<ASCENT, false, false, NOISE>, DescentShape<ASCENT, false>{}, nullptr, none, 0);
}

void launch_descent(float* x, const float* g, int64_t g_stride, float* v, float* S,
                    const float* y, uint16_t* shadow, const ShadowMap* map, int64_t shadow_stride,
                    int64_t stride, int64_t n, int K, const ReplicaScalars& lam, float lr, float mu,
                    int nesterov, const NoiseMap* noise, hipStream_t s, const int32_t* restart) {
  const AscentPass none{};
  if (noise)
    launch_descent_with<ASCENT_NONE, NoiseMap>(x, g, g_stride, v, S, y, shadow, map, shadow_stride, stride, n, K,
                                               lam, lr, mu, nesterov, *noise, s, restart, none);
  else
    launch_descent_with<ASCENT_NONE, NoNoise>(x, g, g_stride, v, S, y, shadow, map, shadow_stride, stride, n, K,
                                              lam, lr, mu, nesterov, NoNoise{}, s, restart, none);
}

void launch_raw_norm(int64_t n, int K, hipStream_t s, int32_t* restart, const AscentPass& up) {
  launch_sumsq_partials(up.g1, up.g1_stride, n, K, up.partials, up.nblk, s, restart);
  if (!up.finish_in_descent())
    launch_norm_finish(up.partials, up.nblk, up.nblk, K, up.rho, up.gamma, up.norms, up.scale, nullptr, 0, nullptr, s);
}

void launch_raw_descent(float* x, const float* g2, int64_t g_stride, float* v, float* S, const float* y,
                        int64_t stride, int64_t n, int K, const ReplicaScalars& lam, float lr, float mu,
                        int nesterov, const NoiseMap* noise, hipStream_t s, const int32_t* restart, const AscentPass& up) {
  auto step = [&](auto ascent, const auto& how) {
    launch_descent_with<decltype(ascent)::value>(x, g2, g_stride, v, S, y, nullptr, nullptr, 0, stride, n, K, lam, lr,
                                                 mu, nesterov, how, s, restart, up);
  };
  auto choose = [&](const auto& how) {
    if (up.xt == nullptr) step(std::integral_constant<int, ASCENT_NONE>{}, how);
    else if (up.finish_in_descent()) step(std::integral_constant<int, ASCENT_SUMS>{}, how);
    else step(std::integral_constant<int, ASCENT_SCALE>{}, how);
  };
  if (noise) choose(*noise);
  else choose(NoNoise{});
}

void launch_grad_mean(const float* src, int64_t src_stride, float* dst, int64_t dst_stride,
                      int64_t n, int K, int copies, hipStream_t s) {
  // dst is this library's own: rows of whole words of four, 16-byte aligned
  grad_mean_kernel<<<blocks_for((n + 3) / 4), kThreads, 0, s>>>(src, src_stride, dst, dst_stride, n / 4, (int)(n % 4), K,
                                                                copies);
}

void launch_center(float* S, float* y, float* gprev, int64_t stride, int64_t n,
                   const DueList& due, float inv_m, float beta, float lr_center, int has_prev,
                   hipStream_t s, int32_t* restart) {
  // this library's own rows, padded with zeros to 64 values: the last word is whole, and stays zero where it pads
  center_kernel<<<blocks_for((n + 3) / 4), kThreads, 0, s>>>(S, y, gprev, stride, (n + 3) / 4, due, inv_m,
                                                             beta, lr_center, has_prev, restart);
}

void launch_broadcast(const float* src, float* dst, int64_t stride, int64_t n, int K, hipStream_t s) {
  // internal buffers only: n and stride are multiples of 4 by construction
  broadcast_kernel<<<blocks_for(n / 4), kThreads, 0, s>>>(src, dst, stride, n / 4, K);
}

void launch_shadow_refresh(const float* x, uint16_t* shadow, const ShadowMap& map, int64_t stride,
                           int64_t shadow_stride, int64_t n, int K, hipStream_t s) {
  dim3 grid(blocks_for(n / 4), K);
  shadow_refresh_kernel<<<grid, kThreads, 0, s>>>(x, shadow, map, stride, shadow_stride, n / 4);
}

void launch_rowmajor_to_b32s(const uint16_t* src, uint16_t* dst, int rows, int cols, int K,
                             hipStream_t s) {
  const int64_t work = (int64_t)rows * ((cols + 7) / 8);
  dim3 grid(blocks_for(work), K);
  rowmajor_to_b32s_kernel<<<grid, kThreads, 0, s>>>(src, dst, rows, cols, b32s_blocks(cols),
                                                    b32s_size(rows, cols));
}

void launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return;
  fill_zero_kernel<<<capped_blocks((int64_t)(bytes / 16)), kThreads, 0, s>>>(
      reinterpret_cast<uint4*>(p), (int64_t)(bytes / 16));
}

void launch_pad_rows(const void* src, void* dst, int64_t rows, int cols, int ld_dst, int elem,
                     hipStream_t s) {
  const unsigned grid = capped_blocks(rows * cols);
  if (elem == 4)
    pad_rows_kernel<float><<<grid, kThreads, 0, s>>>((const float*)src, (float*)dst, rows, cols,
                                                     ld_dst);
  else
    pad_rows_kernel<uint16_t><<<grid, kThreads, 0, s>>>((const uint16_t*)src, (uint16_t*)dst, rows,
                                                        cols, ld_dst);
}

}  // namespace lsam
