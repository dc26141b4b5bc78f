// Kernels around the 3x3 convolution layers of the convolutional model (Section "Experiments":
// the paper's workers train convolutional networks on 32x32x3 images).  A convolution with
// stride 1 and a zero rim of one pixel is run as a GEMM over the unfolded image
//   col[(b,i,j), (u,v,c)] = X[b, i+u-1, j+v-1, c]      (0 outside the image)
// so that the filter bank [out, 3, 3, C] is the GEMM's [out, 9 C] weight matrix and the
// tuned GEMM kernels serve forward, dW and dX unchanged.  This file holds what is left: the
// unfold and its adjoint (a gather: every input pixel sums its up to nine contributions in a
// fixed order), the 2x2 max-pool, and the pool's backward pass fused with the ReLU mask.
// All tensors are fp32, [K][B][H][W][C] with C contiguous; all four kernels are bandwidth
// bound and move 128-bit words, consecutive lanes on consecutive words.
#include <type_traits>

#include "engine.h"
#include "planes.h"

namespace lsam {
namespace {

constexpr int kThreads = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// Writes 4 values as planes at element `at` of each.
template <int NP>
__device__ __forceinline__ void put_planes(unsigned short* p, long long plane, long long at, const f32x4& v) {
  if constexpr (NP > 0) {
    u16x4 w[NP];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      unsigned short t[NP];
      split_planes<NP>(v[r], t);
#pragma unroll
      for (int q = 0; q < NP; ++q) w[q][r] = t[q];
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) *reinterpret_cast<u16x4*>(p + q * plane + at) = w[q];
  }
}

// One bit for each of four values that is positive.
__device__ __forceinline__ unsigned char positive_bits(const f32x4& v) {
  return (unsigned char)((v[0] > 0.f ? 1 : 0) | (v[1] > 0.f ? 2 : 0) | (v[2] > 0.f ? 4 : 0) | (v[3] > 0.f ? 8 : 0));
}

__device__ __forceinline__ f32x4 kept_values(f32x4 v, unsigned bits) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (!(bits >> r & 1)) v[r] = 0.f;
  return v;
}

struct ImgShape {
  int H, W, C;     // one output image of the convolution (H x W positions), C input channels
  int ld;          // pitch of a col row (floats), multiple of 4, >= 9 C
  long long rows;  // B H W
  long long total; // threads needed
  int st;          // stride: the input image is [st H][st W][C]
};

// One thread per 4 values of col.  VEC: C % 4 == 0, they then lie inside one tap.  NP: col is written
// as that many bfloat16 planes, `plane` elements apart (replicas contiguous); 0: as floats.
template <bool VEC, int NP>
__global__ __launch_bounds__(kThreads) void unfold3x3_kernel(const float* __restrict__ X,
                                                             void* __restrict__ col, ImgShape sh,
                                                             long long strideX, long long plane) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= sh.total) return;
  const int words = sh.ld / 4;
  const int q = (int)(idx % words);
  long long m = idx / words;
  const int k = (int)(m / sh.rows);
  m -= (long long)k * sh.rows;
  const int j = (int)(m % sh.W);
  const int i = (int)((m / sh.W) % sh.H);
  const long long b = m / ((long long)sh.W * sh.H);
  const int Hin = sh.st * sh.H, Win = sh.st * sh.W;
  const float* img = X + (long long)k * strideX + b * ((long long)Hin * Win * sh.C);
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    const int e = 4 * q;
    if (e < 9 * sh.C) {
      const int tap = e / sh.C, c = e - tap * sh.C;
      const int ii = sh.st * i + tap / 3 - 1, jj = sh.st * j + tap % 3 - 1;
      if (ii >= 0 && ii < Hin && jj >= 0 && jj < Win)
        o = *reinterpret_cast<const f32x4*>(img + ((long long)ii * Win + jj) * sh.C + c);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = 4 * q + r;
      if (e < 9 * sh.C) {
        const int tap = e / sh.C, c = e - tap * sh.C;
        const int ii = sh.st * i + tap / 3 - 1, jj = sh.st * j + tap % 3 - 1;
        if (ii >= 0 && ii < Hin && jj >= 0 && jj < Win)
          o[r] = img[((long long)ii * Win + jj) * sh.C + c];
      }
    }
  }
  if constexpr (NP == 0) *reinterpret_cast<f32x4*>(static_cast<float*>(col) + idx * 4) = o;
  else put_planes<NP>(static_cast<unsigned short*>(col), plane, idx * 4, o);
}

// Adjoint of the unfold: dX[b,y,x,c] = sum over the taps (u,v) and output positions (i,j) with
// st i + u - 1 = y, st j + v - 1 = x of dcol[(b,i,j), (u,v,c)], taps in (u, v) order; with a
// mask, zero where mask <= 0 (the ReLU output the image came from).
// One thread per 16-byte word of dX; C % 4 == 0.  sh.rows counts the pixels of dX here.
__global__ __launch_bounds__(kThreads) void fold3x3_kernel(const float* __restrict__ dcol,
                                                           float* __restrict__ dX,
                                                           const float* __restrict__ mask, ImgShape sh,
                                                           long long strideCol, long long strideX) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= sh.total) return;
  const int words = sh.C / 4;
  const int c = (int)(idx % words) * 4;
  long long m = idx / words;
  const int k = (int)(m / sh.rows);
  m -= (long long)k * sh.rows;
  const int Hin = sh.st * sh.H, Win = sh.st * sh.W;
  const int x = (int)(m % Win);
  const int y = (int)((m / Win) % Hin);
  const long long b = m / ((long long)Win * Hin);
  const float* src = dcol + (long long)k * strideCol;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    const int yy = y - (tap / 3 - 1), xx = x - (tap % 3 - 1);     // st i and st j
    if (yy >= 0 && xx >= 0 && yy % sh.st == 0 && xx % sh.st == 0) {
      const int ii = yy / sh.st, jj = xx / sh.st;
      if (ii < sh.H && jj < sh.W) {
        const long long mm = (b * sh.H + ii) * sh.W + jj;
        acc += *reinterpret_cast<const f32x4*>(src + mm * sh.ld + tap * sh.C + c);
      }
    }
  }
  const long long at = (long long)k * strideX + m * sh.C + c;
  if (mask != nullptr) {
    const f32x4 keep = *reinterpret_cast<const f32x4*>(mask + at);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (!(keep[r] > 0.f)) acc[r] = 0.f;
  }
  *reinterpret_cast<f32x4*>(dX + at) = acc;
}

struct PoolShape {
  int Ho, Wo, C;    // pooled image
  long long cells;  // K B Ho Wo C/4
};

// Pooled word `idx`: its first channel, its cell (k b, i, j) and where its window's first value lies in the image.
struct PoolCell {
  int c;
  long long cell, base;
};
__device__ __forceinline__ PoolCell pool_cell(long long idx, const PoolShape& sh) {
  const int words = sh.C / 4;
  PoolCell p;
  p.c = (int)(idx % words) * 4;
  p.cell = idx / words;
  const int j = (int)(p.cell % sh.Wo);
  const int i = (int)((p.cell / sh.Wo) % sh.Ho);
  const long long kb = p.cell / ((long long)sh.Wo * sh.Ho);
  p.base = ((kb * 2 * sh.Ho + 2 * i) * (2 * sh.Wo) + 2 * j) * sh.C + p.c;
  return p;
}
// Value t (row-major) of a window.
__device__ __forceinline__ long long pool_offset(int t, const PoolShape& sh) {
  return (t & 1) * sh.C + (t >> 1) * (2LL * sh.Wo * sh.C);
}
// The first maximum of each channel's window, and where it lies: two bits a channel.
__device__ __forceinline__ unsigned first_maximum(const f32x4 (&v)[4], f32x4& m) {
  unsigned arg = 0;
  m = v[0];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    unsigned best = 0;
#pragma unroll
    for (unsigned t = 1; t < 4; ++t)
      if (v[t][r] > m[r]) { m[r] = v[t][r]; best = t; }
    arg |= best << (2 * r);
  }
  return arg;
}
// Gradient of window value t: dP where that is the first maximum and kept.
__device__ __forceinline__ f32x4 unpooled(const f32x4& g, unsigned keep, unsigned arg, unsigned t) {
  f32x4 o;
#pragma unroll
  for (int r = 0; r < 4; ++r) o[r] = (keep >> r & 1) && (arg >> (2 * r) & 3) == t ? g[r] : 0.f;
  return o;
}

// P[b,i,j,c] = max over the 2x2 window of A (a ReLU output), as floats (P null: not) and planes; what the backward pass wants
// of A beside it: `arg`, a byte a word, and the bits of the positive maxima.  One thread per 16-byte word of P.
template <int NP>
__global__ __launch_bounds__(kThreads) void maxpool2_kernel(const float* __restrict__ A,
                                                            float* __restrict__ P, PoolShape sh,
                                                            unsigned char* __restrict__ arg, unsigned char* __restrict__ keep,
                                                            unsigned short* __restrict__ planes, long long plane) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= sh.cells) return;
  const PoolCell w = pool_cell(idx, sh);
  f32x4 v[4], m;
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = *reinterpret_cast<const f32x4*>(A + w.base + pool_offset(t, sh));
  arg[idx] = (unsigned char)first_maximum(v, m);
  keep[idx] = positive_bits(m);
  if (P != nullptr) *reinterpret_cast<f32x4*>(P + idx * 4) = m;
  put_planes<NP>(planes, plane, idx * 4, m);
}

// Backward of ReLU followed by the pool: dA[window] = dP at the window's first maximum if that was positive, else 0, as
// floats (dA null: not) and planes.  From the bits of the forward pass, not from the image (4 bytes a value more): 4 replicas of
// 128 images, 32 channels at 32 x 32: 25 us, 16 so; 64 at 16 x 16 with the planes 13 and 13, 14 together.
template <int NP>
__global__ __launch_bounds__(kThreads) void maxpool2_backward_kernel(const float* __restrict__ dP,
                                                                     const unsigned char* __restrict__ arg,
                                                                     const unsigned char* __restrict__ keep,
                                                                     float* __restrict__ dA, PoolShape sh,
                                                                     unsigned short* __restrict__ planes, long long plane) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= sh.cells) return;
  const PoolCell w = pool_cell(idx, sh);
  const f32x4 g = *reinterpret_cast<const f32x4*>(dP + idx * 4);
  const unsigned a = arg[idx], kept = keep[idx];
#pragma unroll
  for (unsigned t = 0; t < 4; ++t) {
    const f32x4 o = unpooled(g, kept, a, t);
    const long long at = w.base + pool_offset(t, sh);
    if (dA != nullptr) *reinterpret_cast<f32x4*>(dA + at) = o;
    put_planes<NP>(planes, plane, at, o);
  }
}

// Column reductions over the rows of tall matrices [K][rows][C] (C % 4 == 0) are done in two
// fixed-order stages.  First stage: workgroup (chunk, k, column block) covers `chunk_rows` rows
// of 64 columns; thread = (column word w of 16, row group of 16), each group strides over the
// chunk's rows, the groups are added in group order through LDS.  chunk_rows shrinks from 256
// towards 32 until the launch has about a thousand workgroups (short matrices would otherwise
// leave most of the chip idle behind a few long serial sums).
struct ChunkPlan {
  int chunk_rows, chunks, col_blocks;
};
ChunkPlan chunk_plan(long long rows, int C, int K) {
  ChunkPlan p;
  p.col_blocks = (C + 63) / 64;
  p.chunk_rows = 256;
  while (p.chunk_rows > 32 &&
         ((rows + p.chunk_rows - 1) / p.chunk_rows) * p.col_blocks * K < 1024)
    p.chunk_rows /= 2;
  p.chunks = (int)((rows + p.chunk_rows - 1) / p.chunk_rows);
  return p;
}
struct ChunkThread {
  int cw;          // column word (4 columns) of this thread
  int grp;         // row group 0..15
  bool live;       // the column word exists
  long long r0, r1;
};
__device__ __forceinline__ ChunkThread chunk_thread(long long rows, int C, int chunk_rows) {
  ChunkThread t;
  t.cw = blockIdx.z * 16 + (threadIdx.x & 15);
  t.grp = threadIdx.x >> 4;
  t.live = t.cw < C / 4;
  t.r0 = (long long)blockIdx.x * chunk_rows;
  t.r1 = t.r0 + chunk_rows < rows ? t.r0 + chunk_rows : rows;
  return t;
}
// Adds `v` over the 16 row groups in group order; the result is valid for grp == 0.
__device__ __forceinline__ f32x4 combine_groups(f32x4 v, const ChunkThread& t, f32x4* buf) {
  __syncthreads();
  buf[threadIdx.x] = v;
  __syncthreads();
  f32x4 tot = v;
  if (t.grp == 0)
    for (int gq = 1; gq < 16; ++gq) tot += buf[gq * 16 + (threadIdx.x & 15)];
  return tot;
}

// partial[k][chunk][c] = sum of the chunk's rows of A, where `keep` (bits; null: everywhere) is set.
__global__ __launch_bounds__(kThreads) void colsum_partial_kernel(const float* __restrict__ A,
                                                                  const unsigned char* __restrict__ keep,
                                                                  float* __restrict__ partial,
                                                                  long long rows, int N, int chunks,
                                                                  int chunk_rows) {
  __shared__ f32x4 buf[kThreads];
  const ChunkThread t = chunk_thread(rows, N, chunk_rows);
  const int k = blockIdx.y;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (t.live) {
    const long long base = ((long long)k * rows) * N + 4 * t.cw;
    if (keep != nullptr)
      for (long long r = t.r0 + t.grp; r < t.r1; r += 16)
        acc += kept_values(*reinterpret_cast<const f32x4*>(A + base + r * N), keep[(base + r * N) >> 2]);
    else
      for (long long r = t.r0 + t.grp; r < t.r1; r += 16) acc += *reinterpret_cast<const f32x4*>(A + base + r * N);
  }
  const f32x4 tot = combine_groups(acc, t, buf);
  if (t.live && t.grp == 0)
    *reinterpret_cast<f32x4*>(partial + ((long long)k * chunks + blockIdx.x) * N + 4 * t.cw) = tot;
}

// Wt[k][c][(u,v,o)] = W[k][o][(2-u, 2-v, c)]: the filter bank as the weight matrix of the
// convolution that maps the output gradient back to the input (taps mirrored, channels
// swapped).  A 32 x 32 (o, c) tile of one tap per workgroup, transposed through LDS so that both
// the reads (c contiguous) and the writes (o contiguous) are whole 128-byte rows.  32 | Cout.
__global__ __launch_bounds__(kThreads) void flip_filters_kernel(const float* __restrict__ W,
                                                                long long strideW, int ldw,
                                                                float* __restrict__ Wt, int Cout,
                                                                int Cin, int cblocks) {
  __shared__ float tile[32][33];
  const int ob = (blockIdx.x / cblocks) * 32, cb = (blockIdx.x % cblocks) * 32;
  const int tap = blockIdx.y;
  const long long k = blockIdx.z;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const float* src = W + k * strideW + (long long)(8 - tap) * Cin;
#pragma unroll
  for (int r = 0; r < 32; r += 8)
    tile[y + r][x] = cb + x < Cin ? src[(long long)(ob + y + r) * ldw + cb + x] : 0.f;
  __syncthreads();
  float* dst = Wt + k * (long long)Cin * 9 * Cout + (long long)tap * Cout + ob + x;
#pragma unroll
  for (int r = 0; r < 32; r += 8)
    if (cb + y + r < Cin) dst[(long long)(cb + y + r) * 9 * Cout] = tile[x][y + r];
}

// ---- first convolution layer (1..3 input channels) -------------------------------------------------
// With C <= 3 the contraction is 9 C <= 27 long: too short for the plane products, whose 16-byte units of the
// image would straddle taps.  These two kernels gather the image straight into the operands of
// v_mfma_f32_32x32x16_bf16 (the image of one replica is a few MB and stays in cache): rounded values, or the exact split
// of fp32 into three pieces (kernels_conv_gemm.hip), formed in registers.  Lane (l32, h) supplies elements (index
// l32, k = 8 h .. 8 h + 7) of each operand; accumulator element e of a lane belongs to (second operand's index l32,
// first operand's index (e/4)*8 + h*4 + e%4).  What bounds them is vector work per pixel (gather, split), not the
// matrix units and, with few channels, not the memory: on the fp32 units, at a depth of 2 a step with a gather and a decision
// each, they took 2 to 6 times the time of their bytes.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct FirstConv {
  int H, W, Cout;
  float invW, invH;
  long long rows;          // B H W pixels per replica
  long long strideParams;  // floats between replicas' parameter (or gradient) vectors
  int ldw;                 // row pitch of the filter bank [Cout][9 C (+ padding)]
};
constexpr unsigned kOob = 0x7FFFFFF0u;   // byte offset past any operand: the load yields zero

__device__ __forceinline__ void pixel_rc(int p, const FirstConv& f, int& i, int& j) {
  int q = (int)((float)p * f.invW);
  int r = p - q * f.W;
  if (r < 0) { r += f.W; --q; } else if (r >= f.W) { r -= f.W; ++q; }
  j = r;
  const int q2 = (int)((float)q * f.invH);
  int r2 = q - q2 * f.H;
  if (r2 < 0) r2 += f.H; else if (r2 >= f.H) r2 -= f.H;
  i = r2;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t float_rsrc(const float* base, long long n) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(base);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  void* ptr = reinterpret_cast<void*>(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ptr, 0, __builtin_amdgcn_readfirstlane((unsigned)(n * 4)), 0x00020000);
}
__device__ __forceinline__ float load_float(__amdgpu_buffer_rsrc_t rs, unsigned at, int scalar = 0) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, at, scalar, 0));
}

// Eight floats as the NP planes of an operand fragment.
template <int NP>
__device__ __forceinline__ void split_fragment(const float (&x)[8], u32x4 (&f)[NP]) {
  unsigned o[NP][4];
  split_words<NP>(x, o);
  if constexpr (NP == 3) {
    float most = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) most = largest_of(most, x[e]);
    if (past_rounding(most)) split_words_any<NP>(x, o);
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) f[q] = u32x4{o[q][0], o[q][1], o[q][2], o[q][3]};
}
// `at` where bit `bit` of `ok` is set, past every operand elsewhere (two instructions).
__device__ __forceinline__ unsigned if_bit(unsigned ok, int bit, unsigned at) {
  const unsigned m = (unsigned)((int)(ok << (31 - bit)) >> 31);
  return (at & m) | (kOob & ~m);
}
// acc (and, with three planes, low: the five small products) += first x second, smallest products first.
template <int NP>
__device__ __forceinline__ void multiply(const u32x4 (&first)[NP], const u32x4 (&second)[NP], f32x16& acc, f32x16& low) {
  if constexpr (NP == 3) {
    constexpr int xa[5] = {2, 0, 1, 1, 0}, xb[5] = {0, 2, 1, 0, 1};
#pragma unroll
    for (int q = 0; q < 5; ++q)
      low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, first[xa[q]]), __builtin_bit_cast(bf16x8, second[xb[q]]),
                                                    low, 0, 0, 0);
  }
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, first[0]), __builtin_bit_cast(bf16x8, second[0]), acc, 0, 0, 0);
}

// out[k][p][o] = relu(b[o] + sum_t unfolded(p, t) W[o][t]).  A workgroup takes 128 `tiles` consecutive pixels, a quarter a
// wavefront, 32 at a time, and 32 OB channels, whose filters it keeps in LDS as planes; a lane gathers its pixel's values of
// the next 32 under the products of the current ones.  `sums` (may be null): the statistics of the results, a chunk a
// workgroup, as launch_bn_stats leaves them.  4 replicas of 128 images of 32 x 32, on the fp32 units and the statistics beside it,
// then so: 16 channels 33 and 9 us, 21; 64 channels 57 and 22, 41, with rounded operands 31 (4.4 TB/s).
template <int C, int OB, int NP>
__global__ __launch_bounds__(kThreads) void first_conv_forward_kernel(const float* __restrict__ X,
                                                                      const float* __restrict__ params,
                                                                      long long w_off, long long b_off,
                                                                      float* __restrict__ out, FirstConv f, int tiles, int relu,
                                                                      float* __restrict__ sums) {
  constexpr int KC = (9 * C + 15) / 16;        // matrix depths
  __shared__ __attribute__((aligned(16))) unsigned short filters[NP][32 * OB][32];
  __shared__ float wsum[2][4][32 * OB];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int k = blockIdx.y, o0 = blockIdx.z * (32 * OB);
  {
    // rows of 32 values (lanes along t: whole lines of the filter bank); unit u of row o at u ^ (o / 4) % 4
    const float* Wg = params + (long long)k * f.strideParams + w_off;
    for (int e = threadIdx.x; e < OB * 32 * 32; e += kThreads) {
      const int o = e >> 5, t = e & 31;
      unsigned short b[NP];
      split_planes<NP>(t < 9 * C && o0 + o < f.Cout ? Wg[(long long)(o0 + o) * f.ldw + t] : 0.f, b);
#pragma unroll
      for (int q = 0; q < NP; ++q) filters[q][o][(((t >> 3) ^ ((o >> 2) & 3)) << 3) + (t & 7)] = b[q];
    }
  }
  const int rows = (int)f.rows;
  const int first = (blockIdx.x * 4 + wave) * tiles * 32;
  const __amdgpu_buffer_rsrc_t img = float_rsrc(X + (long long)k * f.rows * C, f.rows * C);
  const __amdgpu_buffer_rsrc_t dst = float_rsrc(out + (long long)k * f.rows * f.Cout, f.rows * f.Cout);
  // this lane's values of the unfolded image: where they lie from its pixel's, and which of them lose a rim
  int off[KC][8];
  unsigned masks[2][5] = {};                   // (constants: only the choice by h is left to run time)
#pragma unroll
  for (int kc = 0; kc < KC; ++kc)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      int at[2];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int t = kc * 16 + half * 8 + e, tap = t / C, du = tap / 3, dv = tap - 3 * du;
        const unsigned bit = 1u << (kc * 8 + e);
        at[half] = (((du - 1) * f.W + dv - 1) * C + (t - tap * C)) * 4;
        masks[half][0] |= t < 9 * C ? bit : 0u;
        masks[half][1] |= du == 0 ? bit : 0u;
        masks[half][2] |= du == 2 ? bit : 0u;
        masks[half][3] |= dv == 0 ? bit : 0u;
        masks[half][4] |= dv == 2 ? bit : 0u;
      }
      off[kc][e] = h ? at[1] : at[0];
    }
  const unsigned there = h ? masks[1][0] : masks[0][0], top = h ? masks[1][1] : masks[0][1], bottom = h ? masks[1][2] : masks[0][2],
                 left = h ? masks[1][3] : masks[0][3], right = h ? masks[1][4] : masks[0][4];
  float x[KC][8];
  const auto gather = [&](int p) {
    int i, j;
    pixel_rc(p < rows ? p : 0, f, i, j);
    const unsigned ok = (p < rows ? there : 0u) & ~((i == 0 ? top : 0u) | (i == f.H - 1 ? bottom : 0u) | (j == 0 ? left : 0u) |
                                                    (j == f.W - 1 ? right : 0u));
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int e = 0; e < 8; ++e) x[kc][e] = load_float(img, if_bit(ok, kc * 8 + e, (unsigned)(p * (C * 4) + off[kc][e])));
  };
  float bv[OB], z0[OB], s1[OB], s2[OB];
  bool mine[OB];
#pragma unroll
  for (int q = 0; q < OB; ++q) {
    mine[q] = o0 + 32 * q + l32 < f.Cout;      // (the last block of 32 channels need not be full)
    bv[q] = mine[q] ? (params + (long long)k * f.strideParams + b_off)[o0 + 32 * q + l32] : 0.f;
    z0[q] = s1[q] = s2[q] = 0.f;
  }
  gather(first + l32);
  __syncthreads();
  for (int tile = 0; tile < tiles; ++tile) {
    const int tile0 = first + tile * 32;
    if (tile0 >= rows) break;
    u32x4 fx[KC][NP];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) split_fragment<NP>(x[kc], fx[kc]);
    if (tile + 1 < tiles) gather(tile0 + 32 + l32);
    // acc[e] of lane (l32, h): channel l32 of the block, pixel tile0 + (e/4)*8 + h*4 + e%4, so
    // that a store instruction writes two whole 128-byte rows
#pragma unroll
    for (int q = 0; q < OB; ++q) {
      f32x16 acc, low;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = low[e] = 0.f;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        u32x4 fw[NP];
        const int o = 32 * q + l32;
#pragma unroll
        for (int pl = 0; pl < NP; ++pl)
          fw[pl] = *reinterpret_cast<const u32x4*>(&filters[pl][o][((kc * 2 + h) ^ ((o >> 2) & 3)) << 3]);
        multiply<NP>(fx[kc], fw, acc, low);
      }
      if constexpr (NP == 3) join_sums(acc, low);
      if (tile == 0) z0[q] = __shfl(acc[0], l32, 64) + bv[q];    // the wavefront's first pixel
      const unsigned at = mine[q] ? (unsigned)(tile0 + h * 4) * (unsigned)(f.Cout * 4) + (unsigned)(o0 + 32 * q + l32) * 4u : kOob;
      const auto write = [&](auto whole) {       // (a whole tile of pixels: no pixel is looked at by itself)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int pp = (e / 4) * 8 + e % 4;
          const float z = acc[e] + bv[q];
          if (!decltype(whole)::value && tile0 + h * 4 + pp >= rows) continue;
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, relu && !(z > 0.f) ? 0.f : z), dst, at, pp * f.Cout * 4, 0);
          const float dlt = z - z0[q];
          s1[q] += dlt;
          s2[q] += dlt * dlt;
        }
      };
      if (tile0 + 32 <= rows) write(std::true_type{});
      else write(std::false_type{});
    }
  }
  if (sums == nullptr) return;
  const auto pixels_of = [&](int w) {
    const int left_over = rows - (int)((blockIdx.x * 4 + w) * tiles * 32);
    return left_over < 0 ? 0 : left_over < tiles * 32 ? left_over : tiles * 32;
  };
#pragma unroll
  for (int q = 0; q < OB; ++q) {
    s1[q] += __shfl_xor(s1[q], 32, 64);
    s2[q] += __shfl_xor(s2[q], 32, 64);
    const int n = pixels_of(wave);
    const float inv_n = n > 0 ? 1.f / (float)n : 0.f, m2 = s2[q] - s1[q] * s1[q] * inv_n;
    if (h == 0) {
      wsum[0][wave][32 * q + l32] = z0[q] + s1[q] * inv_n;
      wsum[1][wave][32 * q + l32] = m2 > 0.f ? m2 : 0.f;
    }
  }
  __syncthreads();
  const int c = threadIdx.x;
  if (c < 32 * OB && o0 + c < f.Cout) {
    float mean = 0.f, m2 = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) mean += (float)pixels_of(w) * wsum[0][w][c];
    mean /= (float)((pixels_of(0) + pixels_of(1)) + (pixels_of(2) + pixels_of(3)));
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float dlt = wsum[0][w][c] - mean;
      m2 += wsum[1][w][c] + (float)pixels_of(w) * dlt * dlt;
    }
    float* dst = sums + ((long long)k * gridDim.x + blockIdx.x) * f.Cout + o0 + c;
    dst[0] = mean;
    dst[(long long)gridDim.y * gridDim.x * f.Cout] = m2;
  }
}

// Weight and bias gradient, first stage: workgroup (chunk, k) covers `chunk_px` pixels, a quarter per
// wavefront, 16 at a time, and 32 OB channels (blockIdx.z); partial[k][chunk][o][t] = sum over its pixels of dZ[p][o]
// unfolded(p, t), with t = 9 C standing for the constant 1 (that column is the bias gradient).  The four
// wavefronts' sums are added in wave order through LDS.  NORM: dZ is not read but formed from dY (dout) and Z, which saves the
// normalisation's kernel that wrote it (8 bytes a value more than these loads).  The next 16 pixels' values are requested
// under the products of the current ones.  4 replicas of 128 images of 32 x 32, on the fp32 units and the normalisation's kernel,
// then so: 16 channels 43 and 16 us, 24; 64 channels 57 and 61, 65, with rounded operands 54 (5.0 TB/s).  Few pixels leave it a chain of latencies: with 512 pixels a workgroup
// a step of one 64-channel layer on 4096 pixels took 175 us, with 64 it took 121 (64 to 512, as few as give the launch a
// thousand workgroups).
template <int C, int OB, int NP, bool NORM>
__global__ __launch_bounds__(kThreads) void first_conv_wgrad_kernel(const float* __restrict__ X,
                                                                    const float* __restrict__ dout,
                                                                    float* __restrict__ partial,
                                                                    int chunks, int chunk_px, FirstConv f, FirstNorm norm) {
  __shared__ float red[3][32 * 32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int k = blockIdx.y, ob = blockIdx.z * (32 * OB);
  const int rows = (int)f.rows;
  const __amdgpu_buffer_rsrc_t img = float_rsrc(X + (long long)k * f.rows * C, f.rows * C);
  const __amdgpu_buffer_rsrc_t dz = float_rsrc(dout + (long long)k * f.rows * f.Cout, f.rows * f.Cout);
  const __amdgpu_buffer_rsrc_t zs = NORM ? float_rsrc(norm.z + (long long)k * f.rows * f.Cout, f.rows * f.Cout) : dz;
  const int p0 = blockIdx.x * chunk_px + wave * (chunk_px / 4);
  // this lane's column of the unfolded image: fixed tap and channel
  const int t = l32, tap = t / C, du = tap / 3 - 1, dv = tap % 3 - 1;
  const int shift = ((du * f.W + dv) * C + t - tap * C) * 4;
  f32x16 acc[OB], low[OB];
  unsigned col[OB];                            // this lane's channels; past the last one: out of range
  float mu[OB], scale[OB], base[OB], slope[OB];                // dZ = scale (dY - base - (Z - mu) slope)
#pragma unroll
  for (int q = 0; q < OB; ++q) {
    const int c = ob + 32 * q + l32;
    const bool mine = c < f.Cout;
    col[q] = mine ? (unsigned)c * 4u : kOob;
    if constexpr (NORM) {
      const float* st = norm.stats + (long long)k * 2 * f.Cout;
      const float inv_n = 1.f / (float)rows;
      mu[q] = mine ? st[c] : 0.f;
      const float inv = mine ? st[f.Cout + c] : 0.f;
      scale[q] = mine ? norm.params[k * f.strideParams + norm.gam_off + c] * inv : 0.f;
      slope[q] = mine ? inv * (norm.grad[k * f.strideParams + norm.gam_off + c] * inv_n) : 0.f;
      base[q] = mine ? norm.grad[k * f.strideParams + norm.bet_off + c] * inv_n : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[q][e] = low[q][e] = 0.f;
  }
  float b[8], a[OB][8], z[NORM ? OB : 1][8];
  const bool rows_of_8 = f.W % 8 == 0;         // eight pixels from a multiple of 8 on lie in one row of the image
  const int pixel = f.Cout * 4;
  const auto request = [&](int pstart) {
    const int p8 = pstart + h * 8;
    int i, j;
    pixel_rc(p8 < rows ? p8 : 0, f, i, j);
    if (rows_of_8) {
      const bool ok = t < 9 * C && p8 < rows && (unsigned)(i + du) < (unsigned)f.H;
      const unsigned at = ok ? (unsigned)(p8 * (C * 4) + shift) : kOob;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool off_rim = e == 0 ? dv < 0 && j == 0 : e == 7 && dv > 0 && j + 8 == f.W;
        b[e] = load_float(img, (off_rim ? kOob : at) + e * (C * 4));
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int p = p8 + e;
        const bool ok = t < 9 * C && p < rows && (unsigned)(i + du) < (unsigned)f.H && (unsigned)(j + dv) < (unsigned)f.W;
        b[e] = load_float(img, ok ? (unsigned)(p * (C * 4) + shift) : kOob);
        if (++j == f.W) {
          j = 0;
          if (++i == f.H) i = 0;
        }
      }
    }
    if (t == 9 * C)
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = p8 + e < rows ? 1.f : 0.f;
    // A scalar offset may be left out of the buffer's range check, or be more than the whole buffer: only where all sixteen
    // pixels exist.  A pixel past the last one must read as zero: its value meets b = 0, but 0 times another replica's NaN is NaN.
    if (pstart + 16 <= rows) {
#pragma unroll
      for (int q = 0; q < OB; ++q) {
        const unsigned at = col[q] != kOob ? (unsigned)p8 * (unsigned)pixel + col[q] : kOob;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          a[q][e] = load_float(dz, at, e * pixel);
          if constexpr (NORM) z[q][e] = load_float(zs, at, e * pixel);
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < OB; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned at = p8 + e < rows && col[q] != kOob ? (unsigned)(p8 + e) * (unsigned)pixel + col[q] : kOob;
          a[q][e] = load_float(dz, at);
          if constexpr (NORM) z[q][e] = load_float(zs, at);
        }
    }
  };
  request(p0);
  for (int s = 0; s < chunk_px / 64; ++s) {
    u32x4 fb[NP], fa[OB][NP];
    split_fragment<NP>(b, fb);
#pragma unroll
    for (int q = 0; q < OB; ++q) {
      if constexpr (NORM) {
#pragma unroll
        for (int e = 0; e < 8; ++e) a[q][e] = scale[q] * ((a[q][e] - base[q]) - (z[q][e] - mu[q]) * slope[q]);
      }
      split_fragment<NP>(a[q], fa[q]);
    }
    if (s + 1 < chunk_px / 64) request(p0 + (s + 1) * 16);
#pragma unroll
    for (int q = 0; q < OB; ++q) multiply<NP>(fb, fa[q], acc[q], low[q]);
  }
  // acc[q][e]: o = ob + 32 q + l32, t = (e/4)*8 + h*4 + e%4
#pragma unroll
  for (int q = 0; q < OB; ++q) {
    if constexpr (NP == 3) join_sums(acc[q], low[q]);
    if (wave > 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) red[wave - 1][l32 * 32 + (e / 4) * 8 + h * 4 + e % 4] = acc[q][e];
    }
    __syncthreads();
    if (wave == 0 && ob + 32 * q + l32 < f.Cout) {
      float* dst = partial + (((long long)k * chunks + blockIdx.x) * f.Cout + ob + 32 * q + l32) * 32;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int tt = u * 8 + h * 4;
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int at = l32 * 32 + tt + r;
          v[r] = ((acc[q][u * 4 + r] + red[0][at]) + red[1][at]) + red[2][at];
        }
        *reinterpret_cast<f32x4*>(dst + tt) = v;
      }
    }
    __syncthreads();
  }
}

// Second stage: dW[k][o][t] (t < 9 C) and db[k][o] (t = 9 C) = sum over the chunks.  Workgroup
// (block, k) finishes 64 elements with 16 chains of loads each (chain q adds chunks q, q+16,
// ...), combined pairwise in a fixed tree through LDS; it also writes the sum of the squares of
// what it stored to its own slot.
constexpr int kFinishChains = 16;
__global__ __launch_bounds__(1024) void first_conv_wgrad_finish_kernel(const float* __restrict__ partial,
                                                                       int chunks, int C,
                                                                       float* __restrict__ grad,
                                                                       long long w_off, long long b_off,
                                                                       double* __restrict__ sumsq,
                                                                       long long strideSumsq,
                                                                       FirstConv f, int skip_bias) {
  __shared__ float part[kFinishChains][64];
  const int word = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int k = blockIdx.y;
  const int total = f.Cout * 32;
  const int e = blockIdx.x * 64 + word;       // o * 32 + t; total is a multiple of 64
  float v = 0.f;
  for (int ch = q; ch < chunks; ch += kFinishChains) v += partial[((long long)k * chunks + ch) * total + e];
  part[q][word] = v;
  __syncthreads();
#pragma unroll
  for (int half = kFinishChains / 2; half > 0; half >>= 1) {
    if (q < half) part[q][word] += part[q + half][word];
    __syncthreads();
  }
  if (q == 0) {
    v = part[0][word];
    float* g = grad + (long long)k * f.strideParams;
    const int o = e >> 5, t = e & 31;
    double ssq = 0.0;
    if (t < 9 * C) { g[w_off + (long long)o * f.ldw + t] = v; ssq = (double)v * (double)v; }
    else if (t == 9 * C && !skip_bias) { g[b_off + o] = v; ssq = (double)v * (double)v; }
    if (sumsq != nullptr) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) ssq += __shfl_xor(ssq, off, 64);
      if (word == 0) sumsq[(long long)k * strideSumsq + blockIdx.x] = ssq;
    }
  }
}

// ---- batch normalisation (training mode, per replica and channel over the B H W rows) -------------
// (Appendix "Batch Normalization": each worker uses the statistics of its own minibatch.)
// Z is [K][rows][C] (C % 4 == 0, C <= 1024).  Statistics in one pass over Z that does not lose
// digits when |mean| >> spread: every chunk of rows gets its own mean and its own sum of
// squared deviations from that mean (computed around the chunk's first row); the chunks are
// then combined in double, in a fixed order.
// (Chunks and thread layout: see colsum_partial_kernel.)
__global__ __launch_bounds__(kThreads) void bn_stats_partial_kernel(const float* __restrict__ Z,
                                                                    float* __restrict__ pmean,
                                                                    float* __restrict__ pm2,
                                                                    long long rows, int C, int chunks,
                                                                    int chunk_rows) {
  __shared__ f32x4 buf[kThreads];
  const ChunkThread t = chunk_thread(rows, C, chunk_rows);
  const int k = blockIdx.y;
  const float* base = Z + ((long long)k * rows) * C + 4 * t.cw;
  // One sweep: sums of (z - z0) and (z - z0)^2 with z0 the chunk's first row, a value of the
  // data's own size, so neither sum loses digits to a mean far from zero; then
  //   mean = z0 + s1 / n,   M2 = s2 - s1^2 / n.
  f32x4 s1 = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f}, z0 = {0.f, 0.f, 0.f, 0.f};
  if (t.live) {
    z0 = *reinterpret_cast<const f32x4*>(base + t.r0 * C);
    for (long long r = t.r0 + t.grp; r < t.r1; r += 16) {
      const f32x4 dlt = *reinterpret_cast<const f32x4*>(base + r * C) - z0;
      s1 += dlt;
      s2 += dlt * dlt;
    }
  }
  const f32x4 t1 = combine_groups(s1, t, buf);
  const f32x4 t2 = combine_groups(s2, t, buf);
  if (t.live && t.grp == 0) {
    const float inv_n = 1.f / (float)(t.r1 - t.r0);
    const long long at = ((long long)k * chunks + blockIdx.x) * C + 4 * t.cw;
    *reinterpret_cast<f32x4*>(pmean + at) = z0 + t1 * inv_n;
    f32x4 m2 = t2 - t1 * t1 * inv_n;
#pragma unroll
    for (int r = 0; r < 4; ++r) m2[r] = m2[r] > 0.f ? m2[r] : 0.f;
    *reinterpret_cast<f32x4*>(pm2 + at) = m2;
  }
}

// stats[k][0][c] = mean, stats[k][1][c] = 1 / sqrt(var + eps), var = M2 / rows (biased):
//   mean = sum_i n_i mean_i / rows,   M2 = sum_i [M2_i + n_i (mean_i - mean)^2]
// over the chunks i, in double, in a fixed order.  Next to nothing is read, so what bounds this is
// the chain of loads a thread has to wait for: workgroup (block, k) serves 16 columns with 64 chains
// each (chain q takes chunks q, q + 64, ...), DEPTH chunks in flight per chain, and the first 64 DEPTH chunks stay in
// registers for the second sum: 16 deep, or 4 or 1 where there are no more chunks than that (up to 64 chunks: 4.1 to 4.7 us with
// eight in flight and a loop that ends, 4.5 to 5.0 with the depth of 16, whose skipped chunks are not free).  512 chunks of 64
// columns, four replicas: 18 us with 16 chains and a load at a time, 11 us with eight in flight and read twice, 7.5 us so;
// 128 chunks 14, 5.5 and 5.3.
constexpr int kBnCols = 16, kBnChains = 64;
__device__ __forceinline__ double chain_total(double v, double (*buf)[kBnCols], int col) {
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  __syncthreads();                       // the values of the call before have been read
  if ((threadIdx.x & 63) < kBnCols) buf[threadIdx.x >> 6][col] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kBnCols * kBnChains / 64; ++w) t += buf[w][col];
  return t;
}
template <int DEPTH>
__global__ __launch_bounds__(kBnCols * kBnChains) void bn_stats_finish_kernel(
    const float* __restrict__ pmean, const float* __restrict__ pm2, float* __restrict__ stats,
    long long rows, int C, int chunks, int chunk_rows, float eps) {
  __shared__ double buf[kBnCols * kBnChains / 64][kBnCols];
  const int col = threadIdx.x % kBnCols, q = threadIdx.x / kBnCols;
  const int c = blockIdx.x * kBnCols + col;
  const int k = blockIdx.y;
  const bool live = c < C;
  const double last = (double)(rows - (long long)(chunks - 1) * chunk_rows);
  auto count = [&](int ch) { return ch + 1 < chunks ? (double)chunk_rows : last; };
  const long long base = (long long)k * chunks * C + c;
  float m[DEPTH], v[DEPTH];
  const auto read = [&](int ch0) {
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {
      const int ch = ch0 + i * kBnChains;
      const bool there = live && ch < chunks;
      m[i] = there ? pmean[base + (long long)ch * C] : 0.f;
      v[i] = there ? pm2[base + (long long)ch * C] : 0.f;
    }
  };
  const auto add = [&](int ch0, auto term) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
      if (ch0 + i * kBnChains < chunks) t += term(i, count(ch0 + i * kBnChains));
    return t;
  };
  const auto weighed = [&](int i, double n) { return n * (double)m[i]; };
  constexpr int kRound = kBnChains * DEPTH;
  double s1 = 0.0;
  for (int ch0 = q + kRound; ch0 < chunks; ch0 += kRound) {
    read(ch0);
    s1 += add(ch0, weighed);
  }
  read(q);
  s1 += add(q, weighed);
  const double mean = chain_total(s1, buf, col) / (double)rows;
  const auto spread = [&](int i, double n) {
    const double dlt = (double)m[i] - mean;
    return (double)v[i] + n * dlt * dlt;
  };
  double s2 = add(q, spread);
  for (int ch0 = q + kRound; ch0 < chunks; ch0 += kRound) {
    read(ch0);
    s2 += add(ch0, spread);
  }
  const double m2 = chain_total(s2, buf, col);
  if (live && q == 0) {
    stats[((long long)k * 2) * C + c] = (float)mean;
    stats[((long long)k * 2 + 1) * C + c] = (float)(1.0 / sqrt(m2 / (double)rows + (double)eps));
  }
}

// The shortcut of a residual block as the kernels read it: the block input [B][st H][st W][Cs]
// seen from an output pixel (i, j) and channel c is src[b][st i][st j][c] for c < Cs, 0 beyond.
// A projection shortcut instead: pz [K][rows][C] is the 1x1 convolution of the block input,
// normalised here with its own statistics pstats and gamma_p, beta_p (offsets into params).
struct Shortcut {
  const float* src;     // null: no parameter-free shortcut
  long long stride;     // floats from one replica's block input to the next
  int H, W, Cs, st;     // output image, channels of the block input, pixel step
  const float* pz;      // null: no projection
  const float* pstats;
  long long pgam_off, pbet_off;
};

// What a normalisation's kernels need of one word's columns c.. of replica k, and its output before the ReLU.
struct NormWord {
  f32x4 mu, inv, ga, be;
};
__device__ __forceinline__ NormWord norm_word(const float* __restrict__ stats, const float* __restrict__ params,
                                              long long strideParams, long long gam_off, long long bet_off, int k, int c, int C) {
  NormWord n;
  n.mu = *reinterpret_cast<const f32x4*>(stats + ((long long)k * 2) * C + c);
  n.inv = *reinterpret_cast<const f32x4*>(stats + ((long long)k * 2 + 1) * C + c);
  n.ga = *reinterpret_cast<const f32x4*>(params + k * strideParams + gam_off + c);
  n.be = *reinterpret_cast<const f32x4*>(params + k * strideParams + bet_off + c);
  return n;
}
__device__ __forceinline__ f32x4 normalised(const f32x4& z, const NormWord& n) { return n.ga * ((z - n.mu) * n.inv) + n.be; }
// The shortcut's value of word idx (columns c.. of replica k) added to y.
__device__ __forceinline__ f32x4 with_shortcut(f32x4 y, const Shortcut& sc, const NormWord& proj, long long idx, int k, int c,
                                               int words, long long rows) {
  if (sc.pz != nullptr) {
    y += normalised(*reinterpret_cast<const f32x4*>(sc.pz + idx * 4), proj);
  } else if (sc.src != nullptr && c < sc.Cs) {       // Cs % 4 == 0: a word lies inside or outside
    const long long m = idx / words - (long long)k * rows;       // (b, i, j) of this replica
    long long at = m * sc.Cs + c;
    if (sc.st != 1) {
      const int j = (int)(m % sc.W), i = (int)((m / sc.W) % sc.H);
      const long long b = m / ((long long)sc.W * sc.H);
      at = ((b * (sc.st * sc.H) + sc.st * i) * (sc.st * sc.W) + sc.st * j) * sc.Cs + c;
    }
    y += *reinterpret_cast<const f32x4*>(sc.src + k * sc.stride + at);
  }
  return y;
}
__device__ __forceinline__ f32x4 rectified(f32x4 y) {
#pragma unroll
  for (int r = 0; r < 4; ++r) y[r] = y[r] > 0.f ? y[r] : 0.f;
  return y;
}

// out = relu(gamma (Z - mean) inv_std + beta [+ shortcut]), its planes for the layer that reads it and the bits of its
// positive values.  Bound by its bytes: the floats are written only where something reads them (out null: not at
// all), since a product reads the planes and the gradient that comes back only asks for the sign.  64 channels with one plane,
// 4 replicas of 128 images of 32 x 32: 53.6 us with the floats, 33.4 without (6.3 TB/s).
// One thread per 16-byte word.
template <int NP>
__global__ __launch_bounds__(kThreads) void bn_apply_kernel(const float* __restrict__ Z,
                                                            const float* __restrict__ stats,
                                                            const float* __restrict__ params,
                                                            long long strideParams, long long gam_off,
                                                            long long bet_off, float* __restrict__ out,
                                                            long long rows, int C, long long total,
                                                            Shortcut sc, unsigned short* __restrict__ planes,
                                                            long long plane, unsigned char* __restrict__ keep) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= total) return;
  const int words = C / 4;
  const int c = (int)(idx % words) * 4;
  const int k = (int)(idx / words / rows);
  const NormWord n = norm_word(stats, params, strideParams, gam_off, bet_off, k, c, C);
  const NormWord proj = sc.pz != nullptr ? norm_word(sc.pstats, params, strideParams, sc.pgam_off, sc.pbet_off, k, c, C) : n;
  const f32x4 y = rectified(with_shortcut(normalised(*reinterpret_cast<const f32x4*>(Z + idx * 4), n), sc, proj, idx, k, c, words, rows));
  if (out != nullptr) *reinterpret_cast<f32x4*>(out + idx * 4) = y;
  if (keep != nullptr) keep[idx] = positive_bits(y);
  put_planes<NP>(planes, plane, idx * 4, y);
}

// The same followed by the 2x2 max-pool, one thread per word of the pooled image: the normalised image is not written.  Left for
// the backward pass: Z at each window's first maximum, which of the four that is, and the bits of the positive ones.
// 64 channels, 4 replicas of 128 images of 32 x 32, three planes: 43 and 35 us apart, 37 so; backward 44, 54 and 75 (pool, sums, gradient), 57 so.
template <int NP>
__global__ __launch_bounds__(kThreads) void bn_pool_kernel(const float* __restrict__ Z, const float* __restrict__ stats,
                                                           const float* __restrict__ params, long long strideParams,
                                                           long long gam_off, long long bet_off, float* __restrict__ P,
                                                           float* __restrict__ zmax, long long replica_words, PoolShape sh,
                                                           unsigned char* __restrict__ arg, unsigned char* __restrict__ keep,
                                                           unsigned short* __restrict__ planes, long long plane) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= sh.cells) return;
  const PoolCell w = pool_cell(idx, sh);
  const NormWord n = norm_word(stats, params, strideParams, gam_off, bet_off, (int)(idx / replica_words), w.c, sh.C);
  f32x4 z[4], v[4], m, zm;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    z[t] = *reinterpret_cast<const f32x4*>(Z + w.base + pool_offset(t, sh));
    v[t] = rectified(normalised(z[t], n));
  }
  const unsigned a = first_maximum(v, m);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const unsigned t = a >> (2 * r) & 3;
    zm[r] = t == 0 ? z[0][r] : t == 1 ? z[1][r] : t == 2 ? z[2][r] : z[3][r];
  }
  arg[idx] = (unsigned char)a;
  keep[idx] = positive_bits(m);
  *reinterpret_cast<f32x4*>(zmax + idx * 4) = zm;
  if (P != nullptr) *reinterpret_cast<f32x4*>(P + idx * 4) = m;
  put_planes<NP>(planes, plane, idx * 4, m);
}

// And followed by global average pooling: P[img][c] = mean over the positions, the image itself only as sign bits.  Workgroups
// and order of the sums as in avgpool_kernel.  320 channels at 16 x 16,
// 4 replicas of 128: 54 and 28 us apart, 40 so.
__global__ __launch_bounds__(kThreads) void bn_avgpool_kernel(const float* __restrict__ Z, const float* __restrict__ stats,
                                                              const float* __restrict__ params, long long strideParams,
                                                              long long gam_off, long long bet_off, float* __restrict__ P,
                                                              int HW, int C, int ldp, int images, Shortcut sc,
                                                              unsigned char* __restrict__ keep) {
  __shared__ f32x4 buf[kThreads];
  const int w = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int c = (blockIdx.y * 16 + w) * 4;
  const long long img = blockIdx.x;
  const int k = (int)(img / images), words = C / 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (c < C) {
    const NormWord n = norm_word(stats, params, strideParams, gam_off, bet_off, k, c, C);
    const NormWord proj = sc.pz != nullptr ? norm_word(sc.pstats, params, strideParams, sc.pgam_off, sc.pbet_off, k, c, C) : n;
#pragma unroll 4
    for (int p = grp; p < HW; p += 16) {
      const long long idx = (img * HW + p) * words + c / 4;
      const f32x4 y = rectified(with_shortcut(normalised(*reinterpret_cast<const f32x4*>(Z + idx * 4), n), sc, proj, idx, k, c, words,
                                              (long long)images * HW));
      keep[idx] = positive_bits(y);
      acc += y;
    }
  }
  buf[threadIdx.x] = acc;
  __syncthreads();
  if (grp == 0 && c < C) {
#pragma unroll
    for (int gq = 1; gq < 16; ++gq) acc += buf[gq * 16 + w];
    *reinterpret_cast<f32x4*>(P + img * ldp + c) = acc * (1.f / (float)HW);
  }
}

// The shortcut's share of the block input's gradient: dIn[b][st i][st j][c] += dY[b][i][j][c]
// for c < Cs (dY: gradient of the block output behind its ReLU), where the block input, itself
// a ReLU output `mask`, is positive (mask null: no such condition, the input came from a
// pool).  One thread per 16-byte word of the part of dY that has a counterpart.
__global__ __launch_bounds__(kThreads) void shortcut_backward_kernel(const float* __restrict__ dY,
                                                                     float* __restrict__ dIn,
                                                                     const float* __restrict__ mask,
                                                                     long long rows, int C, Shortcut sc,
                                                                     long long total) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= total) return;
  const int words = sc.Cs / 4;
  const int c = (int)(idx % words) * 4;
  long long m = idx / words;
  const int k = (int)(m / rows);
  m -= (long long)k * rows;
  const int j = (int)(m % sc.W), i = (int)((m / sc.W) % sc.H);
  const long long b = m / ((long long)sc.W * sc.H);
  const long long at = k * sc.stride + ((b * (sc.st * sc.H) + sc.st * i) * (sc.st * sc.W) + sc.st * j) * sc.Cs + c;
  f32x4 g = *reinterpret_cast<const f32x4*>(dY + ((long long)k * rows + m) * C + c);
  if (mask != nullptr) {
    const f32x4 keep = *reinterpret_cast<const f32x4*>(mask + at);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (!(keep[r] > 0.f)) g[r] = 0.f;
  }
  *reinterpret_cast<f32x4*>(dIn + at) += g;
}

// dst[k][b][i][j][c] = src[k][b][2 i][2 j][c]: the pixels a stride-2 1x1 convolution reads, as a
// dense matrix [K][B H W][C].  One thread per 16-byte word of dst.
__global__ __launch_bounds__(kThreads) void subsample2_kernel(const float* __restrict__ src,
                                                              float* __restrict__ dst, long long images,
                                                              int H, int W, int C, long long total) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= total) return;
  const int words = C / 4;
  const int c = (int)(idx % words) * 4;
  long long m = idx / words;
  const int j = (int)(m % W);
  m /= W;
  const int i = (int)(m % H);
  const long long img = m / H;
  const long long at = ((img * (2 * H) + 2 * i) * (2 * W) + 2 * j) * C + c;
  *reinterpret_cast<f32x4*>(dst + idx * 4) = *reinterpret_cast<const f32x4*>(src + at);
}

// dst += src, element by element (n a multiple of 4, both 16-byte aligned).
__global__ __launch_bounds__(kThreads) void add_into_kernel(float* __restrict__ dst,
                                                            const float* __restrict__ src, long long words) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= words) return;
  *reinterpret_cast<f32x4*>(dst + idx * 4) += *reinterpret_cast<const f32x4*>(src + idx * 4);
}

// Global average pooling: P[k][b][c] = mean over the H W positions of A[k][b][.][.][c], P rows of
// pitch ldp; and its backward pass fused with the ReLU the image came from:
// dA[k][b][i][j][c] = dP[k][b][c] / (H W) where A > 0 (A as floats, mask, or its bits, keep; both null: everywhere).  A workgroup sums
// the positions of 16 words of one image in 16 groups (position p in group p mod 16, the groups
// added in order); a thread per word alone walks the image with a load at a time: 128 channels,
// 16 x 16 positions, 512 images took 76 us, 12 us so (5.5 TB/s).
__global__ __launch_bounds__(kThreads) void avgpool_kernel(const float* __restrict__ A, float* __restrict__ P,
                                                           int HW, int C, int ldp) {
  __shared__ f32x4 buf[kThreads];
  const int w = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int c = (blockIdx.y * 16 + w) * 4;
  const long long img = blockIdx.x;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (c < C) {
    const float* a = A + img * (long long)HW * C + c;
#pragma unroll 4
    for (int p = grp; p < HW; p += 16) acc += *reinterpret_cast<const f32x4*>(a + (long long)p * C);
  }
  buf[threadIdx.x] = acc;
  __syncthreads();
  if (grp == 0 && c < C) {
#pragma unroll
    for (int gq = 1; gq < 16; ++gq) acc += buf[gq * 16 + w];
    *reinterpret_cast<f32x4*>(P + img * ldp + c) = acc * (1.f / (float)HW);
  }
}
__global__ __launch_bounds__(kThreads) void avgpool_backward_kernel(const float* __restrict__ dP,
                                                                    const float* __restrict__ mask,
                                                                    const unsigned char* __restrict__ keep,
                                                                    float* __restrict__ dA, long long images,
                                                                    int HW, int C, int ldp) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  const int words = C / 4;
  if (idx >= images * HW * words) return;
  const int c = (int)(idx % words) * 4;
  const long long img = idx / words / HW;
  f32x4 g = *reinterpret_cast<const f32x4*>(dP + img * ldp + c) * (1.f / (float)HW);
  if (keep != nullptr) {
    g = kept_values(g, keep[idx]);
  } else if (mask != nullptr) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(mask + idx * 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (!(a[r] > 0.f)) g[r] = 0.f;
  }
  *reinterpret_cast<f32x4*>(dA + idx * 4) = g;
}

// Word idx, columns c.. of row r of replica k, of the gradient a normalisation's backward pass starts from.
__device__ __forceinline__ f32x4 gradient_word(const GradSource& d, long long idx, int k, int r, int rows, int c) {
  f32x4 g;
  if (d.HW > 0) g = *reinterpret_cast<const f32x4*>(d.g + ((long long)k * (rows / d.HW) + r / d.HW) * d.ld + c) * (1.f / (float)d.HW);
  else g = *reinterpret_cast<const f32x4*>(d.g + idx * 4);
  return d.keep != nullptr ? kept_values(g, d.keep[idx]) : g;
}

// Chunk sums for the backward pass: part[k][chunk][0..C) = sum dY Xh, [C..2C) = sum dY, with
// Xh = (Z - mean) inv_std recomputed from Z.
__global__ __launch_bounds__(kThreads) void bn_backward_partial_kernel(const float* __restrict__ Z, GradSource d,
                                                                       const float* __restrict__ stats,
                                                                       float* __restrict__ part,
                                                                       long long rows, int C, int chunks,
                                                                       int chunk_rows) {
  __shared__ f32x4 buf[kThreads];
  const ChunkThread t = chunk_thread(rows, C, chunk_rows);
  const int k = blockIdx.y;
  f32x4 sg = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
  if (t.live) {
    const f32x4 mu = *reinterpret_cast<const f32x4*>(stats + ((long long)k * 2) * C + 4 * t.cw);
    const f32x4 inv = *reinterpret_cast<const f32x4*>(stats + ((long long)k * 2 + 1) * C + 4 * t.cw);
    const auto walk = [&](const GradSource& src) {
      for (long long r = t.r0 + t.grp; r < t.r1; r += 16) {
        const long long idx = (k * rows + r) * (C / 4) + t.cw;
        const f32x4 dy = gradient_word(src, idx, k, (int)r, (int)rows, 4 * t.cw);
        const f32x4 xh = (*reinterpret_cast<const f32x4*>(Z + idx * 4) - mu) * inv;
        sg += dy * xh;
        sb += dy;
      }
    };
    if (d.HW == 0 && d.keep == nullptr) walk(GradSource{d.g, nullptr, 0, 0});
    else walk(d);
  }
  const f32x4 tg = combine_groups(sg, t, buf);
  const f32x4 tb = combine_groups(sb, t, buf);
  if (t.live && t.grp == 0) {
    float* dst = part + ((long long)k * chunks + blockIdx.x) * 2 * C + 4 * t.cw;
    *reinterpret_cast<f32x4*>(dst) = tg;
    *reinterpret_cast<f32x4*>(dst + C) = tb;
  }
}

// What the gradient of a normalisation's input needs of one word's columns, and that gradient
//   dZ = gamma inv_std (dY - dbeta / N - Xh dgamma / N).
struct NormGradWord {
  f32x4 mu, inv, ga, dga, dbe;
};
__device__ __forceinline__ NormGradWord norm_grad_word(const float* __restrict__ stats, const float* __restrict__ params,
                                                       const float* __restrict__ grad, long long strideParams,
                                                       long long gam_off, long long bet_off, int k, int c, int C) {
  NormGradWord n;
  n.mu = *reinterpret_cast<const f32x4*>(stats + ((long long)k * 2) * C + c);
  n.inv = *reinterpret_cast<const f32x4*>(stats + ((long long)k * 2 + 1) * C + c);
  n.ga = *reinterpret_cast<const f32x4*>(params + k * strideParams + gam_off + c);
  n.dga = *reinterpret_cast<const f32x4*>(grad + k * strideParams + gam_off + c);
  n.dbe = *reinterpret_cast<const f32x4*>(grad + k * strideParams + bet_off + c);
  return n;
}
__device__ __forceinline__ f32x4 norm_gradient(const f32x4& z, const f32x4& dy, const NormGradWord& n, float inv_n) {
  const f32x4 xh = (z - n.mu) * n.inv;
  return n.ga * n.inv * (dy - n.dbe * inv_n - xh * (n.dga * inv_n));
}

// dZ [+ add], written to dZ (null: not at all), which may
// be dY itself or Z (every thread reads its own word of both before it writes), and to its planes.
template <int NP>
__global__ __launch_bounds__(kThreads) void bn_backward_apply_kernel(
    const float* Z, GradSource d, float* dZ, const float* __restrict__ stats,
    const float* __restrict__ params, const float* __restrict__ grad, long long strideParams,
    long long gam_off, long long bet_off, long long rows, int C, long long total, const float* add,
    unsigned short* __restrict__ planes, long long plane) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= total) return;
  const int words = C / 4;
  const int c = (int)(idx % words) * 4;
  const int k = (int)(idx / words / rows), r = (int)(idx / words - k * rows);
  const NormGradWord n = norm_grad_word(stats, params, grad, strideParams, gam_off, bet_off, k, c, C);
  f32x4 o = norm_gradient(*reinterpret_cast<const f32x4*>(Z + idx * 4), gradient_word(d, idx, k, r, (int)rows, c), n,
                          1.f / (float)rows);
  if (add != nullptr) o += *reinterpret_cast<const f32x4*>(add + idx * 4);
  if (dZ != nullptr) *reinterpret_cast<f32x4*>(dZ + idx * 4) = o;
  put_planes<NP>(planes, plane, idx * 4, o);
}

// The same where a pool follows the normalisation, one thread per word of the pooled gradient dP.
template <int NP>
__global__ __launch_bounds__(kThreads) void bn_pool_backward_kernel(
    const float* __restrict__ Z, const float* __restrict__ dP, const unsigned char* __restrict__ arg,
    const unsigned char* __restrict__ keep, float* __restrict__ dZ, const float* __restrict__ stats,
    const float* __restrict__ params, const float* __restrict__ grad, long long strideParams, long long gam_off, long long bet_off,
    long long rows, long long replica_words, PoolShape sh, unsigned short* __restrict__ planes, long long plane) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= sh.cells) return;
  const PoolCell w = pool_cell(idx, sh);
  const NormGradWord n =
      norm_grad_word(stats, params, grad, strideParams, gam_off, bet_off, (int)(idx / replica_words), w.c, sh.C);
  const f32x4 g = *reinterpret_cast<const f32x4*>(dP + idx * 4);
  const unsigned a = arg[idx], kept = keep[idx];
  f32x4 z[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) z[t] = *reinterpret_cast<const f32x4*>(Z + w.base + pool_offset(t, sh));
#pragma unroll
  for (unsigned t = 0; t < 4; ++t) {
    const f32x4 o = norm_gradient(z[t], unpooled(g, kept, a, t), n, 1.f / (float)rows);
    const long long at = w.base + pool_offset(t, sh);
    if (dZ != nullptr) *reinterpret_cast<f32x4*>(dZ + at) = o;
    put_planes<NP>(planes, plane, at, o);
  }
}

unsigned blocks_for(long long total) { return (unsigned)((total + kThreads - 1) / kThreads); }

}  // namespace

int launch_unfold3x3(const float* X, int64_t strideX, void* col, int np, int64_t plane, int ld, int K,
                     int B, int H, int W, int C, int stride, hipStream_t s) {
  ImgShape sh{H, W, C, ld, (long long)B * H * W, 0, stride};
  sh.total = (long long)K * sh.rows * (ld / 4);
  if (ld % 4 || ld < 9 * C || sh.total <= 0 || sh.total >= (1ll << 31) * kThreads || stride < 1 || stride > 2)
    return -1;
  const unsigned grid = blocks_for(sh.total);
  auto run = [&](auto kernel) { kernel<<<grid, kThreads, 0, s>>>(X, col, sh, strideX, plane); };
  if (C % 4 == 0)
    run(np == 0 ? unfold3x3_kernel<true, 0> : np == 1 ? unfold3x3_kernel<true, 1> : unfold3x3_kernel<true, 3>);
  else
    run(np == 0 ? unfold3x3_kernel<false, 0> : np == 1 ? unfold3x3_kernel<false, 1> : unfold3x3_kernel<false, 3>);
  return 0;
}

int launch_fold3x3(const float* dcol, int64_t strideCol, int ld, float* dX, const float* mask,
                   int64_t strideX, int K, int B, int H, int W, int C, int stride, hipStream_t s) {
  ImgShape sh{H, W, C, ld, (long long)B * H * W * stride * stride, 0, stride};
  sh.total = (long long)K * sh.rows * (C / 4);
  if (C % 4 || ld < 9 * C || sh.total <= 0 || sh.total >= (1ll << 31) * kThreads || stride < 1 || stride > 2)
    return -1;
  fold3x3_kernel<<<blocks_for(sh.total), kThreads, 0, s>>>(dcol, dX, mask, sh, strideCol, strideX);
  return 0;
}

void launch_flip_filters(const float* W, int64_t strideW, int ldw, float* Wt, int K, int Cout, int Cin,
                         hipStream_t s) {
  const int cblocks = (Cin + 31) / 32;
  flip_filters_kernel<<<dim3((unsigned)(Cout / 32 * cblocks), 9u, (unsigned)K), kThreads, 0, s>>>(
      W, strideW, ldw, Wt, Cout, Cin, cblocks);
}

// Channel counts that are no multiples of 32 fill these kernels' last block in part; the stored unfolded image
// they would take instead costs more, but for bf16 products of more than 64 channels, which run on the bf16 units
// there, from 5e6 outputs (a step of one such layer, before -> these: fp32, 16 channels 469 -> 356 us, 40 260 ->
// 228, 152 on 2.6e5 pixels 1033 -> 1014; bf16 products 404 -> 361, 260 -> 238; 104 on 3.3e4 pixels 193 -> 187, on 5e4 239 -> 243;
// 152 on 3.3e4 222 -> 221, 184 237 -> 245, 248 on 1.6e4 202 -> 198, on 6.1e4 377 -> 422).
bool first_conv_fits(int C, int Cout, int64_t rows, int K, int round) {
  if (C < 1 || C > 3 || Cout % 8 || Cout > 256 || rows >= (1 << 24)) return false;
  return Cout % 32 == 0 || !round || Cout <= 64 || K * rows * Cout <= 5000000;
}

static int first_chunk_px(int64_t rows, int Cout, int K) {
  int px = 512;
  while (px > 64 && (rows + px - 1) / px * K * ((Cout + 63) / 64) < 1024) px /= 2;
  return px;
}
int first_conv_chunks(int64_t rows, int Cout, int K) {
  const int px = first_chunk_px(rows, Cout, K);
  return (int)((rows + px - 1) / px);
}

static FirstConv first_shape(int H, int W, int Cout, int64_t rows, int64_t strideParams, int ldw) {
  return FirstConv{H, W, Cout, 1.f / (float)W, 1.f / (float)H, rows, strideParams, ldw};
}

// Pixels a workgroup of the forward kernel takes, in 128s: as many (up to 4) as leave the launch a thousand workgroups; what a
// workgroup does first, its filters, then counts least.
static int first_tiles(int64_t rows, int Cout, int K) {
  const int64_t groups = (rows + 127) / 128 * K * ((Cout + 63) / 64);
  return groups >= 4096 ? 4 : groups >= 2048 ? 2 : 1;
}
int launch_first_conv_forward(const float* X, const float* params, int64_t strideParams, int64_t w_off,
                              int64_t b_off, int ldw, float* out, int relu, int round, int K,
                              int64_t rows, int H, int W, int C, int Cout, float* sums, ChunkSums* made, hipStream_t s) {
  if (!first_conv_fits(C, Cout, rows, K, round)) return -1;
  const FirstConv f = first_shape(H, W, Cout, rows, strideParams, ldw);
  const int tiles = first_tiles(rows, Cout, K);
  // (few pixels give few workgroups: one for every 32 channels then)
  const int ob = Cout > 32 && (rows + 127) / 128 * K >= 512 ? 2 : 1;
  const dim3 grid((unsigned)((rows + 128 * tiles - 1) / (128 * tiles)), (unsigned)K, (unsigned)((Cout + 32 * ob - 1) / (32 * ob)));
  auto run = [&](auto kernel) { kernel<<<grid, kThreads, 0, s>>>(X, params, w_off, b_off, out, f, tiles, relu, sums); };
  auto pick = [&](auto o1p1, auto o1p3, auto o2p1, auto o2p3) {
    run(ob == 1 ? (round ? o1p1 : o1p3) : (round ? o2p1 : o2p3));
  };
  if (C == 1) pick(first_conv_forward_kernel<1, 1, 1>, first_conv_forward_kernel<1, 1, 3>, first_conv_forward_kernel<1, 2, 1>, first_conv_forward_kernel<1, 2, 3>);
  else if (C == 2) pick(first_conv_forward_kernel<2, 1, 1>, first_conv_forward_kernel<2, 1, 3>, first_conv_forward_kernel<2, 2, 1>, first_conv_forward_kernel<2, 2, 3>);
  else pick(first_conv_forward_kernel<3, 1, 1>, first_conv_forward_kernel<3, 1, 3>, first_conv_forward_kernel<3, 2, 1>, first_conv_forward_kernel<3, 2, 3>);
  if (made) *made = sums ? ChunkSums{(int)grid.x, 128 * tiles} : ChunkSums{};
  return 0;
}

int launch_first_conv_wgrad(const float* X, const float* dout, const FirstNorm& norm, float* partial, float* grad,
                            int64_t strideParams, int64_t w_off, int64_t b_off, int ldw, int round,
                            int skip_bias, int K, int64_t rows, int H, int W, int C, int Cout,
                            double* sumsq, int64_t sumsq_stride, hipStream_t s) {
  if (!first_conv_fits(C, Cout, rows, K, round)) return -1;
  const FirstConv f = first_shape(H, W, Cout, rows, strideParams, ldw);
  const int chunks = first_conv_chunks(rows, Cout, K), px = first_chunk_px(rows, Cout, K);
  const int ob = Cout > 32 ? 2 : 1;
  const dim3 grid((unsigned)chunks, (unsigned)K, (unsigned)((Cout + 32 * ob - 1) / (32 * ob)));
  auto run = [&](auto kernel) { kernel<<<grid, kThreads, 0, s>>>(X, dout, partial, chunks, px, f, norm); };
  auto pick = [&](auto p1, auto p3, auto p1n, auto p3n) { run(norm.z ? (round ? p1n : p3n) : (round ? p1 : p3)); };
#define LSAM_FIRST_WGRAD(c, o)                                                                                       \
  pick(first_conv_wgrad_kernel<c, o, 1, false>, first_conv_wgrad_kernel<c, o, 3, false>, first_conv_wgrad_kernel<c, o, 1, true>, \
       first_conv_wgrad_kernel<c, o, 3, true>)
  if (C == 1 && ob == 1) LSAM_FIRST_WGRAD(1, 1);
  else if (C == 1) LSAM_FIRST_WGRAD(1, 2);
  else if (C == 2 && ob == 1) LSAM_FIRST_WGRAD(2, 1);
  else if (C == 2) LSAM_FIRST_WGRAD(2, 2);
  else if (ob == 1) LSAM_FIRST_WGRAD(3, 1);
  else LSAM_FIRST_WGRAD(3, 2);
#undef LSAM_FIRST_WGRAD
  first_conv_wgrad_finish_kernel<<<dim3((unsigned)(Cout / 2), (unsigned)K), 1024, 0, s>>>(
      partial, chunks, C, grad, w_off, b_off, sumsq, sumsq_stride, f, skip_bias);
  return Cout / 2;     // sum-of-squares slots written per replica
}

int bn_chunks(int64_t rows, int C, int K) { return chunk_plan(rows, C, K).chunks; }

int launch_bn_stats(const float* Z, float* scratch, const ChunkSums& have, float* stats, int K, int64_t rows, int C, float eps,
                    hipStream_t s) {
  if (C % 4 || C < 4 || C > 4 * kThreads || rows < 1) return -1;
  ChunkSums sums = have;
  const ChunkPlan pl = chunk_plan(rows, C, K);
  if (!sums.chunks) sums = ChunkSums{pl.chunks, pl.chunk_rows};
  float* pmean = scratch;
  float* pm2 = scratch + (long long)K * sums.chunks * C;
  if (!have.chunks)
    bn_stats_partial_kernel<<<dim3((unsigned)pl.chunks, (unsigned)K, (unsigned)pl.col_blocks), kThreads, 0, s>>>(
        Z, pmean, pm2, rows, C, pl.chunks, pl.chunk_rows);
  auto finish = [&](auto kernel) {
    kernel<<<dim3((unsigned)((C + kBnCols - 1) / kBnCols), (unsigned)K), kBnCols * kBnChains, 0, s>>>(pmean, pm2, stats, rows, C,
                                                                                                    sums.chunks, sums.rows, eps);
  };
  finish(sums.chunks <= kBnChains ? bn_stats_finish_kernel<1> : sums.chunks <= 4 * kBnChains ? bn_stats_finish_kernel<4>
                                                                                             : bn_stats_finish_kernel<16>);
  return 0;
}

int launch_add_into(float* dst, const float* src, int64_t n, hipStream_t s) {
  if (n < 4 || n % 4) return -1;
  add_into_kernel<<<blocks_for(n / 4), kThreads, 0, s>>>(dst, src, n / 4);
  return 0;
}

int launch_subsample2(const float* src, float* dst, int64_t images, int H, int W, int C, hipStream_t s) {
  if (C % 4 || C < 4 || H < 1 || W < 1 || images < 1) return -1;
  const long long total = images * H * W * (C / 4);
  subsample2_kernel<<<blocks_for(total), kThreads, 0, s>>>(src, dst, images, H, W, C, total);
  return 0;
}

// The shortcut as the kernels read it; -1: it does not fit the layer.
static int shortcut_of(const ShortcutDesc* d, int64_t rows, int C, Shortcut& sc) {
  sc = Shortcut{nullptr, 0, 1, 1, 0, 1, nullptr, nullptr, 0, 0};
  if (d == nullptr) return 0;
  if (d->pz != nullptr) {
    if (d->pstats == nullptr) return -1;
    sc.pz = d->pz; sc.pstats = d->pstats;
    sc.pgam_off = d->pgam_off; sc.pbet_off = d->pbet_off;
    return 0;
  }
  if (d->Cs % 4 || d->Cs > C || d->H < 1 || d->W < 1 || rows % ((int64_t)d->H * d->W) || d->step < 1 || d->step > 2) return -1;
  sc = Shortcut{d->src, d->stride, d->H, d->W, d->Cs, d->step, nullptr, nullptr, 0, 0};
  return 0;
}

int launch_bn_apply(const float* Z, const float* stats, const float* params, int64_t strideParams, int64_t gam_off, int64_t bet_off,
                    float* out, int K, int64_t rows, int C, const ShortcutDesc* shortcut, const PlaneOut& o, hipStream_t s) {
  Shortcut sc;
  if (C % 4 || C < 4 || rows < 1 || shortcut_of(shortcut, rows, C, sc) != 0) return -1;
  const long long total = (long long)K * rows * (C / 4);
  auto run = [&](auto kernel) {
    kernel<<<blocks_for(total), kThreads, 0, s>>>(Z, stats, params, strideParams, gam_off, bet_off, out, rows, C, total, sc,
                                                  o.p, o.plane, o.keep);
  };
  run(o.np == 0 ? bn_apply_kernel<0> : o.np == 1 ? bn_apply_kernel<1> : bn_apply_kernel<3>);
  return 0;
}

int launch_bn_pool(const float* Z, const float* stats, const float* params, int64_t strideParams, int64_t gam_off, int64_t bet_off,
                   float* P, float* zmax, uint8_t* arg, int K, int64_t images, int H, int W, int C, const PlaneOut& o, hipStream_t s) {
  const long long words = images * (H / 2) * (W / 2) * (C / 4);         // of a replica
  const PoolShape sh{H / 2, W / 2, C, K * words};
  if (C % 4 || C < 4 || H % 2 || W % 2 || words <= 0 || sh.cells >= (1ll << 31) * kThreads || o.keep == nullptr) return -1;
  auto run = [&](auto kernel) {
    kernel<<<blocks_for(sh.cells), kThreads, 0, s>>>(Z, stats, params, strideParams, gam_off, bet_off, P, zmax, words, sh, arg, o.keep,
                                                     o.p, o.plane);
  };
  run(o.np == 0 ? bn_pool_kernel<0> : o.np == 1 ? bn_pool_kernel<1> : bn_pool_kernel<3>);
  return 0;
}

int launch_bn_avgpool(const float* Z, const float* stats, const float* params, int64_t strideParams, int64_t gam_off,
                      int64_t bet_off, float* P, int K, int64_t images, int HW, int C, int ldp, const ShortcutDesc* shortcut,
                      uint8_t* keep, hipStream_t s) {
  Shortcut sc;
  if (C % 4 || C < 4 || HW < 1 || images < 1 || ldp < C || ldp % 4 || shortcut_of(shortcut, images * HW, C, sc) != 0) return -1;
  bn_avgpool_kernel<<<dim3((unsigned)(K * images), (unsigned)((C + 63) / 64)), kThreads, 0, s>>>(
      Z, stats, params, strideParams, gam_off, bet_off, P, HW, C, ldp, (int)images, sc, keep);
  return 0;
}

int launch_shortcut_backward(const float* dY, float* dIn, const float* mask, const ShortcutDesc& d, int K,
                             int64_t rows, int C, hipStream_t s) {
  if (d.Cs % 4 || d.Cs > C || d.Cs < 4 || rows % ((int64_t)d.H * d.W) || d.step < 1 || d.step > 2) return -1;
  const Shortcut sc{nullptr, d.stride, d.H, d.W, d.Cs, d.step, nullptr, nullptr, 0, 0};
  const long long total = (long long)K * rows * (d.Cs / 4);
  shortcut_backward_kernel<<<blocks_for(total), kThreads, 0, s>>>(dY, dIn, mask, rows, C, sc, total);
  return 0;
}

int launch_avgpool(const float* A, float* P, int64_t images, int HW, int C, int ldp, hipStream_t s) {
  if (C % 4 || HW < 1 || ldp < C || ldp % 4) return -1;
  avgpool_kernel<<<dim3((unsigned)images, (unsigned)((C + 63) / 64)), kThreads, 0, s>>>(A, P, HW, C, ldp);
  return 0;
}

int launch_avgpool_backward(const float* dP, const float* mask, const uint8_t* keep, float* dA, int64_t images, int HW, int C,
                            int ldp, hipStream_t s) {
  if (C % 4 || HW < 1 || ldp < C || ldp % 4) return -1;
  avgpool_backward_kernel<<<blocks_for(images * HW * (C / 4)), kThreads, 0, s>>>(dP, mask, keep, dA, images, HW, C, ldp);
  return 0;
}

int launch_bn_backward_partials(const float* Z, const GradSource& dY, const float* stats, float* part, int K,
                                int64_t rows, int C, hipStream_t s) {
  if (C % 4 || C < 4 || C > 4 * kThreads || rows < 1) return -1;
  const ChunkPlan pl = chunk_plan(rows, C, K);
  bn_backward_partial_kernel<<<dim3((unsigned)pl.chunks, (unsigned)K, (unsigned)pl.col_blocks), kThreads, 0,
                               s>>>(Z, dY, stats, part, rows, C, pl.chunks, pl.chunk_rows);
  return pl.chunks;
}

void launch_bn_backward_apply(const float* Z, const GradSource& dY, float* dZ, const float* stats,
                              const float* params, const float* grad, int64_t strideParams,
                              int64_t gam_off, int64_t bet_off, int K, int64_t rows, int C, const float* add,
                              const PlaneOut& o, hipStream_t s) {
  const long long total = (long long)K * rows * (C / 4);
  auto run = [&](auto kernel) {
    kernel<<<blocks_for(total), kThreads, 0, s>>>(Z, dY, dZ, stats, params, grad, strideParams, gam_off, bet_off, rows, C,
                                                  total, add, o.p, o.plane);
  };
  run(o.np == 0 ? bn_backward_apply_kernel<0> : o.np == 1 ? bn_backward_apply_kernel<1> : bn_backward_apply_kernel<3>);
}

void launch_bn_pool_backward(const float* Z, const float* dP, const uint8_t* arg, const uint8_t* keep, float* dZ, const float* stats,
                             const float* params, const float* grad, int64_t strideParams, int64_t gam_off, int64_t bet_off, int K,
                             int64_t images, int H, int W, int C, const PlaneOut& o, hipStream_t s) {
  const long long words = images * (H / 2) * (W / 2) * (C / 4);
  const PoolShape sh{H / 2, W / 2, C, K * words};
  auto run = [&](auto kernel) {
    kernel<<<blocks_for(sh.cells), kThreads, 0, s>>>(Z, dP, arg, keep, dZ, stats, params, grad, strideParams, gam_off, bet_off,
                                                     images * H * W, words, sh, o.p, o.plane);
  };
  run(o.np == 0 ? bn_pool_backward_kernel<0> : o.np == 1 ? bn_pool_backward_kernel<1> : bn_pool_backward_kernel<3>);
}

int colsum_chunks(int64_t rows, int N, int K) { return chunk_plan(rows, N, K).chunks; }

int launch_colsum_partials(const float* A, const uint8_t* keep, int64_t rows, int N, int K, float* partial, hipStream_t s) {
  if (N % 4 || N < 4 || N > 4 * kThreads || rows < 1) return -1;
  const ChunkPlan pl = chunk_plan(rows, N, K);
  colsum_partial_kernel<<<dim3((unsigned)pl.chunks, (unsigned)K, (unsigned)pl.col_blocks), kThreads, 0, s>>>(
      A, keep, partial, rows, N, pl.chunks, pl.chunk_rows);
  return pl.chunks;
}

int launch_maxpool2(const float* A, float* P, uint8_t* arg, int64_t images, int H, int W, int C, const PlaneOut& o, hipStream_t s) {
  const PoolShape sh{H / 2, W / 2, C, images * (H / 2) * (W / 2) * (C / 4)};
  if (C % 4 || H % 2 || W % 2 || sh.cells <= 0 || sh.cells >= (1ll << 31) * kThreads || o.keep == nullptr) return -1;
  auto run = [&](auto kernel) { kernel<<<blocks_for(sh.cells), kThreads, 0, s>>>(A, P, sh, arg, o.keep, o.p, o.plane); };
  run(o.np == 0 ? maxpool2_kernel<0> : o.np == 1 ? maxpool2_kernel<1> : maxpool2_kernel<3>);
  return 0;
}

int launch_maxpool2_backward(const float* dP, const uint8_t* arg, const uint8_t* keep, float* dA, int64_t images, int H,
                             int W, int C, const PlaneOut& o, hipStream_t s) {
  const PoolShape sh{H / 2, W / 2, C, images * (H / 2) * (W / 2) * (C / 4)};
  if (C % 4 || H % 2 || W % 2 || sh.cells <= 0 || sh.cells >= (1ll << 31) * kThreads) return -1;
  auto run = [&](auto kernel) { kernel<<<blocks_for(sh.cells), kThreads, 0, s>>>(dP, arg, keep, dA, sh, o.p, o.plane); };
  run(o.np == 0 ? maxpool2_backward_kernel<0> : o.np == 1 ? maxpool2_backward_kernel<1> : maxpool2_backward_kernel<3>);
  return 0;
}

}  // namespace lsam
