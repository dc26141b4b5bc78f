// Matrix products of the convolution layers on the bf16 matrix units, fp32 accumulate.
//
// Operands are "plane" tensors: every fp32 value x of an image, an output gradient or a filter
// bank is stored as NP bfloat16 values, in NP matrices of the same shape.
//   NP = 1  the value rounded to bfloat16: the arithmetic mode that rounds the operands of every
//           product (what the fp32-storage kernel did while it loaded them).
//   NP = 3  an exact split x = x0 + x1 + x2 (8 + 8 + 8 significand bits, each piece the rounding
//           of what the ones before it leave).  A product is formed from the six leading of the
//           nine cross products, smallest first; what is left out is below 2^-24 of |a||b|, under
//           the rounding of the fp32 accumulation itself, so this is fp32 arithmetic on units that
//           do 16 times the fp32 matrix rate (157 TFLOP/s nominal): six products leave 2.7 times.
// An infinite number, or NaN, is its own leading piece (the others are zero), so what infinite and
// overflowing operands come to is in the sum of the leading products; see join_sums.
// The split is exact from 2^-110 up: bfloat16 ends at 2^-133, so below that the last piece keeps
// what lies above 2^-134 (an operand is then off by at most 2^-134; below 2^-134 it is zero).
//
// The kernel is the ring of the dense bf16 products: buffer_load ... lds straight into a ring of
// NSTAGE k-steps of 32, one barrier per k-step, fragments read one half k-step ahead.  What differs
// is where a lane's 16 bytes come from:
//   ImgK  rows are output pixels, k = (tap, channel): the image is unfolded by address; taps
//         outside the image read out of the buffer's range, which yields zeros;
//   MatK  rows of a stored matrix, k contiguous (filter banks);
//   MatM  k selects the row (output gradients, k = pixel);
//   ImgM  k = pixel, columns are (tap, channel): the image unfolded by address.
// In LDS every operand lies as 32 x 32 blocks of 2 KiB with the unit permutation of b32s.h (a
// lane picks the unit it fetches, the copy itself is linear), so both kinds of fragment reads
// have few bank conflicts (measured: 0 to 13 % of the cycles the LDS is active).
#include <algorithm>
#include <type_traits>

#include "engine.h"
#include "planes.h"

namespace lsam {
namespace {

constexpr int kThreads = 256;
constexpr unsigned kOob = 0x7FFFFFF0u;   // byte offset past any operand: the load yields zeros

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) unsigned char lds_byte;

// How output pixels see the image: pixel (b, i, j) of [oH][oW], tap (a, c) of nu x nv, reads image
// pixel (st i + du0 + a, st j + dv0 + c) of [sH][sW].
// n / d for 0 <= n < 2^31 as the high word of n `magic`, shifted: magic = 2^(31 + l) / d rounded up, l = log2 d rounded up,
// is at most 2^-l of itself too large, which times n stays below 1 / d.  d >= 2.
struct Divisor {
  unsigned magic;
  int shift;
};
inline Divisor divisor(int d) {
  int l = 1;
  while ((1ll << l) < d) ++l;
  return Divisor{(unsigned)(((1ull << (31 + l)) + (unsigned)d - 1) / (unsigned)d), l - 1};
}
__device__ __forceinline__ int divide(int n, const Divisor& d) { return (int)(__umulhi((unsigned)n, d.magic) >> d.shift); }

struct Geometry {
  int C, oH, oW, sH, sW, st, nu, nv, du0, dv0;
  unsigned magicC;                 // 2^32 / C + 1: tap of a contraction index by a high multiply
  Divisor byW, byH, byH2;          // by oW, oH and oH + 2 (weight gradients from patches)
};

struct Params {
  const unsigned short* A; long long strideA, planeA; int ldA; unsigned bytesA;
  const unsigned short* B; long long strideB, planeB; int ldB; unsigned bytesB;
  float* C; long long strideC; int ldC;
  int M, N, Kd, batch;
  int tilesM, tilesN, total, chunks;
  Geometry g;
  int epilogue;
  const float* bias; long long strideBias;
  const float* mask; long long strideMask; int ldMask;
  const unsigned char* keep;                           // the mask as bits, see ConvGemmDesc
  double* sumsq; long long strideSumsq;
  int out_step, out_i, out_j;                          // see ConvGemmDesc
  int ksplit, steps_per_piece; float* partial; long long stridePartial; int ldP;
  const float* add; long long strideAdd; int ldAdd;        // added to the results (may be null)
  int sums; float* sum_part; const float* sum_z; const float* sum_stats;   // see ConvGemmDesc
};

constexpr int waitcnt(int vm, int lgkm) {
  return (vm & 0xF) | ((vm >> 4) << 14) | (0x7 << 4) | ((lgkm & 0xF) << 8);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, unsigned bytes) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(base);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  void* ptr = reinterpret_cast<void*>(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ptr, 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// (b, i, j) of output pixel p
__device__ __forceinline__ void decode(int p, const Geometry& g, int& b, int& i, int& j) {
  const int q = p / g.oW;
  j = p - q * g.oW;
  b = q / g.oH;
  i = q - b * g.oH;
}

// The same by high multiplies (sides of at least 2).
__device__ __forceinline__ void decode_fast(int p, const Geometry& g, int& b, int& i, int& j) {
  const int q = divide(p, g.byW);
  j = p - q * g.oW;
  b = divide(q, g.byH);
  i = q - b * g.oH;
}

// ---- operand loaders ------------------------------------------------------------------------------
// R rows (or columns) of the output; a wavefront instruction fills 1 KiB of LDS = 16 rows of 64
// bytes (k-major) or half a 32 x 32 block (m-major).  Operands shorter than 64 are loaded as 64 (the
// surplus lanes read out of range), so that every wavefront issues the same number of loads.
template <int R>
struct Shape {
  static constexpr int RL = R < 64 ? 64 : R;
  static constexpr int BYTES = RL * 64;               // one plane of one stage
  static constexpr int NLOAD = BYTES / (kThreads * 16);
};

template <int R, int NP, bool SCALAR_TAP>
struct ImgK {
  static constexpr bool KMAJOR = true;
  static constexpr int NLOAD = Shape<R>::NLOAD, BYTES = Shape<R>::BYTES;
  int off[NLOAD], ii[NLOAD], jj[NLOAD];
  int u8[NLOAD];                                       // first channel of this lane's unit in a k-step
  int c0, a, c;                                        // scalar taps: channel, tap row, tap column
  int e0;                                              // otherwise: contraction index of the k-step
  __device__ __forceinline__ void init(const Params& p, int row0, int first_step, int tid) {
    const Geometry& g = p.g;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      const int row = (wave * NLOAD + l) * 16 + (lane >> 2);
      const int u = (lane & 3) ^ ((row >> 2) & 3);
      u8[l] = u * 8;
      const int m = row0 + row;
      int b, i, j;
      decode(m, g, b, i, j);
      ii[l] = (row < R && m < p.M) ? g.st * i : (1 << 20);      // fails every bounds test
      jj[l] = g.st * j;
      off[l] = (int)((((unsigned)(b * g.sH + g.st * i)) * g.sW + g.st * j) * g.C) * 2;
      if (SCALAR_TAP) off[l] += u * 16;
    }
    e0 = first_step * 32;
    if constexpr (SCALAR_TAP) {
      const int tap = e0 / g.C;
      c0 = e0 - tap * g.C;
      a = tap / g.nv;
      c = tap - a * g.nv;
    }
  }
  __device__ __forceinline__ void issue(const Params& p, const __amdgpu_buffer_rsrc_t (&rs)[NP], lds_byte* tile, bool live) {
    const Geometry& g = p.g;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte* dst = tile + wave * NLOAD * 1024;
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      unsigned at;
      if constexpr (SCALAR_TAP) {
        const int du = g.du0 + a, dv = g.dv0 + c;
        const bool ok = live && (unsigned)(ii[l] + du) < (unsigned)g.sH && (unsigned)(jj[l] + dv) < (unsigned)g.sW;
        at = ok ? (unsigned)(off[l] + ((du * g.sW + dv) * g.C + c0) * 2) : kOob;
      } else {
        const int e = e0 + u8[l];
        const int tap = (int)__umulhi((unsigned)e, g.magicC);
        const int ch = e - tap * g.C;
        const int ta = (int)(((unsigned)tap * (g.nv == 3 ? 0x5556u : g.nv == 2 ? 0x8000u : 0x10000u)) >> 16);
        const int du = g.du0 + ta, dv = g.dv0 + tap - ta * g.nv;
        const bool ok = live && e < p.Kd && (unsigned)(ii[l] + du) < (unsigned)g.sH && (unsigned)(jj[l] + dv) < (unsigned)g.sW;
        at = ok ? (unsigned)(off[l] + ((du * g.sW + dv) * g.C + ch) * 2) : kOob;
      }
#pragma unroll
      for (int q = 0; q < NP; ++q)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[q], (__attribute__((address_space(3))) void*)(dst + q * BYTES + l * 1024),
                                                 16, at, 0, 0, 0);
    }
    if constexpr (SCALAR_TAP) {
      c0 += 32;
      if (c0 >= g.C) {
        c0 = 0;
        if (++c == g.nv) { c = 0; ++a; }
      }
    } else {
      e0 += 32;
    }
  }
};

// TAIL: Kd may end inside a k-step with more values of the row behind it (a class of pixels of a stride-2
// input gradient, followed by the next class's filters): they read as zeros.  The image's side is zero
// there as well, but zero times an infinite filter is not.
template <int R, int NP, bool TAIL>
struct MatK {
  static constexpr bool KMAJOR = true;
  static constexpr int NLOAD = Shape<R>::NLOAD, BYTES = Shape<R>::BYTES;
  unsigned off[NLOAD];
  int e;                                               // contraction index of this lane's unit
  __device__ __forceinline__ void init(const Params& p, int row0, int first_step, int tid) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = (lane & 3) ^ ((lane >> 4) & 3);
    e = first_step * 32 + u * 8;
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      const int row = (wave * NLOAD + l) * 16 + (lane >> 2);
      off[l] = (row < R && row0 + row < p.N) ? ((unsigned)(row0 + row) * p.ldB + e) * 2u : kOob;
    }
  }
  __device__ __forceinline__ void issue(const Params& p, const __amdgpu_buffer_rsrc_t (&rs)[NP], lds_byte* tile, bool live) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte* dst = tile + wave * NLOAD * 1024;
    const bool ok = live && (!TAIL || e < p.Kd);
    if (TAIL) e += 32;
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      const unsigned at = ok ? off[l] : kOob;
#pragma unroll
      for (int q = 0; q < NP; ++q)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[q], (__attribute__((address_space(3))) void*)(dst + q * BYTES + l * 1024),
                                                 16, at, 0, 0, 0);
      if (off[l] != kOob) off[l] += 64;
    }
  }
};

// A operand, k selects the row of a matrix [Kd][ldA].
template <int R, int NP>
struct MatM {
  static constexpr bool KMAJOR = false;
  static constexpr int NLOAD = Shape<R>::NLOAD, BYTES = Shape<R>::BYTES;
  unsigned off[NLOAD];
  __device__ __forceinline__ void init(const Params& p, int col0, int first_step, int tid) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      const int chunk = wave * NLOAD + l;
      const int row = (chunk & 1) * 16 + (lane >> 2);
      const int u = (lane & 3) ^ ((row >> 2) & 3);
      const int col = col0 + (chunk >> 1) * 32 + u * 8;
      off[l] = ((chunk >> 1) * 32 < R && col < p.ldA) ? ((unsigned)(first_step * 32 + row) * p.ldA + col) * 2u : kOob;
    }
  }
  __device__ __forceinline__ void issue(const Params& p, const __amdgpu_buffer_rsrc_t (&rs)[NP], lds_byte* tile, bool live) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte* dst = tile + wave * NLOAD * 1024;
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      // rows past Kd lie past the end of the buffer and read as zeros
      const unsigned at = live ? off[l] : kOob;
#pragma unroll
      for (int q = 0; q < NP; ++q)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[q], (__attribute__((address_space(3))) void*)(dst + q * BYTES + l * 1024),
                                                 16, at, 0, 0, 0);
      if (off[l] != kOob) off[l] += (unsigned)p.ldA * 64u;
    }
  }
};

// B operand, k = output pixel, columns n = (tap, channel) of the unfolded image.
template <int R, int NP>
struct ImgM {
  static constexpr bool KMAJOR = false;
  static constexpr int NLOAD = Shape<R>::NLOAD, BYTES = Shape<R>::BYTES;
  // a lane's loads touch at most two rows of a block: pixels of parity chunk & 1
  static constexpr int NPIX = NLOAD > 1 ? 2 : 1;
  int du[NLOAD], dv[NLOAD], coff[NLOAD];               // of the load's column
  int pix[NPIX], i[NPIX], j[NPIX], b[NPIX];
  int di, dj, db;                                      // 32 pixels further
  __device__ __forceinline__ void init(const Params& p, int col0, int first_step, int tid) {
    const Geometry& g = p.g;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      const int chunk = wave * NLOAD + l;
      const int row = (chunk & 1) * 16 + (lane >> 2);
      const int u = (lane & 3) ^ ((row >> 2) & 3);
      const int n = col0 + (chunk >> 1) * 32 + u * 8;
      if ((chunk >> 1) * 32 < R && n < p.N) {
        const int tap = n / g.C, ch = n - tap * g.C;
        du[l] = g.du0 + tap / g.nv;
        dv[l] = g.dv0 + tap % g.nv;
        coff[l] = ((du[l] * g.sW + dv[l]) * g.C + ch) * 2;
      } else {
        du[l] = 1 << 20; dv[l] = 0; coff[l] = 0;
      }
    }
#pragma unroll
    for (int q = 0; q < NPIX; ++q) {
      const int chunk = wave * NLOAD + q;
      pix[q] = first_step * 32 + (chunk & 1) * 16 + (lane >> 2);
      decode(pix[q], g, b[q], i[q], j[q]);
    }
    const int r = 32 / g.oW;
    dj = 32 - r * g.oW;
    db = r / g.oH;
    di = r - db * g.oH;
  }
  __device__ __forceinline__ void issue(const Params& p, const __amdgpu_buffer_rsrc_t (&rs)[NP], lds_byte* tile, bool live) {
    const Geometry& g = p.g;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte* dst = tile + wave * NLOAD * 1024;
    int y[NPIX], x[NPIX], base[NPIX];
#pragma unroll
    for (int q = 0; q < NPIX; ++q) {
      y[q] = (live && pix[q] < p.Kd) ? g.st * i[q] : (1 << 21);
      x[q] = g.st * j[q];
      base[q] = (int)((((unsigned)(b[q] * g.sH + g.st * i[q])) * g.sW + x[q]) * g.C) * 2;
    }
#pragma unroll
    for (int l = 0; l < NLOAD; ++l) {
      const int q = l % NPIX;
      const bool ok = (unsigned)(y[q] + du[l]) < (unsigned)g.sH && (unsigned)(x[q] + dv[l]) < (unsigned)g.sW;
      const unsigned at = ok ? (unsigned)(base[q] + coff[l]) : kOob;
#pragma unroll
      for (int pl = 0; pl < NP; ++pl)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[pl], (__attribute__((address_space(3))) void*)(dst + pl * BYTES + l * 1024),
                                                 16, at, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < NPIX; ++q) {
      pix[q] += 32;
      j[q] += dj;
      const int cj = j[q] >= g.oW ? 1 : 0;
      j[q] -= cj ? g.oW : 0;
      i[q] += di + cj;
      const int ci = i[q] >= g.oH ? 1 : 0;             // di < oH, so once is enough
      i[q] -= ci ? g.oH : 0;
      b[q] += db + ci;
    }
  }
};

// Reads of one wavefront's fragments: T fragments of 32 rows x 16 k, of every plane.
template <int T, int NP, bool KMAJOR, int BYTES>
struct Reader {
  static constexpr int NREAD = NP * T * (KMAJOR ? 1 : 2);
  unsigned rd[2][KMAJOR ? 1 : 2];
  __device__ __forceinline__ void init(int wrow0, int tid) {
    const int lane = tid & 63, l32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      if constexpr (KMAJOR) {
        const int r = wrow0 + l32;
        rd[kc][0] = (unsigned)(r * 64 + (((kc * 2 + h) ^ ((r >> 2) & 3)) * 16));
      } else {
        const int il = lane & 15, gq = lane >> 4;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int kr = kc * 16 + (gq >> 1) * 8 + kk * 4 + (il >> 2);
          const int col = wrow0 + (gq & 1) * 16 + 4 * (il & 3);
          rd[kc][kk] = (unsigned)((col >> 5) * 2048 + kr * 64 + ((((col & 31) >> 3) ^ ((kr >> 2) & 3)) << 4) + (col & 7) * 2);
        }
      }
    }
  }
  __device__ __forceinline__ void read(const lds_byte* tile, int kc, u32x4 (&f)[NP][T]) const {
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if constexpr (KMAJOR) {
          f[q][t] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(tile + q * BYTES + rd[kc][0] + t * 2048);
        } else {
#if defined(__HIP_DEVICE_COMPILE__)
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4*)(tile + q * BYTES + rd[kc][0] + t * 2048));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) s16x4*)(tile + q * BYTES + rd[kc][1] + t * 2048));
          const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
          f[q][t][0] = l2[0]; f[q][t][1] = l2[1]; f[q][t][2] = h2[0]; f[q][t][3] = h2[1];
#endif
        }
      }
  }
};

template <int MASK, int N, int M, int I>
struct Interleave {
  static __device__ __forceinline__ void run() {
    constexpr int ops = N * (I + 1) / M - N * I / M;
    if constexpr (ops > 0) __builtin_amdgcn_sched_group_barrier(MASK, ops, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (I + 1 < M) Interleave<MASK, N, M, I + 1>::run();
  }
};

// Writes a workgroup's results, rows tm0.., columns tn0..: four wavefronts, WM of them below each other, each with TM x TN
// blocks of 32 x 32, as the launch asks.  A wavefront passes 32-row strips through its private piece of LDS (strips: a pair of
// pieces each) and writes rows, consecutive lanes on consecutive 16 bytes (bias, mask and addend are read the same way).
// The column sums a normalisation wants are taken on the way, from results that would be read again for them:
// a lane keeps its four columns, the lanes of a column and then the wavefronts are added in a fixed order, one chunk of rows a
// workgroup.  Patches of 64 channels with one plane, 4 replicas of 128 images of 32 x 32: forward 63 us and 22 for the kernel that read
// Z again, 66 together; input gradient with bits 84 and 53 for dY and Z, 116 together.
// PLAIN: nothing of that, as for weight gradients and pieces of a cut contraction; what the others need, left in, cost a launch
// of those 0.7 to 1.9 us.
template <int TM, int TN, int WM, bool PLAIN>
__device__ __forceinline__ void store_tile(const Params& p, const f32x16 (&acc)[TM][TN], float* strips0, float* strips1, int tm0,
                                           int tn0, int bat, int piece, int t_in, int chunk, int chunks) {
  constexpr int WN = 4 / WM;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, h = lane >> 5;
  const int m0 = tm0 + wave / WN * (TM * 32), n0 = tn0 + wave % WN * (TN * 32);
  const auto strips = [&](int w) { return (w >> 1 ? strips1 : strips0) + (w & 1) * (32 * (TN * 32 + 4)); };
  float* stage = strips(wave);
  const bool split_mode = p.ksplit > 1;
  float* C = split_mode ? p.partial + (long long)piece * p.stridePartial + (long long)bat * p.M * p.ldP
                        : p.C + (long long)bat * p.strideC;
  const int ldC = split_mode ? p.ldP : p.ldC;
  const bool has_bias = !PLAIN && !split_mode && (p.epilogue == EPI_BIAS || p.epilogue == EPI_BIAS_RELU);
  const bool relu = !PLAIN && !split_mode && p.epilogue == EPI_BIAS_RELU;
  const bool masked = !PLAIN && !split_mode && p.epilogue == EPI_MASK;
  const float* mask = masked && p.keep == nullptr ? p.mask + (long long)bat * p.strideMask : nullptr;
  const unsigned char* keep = masked && p.keep != nullptr ? p.keep + (long long)bat * p.strideMask / 4 : nullptr;
  // (of a stride-2 input gradient, the class of even rows and columns)
  const bool adds = !PLAIN && !split_mode && p.add != nullptr && p.out_i == 0 && p.out_j == 0;
  const float* add = adds ? p.add + (long long)bat * p.strideAdd : nullptr;
  constexpr int PITCH = TN * 32 + 4;
  constexpr int LANES_PER_ROW = TN * 8;
  constexpr int ROWS_PER_PASS = 64 / LANES_PER_ROW;
  constexpr int PASSES = (32 + ROWS_PER_PASS - 1) / ROWS_PER_PASS;
  constexpr int GRP = PASSES < 4 ? PASSES : 4;
  const int c4 = (lane % LANES_PER_ROW) * 4;
  const int rsub = lane / LANES_PER_ROW;
  const int n = n0 + c4;
  float ssq = 0.f;
  const auto row_of = [&](int pass, int i) {        // the result's row, < 0 for none; N is a multiple of 4
    const int rr = pass * ROWS_PER_PASS + rsub, m = m0 + i * 32 + rr;
    return pass < PASSES && rr < 32 && rsub < ROWS_PER_PASS && m < p.M && n < p.N ? m : -1;
  };
  const auto placed = [&](int m) {                  // where a stride-2 input gradient's class writes it
    if (PLAIN || p.out_step <= 1) return m;
    int b, oi, oj;
    decode(m, p.g, b, oi, oj);
    return ((b * p.g.oH + oi) * 2 + p.out_i) * (2 * p.g.oW) + 2 * oj + p.out_j;
  };
  f32x4 bv = {0.f, 0.f, 0.f, 0.f};
  if (has_bias && n < p.N) bv = *reinterpret_cast<const f32x4*>(p.bias + (long long)bat * p.strideBias + n);
  f32x4 mu = {0.f, 0.f, 0.f, 0.f}, inv = mu, s1 = mu, s2 = mu;      // of the sums; mu of statistics: their shift
  const bool backward_sums = !PLAIN && p.sums == 2;
  if (backward_sums && n < p.N) {
    mu = *reinterpret_cast<const f32x4*>(p.sum_stats + (long long)bat * 2 * p.N + n);
    inv = *reinterpret_cast<const f32x4*>(p.sum_stats + ((long long)bat * 2 + 1) * p.N + n);
  }
  const float* sz = backward_sums ? p.sum_z + (long long)bat * p.strideC : nullptr;
  if (p.sums == 1 && adds && m0 < p.M && n < p.N) mu = *reinterpret_cast<const f32x4*>(add + (long long)m0 * p.ldAdd + n);
  // Waited for here: a wait in front of the sum of every pass would also wait for the stores of the pass
  // before (16 channels at 32 x 32 with three planes, 4 replicas of 128: 40.4 us a launch so, 37.9 us here;
  // patches of 64 channels with one plane 12 % of the launch).
  __builtin_amdgcn_s_waitcnt(waitcnt(0, 15));
  // What the results meet in memory (addend, mask, Z) is requested for GRP passes at a time, a group ahead of the stores: a load
  // after a group's stores is waited for together with them (the launch of 116 us above 122 without, with three planes 222 and 230).
  // Results that meet nothing are written without those
  // registers and branches (152 channels from 27 with one plane, 4 replicas of 64 at 32 x 32, where the
  // stores are the launch: 55 us with them, 42 without).
  // (A mask comes as bits where the layer below is normalised: read as floats it was as long a stream as the results, patches
  // of 64 channels with one plane, 4 replicas of 128 images of 32 x 32, 104 us a launch, 84 with bits, 63 without a mask.  Z is
  // met only beside bits, so it shares the mask's registers.)
  constexpr int GROUPS = (PASSES + GRP - 1) / GRP;      // of a strip
  const auto write = [&](auto meets, auto sums) {
    constexpr bool MEETS = decltype(meets)::value, SUMS = decltype(sums)::value;
    f32x4 other[MEETS ? 2 : 1][GRP], ad[MEETS ? 2 : 1][GRP];
    unsigned bits[MEETS ? 2 : 1][GRP];
    int row[2][GRP];
    const auto request = [&](int g) {
#pragma unroll
      for (int u = 0; u < GRP; ++u) {
        int& r = row[g & 1][u];
        r = row_of(g % GROUPS * GRP + u, g / GROUPS);
        if (r < 0) continue;
        if constexpr (MEETS) {
          if (adds) ad[g & 1][u] = *reinterpret_cast<const f32x4*>(add + (long long)r * p.ldAdd + n);
          r = placed(r);
          if (keep != nullptr) bits[g & 1][u] = keep[((long long)r * p.ldMask + n) >> 2];
          else if (masked) other[g & 1][u] = *reinterpret_cast<const f32x4*>(mask + (long long)r * p.ldMask + n);
          if (SUMS && backward_sums) other[g & 1][u] = *reinterpret_cast<const f32x4*>(sz + (long long)r * ldC + n);
        } else {
          r = placed(r);
        }
      }
    };
    if constexpr (MEETS) request(0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 v;
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = acc[i][j][q * 4 + r];
          *reinterpret_cast<f32x4*>(stage + l32 * PITCH + j * 32 + q * 8 + h * 4) = v;
        }
      // statistics are sums around the wavefront's first row, a value of the data's own size
      if (SUMS && !backward_sums && i == 0) mu += *reinterpret_cast<const f32x4*>(stage + c4) + bv;
#pragma unroll
      for (int gs = 0; gs < GROUPS; ++gs) {
        const int g = i * GROUPS + gs, at = MEETS ? g & 1 : 0;
        if constexpr (!MEETS) request(g);
        else if (g + 1 < TM * GROUPS) request(g + 1);
#pragma unroll
        for (int u = 0; u < GRP; ++u) {
          const int r = row[g & 1][u];
          if (r < 0) continue;
          f32x4 v = *reinterpret_cast<const f32x4*>(stage + ((gs * GRP + u) * ROWS_PER_PASS + rsub) * PITCH + c4);
          v += bv;
          if (MEETS && adds) v += ad[at][u];
          if (relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
          }
          if (MEETS && keep != nullptr) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (!(bits[at][u] >> e & 1)) v[e] = 0.f;
          } else if (MEETS && masked) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (!(other[at][u][e] > 0.f)) v[e] = 0.f;
          }
          *reinterpret_cast<f32x4*>(C + (long long)r * ldC + n) = v;
          if (SUMS && MEETS && backward_sums) {
            s1 += v * ((other[at][u] - mu) * inv);
            s2 += v;
          } else if (SUMS) {
            const f32x4 dlt = v - mu;
            s1 += dlt;
            s2 += dlt * dlt;
          } else {
            ssq += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
          }
        }
      }
    }
  };
  const bool meets = adds || masked || backward_sums;
  if constexpr (PLAIN) {
    write(std::false_type{}, std::false_type{});
  } else if (p.sums != 0) {
    if (meets) write(std::true_type{}, std::true_type{});
    else write(std::false_type{}, std::true_type{});
  } else {
    if (meets) write(std::true_type{}, std::false_type{});
    else write(std::false_type{}, std::false_type{});
  }
  if (!PLAIN && p.sums != 0) {
    const auto rows_of = [&](int wm) {
      const int left = p.M - (tm0 + wm * (TM * 32));
      return left < 0 ? 0 : left < TM * 32 ? left : TM * 32;
    };
#pragma unroll
    for (int off = LANES_PER_ROW; off < 64; off <<= 1)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s1[r] += __shfl_xor(s1[r], off, 64);
        s2[r] += __shfl_xor(s2[r], off, 64);
      }
    if (!backward_sums) {
      const int rows = rows_of(wave / WN);
      const float inv_n = rows > 0 ? 1.f / (float)rows : 0.f;
      const f32x4 m2 = s2 - s1 * s1 * inv_n;
      s1 = mu + s1 * inv_n;
#pragma unroll
      for (int r = 0; r < 4; ++r) s2[r] = m2[r] > 0.f ? m2[r] : 0.f;
    }
    if (rsub == 0) {
      *reinterpret_cast<f32x4*>(stage + c4) = s1;
      *reinterpret_cast<f32x4*>(stage + TN * 32 + c4) = s2;
    }
    __syncthreads();
    const int c = tid % (TN * 32), wn = tid / (TN * 32);
    if (wn < WN && tn0 + tid < p.N) {
      float a = 0.f, b = 0.f, rows = 0.f;
#pragma unroll
      for (int wm = 0; wm < WM; ++wm) {
        const float* from = strips(wm * WN + wn) + c;
        const float nw = backward_sums ? 1.f : (float)rows_of(wm);
        a += nw * from[0];
        rows += nw;
        if (backward_sums) b += from[TN * 32];
      }
      const long long N = p.N;
      if (backward_sums) {
        float* dst = p.sum_part + ((long long)bat * chunks + chunk) * 2 * N + tn0 + tid;
        dst[0] = a;
        dst[N] = b;
      } else {
        a /= rows;
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) {
          const float* from = strips(wm * WN + wn) + c;
          const float dlt = from[0] - a;
          b += from[TN * 32] + (float)rows_of(wm) * dlt * dlt;
        }
        float* dst = p.sum_part + ((long long)bat * chunks + chunk) * N + tn0 + tid;
        dst[0] = a;
        dst[(long long)p.batch * chunks * N] = b;
      }
    }
  }
  if (p.sumsq != nullptr && !split_mode) {
    __shared__ double part[4];
    double tot = (double)ssq;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    if (lane == 0) part[wave] = tot;
    __syncthreads();
    if (tid == 0) p.sumsq[(long long)bat * p.strideSumsq + t_in] = (part[0] + part[1]) + (part[2] + part[3]);
  }
}

enum Kind { kForward = 0, kForwardAnyC = 1, kWeightGrad = 2 };

template <int NP, int KIND, int BM> struct PickA { typedef ImgK<BM, NP, KIND == kForward> type; };
template <int NP, int BM> struct PickA<NP, kWeightGrad, BM> { typedef MatM<BM, NP> type; };
template <int NP, int KIND, int BN> struct PickB { typedef MatK<BN, NP, KIND == kForwardAnyC> type; };
template <int NP, int BN> struct PickB<NP, kWeightGrad, BN> { typedef ImgM<BN, NP> type; };

template <int NP, int KIND, int BM, int BN, int WM, int NSTAGE, bool PLAIN>
__device__ __forceinline__ void conv_gemm_workgroup(Params& p) {
  static_assert(NSTAGE >= 2 && NSTAGE <= 4, "ring of 2 to 4 stages");
  typedef typename PickA<NP, KIND, BM>::type OpA;
  typedef typename PickB<NP, KIND, BN>::type OpB;
  constexpr int WN = 4 / WM;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  static_assert(TM >= 1 && TN >= 1, "a wavefront takes whole 32 x 32 tiles");
  constexpr int A_BYTES = NP * OpA::BYTES, STAGE = A_BYTES + NP * OpB::BYTES;
  constexpr int EPI_PITCH = TN * 32 + 4;
  constexpr int EPI_BYTES = 2 * 32 * EPI_PITCH * 4;            // strips of two wavefronts
  constexpr int ST0 = STAGE > EPI_BYTES ? STAGE : EPI_BYTES;
  __shared__ __attribute__((aligned(1024))) unsigned char st0[ST0];
  __shared__ __attribute__((aligned(1024))) unsigned char st1[ST0];
  __shared__ __attribute__((aligned(1024))) unsigned char st2[NSTAGE > 2 ? STAGE : 1024];
  __shared__ __attribute__((aligned(1024))) unsigned char st3[NSTAGE > 3 ? STAGE : 1024];

  // contiguous tile range per XCD; inside a replica bands of 8 tile rows, row fastest (the
  // workgroups running together share operand panels in one XCD's L2).  The pieces of a split
  // contraction are the outermost index: neighbours then read the same pixels.
  const int logical = (blockIdx.x % 8) * p.chunks + blockIdx.x / 8;
  if (logical >= p.total) return;
  const int per_rep = p.tilesM * p.tilesN;
  int index = logical;
  if constexpr (KIND != kWeightGrad) {
    if (p.out_step == 2) {
      // four classes of pixels (see ConvGemmDesc), side by side: neighbours read the same pixels,
      // and every part of the grid has the same mix of one to four taps
      const int cls = 3 - (logical & 3), odd_i = cls >> 1, odd_j = cls & 1;
      index = logical >> 2;
      const int before = cls == 0 ? 0 : 2 * cls - 1;   // taps of the classes in front: 0, 1, 3, 5
      p.g.nu = 1 + odd_i; p.g.nv = 1 + odd_j; p.g.du0 = p.g.dv0 = 0;
      p.Kd = p.g.nu * p.g.nv * p.g.C;
      p.B += before * p.g.C; p.bytesB -= (unsigned)(before * p.g.C * 2);
      p.out_i = odd_i; p.out_j = odd_j;
    }
  }
  int rest = index / per_rep;
  const int t_in = index - rest * per_rep;
  const int piece = rest % p.ksplit;
  const int bat = rest / p.ksplit;
  constexpr int GROUP_M = 8;
  const int band = t_in / (GROUP_M * p.tilesN);
  const int first_m = band * GROUP_M;
  const int gsize = p.tilesM - first_m < GROUP_M ? p.tilesM - first_m : GROUP_M;
  const int tin = t_in - band * GROUP_M * p.tilesN;
  const int m0 = (first_m + tin % gsize) * BM, n0 = (tin / gsize) * BN;

  const unsigned short* Ab = p.A + (long long)bat * p.strideA;
  const unsigned short* Bb = p.B + (long long)bat * p.strideB;
  __amdgpu_buffer_rsrc_t ra[NP], rb[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    ra[q] = make_rsrc(Ab + q * p.planeA, p.bytesA);
    rb[q] = make_rsrc(Bb + q * p.planeB, p.bytesB);
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);

  const int all = (p.Kd + 31) / 32;
  const int first = piece * p.steps_per_piece;
  const int ksteps = all - first < p.steps_per_piece ? all - first : p.steps_per_piece;

  OpA oa; OpB ob;
  oa.init(p, m0, first, tid);
  ob.init(p, n0, first, tid);
  Reader<TM, NP, OpA::KMAJOR, OpA::BYTES> qa;
  Reader<TN, NP, OpB::KMAJOR, OpB::BYTES> qb;
  qa.init(wm0, tid);
  qb.init(wn0, tid);
  constexpr int NL = NP * (OpA::NLOAD + OpB::NLOAD);
  constexpr int ND = decltype(qa)::NREAD + decltype(qb)::NREAD;
  constexpr int NPROD = NP == 1 ? 1 : 6;
  constexpr int NM = NPROD * TM * TN;

  // NP = 3: the product of the leading pieces has accumulators of its own.  The other five are
  // 2^-8 of it and less, so adding them up separately costs nothing in their own sum and takes
  // five of six roundings off the large one (relative error of 576-term sums: 2.5e-7 with one set
  // of accumulators, fp32 FMA chain 4e-7).  They start from zero, and the bias is added last: a sum
  // that holds the bias already rounds each of its steps at the bias's size.
  f32x16 acc[TM][TN], low[NP > 1 ? TM : 1][NP > 1 ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[i][j][e] = 0.f;
        if constexpr (NP > 1) low[i][j][e] = 0.f;
      }

  u32x4 fa[2][NP][TM], fb[2][NP][TN];
  auto mfma_chunk = [&](int buf) {
    // cross products of the planes, smallest first
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int q = 6 - NPROD; q < 6; ++q)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          f32x16& to = (NP > 1 && q < 5) ? low[NP > 1 ? i : 0][NP > 1 ? j : 0] : acc[i][j];
          to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[buf][pb[q]][j]),
                                                       __builtin_bit_cast(bf16x8, fa[buf][pa[q]][i]), to, 0, 0, 0);
        }
  };
  lds_byte* s0 = (lds_byte*)st0;
  lds_byte* s1 = (lds_byte*)st1;
  lds_byte* s2 = (lds_byte*)st2;
  lds_byte* s3 = (lds_byte*)st3;

  // k-steps past the last one are requested out of range (zeros), which keeps the number of
  // loads in flight, and so the wait counts, the same in every step
  oa.issue(p, ra, s0, 0 < ksteps); ob.issue(p, rb, s0 + A_BYTES, 0 < ksteps);
  oa.issue(p, ra, s1, 1 < ksteps); ob.issue(p, rb, s1 + A_BYTES, 1 < ksteps);
  if constexpr (NSTAGE > 2) { oa.issue(p, ra, s2, 2 < ksteps); ob.issue(p, rb, s2 + A_BYTES, 2 < ksteps); }
  if constexpr (NSTAGE > 3) { oa.issue(p, ra, s3, 3 < ksteps); ob.issue(p, rb, s3 + A_BYTES, 3 < ksteps); }
  __builtin_amdgcn_s_waitcnt(waitcnt((NSTAGE - 1) * NL, 15));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  qa.read(s0, 0, fa[0]);
  qb.read(s0 + A_BYTES, 0, fb[0]);

  // One k-step on stage CUR; NEXT holds the following one; the step NSTAGE ahead is requested
  // into CUR as soon as every wavefront has taken its last fragment out of it.
#define LSAM_CONV_STEP(CUR, NEXT)                                                         \
  {                                                                                       \
    qa.read(CUR, 1, fa[1]);                                                               \
    qb.read(CUR + A_BYTES, 1, fb[1]);                                                     \
    mfma_chunk(0);                                                                        \
    Interleave<0x100, ND, NM, 0>::run();                                                  \
    __builtin_amdgcn_s_waitcnt(waitcnt((NSTAGE - 2) * NL, 0));                            \
    asm volatile("" ::: "memory");                                                        \
    __builtin_amdgcn_s_barrier();                                                         \
    asm volatile("" ::: "memory");                                                        \
    oa.issue(p, ra, CUR, ks + NSTAGE < ksteps);                                           \
    ob.issue(p, rb, CUR + A_BYTES, ks + NSTAGE < ksteps);                                 \
    qa.read(NEXT, 0, fa[0]);                                                              \
    qb.read(NEXT + A_BYTES, 0, fb[0]);                                                    \
    mfma_chunk(1);                                                                        \
    Interleave<0x120, ND + NL, NM, 0>::run();                                             \
    if (++ks >= ksteps) break;                                                            \
  }
  for (int ks = 0;;) {
    LSAM_CONV_STEP(s0, s1)
    if constexpr (NSTAGE == 2) {
      LSAM_CONV_STEP(s1, s0)
    } else if constexpr (NSTAGE == 3) {
      LSAM_CONV_STEP(s1, s2)
      LSAM_CONV_STEP(s2, s0)
    } else {
      LSAM_CONV_STEP(s1, s2)
      LSAM_CONV_STEP(s2, s3)
      LSAM_CONV_STEP(s3, s0)
    }
  }
#undef LSAM_CONV_STEP
  __builtin_amdgcn_s_waitcnt(waitcnt(0, 0));           // nothing may still be writing LDS
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  if constexpr (NP > 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        join_sums(acc[i][j], low[i][j]);
  }

  const bool classes = KIND != kWeightGrad && p.out_step == 2;
  store_tile<TM, TN, WM, PLAIN>(p, acc, reinterpret_cast<float*>(st0), reinterpret_cast<float*>(st1), m0, n0, bat, piece, t_in,
                                classes ? m0 / BM * 4 + p.out_i * 2 + p.out_j : m0 / BM, classes ? 4 * p.tilesM : p.tilesM);
}
template <int NP, int KIND, int BM, int BN, int WM, int NSTAGE, int OCC>
__global__ __launch_bounds__(kThreads, OCC) void conv_gemm_kernel(Params p) {
  conv_gemm_workgroup<NP, KIND, BM, BN, WM, NSTAGE, KIND == kWeightGrad>(p);
}
// (of a cut contraction)
template <int NP, int KIND, int BM, int BN, int WM, int NSTAGE, int OCC, bool PIECE>
__global__ __launch_bounds__(kThreads, OCC) void conv_gemm_kernel(Params p) {
  conv_gemm_workgroup<NP, KIND, BM, BN, WM, NSTAGE, PIECE>(p);
}

// A uniform value the compiler may not compute with ahead of time: without it the addresses of all
// unrolled stages are formed in front of the loop and kept, more scalar registers than there are.
__device__ __forceinline__ int opaque(int v) {
  int t = __builtin_amdgcn_readfirstlane(v);
  asm volatile("" : "+s"(t));
  return __builtin_amdgcn_readfirstlane(t);
}

// Load x (plane x / NLA, round x % NLA) of the patch of the channel block that starts `at` bytes into
// a pixel; bytes: size of a plane of the image, 0 if the block does not exist (everything is then
// out of range, which yields zeros).  Surplus loads of the last round go to `spill`.
template <int NCHUNK, int NLA>
__device__ __forceinline__ void issue_patch(const unsigned short* base, long long plane, unsigned bytes, lds_byte* buf,
                                            lds_byte* spill, const unsigned (&off)[NLA], int wave, int x, int at) {
  const int q = x / NLA, l = x % NLA, chunk = wave + 4 * l;
  lds_byte* dst = chunk < NCHUNK ? buf + (q * NCHUNK + chunk) * 1024 : spill;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base + q * plane, bytes), (__attribute__((address_space(3))) void*)dst, 16,
                                           off[l], at, 0, 0);
}
// Filters of one stage, one plane: the three taps that start at byte `at` of a filter, C2 bytes each;
// [tap][64 rows][64 bytes].
__device__ __forceinline__ void issue_filters(const unsigned short* base, unsigned bytes, lds_byte* buf, unsigned off, int wave,
                                              int at, int C2) {
#pragma unroll
  for (int x = 0; x < 3; ++x)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base, bytes),
                                             (__attribute__((address_space(3))) void*)(buf + x * 4096 + wave * 1024), 16, off,
                                             at + x * C2, 0, 0);
}
// The same for stages of 16 channels of one tap, three planes: rows (wave % 2) * 32.. of plane
// wave / 2, and of plane 2 for the first two wavefronts; [plane][64 rows][32 bytes].
__device__ __forceinline__ void issue_split_filters(const unsigned short* base, long long plane, unsigned bytes, lds_byte* buf,
                                                    lds_byte* spill, unsigned off, int wave, int at) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base + (wave >> 1) * plane, bytes),
                                           (__attribute__((address_space(3))) void*)(buf + wave * 1024), 16, off, at, 0, 0);
  lds_byte* dst = wave < 2 ? buf + 4096 + wave * 1024 : spill;
  __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base + 2 * plane, wave < 2 ? bytes : 0u),
                                           (__attribute__((address_space(3))) void*)dst, 16, off, at, 0, 0);
}

// ---- forward product and input gradient of 3x3 layers with stride 1, image patches in LDS -----------
// The ring above fetches every pixel nine times, once per tap, and at these tile sizes waits for
// the path into LDS.  Here a workgroup takes 256 consecutive pixels x 64 columns and keeps, per 32
// channels, the patch of the zero-rimmed image those pixels touch: NCHUNK x 16 slots of 64 bytes
// (a slot is a pixel of the rimmed image; slots outside the image read as zeros).  A tap is then
// a constant shift of the slot, and the nine taps read the same patch.  The filters of TPS taps
// (12 KiB) come through a ring of two stages; the patch of the next 32 channels is requested
// during the first stages of the current one into the other of two patch buffers.
//   Bytes into LDS per 32 channels: 22 + 37 KiB a plane (32 x 32 image) against 180 for the ring.
// Four wavefronts below each other, 64 x 64 results each: 64 bytes of LDS reads per clock and
// compute unit at the full matrix rate (64 x 32 per wavefront would need 96 of the 128).
template <int NCHUNK, bool PLAIN>
__device__ __forceinline__ void patch_workgroup(Params& p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NP = 1, BM = 256, BN = 64, TM = 2, TN = 2;
  constexpr int TPS = 3;                               // taps per stage of filters
  constexpr int S = 9 / TPS;                           // stages per 32 channels
  constexpr int NLA = (NCHUNK + 3) / 4;                // patch loads per wavefront and plane
  constexpr int NA = NLA * NP;                         // ... in all, AG per stage from the first one on
  constexpr int AG = (NA + S - 2) / (S - 1);
  static_assert((NA + AG - 1) / AG <= S - 1, "the patch is requested before the last stage");
  constexpr int A_BYTES = NP * NCHUNK * 1024, B_BYTES = 3 * 4096;
  constexpr int EPI_PITCH = BN + 4;
  static_assert(A_BYTES >= 2 * 32 * EPI_PITCH * 4, "room for the epilogue's strips");
  __shared__ __attribute__((aligned(1024))) unsigned char pa0[A_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char pa1[A_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char pb0[B_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char pb1[B_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char spill[1024];   // surplus loads of the last round end here

  const int logical = (blockIdx.x % 8) * p.chunks + blockIdx.x / 8;
  if (logical >= p.total) return;
  // (quotients come from the vector unit: back to scalars, the addresses below depend on them)
  const int per_rep = p.tilesM * p.tilesN;
  const int rest = __builtin_amdgcn_readfirstlane(logical / per_rep);
  const int t_in = logical - rest * per_rep;
  const int bat = __builtin_amdgcn_readfirstlane(rest / p.ksplit);
  const int piece = rest - bat * p.ksplit;
  const int t_row = __builtin_amdgcn_readfirstlane(t_in / p.tilesN);
  // column tiles of one row tile are neighbours: they read the same patch
  const int m0 = t_row * BM, n0 = (t_in - t_row * p.tilesN) * BN;

  const unsigned short* Ab = p.A + (long long)bat * p.strideA;
  const unsigned short* Bb = p.B + (long long)bat * p.strideB;
  const Geometry& g = p.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int wm0 = wave * 64;
  const int W2 = g.oW + 2, H2 = g.oH + 2;

  const int blocks = g.C / 32;                          // 32-channel blocks of the contraction
  const int first = piece * p.steps_per_piece;
  const int nblk = blocks - first < p.steps_per_piece ? blocks - first : p.steps_per_piece;

  // rimmed row of the tile's first slot
  int pr0;
  {
    int b, i, j;
    decode(m0, g, b, i, j);
    pr0 = __builtin_amdgcn_readfirstlane(b * H2 + i);
  }
  // global offset of this lane's 16 bytes of slot (wave + 4 l) * 16 + lane / 4
  unsigned aoff[NLA];
  const int images = p.M / (g.oH * g.oW);
#pragma unroll
  for (int l = 0; l < NLA; ++l) {
    const int slot = (wave + 4 * l) * 16 + (lane >> 2);
    const int u = (lane & 3) ^ ((slot >> 2) & 3);
    const int r = slot / W2, col = slot - r * W2 - 1;
    const int pr = pr0 + r, b = pr / H2, i = pr - b * H2 - 1;
    const bool ok = (unsigned)i < (unsigned)g.oH && (unsigned)col < (unsigned)g.oW && b < images && wave + 4 * l < NCHUNK;
    aoff[l] = ok ? ((unsigned)((b * g.oH + i) * g.oW + col) * g.C + u * 8) * 2u : kOob;
  }
  unsigned boff;
  {
    const int row = wave * 16 + (lane >> 2);
    const int u = (lane & 3) ^ ((row >> 2) & 3);
    boff = n0 + row < p.N ? ((unsigned)(n0 + row) * p.ldB + u * 8) * 2u : kOob;
  }
  lds_byte* a0 = (lds_byte*)pa0;
  lds_byte* a1 = (lds_byte*)pa1;
  lds_byte* b0 = (lds_byte*)pb0;
  lds_byte* b1 = (lds_byte*)pb1;
  lds_byte* sp = (lds_byte*)spill;
  // slot of this lane's pixel in each of the wavefront's two 32-row strips
  int slot[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    int m = m0 + wm0 + i * 32 + l32;
    if (m >= p.M) m = p.M - 1;
    int b, y, x;
    decode(m, g, b, y, x);
    slot[i] = (b * H2 + y + 1 - pr0) * W2 + x + 1;
  }
  const unsigned brd = (unsigned)(l32 * 64 + ((h ^ ((l32 >> 2) & 3)) * 16));

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  u32x4 fa[2][NP][TM], fb[2][NP][TN];
  unsigned ard[TM];                                     // LDS offset of the current tap's first half
  // fragments of sub-step u (tap u / 2 of the stage, half u % 2) of stage s
  auto read_frags = [&](const lds_byte* abuf, const lds_byte* bbuf, int s, int u, int buf) {
    const int tap = s * TPS + u / 2;
    if (u % 2 == 0) {
      const int shift = (tap / 3 - 1) * W2 + tap % 3 - 1;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const unsigned t = (unsigned)(slot[i] + shift);
        ard[i] = (t << 6) | (((t << 2) & 48u) ^ (unsigned)(h << 4));
      }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[buf][q][i] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(
            abuf + q * NCHUNK * 1024 + (u % 2 ? ard[i] ^ 32u : ard[i]));
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[buf][q][j] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(
            bbuf + (NP == 1 ? u / 2 : q) * 4096 + j * 2048 + (u % 2 ? brd ^ 32u : brd));
    }
  };
  auto mfma = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[buf][0][j]),
                                                            __builtin_bit_cast(bf16x8, fa[buf][0][i]), acc[i][j], 0, 0, 0);
  };
  constexpr int ND = NP * (TM + TN), NM = TM * TN;

#pragma unroll
  for (int x = 0; x < NA; ++x) issue_patch<NCHUNK>(Ab, 0, p.bytesA, a0, sp, aoff, wave, x, first * 64);
  issue_filters(Bb, p.bytesB, b0, boff, wave, first * 64, g.C * 2);
  issue_filters(Bb, p.bytesB, b1, boff, wave, TPS * g.C * 2 + first * 64, g.C * 2);
  __builtin_amdgcn_s_waitcnt(waitcnt(3, 15));           // the patch and stage 0
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_frags(a0, b0, 0, 0, 0);

  // One 32-channel block on patch CUR: S stages, their filters alternating between BX and BY.  A
  // stage's last sub-step follows the barrier after which its filter buffer is free: the stage
  // two further is requested into it, and (first stages) a share of the next block's patch into
  // NEXT, free since the previous block's last barrier.  Loads of the newest group that may
  // still be in flight at a stage's barrier: the patch share behind its filters.
#define LSAM_PATCH_STAGE(CUR, NEXT, BC, BN_, s)                                                                       \
  {                                                                                                                   \
    constexpr int U = 2 * TPS;                                                                                        \
    _Pragma("unroll") for (int u = 0; u + 1 < U; ++u) {                                                               \
      read_frags(CUR, BC, s, u + 1, (u + 1) & 1);                                                                     \
      mfma(u & 1);                                                                                                    \
      Interleave<0x100, ND, NM, 0>::run();                                                                            \
    }                                                                                                                 \
    constexpr int left = NA - ((s) - 1) * AG;                                                                         \
    constexpr int behind = (s) == 0 || (s) == S - 1 || left < 0 ? 0 : (left < AG ? left : AG);                        \
    __builtin_amdgcn_s_waitcnt(waitcnt(behind, 0));                                                                   \
    asm volatile("" ::: "memory");                                                                                    \
    __builtin_amdgcn_s_barrier();                                                                                     \
    asm volatile("" ::: "memory");                                                                                    \
    const int bn = (s) + 2 < S ? blk : blk + 1;                                                                       \
    issue_filters(Bb, bn < nblk ? p.bytesB : 0u, BC, boff, wave, ((s) + 2) % S * TPS * (g.C * 2) + (first + bn) * 64, g.C * 2); \
    _Pragma("unroll") for (int x = (s) * AG; x < (s) * AG + AG; ++x)                                                  \
      if (x < NA && (s) < S - 1)                                                                                      \
        issue_patch<NCHUNK>(Ab, 0, blk + 1 < nblk ? p.bytesA : 0u, NEXT, sp, aoff, wave, x, (first + blk + 1) * 64);  \
    read_frags((s) + 1 < S ? CUR : NEXT, BN_, ((s) + 1) % S, 0, 0);                                                   \
    mfma(1);                                                                                                          \
    constexpr int share = (s) == S - 1 || NA - (s) * AG < 0 ? 0 : (NA - (s) * AG < AG ? NA - (s) * AG : AG);          \
    Interleave<0x120, ND + 3 + share, NM, 0>::run();                                                                  \
  }
#define LSAM_PATCH_BLOCK(CUR, NEXT, BX, BY)                                                                           \
  {                                                                                                                   \
    LSAM_PATCH_STAGE(CUR, NEXT, BX, BY, 0)                                                                            \
    LSAM_PATCH_STAGE(CUR, NEXT, BY, BX, 1)                                                                            \
    LSAM_PATCH_STAGE(CUR, NEXT, BX, BY, 2)                                                                            \
  }
  for (int blk = 0;;) {
    LSAM_PATCH_BLOCK(a0, a1, b0, b1)
    if (++blk >= nblk) break;
    LSAM_PATCH_BLOCK(a1, a0, b1, b0)
    if (++blk >= nblk) break;
  }
#undef LSAM_PATCH_BLOCK
#undef LSAM_PATCH_STAGE
  __builtin_amdgcn_s_waitcnt(waitcnt(0, 0));            // nothing may still be writing LDS
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  store_tile<TM, TN, 4, PLAIN>(p, acc, reinterpret_cast<float*>(pa0), reinterpret_cast<float*>(pa1), m0, n0, bat, piece, t_in, t_row,
                               p.tilesM);
#endif
}
// Pieces of a cut contraction, and (WHOLE) whole ones.
template <int NCHUNK>
__global__ __launch_bounds__(kThreads, 2) void conv_patch_kernel(Params p) {
  patch_workgroup<NCHUNK, true>(p);
}
template <int NCHUNK, bool WHOLE>
__global__ __launch_bounds__(kThreads, 2) void conv_patch_kernel(Params p) {
  patch_workgroup<NCHUNK, !WHOLE>(p);
}

// The same with three planes.  A workgroup takes TM x 128 pixels and blocks of 16 channels (one
// matrix depth): two patches of NCHUNK x 32 slots of 32 bytes a plane and two stages of filters (one
// tap, 6 KiB) are 80 KiB, so two workgroups share a compute unit and one's first loads and
// write-out run under the other's products (one workgroup of 32-channel blocks, all 160 KiB of
// LDS: 276 against 222 us on 64 channels at 32 x 32).  A 16-byte unit of slot t lies at position
// u ^ (t / 8) % 2: 16 consecutive slots read without bank conflicts at any shift.  A strip of 32 pixels
// is not always that: where it runs over the end of an image row its slots jump by two, and the
// reads collide (measured: 15 to 19 % of the cycles the LDS is active are conflicts with 32-wide
// images, 39 % with 16-wide and 8-wide ones; one plane 19 to 23 % and 49 %).
// Per stage (a tap at one matrix depth) and wavefront: 6 TM TN products, 3 (TM + TN) fragment reads.
// TN = 1 serves layers of up to 32 columns (half of the filter rows it requests do not exist and
// cost no traffic): 16 channels at 32 x 32, 4 replicas of 128: 38 us,
// 56 by the ring (which fetches every pixel nine times).
// A last column of tiles with 32 columns or fewer left takes the same steps on half a tile: 160 columns are 2.5 tiles of
// work and not 3.  A kernel of its own: with both bodies in one the others were 0.3 % slower.  Steps of two layers, 4
// replicas of 64 images, whole / half tiles: 32 x 32, 80 channels 1749 / 1730 us, 96 1980 / 1921, 160 4208 / 4127; 20 x 20, 160
// 2327 / 2288.  Between one and two rounds of the 512 workgroups that fit the chip whole tiles stay: 160 channels at
// 16 x 16, 768 workgroups, 1203 / 1232.
template <int TM, int TN, int NCHUNK, bool PLAIN>
__device__ __forceinline__ void split_patch_tile(const Params& p, lds_byte* a0, lds_byte* a1, lds_byte* b0, lds_byte* b1,
                                                 lds_byte* sp, int m0, int n0, int bat, int piece, int t_in, int t_row) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NP = 3, BN = TN * 32, S = 9;
  constexpr int NLA = (NCHUNK + 3) / 4, NA = NLA * NP, AG = (NA + S - 2) / (S - 1);
  const unsigned short* Ab = p.A + (long long)bat * p.strideA;
  const unsigned short* Bb = p.B + (long long)bat * p.strideB;
  const Geometry& g = p.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int H2 = g.oH + 2;
  int W2 = g.oW + 2, C2 = g.C * 2;

  const int blocks = g.C / 16;
  const int first = piece * p.steps_per_piece;
  const int nblk = blocks - first < p.steps_per_piece ? blocks - first : p.steps_per_piece;

  int pr0;                                               // rimmed row of the tile's first slot
  {
    int b, i, j;
    decode(m0, g, b, i, j);
    pr0 = __builtin_amdgcn_readfirstlane(b * H2 + i);
  }
  unsigned aoff[NLA];
  const int images = p.M / (g.oH * g.oW);
#pragma unroll
  for (int l = 0; l < NLA; ++l) {
    const int slot = (wave + 4 * l) * 32 + (lane >> 1);
    const int u = (lane & 1) ^ ((slot >> 3) & 1);
    const int r = slot / W2, col = slot - r * W2 - 1;
    const int pr = pr0 + r, b = pr / H2, i = pr - b * H2 - 1;
    const bool ok = (unsigned)i < (unsigned)g.oH && (unsigned)col < (unsigned)g.oW && b < images && wave + 4 * l < NCHUNK;
    aoff[l] = ok ? ((unsigned)((b * g.oH + i) * g.oW + col) * g.C + u * 8) * 2u : kOob;
  }
  // a wavefront's two loads of a filter stage: rows (wave % 2) * 32.. of plane wave / 2, and, for the
  // first two wavefronts, of plane 2
  unsigned boff;
  {
    const int row = (wave & 1) * 32 + (lane >> 1);
    const int u = (lane & 1) ^ ((row >> 3) & 1);
    boff = row < BN && n0 + row < p.N ? ((unsigned)(n0 + row) * p.ldB + u * 8) * 2u : kOob;
  }
  int slot[TM];                                          // of this lane's pixel in each 32-row strip
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    int m = m0 + wave * (TM * 32) + i * 32 + l32;
    if (m >= p.M) m = p.M - 1;
    int b, y, x;
    decode(m, g, b, y, x);
    slot[i] = (b * H2 + y + 1 - pr0) * W2 + x + 1;
  }
  const unsigned brd = (unsigned)(l32 * 32 + ((h ^ ((l32 >> 3) & 1)) * 16));

  f32x16 acc[TM][TN], low[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.f;

  u32x4 fa[2][NP][TM], fb[2][NP][TN];
  auto read_frags = [&](const lds_byte* abuf, const lds_byte* bbuf, int tap, int buf) {
    const int shift = (tap / 3 - 1) * W2 + tap % 3 - 1;
    unsigned rd[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const unsigned t = (unsigned)(slot[i] + shift);
      rd[i] = (t << 5) | (((t << 1) & 16u) ^ (unsigned)(h << 4));
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[buf][q][i] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(abuf + q * NCHUNK * 1024 + rd[i]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[buf][q][j] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(bbuf + q * 2048 + j * 1024 + brd);
    }
  };
  auto mfma = [&](int buf) {
    constexpr int xa[6] = {2, 0, 1, 1, 0, 0}, xb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          f32x16& to = q < 5 ? low[i][j] : acc[i][j];
          to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[buf][xb[q]][j]),
                                                       __builtin_bit_cast(bf16x8, fa[buf][xa[q]][i]), to, 0, 0, 0);
        }
  };
  constexpr int ND = NP * (TM + TN), NM = 6 * TM * TN;

#pragma unroll
  for (int x = 0; x < NA; ++x) issue_patch<NCHUNK>(Ab, p.planeA, p.bytesA, a0, sp, aoff, wave, x, first * 32);
  issue_split_filters(Bb, p.planeB, p.bytesB, b0, sp, boff, wave, first * 32);
  issue_split_filters(Bb, p.planeB, p.bytesB, b1, sp, boff, wave, C2 + first * 32);
  __builtin_amdgcn_s_waitcnt(waitcnt(2, 15));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_frags(a0, b0, 0, 0);

  // Stage s of a 16-channel block on patch CUR, filters in BC, fragments in register set F.  After its
  // barrier every wavefront holds the stage's fragments, so the filters two stages on and a share
  // of the next block's patch are requested (BC and NEXT are free) and the next stage's
  // fragments read under the products.  At the barrier the newest patch share may be in flight.
#define LSAM_SPLIT_STAGE(CUR, NEXT, BC, BX, s, F)                                                                     \
  {                                                                                                                   \
    constexpr int before = (s) == 0 ? 0 : NA - ((s) - 1) * AG, share = NA - (s) * AG;                                 \
    constexpr int behind = before < 0 ? 0 : (before < AG ? before : AG);                                              \
    constexpr int now = share < 0 ? 0 : (share < AG ? share : AG);                                                    \
    __builtin_amdgcn_s_waitcnt(waitcnt(behind, 0));                                                                   \
    asm volatile("" ::: "memory");                                                                                    \
    __builtin_amdgcn_s_barrier();                                                                                     \
    asm volatile("" ::: "memory");                                                                                    \
    wave = opaque(wave); W2 = opaque(W2); C2 = opaque(C2);                                                            \
    const int bn = (s) + 2 < S ? blk : blk + 1;                                                                       \
    issue_split_filters(Bb, p.planeB, bn < nblk ? p.bytesB : 0u, BC, sp, boff, wave,                                  \
                        ((s) + 2) % S * C2 + (first + bn) * 32);                                                      \
    _Pragma("unroll") for (int x = (s) * AG; x < (s) * AG + now; ++x)                                                 \
        issue_patch<NCHUNK>(Ab, p.planeA, blk + 1 < nblk ? p.bytesA : 0u, NEXT, sp, aoff, wave, x, (first + blk + 1) * 32); \
    read_frags((s) + 1 < S ? CUR : NEXT, BX, ((s) + 1) % S, (F) ^ 1);                                                 \
    mfma(F);                                                                                                          \
    Interleave<0x120, ND + 2 + now, NM, 0>::run();                                                                    \
  }
#define LSAM_SPLIT_BLOCK(CUR, NEXT, BX, BY, F)                                                                        \
  {                                                                                                                   \
    LSAM_SPLIT_STAGE(CUR, NEXT, BX, BY, 0, F)                                                                         \
    LSAM_SPLIT_STAGE(CUR, NEXT, BY, BX, 1, (F) ^ 1)                                                                   \
    LSAM_SPLIT_STAGE(CUR, NEXT, BX, BY, 2, F)                                                                         \
    LSAM_SPLIT_STAGE(CUR, NEXT, BY, BX, 3, (F) ^ 1)                                                                   \
    LSAM_SPLIT_STAGE(CUR, NEXT, BX, BY, 4, F)                                                                         \
    LSAM_SPLIT_STAGE(CUR, NEXT, BY, BX, 5, (F) ^ 1)                                                                   \
    LSAM_SPLIT_STAGE(CUR, NEXT, BX, BY, 6, F)                                                                         \
    LSAM_SPLIT_STAGE(CUR, NEXT, BY, BX, 7, (F) ^ 1)                                                                   \
    LSAM_SPLIT_STAGE(CUR, NEXT, BX, BY, 8, F)                                                                         \
  }
  // the barrier of the last stage, whose products read on into NEXT, leaves what the stage before it
  // requested in flight: that must be none of the patch
  static_assert(AG * (S - 2) >= NA, "the patch is requested before the last stage but one");
  int blk = 0;
  while (blk + 1 < nblk) {
    LSAM_SPLIT_BLOCK(a0, a1, b0, b1, 0)
    ++blk;
    LSAM_SPLIT_BLOCK(a1, a0, b1, b0, 1)
    ++blk;
  }
  if (blk < nblk) LSAM_SPLIT_BLOCK(a0, a1, b0, b1, 0)
#undef LSAM_SPLIT_BLOCK
#undef LSAM_SPLIT_STAGE
  __builtin_amdgcn_s_waitcnt(waitcnt(0, 0));            // nothing may still be writing LDS
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      join_sums(acc[i][j], low[i][j]);
  store_tile<TM, TN, 4, PLAIN>(p, acc, (float*)a0, (float*)a1, m0, n0, bat, piece, t_in, t_row, p.tilesM);
#endif
}

template <int TM, int TN, int NCHUNK, bool NARROW_LAST, bool PLAIN>
__device__ __forceinline__ void split_patch_workgroup(const Params& p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NP = 3, BM = TM * 128, BN = TN * 32;
  constexpr int A_BYTES = NP * NCHUNK * 1024, B_BYTES = NP * 2048;
  constexpr int EPI_PITCH = BN + 4;
  static_assert(A_BYTES >= 2 * 32 * EPI_PITCH * 4, "room for the epilogue's strips");
  __shared__ __attribute__((aligned(1024))) unsigned char pa0[A_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char pa1[A_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char pb0[B_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char pb1[B_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char spill[1024];   // surplus loads end here

  const int logical = (blockIdx.x % 8) * p.chunks + blockIdx.x / 8;
  if (logical >= p.total) return;
  // (quotients come from the vector unit: back to scalars, the addresses below depend on them)
  const int per_rep = p.tilesM * p.tilesN;
  const int rest = __builtin_amdgcn_readfirstlane(logical / per_rep);
  const int t_in = logical - rest * per_rep;
  const int bat = __builtin_amdgcn_readfirstlane(rest / p.ksplit);
  const int piece = rest - bat * p.ksplit;
  const int t_row = __builtin_amdgcn_readfirstlane(t_in / p.tilesN);
  const int m0 = t_row * BM, n0 = (t_in - t_row * p.tilesN) * BN;   // neighbours read the same patch

  lds_byte* a0 = (lds_byte*)pa0;
  lds_byte* a1 = (lds_byte*)pa1;
  lds_byte* b0 = (lds_byte*)pb0;
  lds_byte* b1 = (lds_byte*)pb1;
  lds_byte* sp = (lds_byte*)spill;
  if (NARROW_LAST && p.N - n0 <= 32) split_patch_tile<TM, 1, NCHUNK, PLAIN>(p, a0, a1, b0, b1, sp, m0, n0, bat, piece, t_in, t_row);
  else split_patch_tile<TM, TN, NCHUNK, PLAIN>(p, a0, a1, b0, b1, sp, m0, n0, bat, piece, t_in, t_row);
#endif
}
template <int TM, int TN, int NCHUNK>
__global__ __launch_bounds__(kThreads, 2) void conv_split_patch_kernel(Params p) {
  split_patch_workgroup<TM, TN, NCHUNK, false, true>(p);
}
template <int TM, int TN, int NCHUNK, bool WHOLE>
__global__ __launch_bounds__(kThreads, 2) void conv_split_patch_kernel(Params p) {
  split_patch_workgroup<TM, TN, NCHUNK, false, !WHOLE>(p);
}
template <int TM, int TN, int NCHUNK>
__global__ __launch_bounds__(kThreads, 2) void conv_split_patch_narrow_last_kernel(Params p) {
  split_patch_workgroup<TM, TN, NCHUNK, true, true>(p);
}
template <int TM, int TN, int NCHUNK, bool WHOLE>
__global__ __launch_bounds__(kThreads, 2) void conv_split_patch_narrow_last_kernel(Params p) {
  split_patch_workgroup<TM, TN, NCHUNK, true, !WHOLE>(p);
}

// ---- weight gradient of 3x3 layers with stride 1, image patches in LDS ------------------
// The ring forms 64 x 128 results from operands that pass through LDS once per 64 rows resp. per
// tap, 1152 bytes a pixel, and waits for the caches that deliver them (160 channels at 32 x 32,
// 4 replicas of 128: 9.6 TB/s out of L2 at 106 TFLOP/s).  Here a workgroup takes 32 OB output channels x 32
// input channels x all nine taps: PX pixels of the gradient and the patch of the zero-rimmed
// image they touch (NCHUNK x 16 slots of 64 bytes a plane, a tap a constant shift of the slot) feed
// nine products, 790 bytes a pixel for 64 x 288 results.  Eight wavefronts, two to a matrix unit:
// each owns one 32-channel block of the gradient, every PG-th matrix depth of 16 pixels and five or
// four of the taps, and the two that share a unit have nine between them (all nine in one
// wavefront are 288 accumulators, more than its 256 registers for them).  Three stages in LDS, the
// loads of the one after the next under the products of the current one (with two stages they
// have to wait for a second barrier, and the matrix units for them: 45 % busy).  The PG sums are added through LDS at the end and the launch leaves one partial
// result per piece of the contraction.  4 replicas of 128, ring -> here: 64 channels at 32 x 32 320 ->
// 218 us (177 TFLOP/s), 160 channels 2270 -> 1440, 320 channels at 16 x 16 1400 -> 1020.
template <int NLA>
__device__ __forceinline__ void patch_offsets(const Geometry& g, int px0, int images, const int (&row)[NLA],
                                              const int (&col)[NLA], unsigned (&off)[NLA]) {
  const int H2 = g.oH + 2;
  int b0, i0, j0;
  decode_fast(px0, g, b0, i0, j0);
  const int pr0 = __builtin_amdgcn_readfirstlane(b0 * H2 + i0);
#pragma unroll
  for (int l = 0; l < NLA; ++l) {
    const int pr = pr0 + row[l], b = divide(pr, g.byH2), i = pr - b * H2 - 1;
    const bool ok = (unsigned)i < (unsigned)g.oH && b < images && col[l] >= 0;
    off[l] = ok ? (unsigned)(b * g.oH + i) * (unsigned)(g.oW * g.C * 2) + (unsigned)col[l] : kOob;
  }
}
// Load x of a stage: planes of the patch (NLA each), then of the gradient; `ahead`: bytes in front of the
// stage's first row of the gradient.
template <int NP, int OB, int PX, int NCHUNK, int NLA>
__device__ __forceinline__ void issue_wgrad(const Params& p, const unsigned short* Ab, const unsigned short* Bb, lds_byte* buf,
                                            lds_byte* spill, bool live, const unsigned (&off)[NLA], unsigned zoff, unsigned ahead,
                                            int wave, int x) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (x < NP * NLA) {
    const int q = x / NLA, l = x % NLA, chunk = wave + 8 * l;
    lds_byte* dst = chunk < NCHUNK ? buf + (q * NCHUNK + chunk) * 1024 : spill;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(Bb + q * p.planeB, live ? p.bytesB : 0u),
                                             (__attribute__((address_space(3))) void*)dst, 16, off[l], 0, 0, 0);
  } else {
    const int q = x - NP * NLA;
    lds_byte* dst = wave < OB * PX / 16 ? buf + NP * NCHUNK * 1024 + q * (OB * PX * 64) + wave * 1024 : spill;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(Ab + q * p.planeA, live ? p.bytesA : 0u),
                                             (__attribute__((address_space(3))) void*)dst, 16,
                                             zoff == kOob ? kOob : zoff + ahead, 0, 0, 0);
  }
#endif
}

__device__ __forceinline__ u32x4 read_transposed(const lds_byte* at0, const lds_byte* at1) {
  u32x4 f = {0u, 0u, 0u, 0u};
#if defined(__HIP_DEVICE_COMPILE__)
  const u32x2 l2 = __builtin_bit_cast(
      u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at0));
  const u32x2 h2 = __builtin_bit_cast(
      u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at1));
  f[0] = l2[0]; f[1] = l2[1]; f[2] = h2[0]; f[3] = h2[1];
#endif
  return f;
}

template <int NP, int OB, int PX, int NCHUNK>
__global__ __launch_bounds__(512, 2) void conv_wgrad_kernel(Params p) {
  constexpr int PG = 4 / OB, CH = PX / 16 / PG, NT = 5;   // CH: matrix depths per wavefront and stage
  constexpr int NLA = (NCHUNK + 7) / 8, NL = NP * (NLA + 1);
  constexpr int X_BYTES = NP * NCHUNK * 1024, Z_PLANE = OB * PX * 64, USED = X_BYTES + NP * Z_PLANE;
  constexpr int SUMS = NT * 16 * 64;                       // floats of a wavefront's sums
  constexpr int STAGE = USED > 2 * SUMS * 4 ? USED : 2 * SUMS * 4;
  static_assert(OB * PX <= 128, "a load of the gradient per wavefront and plane");
  __shared__ __attribute__((aligned(1024))) unsigned char st0[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char st1[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char st2[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char spill[1024];

  const int logical = (blockIdx.x % 8) * p.chunks + blockIdx.x / 8;
  if (logical >= p.total) return;
  const int per_rep = p.tilesM * p.tilesN;
  const int rest = __builtin_amdgcn_readfirstlane(logical / per_rep);
  const int t_in = logical - rest * per_rep;
  const int bat = __builtin_amdgcn_readfirstlane(rest / p.ksplit);
  const int piece = rest - bat * p.ksplit;
  const int t_row = __builtin_amdgcn_readfirstlane(t_in / p.tilesN);
  const int m0 = t_row * (OB * 32), c0 = (t_in - t_row * p.tilesN) * 32;

  const unsigned short* Ab = p.A + (long long)bat * p.strideA;
  const unsigned short* Bb = p.B + (long long)bat * p.strideB;
  const Geometry& g = p.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ob = wave % OB, pg = wave / OB % PG, tg = wave / 4;   // output channels, pixels, taps
  const int H2 = g.oH + 2, W2 = g.oW + 2;
  const int images = p.Kd / (g.oH * g.oW);

  const int all = (p.Kd + PX - 1) / PX;                    // stages of the whole contraction
  const int first = piece * p.steps_per_piece;
  const int n = all - first < p.steps_per_piece ? all - first : p.steps_per_piece;

  int row[NLA], col[NLA];                                  // this lane's patch slots: rimmed row, byte offset in the row
#pragma unroll
  for (int l = 0; l < NLA; ++l) {
    const int slot = (wave + 8 * l) * 16 + (lane >> 2);
    row[l] = slot / W2;
    const int x = slot - row[l] * W2 - 1;
    col[l] = (unsigned)x < (unsigned)g.oW && wave + 8 * l < NCHUNK && c0 + (lane & 3) * 8 < g.C
                 ? (x * g.C + c0 + (lane & 3) * 8) * 2 : -1;
  }
  unsigned zoff;
  {
    const int blk = wave / (PX / 16), r = wave % (PX / 16) * 16 + (lane >> 2);
    const int c = m0 + blk * 32 + (lane & 3) * 8;
    zoff = blk < OB && c < p.ldA ? ((unsigned)r * p.ldA + c) * 2u : kOob;
  }
  lds_byte* s0 = (lds_byte*)st0;
  lds_byte* s1 = (lds_byte*)st1;
  lds_byte* s2 = (lds_byte*)st2;
  lds_byte* sp = (lds_byte*)spill;

  // transposing reads: lane -> pixel kr (+ 4) of the depth, four channels from colb / 2 on
  const int il = lane & 15, gq = lane >> 4;
  const int kr = (gq >> 1) * 8 + (il >> 2);
  const int colb = ((gq & 1) * 16 + 4 * (il & 3)) * 2;
  int shift[NT];                                           // of this wavefront's taps, in bytes (the tenth: unused)
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int tap = tg * NT + i < 9 ? tg * NT + i : 8;
    shift[i] = (tap / 3 * W2 + tap % 3) * 64;
  }

  f32x16 acc[NT], low[NP == 3 ? NT : 1];                   // low: the small products of a split
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      acc[t][e] = 0.f;
      if constexpr (NP == 3) low[t][e] = 0.f;
    }

  // What a stage needs in addresses is worked out under the products of the stages before it: the
  // offsets of its patch two stages ahead, its pixels' slots (of tap (0, 0)) one.
  unsigned off[NLA];
  int xs[CH][2], zs[CH][2];
  auto slots_of = [&](int px0) {
    int b, y, x;
    decode_fast(px0, g, b, y, x);
    const int pr0 = b * H2 + y;
#pragma unroll
    for (int cc = 0; cc < CH; ++cc)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        decode_fast(px0 + (pg + PG * cc) * 16 + kr + kk * 4, g, b, y, x);
        xs[cc][kk] = ((b * H2 + y - pr0) * W2 + x) * 64 + colb;
      }
  };
#pragma unroll
  for (int cc = 0; cc < CH; ++cc)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) zs[cc][kk] = X_BYTES + (ob * PX + (pg + PG * cc) * 16 + kr + kk * 4) * 64 + colb;
  const unsigned step = (unsigned)(p.ldA * 2) * PX;        // bytes of a stage's rows of the gradient
  patch_offsets(g, first * PX, images, row, col, off);
#pragma unroll
  for (int x = 0; x < NL; ++x) issue_wgrad<NP, OB, PX, NCHUNK>(p, Ab, Bb, s0, sp, true, off, zoff, first * step, wave, x);
  patch_offsets(g, (first + 1) * PX, images, row, col, off);
#pragma unroll
  for (int x = 0; x < NL; ++x) issue_wgrad<NP, OB, PX, NCHUNK>(p, Ab, Bb, s1, sp, 1 < n, off, zoff, (first + 1) * step, wave, x);
  patch_offsets(g, (first + 2) * PX, images, row, col, off);
  slots_of(first * PX);
  constexpr int LPS = (NL + CH * (NT - 1) - 1) / (CH * (NT - 1));   // loads under a step's products

  auto compute = [&](const lds_byte* buf, lds_byte* fill, int st) {
    u32x4 fa[2][NP], fb[2][NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      fa[0][q] = read_transposed(buf + zs[0][0] + q * Z_PLANE, buf + zs[0][1] + q * Z_PLANE);
      fb[0][q] = read_transposed(buf + xs[0][0] + shift[0] + q * NCHUNK * 1024, buf + xs[0][1] + shift[0] + q * NCHUNK * 1024);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 4 * NP, 0);
#pragma unroll
    for (int t = 0; t < CH * NT; ++t) {
      const int cc = t / NT, i = t % NT, nt = t + 1, nc = nt / NT;
      if (nt < CH * NT) {
        if (nc != cc)
#pragma unroll
          for (int q = 0; q < NP; ++q)
            fa[nc & 1][q] = read_transposed(buf + zs[nc][0] + q * Z_PLANE, buf + zs[nc][1] + q * Z_PLANE);
#pragma unroll
        for (int q = 0; q < NP; ++q)
          fb[nt & 1][q] = read_transposed(buf + xs[nc][0] + shift[nt % NT] + q * NCHUNK * 1024,
                                          buf + xs[nc][1] + shift[nt % NT] + q * NCHUNK * 1024);
      }
      const int x0 = (cc * (NT - 1) + i) * LPS;
      if (i < NT - 1)
#pragma unroll
        for (int x = x0; x < x0 + LPS; ++x)
          if (x < NL)
            issue_wgrad<NP, OB, PX, NCHUNK>(p, Ab, Bb, fill, sp, st + 2 < n, off, zoff, (first + st + 2) * step, wave, x);
      if (i < NT - 1 || tg == 0) {
        if constexpr (NP == 3) {
          constexpr int xa[5] = {2, 0, 1, 1, 0}, xb[5] = {0, 2, 1, 0, 1};
#pragma unroll
          for (int q = 0; q < 5; ++q)
            low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[t & 1][xb[q]]),
                                                             __builtin_bit_cast(bf16x8, fa[cc & 1][xa[q]]), low[i], 0, 0, 0);
        }
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[t & 1][0]),
                                                         __builtin_bit_cast(bf16x8, fa[cc & 1][0]), acc[i], 0, 0, 0);
        if (i < NT - 1) Interleave<0x120, 2 * NP + LPS, NP == 3 ? 6 : 1, 0>::run();
      }
    }
  };

  // After a stage's barrier every wavefront is through with the stage before, whose place the one
  // after the next takes.
#define LSAM_WGRAD_STAGE(CUR, FILL)                                                                                   \
  {                                                                                                                   \
    __builtin_amdgcn_s_waitcnt(waitcnt(NL, 0));                                                                       \
    asm volatile("" ::: "memory");                                                                                    \
    __builtin_amdgcn_s_barrier();                                                                                     \
    asm volatile("" ::: "memory");                                                                                    \
    compute(CUR, FILL, st);                                                                                           \
    slots_of((first + st + 1) * PX);                                                                                  \
    patch_offsets(g, (first + st + 3) * PX, images, row, col, off);                                                   \
    if (++st >= n) break;                                                                                             \
  }
  for (int st = 0;;) {
    LSAM_WGRAD_STAGE(s0, s2)
    LSAM_WGRAD_STAGE(s1, s0)
    LSAM_WGRAD_STAGE(s2, s1)
  }
#undef LSAM_WGRAD_STAGE
  __builtin_amdgcn_s_waitcnt(waitcnt(0, 0));            // nothing may still be writing LDS
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if constexpr (NP == 3) {
#pragma unroll
    for (int t = 0; t < NT; ++t) join_sums(acc[t], low[t]);
  }
  // the sums of pixel groups half.. to those of groups 0..half - 1
#pragma unroll
  for (int half = PG / 2; half >= 1; half /= 2) {
    const int slot = (pg % half * OB + ob) * 2 + tg;       // at most four
    float* at = reinterpret_cast<float*>(slot & 1 ? st1 : st0) + (slot >> 1) * SUMS + lane;
    if (pg >= half && pg < 2 * half) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) at[(t * 16 + e) * 64] = acc[t][e];
    }
    __syncthreads();
    if (pg < half) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] += at[(t * 16 + e) * 64];
    }
    __syncthreads();
  }
  const int m = m0 + ob * 32 + (lane & 31);
  if (pg == 0 && m < p.M) {
    float* C = p.partial + (long long)piece * p.stridePartial + ((long long)bat * p.M + m) * p.ldP;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (tg * NT + t >= 9) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = c0 + q * 8 + (lane >> 5) * 4;
        f32x4 v = {acc[t][q * 4], acc[t][q * 4 + 1], acc[t][q * 4 + 2], acc[t][q * 4 + 3]};
        if (c < g.C) *reinterpret_cast<f32x4*>(C + (tg * NT + t) * g.C + c) = v;
      }
    }
  }
}

// Every specialisation that is launched is instantiated explicitly (the compiler does not emit the
// host-side launch stubs of all implicit instantiations of such a kernel).
#define LSAM_CONV_KERNEL(...) template __global__ void conv_gemm_kernel<__VA_ARGS__>(Params);
LSAM_CONV_KERNEL(1, kForward, 128, 128, 2, 4, 2)
LSAM_CONV_KERNEL(1, kForward, 128, 128, 2, 4, 2, true)
LSAM_CONV_KERNEL(1, kForward, 256, 128, 2, 3, 2)
LSAM_CONV_KERNEL(1, kForward, 256, 128, 2, 3, 2, true)
LSAM_CONV_KERNEL(1, kForward, 256, 64, 4, 3, 2)
LSAM_CONV_KERNEL(1, kForward, 256, 64, 4, 3, 2, true)
LSAM_CONV_KERNEL(1, kForward, 256, 32, 4, 3, 2)
LSAM_CONV_KERNEL(1, kForward, 256, 32, 4, 3, 2, true)
LSAM_CONV_KERNEL(1, kForwardAnyC, 128, 128, 2, 4, 2)
LSAM_CONV_KERNEL(1, kForwardAnyC, 128, 128, 2, 4, 2, true)
LSAM_CONV_KERNEL(1, kForwardAnyC, 256, 128, 2, 3, 2)
LSAM_CONV_KERNEL(1, kForwardAnyC, 256, 128, 2, 3, 2, true)
LSAM_CONV_KERNEL(1, kForwardAnyC, 256, 64, 4, 3, 2)
LSAM_CONV_KERNEL(1, kForwardAnyC, 256, 64, 4, 3, 2, true)
LSAM_CONV_KERNEL(1, kForwardAnyC, 256, 32, 4, 3, 2)
LSAM_CONV_KERNEL(1, kForwardAnyC, 256, 32, 4, 3, 2, true)
LSAM_CONV_KERNEL(1, kWeightGrad, 128, 128, 2, 4, 2)
LSAM_CONV_KERNEL(1, kWeightGrad, 64, 128, 2, 4, 2)
LSAM_CONV_KERNEL(1, kWeightGrad, 32, 128, 1, 4, 2)
LSAM_CONV_KERNEL(3, kForward, 128, 64, 2, 2, 2)
LSAM_CONV_KERNEL(3, kForward, 128, 64, 2, 2, 2, true)
LSAM_CONV_KERNEL(3, kForward, 128, 32, 4, 2, 2)
LSAM_CONV_KERNEL(3, kForward, 128, 32, 4, 2, 2, true)
LSAM_CONV_KERNEL(3, kForwardAnyC, 128, 64, 2, 2, 2)
LSAM_CONV_KERNEL(3, kForwardAnyC, 128, 64, 2, 2, 2, true)
LSAM_CONV_KERNEL(3, kForwardAnyC, 128, 32, 4, 2, 2)
LSAM_CONV_KERNEL(3, kForwardAnyC, 128, 32, 4, 2, 2, true)
LSAM_CONV_KERNEL(3, kWeightGrad, 64, 128, 2, 2, 2)
LSAM_CONV_KERNEL(3, kWeightGrad, 32, 128, 1, 2, 2)

template __global__ void conv_patch_kernel<22>(Params);
template __global__ void conv_patch_kernel<22, true>(Params);
template __global__ void conv_patch_kernel<26>(Params);
template __global__ void conv_patch_kernel<26, true>(Params);
template __global__ void conv_split_patch_kernel<2, 2, 11>(Params);
template __global__ void conv_split_patch_kernel<2, 2, 11, true>(Params);
template __global__ void conv_split_patch_narrow_last_kernel<2, 2, 11>(Params);
template __global__ void conv_split_patch_narrow_last_kernel<2, 2, 11, true>(Params);
template __global__ void conv_split_patch_kernel<1, 2, 10>(Params);
template __global__ void conv_split_patch_kernel<1, 2, 10, true>(Params);
template __global__ void conv_split_patch_narrow_last_kernel<1, 2, 10>(Params);
template __global__ void conv_split_patch_narrow_last_kernel<1, 2, 10, true>(Params);
template __global__ void conv_split_patch_kernel<2, 1, 11>(Params);
template __global__ void conv_split_patch_kernel<2, 1, 11, true>(Params);
template __global__ void conv_split_patch_kernel<1, 1, 10>(Params);
template __global__ void conv_split_patch_kernel<1, 1, 10, true>(Params);
template __global__ void conv_wgrad_kernel<3, 2, 64, 9>(Params);
template __global__ void conv_wgrad_kernel<3, 1, 64, 9>(Params);
template __global__ void conv_wgrad_kernel<1, 2, 64, 9>(Params);
template __global__ void conv_wgrad_kernel<1, 1, 64, 9>(Params);

// ---- planes --------------------------------------------------------------------------------------
// dst planes of n values (a multiple of 4), 4 to a thread.  Bound by its (4 + 2 NP) bytes a value.
template <int NP>
__global__ __launch_bounds__(kThreads) void split_kernel(const float* __restrict__ src, unsigned short* __restrict__ dst,
                                                         long long plane, long long words) {
  const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (idx >= words) return;
  const f32x4 v = *reinterpret_cast<const f32x4*>(src + idx * 4);
  u16x4 o[NP];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    unsigned short t[NP];
    split_planes<NP>(v[r], t);
#pragma unroll
    for (int q = 0; q < NP; ++q) o[q][r] = t[q];
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) *reinterpret_cast<u16x4*>(dst + q * plane + idx * 4) = o[q];
}

// Planes of all filter banks of a model, one launch (a launch per bank and pass cost more than
// the copies).  Workgroups are dealt out bank by bank (FilterBank::first); a bank is copied with its
// rows padded to pitch ldp by zeros, or mirrored and transposed for the input gradient:
//   dst[c][tap * rows + o] = W[o][source(tap) * cols + c],
// source(tap) = taps - 1 - tap, or the order in which the classes of a stride-2 gradient follow each other,
// in 32 x 32 (o, c) tiles of one tap, transposed through LDS so that reads and writes are both rows.
template <int NP>
__global__ __launch_bounds__(kThreads) void filters_kernel(const float* __restrict__ params, long long strideParams,
                                                           const FilterBank* __restrict__ banks, int n,
                                                           unsigned short* __restrict__ dst, long long plane) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (banks[mid].first <= (int)blockIdx.x) lo = mid;
    else hi = mid - 1;
  }
  const FilterBank f = banks[lo];
  const int block = blockIdx.x - f.first;
  const long long k = blockIdx.y;
  const float* W = params + k * strideParams + f.src;
  if (f.taps == 0) {
    const int words = f.ldp / 4;
    const int idx = block * kThreads + threadIdx.x;
    if (idx < f.rows * words) {
      const int o = idx / words, c = (idx - o * words) * 4;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (c < f.cols) v = *reinterpret_cast<const f32x4*>(W + (long long)o * f.ldw + c);     // cols % 4 == 0
      u16x4 t[NP];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        unsigned short b[NP];
        split_planes<NP>(v[r], b);
#pragma unroll
        for (int q = 0; q < NP; ++q) t[q][r] = b[q];
      }
      unsigned short* to = dst + f.dst + (k * f.rows + o) * f.ldp + c;
#pragma unroll
      for (int q = 0; q < NP; ++q) *reinterpret_cast<u16x4*>(to + q * plane) = t[q];
    }
  } else {
    __shared__ float tile[32][33];
    const int cblocks = (f.cols + 31) / 32;
    const int tap = block % f.taps, ot = block / f.taps / cblocks, ct = block / f.taps % cblocks;
    const int ob = ot * 32, cb = ct * 32;
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    // (stride 2: the centre; its row's and its column's other two; the corners)
    const int from = f.taps == 9 && f.stride == 2 ? (int)(0x026817354ull >> (4 * tap) & 15) : f.taps - 1 - tap;
    const float* src = W + (long long)from * f.cols;
#pragma unroll
    for (int r = 0; r < 32; r += 8)
      tile[y + r][x] = (cb + x < f.cols && ob + y + r < f.rows) ? src[(long long)(ob + y + r) * f.ldw + cb + x] : 0.f;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 32; r += 8) {
      const int c = cb + y + r;
      if (c >= f.cols) continue;
      unsigned short b[NP];
      split_planes<NP>(tile[x][y + r], b);
      unsigned short* row = dst + f.dst + (k * f.cols + c) * f.ldp;
      if (ob + x < f.rows) {
#pragma unroll
        for (int q = 0; q < NP; ++q) row[q * plane + tap * f.rows + ob + x] = b[q];
      }
      // the row's padding: written by the workgroups of the last tap's last output block
      if (tap == f.taps - 1 && ob + 32 >= f.rows) {
        for (int z = f.taps * f.rows + x; z < f.ldp; z += 32)
#pragma unroll
          for (int q = 0; q < NP; ++q) row[q * plane + z] = 0;
      }
    }
  }
}

unsigned blocks_for(long long n) { return (unsigned)((n + kThreads - 1) / kThreads); }

struct Tile { int bm, bn; };

int tiled(Params& p, int bm, int bn) {
  p.tilesM = (p.M + bm - 1) / bm;
  p.tilesN = (p.N + bn - 1) / bn;
  p.total = p.tilesM * p.tilesN * p.batch * p.ksplit * (p.out_step == 2 ? 4 : 1);
  p.chunks = (p.total + 7) / 8;
  return p.tilesM * p.tilesN;
}

template <int NP, int KIND, int BM, int BN, int WM, int NSTAGE, int OCC>
int run(Params& p, hipStream_t s) {
  const int slots = tiled(p, BM, BN);
  if constexpr (KIND != kWeightGrad) {
    if (p.ksplit > 1) {
      conv_gemm_kernel<NP, KIND, BM, BN, WM, NSTAGE, OCC, true><<<p.chunks * 8, kThreads, 0, s>>>(p);
      return slots;
    }
  }
  conv_gemm_kernel<NP, KIND, BM, BN, WM, NSTAGE, OCC><<<p.chunks * 8, kThreads, 0, s>>>(p);
  return slots;
}

template <int KIND>
int run_forward(Params& p, const Tile& t, int np, hipStream_t s) {
  if (np == 1) {
    if (t.bm == 256 && t.bn == 128) return run<1, KIND, 256, 128, 2, 3, 2>(p, s);
    if (t.bn == 128) return run<1, KIND, 128, 128, 2, 4, 2>(p, s);
    if (t.bn == 64) return run<1, KIND, 256, 64, 4, 3, 2>(p, s);
    return run<1, KIND, 256, 32, 4, 3, 2>(p, s);
  }
  if (t.bn == 64) return run<3, KIND, 128, 64, 2, 2, 2>(p, s);
  return run<3, KIND, 128, 32, 4, 2, 2>(p, s);
}
int run_weight_grad(Params& p, const Tile& t, int np, hipStream_t s) {
  if (np == 1) {
    if (t.bm == 128) return run<1, kWeightGrad, 128, 128, 2, 4, 2>(p, s);
    if (t.bm == 64) return run<1, kWeightGrad, 64, 128, 2, 4, 2>(p, s);
    return run<1, kWeightGrad, 32, 128, 1, 4, 2>(p, s);
  }
  if (t.bm == 64) return run<3, kWeightGrad, 64, 128, 2, 2, 2>(p, s);
  return run<3, kWeightGrad, 32, 128, 1, 2, 2>(p, s);
}

enum PatchKind { kNoPatch = 0, kPatch22, kPatch26, kSplitPatch256, kSplitPatch128, kSplitNarrow256, kSplitNarrow128, kWgrad64, kWgrad32 };
int run_patch(Params& p, int kind, int np, hipStream_t s) {
  if (kind == kWgrad64 || kind == kWgrad32) {
    tiled(p, kind == kWgrad64 ? 64 : 32, 9 * 32);            // N = 9 C: a column of tiles per 32 channels
    const unsigned grid = (unsigned)p.chunks * 8;
    if (np == 1 && kind == kWgrad64) conv_wgrad_kernel<1, 2, 64, 9><<<grid, 512, 0, s>>>(p);
    else if (np == 1) conv_wgrad_kernel<1, 1, 64, 9><<<grid, 512, 0, s>>>(p);
    else if (kind == kWgrad64) conv_wgrad_kernel<3, 2, 64, 9><<<grid, 512, 0, s>>>(p);
    else conv_wgrad_kernel<3, 1, 64, 9><<<grid, 512, 0, s>>>(p);
    return 0;                                                // partial sums only
  }
  const int slots = tiled(p, kind == kSplitPatch128 || kind == kSplitNarrow128 ? 128 : 256,
                          kind == kSplitNarrow256 || kind == kSplitNarrow128 ? 32 : 64);
  const unsigned grid = (unsigned)p.chunks * 8;
  const bool narrow_last = (p.N - 1) % 64 < 32 && (p.total <= 512 || p.total >= 1024);
  auto go = [&](auto piece, auto whole) { (p.ksplit > 1 ? +piece : +whole)<<<grid, kThreads, 0, s>>>(p); };
  if (kind == kPatch22) go(conv_patch_kernel<22>, conv_patch_kernel<22, true>);
  else if (kind == kPatch26) go(conv_patch_kernel<26>, conv_patch_kernel<26, true>);
  else if (kind == kSplitPatch256 && narrow_last) go(conv_split_patch_narrow_last_kernel<2, 2, 11>, conv_split_patch_narrow_last_kernel<2, 2, 11, true>);
  else if (kind == kSplitPatch256) go(conv_split_patch_kernel<2, 2, 11>, conv_split_patch_kernel<2, 2, 11, true>);
  else if (kind == kSplitPatch128 && narrow_last) go(conv_split_patch_narrow_last_kernel<1, 2, 10>, conv_split_patch_narrow_last_kernel<1, 2, 10, true>);
  else if (kind == kSplitPatch128) go(conv_split_patch_kernel<1, 2, 10>, conv_split_patch_kernel<1, 2, 10, true>);
  else if (kind == kSplitNarrow256) go(conv_split_patch_kernel<2, 1, 11>, conv_split_patch_kernel<2, 1, 11, true>);
  else go(conv_split_patch_kernel<1, 1, 10>, conv_split_patch_kernel<1, 1, 10, true>);
  return slots;
}

struct ConvPlan {
  Tile tile;
  int patch;              // PatchKind: the patch kernel that serves the launch, or the ring
  int splits, steps, ldP; // steps: k-steps of 32 (patch kernels: blocks of 32 or 16 channels) per piece
  size_t ws_bytes;
};

// Slots of the largest patch a tile of bm consecutive pixels can touch: its image rows, the rows
// above and below, and two more at every boundary between images it contains.  Square images whose
// patches fit the kernels there are: three planes, forward and dX, sides of 4 to 30, 32, 33 and 64, dW
// 4, 6 to 11, 16 and 32; one plane, forward and dX, 8, 12 to 22, 24, 32 and 64.  Others take the ring.
int patch_slots(int bm, int H, int W) {
  int rows, inside;
  if (bm % W == 0) {
    rows = bm / W;
    inside = H % rows == 0 ? 0 : rows % H == 0 ? rows / H - 1 : (rows + H - 2) / H;
  } else {
    rows = (bm - 2) / W + 2;
    inside = (rows + H - 2) / H;
  }
  return (rows + 2 + 2 * inside) * (W + 2);
}

ConvPlan conv_plan(const ConvGemmDesc& d) {
  ConvPlan pl{{128, 128}, 0, 1, 0, 0, 0};
  auto count = [&](int bm, int bn) { return (long long)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * d.batch; };
  // Tiles by measurement (4 replicas, batch 128).  One plane: 256 x 128 while that gives every
  // compute unit its two workgroups (128 channels at 16 x 16: 53 us against 62 with 128 x 128; 256
  // at 8 x 8, 256 tiles: 70 against 54).  Three planes: the LDS holds two workgroups of 128 x 64
  // (227 us at 128 channels, 16 x 16) or one of 128 x 128 (251).
  if (!d.wgrad) {
    if (d.np == 1)
      pl.tile = d.N > 64 ? (count(256, 128) >= 384 ? Tile{256, 128} : Tile{128, 128}) : d.N > 32 ? Tile{256, 64} : Tile{256, 32};
    else
      pl.tile = d.N > 32 ? Tile{128, 64} : Tile{128, 32};
  } else {
    pl.tile = d.M > 64 && d.np == 1 ? Tile{128, 128} : d.M > 32 ? Tile{64, 128} : Tile{32, 128};
  }
  const PlaneImage& im = d.image;
  if (!d.wgrad && im.nu == 3 && im.nv == 3 && im.st == 1 && d.out_step == 1 &&
      im.C % (d.np == 1 ? 32 : 16) == 0 && (d.np == 3 || d.N > 32)) {
    const int s256 = patch_slots(256, im.oH, im.oW), s128 = patch_slots(128, im.oH, im.oW);
    if (d.np == 1) pl.patch = s256 <= 22 * 16 ? kPatch22 : s256 <= 26 * 16 ? kPatch26 : kNoPatch;
    else if (d.N > 32) pl.patch = s256 <= 11 * 32 ? kSplitPatch256 : s128 <= 10 * 32 ? kSplitPatch128 : kNoPatch;
    else pl.patch = s256 <= 11 * 32 ? kSplitNarrow256 : s128 <= 10 * 32 ? kSplitNarrow128 : kNoPatch;
    if (pl.patch) {
      const Tile t{pl.patch == kSplitPatch128 || pl.patch == kSplitNarrow128 ? 128 : 256, d.N > 32 ? 64 : 32};
      // Fewer than 64 of the three-plane patches' large tiles leave the chip idle, where the ring's smaller ones can also cut
      // the contraction (two layers at 16 x 16, patches / ring: 48 channels, 26 tiles 359 / 320 us, 80, 32 tiles 370 / 348, 112, 32
      // tiles 392 / 364; 160, 78 tiles 491 / 523).  Layers of whole blocks of 32 channels, which had these patches before
      // other counts did, would gain 3 to 5 % there too (64, 26 tiles 372 / 347) and are left as they are.
      if (d.np == 3 && (im.C % 32 || d.N % 32) && count(t.bm, t.bn) < 64) pl.patch = kNoPatch;
      else pl.tile = t;
    }
  }
  // Weight gradients: the patch kernel always leaves partial sums.  Its workgroups have a compute unit to
  // themselves and equal work, so the contraction is cut for one, two or four full rounds of 256,
  // the first that keeps 93 % of the units busy.
  if (d.wgrad && im.nu == 3 && im.nv == 3 && im.st == 1 && im.oW >= 2 && im.oH >= 2) {
    const bool wide = d.M > 32;
    const int px = 64;
    const long long tiles = (long long)((d.M + (wide ? 63 : 31)) / (wide ? 64 : 32)) * ((im.C + 31) / 32) * d.batch;
    const int stages = (d.Kd + px - 1) / px;
    long long pieces = 0;
    for (int r = 1; r <= 4; r *= 2) {
      pieces = 256LL * r / tiles;
      if (pieces * tiles >= 238LL * r) break;
    }
    if (pieces > 64) pieces = 64;
    if (pieces > stages / 4) pieces = stages / 4;
    if (patch_slots(px, im.oH, im.oW) <= 9 * 16 && pieces >= 2) {
      pl.patch = wide ? kWgrad64 : kWgrad32;
      pl.steps = (int)((stages + pieces - 1) / pieces);
      pl.splits = (stages + pl.steps - 1) / pl.steps;
      pl.ldP = d.N;
      pl.ws_bytes = (size_t)pl.splits * d.batch * d.M * pl.ldP * 4;
      if (pl.splits >= 2) return pl;
      pl = ConvPlan{pl.tile, 0, 1, 0, 0, 0};
    }
  }
  const int per_block = pl.patch ? (d.np == 1 ? 32 : 16) : 0;
  const int all = pl.patch ? im.C / per_block : (d.Kd + 31) / 32;
  const long long tiles = count(pl.tile.bm, pl.tile.bn);
  const int target = 512;                                   // workgroups that fit the chip
  pl.steps = all;
  if (tiles < target && all >= (pl.patch ? 4 : 16) && d.out_step == 1) {
    long long want = (target + tiles - 1) / tiles;
    long long cap = pl.patch ? all / 2 : all / 8;
    long long sp = want < cap ? want : cap;
    if (sp > 64) sp = 64;
    if (sp > 1) {
      pl.steps = (int)((all + sp - 1) / sp);
      pl.splits = (all + pl.steps - 1) / pl.steps;
      pl.ldP = (d.N + 3) / 4 * 4;
      pl.ws_bytes = (size_t)pl.splits * d.batch * d.M * pl.ldP * 4;
    }
  }
  if (pl.splits == 1) { pl.steps = all; pl.ws_bytes = 0; }
  return pl;
}

}  // namespace

size_t conv_gemm_splitk_bytes(const ConvGemmDesc& d) { return conv_plan(d).ws_bytes; }

int launch_conv_gemm(const ConvGemmDesc& d, hipStream_t s, int* sumsq_slots, ChunkSums* made) {
  if (d.np != 1 && d.np != 3) return -1;
  if (d.M <= 0 || d.N <= 0 || d.Kd <= 0 || d.batch <= 0 || d.N % 4 || d.ldC % 4 || d.strideC % 4) return -1;
  const PlaneImage& im = d.image;
  const long long out_px = d.wgrad ? d.Kd : d.M;
  if (im.C < 8 || im.C % 8 || im.oH < 1 || im.oW < 1 || im.sH < 1 || im.sW < 1 || im.st < 1 || im.nu < 1 || im.nu > 3 ||
      im.nv < 1 || im.nv > 3 || out_px % ((long long)im.oH * im.oW))
    return -1;
  const int taps = im.nu * im.nv;
  const long long img_elems = out_px / ((long long)im.oH * im.oW) * im.sH * im.sW * im.C;
  if ((d.wgrad ? d.N : d.Kd) != taps * im.C) return -1;
  const bool scalar_tap = im.C % 32 == 0;
  // the other operand: filters [N][ld] resp. output gradient [Kd][ld]
  const long long rows = d.wgrad ? d.Kd : d.N;
  if (d.ld % 8 || (d.wgrad ? d.ld != d.M : d.ld < (d.Kd + 31) / 32 * 32)) return -1;
  if (d.out_step != 1 && (d.out_step != 2 || d.wgrad || im.st != 1 || taps != 9 || im.oH != im.sH || im.oW != im.sW ||
                          d.sumsq != nullptr || out_px >= (1 << 29)))
    return -1;
  // 32-bit byte offsets; a k-step may reach up to 32 rows past the end
  if (img_elems * 2 >= 0x7FFF0000LL || (rows + 32) * d.ld * 2 >= 0x7FFF0000LL) return -1;
  if (((uintptr_t)im.p & 15) || ((uintptr_t)d.other & 15) || (im.stride % 8) || (im.plane % 8) || (d.other_stride % 8) ||
      (d.other_plane % 8) || ((uintptr_t)d.C & 15))
    return -1;
  if (d.epilogue == EPI_MASK && (d.ldMask % 4 || d.strideMask % 4 || (!d.keep && ((uintptr_t)d.mask & 15)))) return -1;
  if (d.add && (d.wgrad || d.ldAdd % 4 || d.strideAdd % 4 || ((uintptr_t)d.add & 15))) return -1;
  if ((d.epilogue == EPI_BIAS || d.epilogue == EPI_BIAS_RELU) && (((uintptr_t)d.bias & 15) || d.strideBias % 4)) return -1;
  Params p{};
  const unsigned image_bytes = (unsigned)(img_elems * 2), other_bytes = (unsigned)(rows * d.ld * 2);
  if (!d.wgrad) {
    p.A = im.p; p.strideA = im.stride; p.planeA = im.plane; p.bytesA = image_bytes;
    p.B = d.other; p.strideB = d.other_stride; p.planeB = d.other_plane; p.ldB = d.ld; p.bytesB = other_bytes;
  } else {
    p.A = d.other; p.strideA = d.other_stride; p.planeA = d.other_plane; p.ldA = d.ld; p.bytesA = other_bytes;
    p.B = im.p; p.strideB = im.stride; p.planeB = im.plane; p.bytesB = image_bytes;
  }
  p.C = d.C; p.strideC = d.strideC; p.ldC = d.ldC;
  p.M = d.M; p.N = d.N; p.Kd = d.Kd; p.batch = d.batch;
  p.g = Geometry{im.C, im.oH, im.oW, im.sH, im.sW, im.st, im.nu, im.nv, im.du0, im.dv0,
                 (unsigned)((1ull << 32) / (unsigned)im.C + 1), divisor(im.oW), divisor(im.oH),
                 divisor(im.oH + 2)};
  p.epilogue = d.epilogue;
  p.out_step = d.out_step;
  p.bias = d.bias; p.strideBias = d.strideBias;
  p.mask = d.mask; p.strideMask = d.strideMask; p.ldMask = d.ldMask; p.keep = d.keep;
  p.add = d.add; p.strideAdd = d.strideAdd; p.ldAdd = d.ldAdd;
  p.sumsq = d.sumsq; p.strideSumsq = d.sumsq_stride;
  if (d.sums != 0 && (d.wgrad || d.ldC != d.N || ((uintptr_t)d.sum_part & 15) ||
                      (d.sums == 2 && ((d.epilogue == EPI_MASK && !d.keep) || ((uintptr_t)d.sum_z & 15) || ((uintptr_t)d.sum_stats & 15)))))
    return -1;
  ConvPlan pl = conv_plan(d);
  const bool room = d.splitk_ws != nullptr && d.splitk_bytes >= pl.ws_bytes && ((uintptr_t)d.splitk_ws & 15) == 0;
  if (d.wgrad && pl.patch && !room) pl.patch = kNoPatch, pl.splits = 1, pl.steps = (d.Kd + 31) / 32;
  p.ksplit = 1; p.steps_per_piece = pl.steps * pl.splits;     // all of it
  if (pl.splits > 1 && room) {
    p.ksplit = pl.splits; p.steps_per_piece = pl.steps;
    p.partial = d.splitk_ws; p.ldP = pl.ldP;
    p.stridePartial = (long long)d.batch * d.M * pl.ldP;
  }
  if (p.ksplit == 1) { p.sums = d.sums; p.sum_part = d.sum_part; p.sum_z = d.sum_z; p.sum_stats = d.sum_stats; }
  int slots = pl.patch ? run_patch(p, pl.patch, d.np, s)
              : d.wgrad ? run_weight_grad(p, pl.tile, d.np, s)
              : scalar_tap ? run_forward<kForward>(p, pl.tile, d.np, s) : run_forward<kForwardAnyC>(p, pl.tile, d.np, s);
  if (p.ksplit > 1 && d.list && d.list->n < ReduceList::kMax && d.N % 4 == 0 && p.ldP % 4 == 0) {
    ReduceList& list = *d.list;
    const int blocks = (int)(((long long)d.M * (p.ldP / 4) + kThreads - 1) / kThreads);
    list.job[list.n++] = ReduceList::Job{p.partial, p.stridePartial, d.C, d.strideC, d.M, d.N, d.ldC, p.ldP, p.ksplit, list.blocks, d.list_slot};
    list.blocks += blocks;
    slots = blocks;
  } else if (p.ksplit > 1) {
    GemmDesc r{};
    r.C = d.C; r.strideC = d.strideC; r.ldC = d.ldC; r.M = d.M; r.N = d.N; r.batch = d.batch;
    r.epilogue = d.epilogue; r.bias = d.bias; r.strideBias = d.strideBias;
    r.mask = d.mask; r.strideMask = d.strideMask; r.ldMask = d.ldMask; r.keep = d.keep;
    r.add = d.add; r.strideAdd = d.strideAdd; r.ldAdd = d.ldAdd;
    r.sumsq = d.sumsq; r.sumsq_stride = d.sumsq_stride;
    slots = launch_splitk_reduce(r, p.partial, p.ksplit, p.stridePartial, p.ldP, s);
  }
  if (sumsq_slots) *sumsq_slots = slots;
  if (made) *made = p.sums ? ChunkSums{p.tilesM * (p.out_step == 2 ? 4 : 1), pl.tile.bm} : ChunkSums{};
  return 0;
}

int conv_gemm_sum_chunks(int64_t rows) { return (int)(rows / 128) + 8; }

int launch_split_planes(const float* src, uint16_t* dst, int np, int64_t plane, int64_t n, hipStream_t s) {
  if (n < 4 || n % 4 || plane % 8 || ((uintptr_t)src & 15) || ((uintptr_t)dst & 15)) return -1;
  if (np == 1) split_kernel<1><<<blocks_for(n / 4), kThreads, 0, s>>>(src, dst, plane, n / 4);
  else split_kernel<3><<<blocks_for(n / 4), kThreads, 0, s>>>(src, dst, plane, n / 4);
  return 0;
}

int filter_bank_blocks(const FilterBank& f) {
  if (f.taps == 0) return (int)(((long long)f.rows * (f.ldp / 4) + kThreads - 1) / kThreads);
  return (f.rows + 31) / 32 * ((f.cols + 31) / 32) * f.taps;
}

int launch_filters(const float* params, int64_t strideParams, const FilterBank* banks, int n, int blocks, uint16_t* dst,
                   int np, int64_t plane, int K, hipStream_t s) {
  if (n < 1 || blocks < 1) return -1;
  const dim3 grid((unsigned)blocks, (unsigned)K);
  if (np == 1) filters_kernel<1><<<grid, kThreads, 0, s>>>(params, strideParams, banks, n, dst, plane);
  else filters_kernel<3><<<grid, kThreads, 0, s>>>(params, strideParams, banks, n, dst, plane);
  return 0;
}

}  // namespace lsam
