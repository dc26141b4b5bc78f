// Pieces of the fp32 dense model's backward pass that run as kernels of their own or as workgroups of
// the launch that takes a whole pass's gradients (kernels_gemm.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace lsam {

constexpr int kHeadMaxC = 16;       // classes of the narrow head
typedef float hf4 __attribute__((ext_vector_type(4)));

// db[n] = sum_b dz[b][n] for the 64 columns from 64 * block on.  Share w of WAVES takes every WAVES-th row from w
// on, as four chains; `part`: WAVES * 64 floats of LDS.  WAVES / ROLES wavefronts, each with ROLES shares: what
// bounds it is the chain of loads a wavefront waits for, and a wavefront with four shares has sixteen under way.
template <int WAVES, int ROLES = 1>
__device__ __forceinline__ void column_sums(const float* dz, long long ld, float* db, int B, int N, int block, float* part,
                                            double* sumsq) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = block * 64 + lane;
  float s[ROLES][4] = {};
  auto share = [&](int r) { return wave + r * (WAVES / ROLES); };
  if (n < N) {
    auto at = [&](int b) { return dz[(long long)b * ld + n]; };
    int base = 0;
    for (; base + 4 * WAVES <= B; base += 4 * WAVES)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < ROLES; ++r) s[r][i] += at(base + share(r) + i * WAVES);
#pragma unroll
    for (int r = 0; r < ROLES; ++r) {
      int b = base + share(r);
      if (b + 3 * WAVES < B) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s[r][i] += at(b + i * WAVES);
        b += 4 * WAVES;
      }
      for (; b < B; b += WAVES) s[r][0] += at(b);
    }
  }
#pragma unroll
  for (int r = 0; r < ROLES; ++r) part[share(r) * 64 + lane] = (s[r][0] + s[r][1]) + (s[r][2] + s[r][3]);
  __syncthreads();
  if (wave == 0) {
    float r = 0.f;
    if (n < N) {
#pragma unroll
      for (int w = 0; w < WAVES; w += 4)
        r += (part[w * 64 + lane] + part[(w + 1) * 64 + lane]) + (part[(w + 2) * 64 + lane] + part[(w + 3) * 64 + lane]);
      db[n] = r;
    }
    if (sumsq != nullptr) {        // sum of the squares of these 64 results
      double q = (double)r * (double)r;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off, 64);
      if (lane == 0) *sumsq = q;
    }
  }
}

// The narrow head's dW[c][j] = sum_b dz[b][c] A[b][j] for the 16 columns from 16 * block on, and (block 0)
// db[c] = sum_b dz[b][c], of one replica, by 256 threads.  Thread = (column, one of 16 row groups); the row
// groups are combined in a fixed order through LDS: head_grad_lds(B, ld_dz) bytes, 16-byte aligned.
inline __host__ __device__ int head_grad_lds(int B, int ld_dz) {
  return (16 * kHeadMaxC * 17 + B * ld_dz) * 4 + 4 * 8;
}
__device__ __forceinline__ void head_weight_grad(const float* dz, int ld_dz, const float* A, int ldA, float* dW, int ldw,
                                                 float* db, int B, int C, int in, int block, float* lds, double* sumsq) {
  double* ssq_part = reinterpret_cast<double*>(lds);
  float* part = lds + 8;                                 // [16][kHeadMaxC][17]
  float* dzs = part + 16 * kHeadMaxC * 17;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = tid & 15, rg = tid >> 4;
  for (int i = tid; i < B * ld_dz / 4; i += 256) reinterpret_cast<hf4*>(dzs)[i] = reinterpret_cast<const hf4*>(dz)[i];
  const int j = block * 16 + col;
  const float* ak = A + j;
  float acc[kHeadMaxC];
#pragma unroll
  for (int c = 0; c < kHeadMaxC; ++c) acc[c] = 0.f;
  __syncthreads();
  if (j < in) {
#pragma unroll 8
    for (int b = rg; b < B; b += 16) {
      const float av = ak[(long long)b * ldA];
#pragma unroll
      for (int c = 0; c < kHeadMaxC; ++c)
        if (c < C) acc[c] += dzs[b * ld_dz + c] * av;
    }
  }
#pragma unroll
  for (int c = 0; c < kHeadMaxC; ++c) part[(rg * kHeadMaxC + c) * 17 + col] = acc[c];
  __syncthreads();
  float ssq = 0.f;
  {
    const int c = tid >> 4;                 // thread = (class, column)
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) v += part[(q * kHeadMaxC + c) * 17 + col];
    if (c < C && j < in) {
      dW[(long long)c * ldw + j] = v;
      ssq += v * v;
    }
  }
  if (block == 0 && tid < C) {
    float s0 = 0.f, s1 = 0.f;
    int b = 0;
    for (; b + 1 < B; b += 2) { s0 += dzs[b * ld_dz + tid]; s1 += dzs[(b + 1) * ld_dz + tid]; }
    if (b < B) s0 += dzs[b * ld_dz + tid];
    const float sb = s0 + s1;
    db[tid] = sb;
    ssq += sb * sb;
  }
  if (sumsq != nullptr) {
    double q = (double)ssq;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) q += __shfl_xor(q, off, 64);
    if (lane == 0) ssq_part[wave] = q;
    __syncthreads();
    if (tid == 0) *sumsq = (ssq_part[0] + ssq_part[1]) + (ssq_part[2] + ssq_part[3]);
  }
}

// Four neighbouring sums of a split contraction's n pieces, `stride` apart: one chain below eight pieces,
// four interleaved ones from there on (the order of the reduce kernel).
__device__ __forceinline__ hf4 split_sum(const float* p, long long stride, int n) {
  auto at = [&](int s) { return *reinterpret_cast<const hf4*>(p + (long long)s * stride); };
  hf4 v[4] = {};
  if (n < 8) {
    for (int s = 0; s < n; ++s) v[0] += at(s);
    return v[0];
  }
  for (int s = 0; s < n; s += 4)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (s + q < n) v[q] += at(s + q);
  return (v[0] + v[1]) + (v[2] + v[3]);
}

}  // namespace lsam
