// fp32 GEMM with fp32 products and sums for the fp32 MLP workload (gradients agree with the fp64 reference to 1e-5).
// Same operand convention as the bf16 kernel: D[i][j] = sum_k A(i,k) B(j,k), either operand optionally stored
// reduction-index-slow.
//
// What bounds these products is latency: a layer of the batch-32 workload is 4 MFLOP over 256 KB.  A workgroup owns one
// T x T tile (T = 16 or 32), its four waves take the reduction in turns of KC = 64 or 32 k values (wave w: chunks w, w + 4,
// ...), straight from global memory into the fp32 matrix instructions: no LDS round trip and no barrier before the
// end, all loads of a chunk in flight at once and the next chunk's issued before the current one is multiplied.  A lane
// loads 4 consecutive k values of its row (or 4 k-rows of its column); matrix instruction j then takes value j of every
// lane, the same permutation of k on both sides.  At the end the four partial tiles meet in LDS and are added in wave
// order.  Against the former 64 x 64 LDS tiles (four workgroups and 16 barrier-separated slices for [32 x 256] over 256, 45 us
// of which 2 are left) the full step of four layers of 256 at batch 32 went from 314 to 48 us (14 launches; the host needs
// 44 us to issue them), of eight layers of 1024 at batch 512 from 3637 to 508 us.
#include "kernels.h"

namespace et {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int T> struct Acc;
template <> struct Acc<16> { typedef f32x4 type; };
template <> struct Acc<32> { typedef f32x16 type; };
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 mma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// U quadruples of k values of one row (or column) of an operand, k = k0 + u * KU + q * 4 + 0..3, zero outside the matrix
template <int T, int U, bool TR>
__device__ __forceinline__ void load_quads(const float* base, int ld, int row, int rows, int k0, int q, int K, bool vec, f32x4 (&v)[U]) {
  constexpr int KU = 256 / T;   // k values covered by the wave with one quadruple per lane
  const bool in = row < rows;
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int k = k0 + u * KU + q * 4;
    if (!TR && vec && in && k + 4 <= K) {
      v[u] = *(const f32x4*)(base + (long long)row * ld + k);
    } else {
#pragma unroll
      for (int j = 0; j < 4; j++)
        v[u][j] = in && k + j < K ? (TR ? base[(long long)(k + j) * ld + row] : base[(long long)row * ld + k + j]) : 0.f;
    }
  }
}

template <int T, bool AT, bool BT>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Desc g) {
  constexpr int U = 4, KU = 256 / T, KC = U * KU;
  __shared__ float part[4][T * T];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  const int r = lane % T, q = lane / T;
  const bool va = (g.lda & 3) == 0 && ((uintptr_t)g.A & 15) == 0, vb = (g.ldb & 3) == 0 && ((uintptr_t)g.B & 15) == 0;
  typename Acc<T>::type acc = {};
  f32x4 a[U], b[U], an[U], bn[U];
  int k0 = wave * KC;
  if (k0 < g.K) {
    load_quads<T, U, AT>(g.A, g.lda, m0 + r, g.M, k0, q, g.K, va, a);
    load_quads<T, U, BT>(g.B, g.ldb, n0 + r, g.N, k0, q, g.K, vb, b);
  }
  for (; k0 < g.K; k0 += 4 * KC) {
    const int kn = k0 + 4 * KC;
    if (kn < g.K) {
      load_quads<T, U, AT>(g.A, g.lda, m0 + r, g.M, kn, q, g.K, va, an);
      load_quads<T, U, BT>(g.B, g.ldb, n0 + r, g.N, kn, q, g.K, vb, bn);
    }
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int j = 0; j < 4; j++) acc = mma(a[u][j], b[u][j], acc);
#pragma unroll
    for (int u = 0; u < U; u++) { a[u] = an[u]; b[u] = bn[u]; }
  }
  // accumulator x of a lane is element (row, lane % T) of the tile, row = (x / 4) * (256 / T) + (lane / T) * 4 + x % 4
#pragma unroll
  for (int x = 0; x < T * T / 64; x++) part[wave][((x / 4) * (256 / T) + q * 4 + x % 4) * T + r] = acc[x];
  __syncthreads();
#pragma unroll
  for (int o = 0; o < T * T / 256; o++) {
    const int e = o * 256 + threadIdx.x;
    const int row = m0 + e / T, col = n0 + e % T;
    if (row >= g.M || col >= g.N) continue;
    float v = ((part[0][e] + part[1][e]) + part[2][e]) + part[3][e];
    const long long ci = (long long)row * g.ldc + col;
    if (g.relu_out) v = fmaxf(v, 0.f);
    if (g.mask) v = g.mask[ci] > 0.f ? v : 0.f;
    g.C[ci] = v;
  }
}

template <int T>
void launch(const GemmF32Desc& d, hipStream_t s) {
  const dim3 grid((d.N + T - 1) / T, (d.M + T - 1) / T), block(256);
  if (d.a_t && d.b_t) hipLaunchKernelGGL((gemm_f32_kernel<T, true, true>), grid, block, 0, s, d);
  else if (d.a_t) hipLaunchKernelGGL((gemm_f32_kernel<T, true, false>), grid, block, 0, s, d);
  else if (d.b_t) hipLaunchKernelGGL((gemm_f32_kernel<T, false, true>), grid, block, 0, s, d);
  else hipLaunchKernelGGL((gemm_f32_kernel<T, false, false>), grid, block, 0, s, d);
}

}  // namespace

hipError_t gemm_f32(const GemmF32Desc& d, hipStream_t s) {
  if (!d.A || !d.B || !d.C || d.M <= 0 || d.N <= 0 || d.K <= 0 || d.ldc < d.N) return hipErrorInvalidValue;
  if ((!d.a_t && d.lda < d.K) || (d.a_t && d.lda < d.M) || (!d.b_t && d.ldb < d.K) || (d.b_t && d.ldb < d.N))
    return hipErrorInvalidValue;
  // 32 x 32 tiles halve the operand reads; with fewer than two per CU the smaller tiles bring more waves
  const long long tiles32 = (long long)((d.M + 31) / 32) * ((d.N + 31) / 32);
  if (tiles32 >= 512) launch<32>(d, s);
  else launch<16>(d, s);
  return hipGetLastError();
}

}  // namespace et
