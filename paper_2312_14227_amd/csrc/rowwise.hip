// HBM-bound kernels of the training step: LayerNorm forward/backward, softmax forward/backward,
// cross-entropy, column and batch reductions (bias / LayerNorm gain and shift / embedding
// gradients, Sections 5.1 and 5.2), embedding assembly.  One 64-lane wave owns one row in the
// row-wise kernels; reductions inside a wave use cross-lane shuffles, all sums have a fixed
// order so results are bit-reproducible.
#include "kernels.h"

namespace et {
namespace {

constexpr int WAVE = 64;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, WAVE));
  return v;
}

typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------------------------
// column sums, stage 1: a block of 8 column-threads (8 columns each) x 32 row-threads sums
// cs_rows() rows of 64 columns; stage 2 adds the row-chunk partials in ascending order
// ---------------------------------------------------------------------------------------------
// (narrow matrices, at most 16 or 32 columns, take 2 or 4 column-threads instead, so that no thread is idle)
__host__ __device__ inline int cs_threads(int cols) { return cols <= 16 ? 2 : cols <= 32 ? 4 : 8; }
// rows per chunk: about 2048 workgroups per launch (a multiple of 32 rows, 64 to 1024; 128 rows are a step of the narrow form), so that a tall narrow
// matrix and a short wide one both fill the chip; the same function sizes the partial buffer
__host__ __device__ inline int cs_rows(int rows, int cols) {
  const int cs_cols = cs_threads(cols) * 8;
  const int col_blocks = (cols + cs_cols - 1) / cs_cols;
  const int chunks_wanted = 2048 / col_blocks > 0 ? 2048 / col_blocks : 1;
  int per = ((rows + chunks_wanted - 1) / chunks_wanted + 31) & ~31;
  return per < 64 ? 64 : (per > 1024 ? 1024 : per);
}

template <int CT, bool F32IN, bool XHAT>
__global__ __launch_bounds__(256) void colsum_stage1(const bf16* __restrict__ d16, const float* __restrict__ d32,
                                                     long long d_stride, const float* __restrict__ h,
                                                     long long h_stride, const float* __restrict__ mean,
                                                     const float* __restrict__ rstd, long long stat_stride,
                                                     float* __restrict__ partials, int rows, int cols) {
  constexpr int CS_COLS = CT * 8, RT = 256 / CT;
  __shared__ float red[RT][CS_COLS + 1];
  const int cx = threadIdx.x % CT, ry = threadIdx.x / CT;
  const int c0 = blockIdx.x * CS_COLS + cx * 8;
  const int chunk_rows = cs_rows(rows, cols);
  const int r_begin = blockIdx.y * chunk_rows, r_end = min(rows, r_begin + chunk_rows);
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; j++) acc[j] = 0.f;
  if (c0 < cols) {
    for (int r = r_begin + ry; r < r_end; r += RT) {
      float v[8];
      if (F32IN) {
        const float4 a = *(const float4*)(d32 + (long long)r * d_stride + c0);
        const float4 b = *(const float4*)(d32 + (long long)r * d_stride + c0 + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
      } else {
        const bf16x8 a = *(const bf16x8*)(d16 + (long long)r * d_stride + c0);
#pragma unroll
        for (int j = 0; j < 8; j++) v[j] = (float)a[j];
      }
      if (XHAT) {
        const float mu = mean[r * stat_stride], rs = rstd[r * stat_stride];
        const float4 a = *(const float4*)(h + (long long)r * h_stride + c0);
        const float4 b = *(const float4*)(h + (long long)r * h_stride + c0 + 4);
        v[0] *= (a.x - mu) * rs; v[1] *= (a.y - mu) * rs; v[2] *= (a.z - mu) * rs; v[3] *= (a.w - mu) * rs;
        v[4] *= (b.x - mu) * rs; v[5] *= (b.y - mu) * rs; v[6] *= (b.z - mu) * rs; v[7] *= (b.w - mu) * rs;
      }
#pragma unroll
      for (int j = 0; j < 8; j++) acc[j] += v[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 8; j++) red[ry][cx * 8 + j] = acc[j];
  __syncthreads();
  if (threadIdx.x < CS_COLS) {
    const int c = blockIdx.x * CS_COLS + threadIdx.x;
    if (c < cols) {
      float s = red[0][threadIdx.x];
#pragma unroll
      for (int k = 1; k < RT; k++) s += red[k][threadIdx.x];
      partials[(long long)blockIdx.y * cols + c] = s;
    }
  }
}

// Second step of many column sums at once: a workgroup adds the partial rows of 16 columns of one job, 64 threads per
// four columns taking every 64th row, then in a fixed tree.  One launch for a whole backward pass: as a launch per sum this
// step was 4.7 us each, 100 of them in a full ViT-B step.
constexpr int MAX_JOBS = 120;   // (kernel arguments: 32 bytes each)
struct SumJobs {
  int n;
  SumJob job[MAX_JOBS];
};
__global__ __launch_bounds__(256) void sum_finish_kernel(SumJobs jobs) {
  __shared__ __attribute__((aligned(16))) float red[64][20];
  __shared__ float red2[16][17];
  int lo = 0, hi = jobs.n - 1;   // the job this workgroup belongs to: the last with block0 <= blockIdx.x
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs.job[mid].block0 <= (int)blockIdx.x) lo = mid;
    else hi = mid - 1;
  }
  const SumJob j = jobs.job[lo];
  const int quad = threadIdx.x & 3, part = threadIdx.x >> 2;
  const int c0 = ((int)blockIdx.x - j.block0) * 16 + quad * 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c0 < j.cols) {
#pragma unroll 4
    for (int r = part; r < j.rows; r += 64) {
      const float4 v = *(const float4*)(j.part + (long long)r * j.cols + c0);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
  }
  *(float4*)&red[part][quad * 4] = s;
  __syncthreads();
  const int col = threadIdx.x & 15, grp = threadIdx.x >> 4;
  red2[grp][col] = ((red[grp * 4][col] + red[grp * 4 + 1][col]) + red[grp * 4 + 2][col]) + red[grp * 4 + 3][col];
  __syncthreads();
  const int c = ((int)blockIdx.x - j.block0) * 16 + (int)threadIdx.x;
  if (threadIdx.x < 16 && c < j.cols) {
    float t = red2[0][threadIdx.x];
#pragma unroll
    for (int g = 1; g < 16; g++) t += red2[g][threadIdx.x];
    j.out[c] = t;
  }
}

__global__ void batchsum_kernel(const float* __restrict__ d, float* __restrict__ out, int B, long long batch_stride,
                                int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = d[i];
  for (int b = 1; b < B; b++) s += d[(long long)b * batch_stride + i];
  out[i] = s;
}

// ---------------------------------------------------------------------------------------------
// softmax rows (attention probabilities) and its backward
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void softmax_rows_kernel(const float* __restrict__ s, bf16* __restrict__ p, int rows,
                                                           int cols, int ld) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* x = s + (long long)row * ld;
  bf16* o = p + (long long)row * ld;
  float mx = -INFINITY;
  for (int i = lane; i < cols; i += WAVE) mx = fmaxf(mx, x[i]);
  mx = wave_max(mx);
  float sum = 0.f;
  for (int i = lane; i < cols; i += WAVE) sum += __expf(x[i] - mx);
  const float inv = 1.f / wave_sum(sum);
  for (int i = lane; i < ld; i += WAVE) o[i] = (bf16)(i < cols ? __expf(x[i] - mx) * inv : 0.f);
}

__global__ __launch_bounds__(256) void softmax_bwd_rows_kernel(const float* __restrict__ dp, const bf16* __restrict__ p,
                                                               bf16* __restrict__ ds, float scale, int rows, int cols,
                                                               int ld) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* g = dp + (long long)row * ld;
  const bf16* pr = p + (long long)row * ld;
  bf16* o = ds + (long long)row * ld;
  float dot = 0.f;
  for (int i = lane; i < cols; i += WAVE) dot += g[i] * (float)pr[i];
  dot = wave_sum(dot);
  for (int i = lane; i < ld; i += WAVE) o[i] = (bf16)(i < cols ? scale * (float)pr[i] * (g[i] - dot) : 0.f);
}

// ---------------------------------------------------------------------------------------------
// mean softmax cross-entropy and its gradient: one wave per row (4 rows per block) writes the
// gradient and the row's loss term; a second one-wave kernel adds the terms in ascending order
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void xent_rows_kernel(const float* __restrict__ logits, const int32_t* __restrict__ y,
                                                        int B, int C, float* __restrict__ row_loss,
                                                        float* __restrict__ dl, bf16* __restrict__ dl16, int ld16) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= B) return;
  const float invB = 1.f / (float)B;
  const float* x = logits + (long long)r * C;
  float mx = -INFINITY;
  for (int i = lane; i < C; i += WAVE) mx = fmaxf(mx, x[i]);
  mx = wave_max(mx);
  float sum = 0.f;
  for (int i = lane; i < C; i += WAVE) sum += expf(x[i] - mx);
  sum = wave_sum(sum);
  const float lse = logf(sum) + mx;
  const int label = y[r];
  if (lane == 0) row_loss[r] = lse - x[label];
  for (int i = lane; i < ld16; i += WAVE) {
    float gval = 0.f;
    if (i < C) {
      gval = (expf(x[i] - lse) - (i == label ? 1.f : 0.f)) * invB;
      dl[(long long)r * C + i] = gval;
    }
    if (dl16) dl16[(long long)r * ld16 + i] = (bf16)gval;
  }
}

__global__ __launch_bounds__(64) void xent_loss_kernel(const float* __restrict__ row_loss, int B, float* __restrict__ loss) {
  if (threadIdx.x != 0) return;
  float acc = 0.f;
  for (int r = 0; r < B; r++) acc += row_loss[r];
  *loss = acc / (float)B;
}

// ---------------------------------------------------------------------------------------------
// embedding assembly, CLS-row drop, fill
// ---------------------------------------------------------------------------------------------
__global__ void embed_assemble_kernel(const float* __restrict__ e, const bf16* __restrict__ cls,
                                      const bf16* __restrict__ pos, float* __restrict__ h0, int B, int T, int D) {
  const long long i4 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int d4 = D >> 2;
  if (i4 >= (long long)B * T * d4) return;
  const int c = (int)(i4 % d4) * 4;
  const long long bt = i4 / d4;
  const int t = (int)(bt % T);
  const long long b = bt / T;
  const bf16x4 pv = *(const bf16x4*)(pos + (long long)t * D + c);
  float4 r;
  if (t == 0) {
    const bf16x4 cv = *(const bf16x4*)(cls + c);
    r = make_float4((float)cv[0], (float)cv[1], (float)cv[2], (float)cv[3]);
  } else {
    r = *(const float4*)(e + (b * (T - 1) + (t - 1)) * D + c);
  }
  r.x += (float)pv[0]; r.y += (float)pv[1]; r.z += (float)pv[2]; r.w += (float)pv[3];
  *(float4*)(h0 + bt * D + c) = r;
}

__global__ void gather_patch_rows_kernel(const float* __restrict__ d, bf16* __restrict__ out, int B, int T, int D) {
  const long long i4 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int d4 = D >> 2;
  if (i4 >= (long long)B * (T - 1) * d4) return;
  const int c = (int)(i4 % d4) * 4;
  const long long bp = i4 / d4;
  const int p = (int)(bp % (T - 1));
  const long long b = bp / (T - 1);
  const float4 v = *(const float4*)(d + (b * T + p + 1) * D + c);
  bf16x4 q;
  q[0] = (bf16)v.x; q[1] = (bf16)v.y; q[2] = (bf16)v.z; q[3] = (bf16)v.w;
  *(bf16x4*)(out + bp * D + c) = q;
}

__global__ void fill_zero_kernel(uint4* __restrict__ p, size_t n16, unsigned char* __restrict__ tail, size_t ntail) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
inline bool al8(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7) == 0; }

}  // namespace

int colsum_parts(int rows, int cols) {
  const int per = cs_rows(rows, cols);
  return (rows + per - 1) / per;
}

hipError_t colsum_part(const bf16* d, const float* d_f32, long long d_stride, const float* h, long long h_stride, const float* mean,
                       const float* rstd, long long stat_stride, float* part, int rows, int cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0 || (cols & 7) || (d_stride & 7) || (h && (h_stride & 3)) || (!d && !d_f32) || !part) return hipErrorInvalidValue;
  if ((d && !al16(d)) || (d_f32 && !al16(d_f32)) || (h && !al16(h)) || !al16(part)) return hipErrorInvalidValue;
  const int ct = cs_threads(cols);
  const dim3 grid((cols + ct * 8 - 1) / (ct * 8), colsum_parts(rows, cols)), block(256);
#define ET_CT(CT, F32IN, XHAT) \
  hipLaunchKernelGGL((colsum_stage1<CT, F32IN, XHAT>), grid, block, 0, s, d, d_f32, d_stride, h, h_stride, mean, rstd, stat_stride, part, rows, cols)
#define ET_CS(F32IN, XHAT)                      \
  do {                                          \
    if (ct == 2) ET_CT(2, F32IN, XHAT);         \
    else if (ct == 4) ET_CT(4, F32IN, XHAT);    \
    else ET_CT(8, F32IN, XHAT);                 \
  } while (0)
  if (d_f32) {
    if (h) ET_CS(true, true);
    else ET_CS(true, false);
  } else {
    if (h) ET_CS(false, true);
    else ET_CS(false, false);
  }
#undef ET_CS
#undef ET_CT
  return hipGetLastError();
}

hipError_t sum_finish(SumJob* jobs, int n, hipStream_t s, int* launches) {
  *launches = 0;
  for (int i = 0; i < n; i += MAX_JOBS) {
    SumJobs a;
    a.n = n - i < MAX_JOBS ? n - i : MAX_JOBS;
    int blocks = 0;
    for (int k = 0; k < a.n; k++) {
      a.job[k] = jobs[i + k];
      if (!a.job[k].part || !a.job[k].out || a.job[k].rows < 1 || a.job[k].cols < 4 || (a.job[k].cols & 3) || !al16(a.job[k].part))
        return hipErrorInvalidValue;
      a.job[k].block0 = blocks;
      blocks += (a.job[k].cols + 15) / 16;
    }
    hipLaunchKernelGGL(sum_finish_kernel, dim3(blocks), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    (*launches)++;
  }
  return hipSuccess;
}

hipError_t batchsum(const float* d, float* out, int B, long long batch_stride, int n, hipStream_t s) {
  if (B <= 0 || n <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(batchsum_kernel, dim3((n + 255) / 256), dim3(256), 0, s, d, out, B, batch_stride, n);
  return hipGetLastError();
}

hipError_t softmax_rows(const float* sc, bf16* p, int rows, int cols, int ld, hipStream_t s) {
  if (rows <= 0 || cols <= 0 || ld < cols) return hipErrorInvalidValue;
  hipLaunchKernelGGL(softmax_rows_kernel, dim3((rows + 3) / 4), dim3(256), 0, s, sc, p, rows, cols, ld);
  return hipGetLastError();
}

hipError_t softmax_bwd_rows(const float* dp, const bf16* p, bf16* ds, float scale, int rows, int cols, int ld,
                            hipStream_t s) {
  if (rows <= 0 || cols <= 0 || ld < cols) return hipErrorInvalidValue;
  hipLaunchKernelGGL(softmax_bwd_rows_kernel, dim3((rows + 3) / 4), dim3(256), 0, s, dp, p, ds, scale, rows, cols, ld);
  return hipGetLastError();
}

hipError_t xent(const float* logits, const int32_t* y, int B, int C, float* loss, float* dlogits, bf16* dlogits_bf16,
                int ld16, hipStream_t s) {
  if (B <= 0 || C <= 0 || ld16 < C) return hipErrorInvalidValue;
  float* row_loss = loss + 64;
  hipLaunchKernelGGL(xent_rows_kernel, dim3((B + 3) / 4), dim3(256), 0, s, logits, y, B, C, row_loss, dlogits,
                     dlogits_bf16, ld16);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(xent_loss_kernel, dim3(1), dim3(64), 0, s, row_loss, B, loss);
  return hipGetLastError();
}

hipError_t embed_assemble(const float* e, const bf16* cls, const bf16* pos, float* h0, int B, int T, int D,
                          hipStream_t s) {
  if ((D & 3) || !al16(e) || !al8(cls) || !al8(pos) || !al16(h0)) return hipErrorInvalidValue;
  const long long n = (long long)B * T * (D / 4);
  hipLaunchKernelGGL(embed_assemble_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, e, cls, pos, h0, B, T, D);
  return hipGetLastError();
}

hipError_t gather_patch_rows(const float* d, bf16* out, int B, int T, int D, hipStream_t s) {
  if ((D & 3) || !al16(d) || !al8(out)) return hipErrorInvalidValue;
  const long long n = (long long)B * (T - 1) * (D / 4);
  hipLaunchKernelGGL(gather_patch_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d, out, B, T, D);
  return hipGetLastError();
}

hipError_t fill_zero(void* p, size_t bytes, hipStream_t s) {
  if (!al16(p)) return hipErrorInvalidValue;
  if (bytes == 0) return hipSuccess;
  const size_t n16 = bytes / 16, ntail = bytes % 16;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)p, n16,
                     (unsigned char*)p + n16 * 16, ntail);
  return hipGetLastError();
}

}  // namespace et
