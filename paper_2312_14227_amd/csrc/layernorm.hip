// LayerNorm forward and backward.  One 64-lane wave owns one row and holds it in registers (V float4 per lane, rows of up to
// V * 256 elements, lanes beyond the end idle); reductions inside a wave use cross-lane shuffles, all sums have a fixed order.
//
// The backward kernel produces everything that hangs on the same reads: the input gradient joined by the residual
// branch, and, where asked for, the column sums that are the gradients of the gain, the shift and the bias whose
// gradient stream this is (the projection or second MLP bias in front of the LayerNorm's input).  It is bound by HBM
// (16 bytes per element); the three sums as kernels of their own read 20 more and cost two launches each.
#include "kernels.h"

namespace et {
namespace {

constexpr int WAVE = 64;
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

// out = (h - mean) * rstd * gain + shift, statistics in fp32 (two passes over the registers)
template <int V>
__global__ __launch_bounds__(256) void layernorm_fwd_kernel(const float* __restrict__ h, long long in_stride, const bf16* __restrict__ gain,
                                                            const bf16* __restrict__ shift, float eps, bf16* __restrict__ out,
                                                            float* __restrict__ mean, float* __restrict__ rstd, int rows, int D) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, n4 = D >> 2;
  if (row >= rows) return;
  const float4* x = (const float4*)(h + (long long)row * in_stride);
  float4 v[V];
  bf16x4 g[V], b[V];
#pragma unroll
  for (int j = 0; j < V; j++) {
    const int i = lane + j * WAVE;
    v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < n4) {
      v[j] = x[i];
      g[j] = ((const bf16x4*)gain)[i];
      b[j] = ((const bf16x4*)shift)[i];
    }
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < V; j++) s += (v[j].x + v[j].y) + (v[j].z + v[j].w);
  const float mu = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < V; j++) {
    if (lane + j * WAVE >= n4) continue;
    const float a = v[j].x - mu, bb = v[j].y - mu, c = v[j].z - mu, d = v[j].w - mu;
    q += (a * a + bb * bb) + (c * c + d * d);
  }
  const float rs = 1.f / sqrtf(wave_sum(q) / (float)D + eps);
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
  bf16x4* o = (bf16x4*)(out + (long long)row * D);
#pragma unroll
  for (int j = 0; j < V; j++) {
    if (lane + j * WAVE >= n4) continue;
    bf16x4 r;
    r[0] = (bf16)((v[j].x - mu) * rs * (float)g[j][0] + (float)b[j][0]);
    r[1] = (bf16)((v[j].y - mu) * rs * (float)g[j][1] + (float)b[j][1]);
    r[2] = (bf16)((v[j].z - mu) * rs * (float)g[j][2] + (float)b[j][2]);
    r[3] = (bf16)((v[j].w - mu) * rs * (float)g[j][3] + (float)b[j][3]);
    o[lane + j * WAVE] = r;
  }
}

// with xhat = (h - mean) * rstd, t = d * gain:  dh = skip + rstd * (t - mean(t) - xhat * mean(t * xhat))
// SUMS: workgroup w leaves its rows' sums of d * xhat, d and dh in row w of part_gain, part_shift, part_bias
template <int V, bool SUMS>
__global__ __launch_bounds__(SUMS ? 512 : 256) void layernorm_bwd_kernel(LayerNormBwd a) {
  constexpr int NW = SUMS ? 8 : 4;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n4 = a.D >> 2;
  float4 sg[SUMS ? V : 1], ss[SUMS ? V : 1], sb[SUMS ? V : 1];
#pragma unroll
  for (int j = 0; j < (SUMS ? V : 1); j++) sg[j] = ss[j] = sb[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int row = blockIdx.x * NW + wave; row < a.rows; row += gridDim.x * NW) {
    const float4* x = (const float4*)(a.h + (long long)row * a.h_stride);
    const bf16x4* d4 = (const bf16x4*)(a.d + (long long)row * a.d_stride);
    const bool with_skip = a.skip && (a.skip_period <= 1 || row % a.skip_period == 0);
    const float4* sk = (const float4*)(a.skip + (long long)row * a.out_stride);
    float4 v[V], k[V];
    bf16x4 dv[V], g[V];
#pragma unroll
    for (int j = 0; j < V; j++) {
      const int i = lane + j * WAVE;
      k[j] = v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int e = 0; e < 4; e++) dv[j][e] = g[j][e] = (bf16)0.f;
      if (i < n4) {
        v[j] = x[i];
        dv[j] = d4[i];
        g[j] = ((const bf16x4*)a.gain)[i];
        if (with_skip) k[j] = sk[i];
      }
    }
    const float mu = a.mean[(long long)row * a.stat_stride], rs = a.rstd[(long long)row * a.stat_stride];
    float t[V][4];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < V; j++) {   // (v becomes xhat; the idle lanes' values are multiplied by zeros)
      v[j].x = (v[j].x - mu) * rs; v[j].y = (v[j].y - mu) * rs; v[j].z = (v[j].z - mu) * rs; v[j].w = (v[j].w - mu) * rs;
#pragma unroll
      for (int e = 0; e < 4; e++) t[j][e] = (float)dv[j][e] * (float)g[j][e];
      s1 += (t[j][0] + t[j][1]) + (t[j][2] + t[j][3]);
      s2 += (t[j][0] * v[j].x + t[j][1] * v[j].y) + (t[j][2] * v[j].z + t[j][3] * v[j].w);
    }
    const float m1 = wave_sum(s1) / (float)a.D, m2 = wave_sum(s2) / (float)a.D;
    float4* o = (float4*)(a.dh + (long long)row * a.out_stride);
    bf16x4* o16 = (bf16x4*)(a.dh16 + (long long)row * a.out_stride);
#pragma unroll
    for (int j = 0; j < V; j++) {
      if (lane + j * WAVE >= n4) continue;
      float4 r;
      r.x = rs * (t[j][0] - m1 - v[j].x * m2) + k[j].x;
      r.y = rs * (t[j][1] - m1 - v[j].y * m2) + k[j].y;
      r.z = rs * (t[j][2] - m1 - v[j].z * m2) + k[j].z;
      r.w = rs * (t[j][3] - m1 - v[j].w * m2) + k[j].w;
      o[lane + j * WAVE] = r;
      bf16x4 q;
      q[0] = (bf16)r.x; q[1] = (bf16)r.y; q[2] = (bf16)r.z; q[3] = (bf16)r.w;
      o16[lane + j * WAVE] = q;
      if (SUMS) {
        const float d0 = (float)dv[j][0], d1 = (float)dv[j][1], d2 = (float)dv[j][2], d3 = (float)dv[j][3];
        float4 &G = sg[SUMS ? j : 0], &S = ss[SUMS ? j : 0], &B = sb[SUMS ? j : 0];
        G.x += d0 * v[j].x; G.y += d1 * v[j].y; G.z += d2 * v[j].z; G.w += d3 * v[j].w;
        S.x += d0; S.y += d1; S.z += d2; S.w += d3;
        B.x += r.x; B.y += r.y; B.z += r.z; B.w += r.w;
      }
    }
  }
  if constexpr (SUMS) {
    // the eight waves' sums meet in LDS, one of the three at a time, and are added in wave order
    __shared__ float4 red[NW][V * WAVE];
    auto leave = [&](const float4 (&s)[SUMS ? V : 1], float* part) {
      if (!part) return;
#pragma unroll
      for (int j = 0; j < V; j++) red[wave][lane + j * WAVE] = s[SUMS ? j : 0];
      __syncthreads();
      for (int i = threadIdx.x; i < n4; i += 512) {
        float4 u = red[0][i];
#pragma unroll
        for (int w = 1; w < NW; w++) { const float4 y = red[w][i]; u.x += y.x; u.y += y.y; u.z += y.z; u.w += y.w; }
        ((float4*)(part + (long long)blockIdx.x * a.D))[i] = u;
      }
      __syncthreads();
    };
    leave(sg, a.part_gain);
    leave(ss, a.part_shift);
    leave(sb, a.part_bias);
  }
}

// rows of more than 2048 elements: the same formulas, the row read from memory in every pass
__global__ __launch_bounds__(256) void layernorm_fwd_any_kernel(const float* __restrict__ h, long long in_stride, const bf16* __restrict__ gain,
                                                                const bf16* __restrict__ shift, float eps, bf16* __restrict__ out,
                                                                float* __restrict__ mean, float* __restrict__ rstd, int rows, int D) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* x = h + (long long)row * in_stride;
  float s = 0.f;
  for (int i = lane; i < D; i += WAVE) s += x[i];
  const float mu = wave_sum(s) / (float)D;
  float q = 0.f;
  for (int i = lane; i < D; i += WAVE) q += (x[i] - mu) * (x[i] - mu);
  const float rs = 1.f / sqrtf(wave_sum(q) / (float)D + eps);
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
  for (int i = lane; i < D; i += WAVE) out[(long long)row * D + i] = (bf16)((x[i] - mu) * rs * (float)gain[i] + (float)shift[i]);
}
__global__ __launch_bounds__(256) void layernorm_bwd_any_kernel(LayerNormBwd a) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= a.rows) return;
  const float* x = a.h + (long long)row * a.h_stride;
  const bf16* d = a.d + (long long)row * a.d_stride;
  const bool with_skip = a.skip && (a.skip_period <= 1 || row % a.skip_period == 0);
  const float mu = a.mean[(long long)row * a.stat_stride], rs = a.rstd[(long long)row * a.stat_stride];
  float s1 = 0.f, s2 = 0.f;
  for (int i = lane; i < a.D; i += WAVE) {
    const float t = (float)d[i] * (float)a.gain[i];
    s1 += t;
    s2 += t * ((x[i] - mu) * rs);
  }
  const float m1 = wave_sum(s1) / (float)a.D, m2 = wave_sum(s2) / (float)a.D;
  for (int i = lane; i < a.D; i += WAVE) {
    const long long o = (long long)row * a.out_stride + i;
    const float r = rs * ((float)d[i] * (float)a.gain[i] - m1 - (x[i] - mu) * rs * m2) + (with_skip ? a.skip[o] : 0.f);
    a.dh[o] = r;
    a.dh16[o] = (bf16)r;
  }
}

inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
inline bool al8(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 7) == 0; }

template <int V>
void launch_bwd(const LayerNormBwd& a, hipStream_t s) {
  if (a.part_gain || a.part_shift || a.part_bias)
    hipLaunchKernelGGL((layernorm_bwd_kernel<V, true>), dim3(layernorm_bwd_parts(a.rows)), dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((layernorm_bwd_kernel<V, false>), dim3((a.rows + 3) / 4), dim3(256), 0, s, a);
}

}  // namespace

hipError_t layernorm_fwd(const float* h, long long in_stride, const bf16* gain, const bf16* shift, float eps, bf16* out,
                         float* mean, float* rstd, int rows, int D, hipStream_t s) {
  if (rows <= 0 || D <= 0 || (D & 3) || (in_stride & 3) || !al16(h) || !al8(gain) || !al8(shift) || !al8(out))
    return hipErrorInvalidValue;
  const dim3 grid((rows + 3) / 4), block(256);
  switch ((D + 255) / 256) {
#define ET_LN(V) \
    case V: hipLaunchKernelGGL(layernorm_fwd_kernel<V>, grid, block, 0, s, h, in_stride, gain, shift, eps, out, mean, rstd, rows, D); break;
    ET_LN(1) ET_LN(2) ET_LN(3) ET_LN(4) ET_LN(5) ET_LN(6) ET_LN(7) ET_LN(8)
#undef ET_LN
    default: hipLaunchKernelGGL(layernorm_fwd_any_kernel, grid, block, 0, s, h, in_stride, gain, shift, eps, out, mean, rstd, rows, D);
  }
  return hipGetLastError();
}

// two workgroups of eight rows at a time per CU; fewer rows, fewer workgroups
int layernorm_bwd_parts(int rows) { return rows >= 512 * 8 ? 512 : (rows + 7) / 8; }

hipError_t layernorm_bwd(const LayerNormBwd& a, hipStream_t s) {
  if (a.rows <= 0 || a.D <= 0 || (a.D & 3) || (a.d_stride & 3) || (a.h_stride & 3) || (a.out_stride & 3) ||
      !al16(a.h) || !al8(a.d) || !al8(a.gain) || !al16(a.dh) || !a.dh16 || !al8(a.dh16) || (a.skip && !al16(a.skip)) || !al16(a.part_gain) ||
      !al16(a.part_shift) || !al16(a.part_bias))
    return hipErrorInvalidValue;
  switch ((a.D + 255) / 256) {
#define ET_LN(V) case V: launch_bwd<V>(a, s); break;
    ET_LN(1) ET_LN(2) ET_LN(3) ET_LN(4) ET_LN(5) ET_LN(6) ET_LN(7) ET_LN(8)
#undef ET_LN
    default:
      if (a.part_gain || a.part_shift || a.part_bias) return hipErrorInvalidValue;   // (LAYERNORM_SUMS_MAX_D)
      hipLaunchKernelGGL(layernorm_bwd_any_kernel, dim3((a.rows + 3) / 4), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace et
