// Backward of a per-channel affine y = act(z * gain + shift) on NHWC rows [M][C], in one pass over the gradient:
//   m = ((d + add) where the activation is open), rounded to bf16 as a stored tensor would be;
//   sums over the rows of m (shift) and of m * z (gain), and m * gain for the convolution in front of the affine.
// Bound by HBM and, on small maps, by latency.  The masking and the shortcut's addend used to be a pass of their own (read d, add,
// y, write m); here they cost at most the addend's read: where z is at hand the activation's openness is computed from it, with
// the expression and rounding of the forward pass, and y is not read.
// A workgroup is cw groups of 8 channels x pw rows, cw = C / 8 wherever that is at most 32, so that neighbouring rows follow
// without a gap and no thread idles (C = 96, 144: 1.5 and 2.25 blocks of 64 columns before).  One row per thread and
// step: four loaded at a time are no faster on large maps ([401408 x 96], three passes: 49.3 and 50.9 us = 4.7 TB/s) and, with four
// times the code and a quarter of the workgroups, slower on small ones ([1014 x 1024] with the mask 3.6 and 5.1 us).
// The order of a sum depends on rows and C only, not on which of the outputs are wanted.
#include <algorithm>

#include "kernels.h"

namespace et {
namespace {

typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

struct Plan { int cw, pw, tiles, per, chunks; };

// About 1024 workgroups (four per CU).
Plan plan_of(long long rows, int cols) {
  Plan p;
  const int c8n = cols >> 3;
  p.cw = std::min(c8n, 32);
  if (c8n > 32)
    for (int q = 32; q > 16; q--)
      if (c8n % q == 0) { p.cw = q; break; }
  p.pw = 256 / p.cw;
  p.tiles = (c8n + p.cw - 1) / p.cw;
  const int wanted = std::max(1, 1024 / p.tiles);
  p.per = (int)((rows + (long long)wanted * p.pw - 1) / ((long long)wanted * p.pw) * p.pw);
  p.chunks = (int)((rows + p.per - 1) / p.per);
  return p;
}

enum Mask : int { OPEN = 0, FROM_Y = 1, FROM_Z = 2 };
enum Z : int { NO_Z = 0, Z_BF16 = 1, Z_F32 = 2 };

template <int MASK, int ZK, bool ADD>
__global__ __launch_bounds__(256) void affine_back_kernel(AffineBack a, Plan pl) {
  __shared__ __attribute__((aligned(16))) float red[2][256 * 8];
  __shared__ float part[2][256];
  const int c = threadIdx.x % pl.cw, p = threadIdx.x / pl.cw;
  const int tile = blockIdx.x % pl.tiles, chunk = blockIdx.x / pl.tiles;
  const int c0 = (tile * pl.cw + c) * 8;
  const int r_begin = chunk * pl.per, r_end = min(a.rows, r_begin + pl.per);
  const bool on = p < pl.pw && c0 < a.cols;
  float sum[8], mul[8];
#pragma unroll
  for (int j = 0; j < 8; j++) sum[j] = mul[j] = 0.f;
  if (on) {
    bf16x8 gn = {}, sh = {};   // (widened where they are used: the first rows are requested before these have arrived)
    if (MASK == FROM_Z || a.dout) gn = *(const bf16x8*)(a.gain + c0);
    if (MASK == FROM_Z) sh = *(const bf16x8*)(a.shift + c0);
    for (int r = r_begin + p; r < r_end; r += pl.pw) {
      const long long at = (long long)r * a.cols + c0;
      const bf16x8 d = *(const bf16x8*)(a.d + at);
      bf16x8 b = {}, y = {}, z = {}, m, o;
      float zf[8];
      if (ADD) b = *(const bf16x8*)(a.add + at);
      if (MASK == FROM_Y) y = *(const bf16x8*)(a.y + at);
      if (ZK == Z_BF16) z = *(const bf16x8*)(a.z + at);
      if (ZK == Z_F32) {
        *(float4*)zf = *(const float4*)(a.z32 + at);
        *(float4*)(zf + 4) = *(const float4*)(a.z32 + at + 4);
      }
#pragma unroll
      for (int j = 0; j < 8; j++) {
        const float zz = ZK == Z_F32 ? zf[j] : (float)z[j];
        bf16 v = d[j];
        if (ADD) v = (bf16)((float)v + (float)b[j]);
        if (MASK != OPEN) {
          const float act = MASK == FROM_Y ? (float)y[j] : (float)(bf16)fminf(fmaxf(fmaf(zz, (float)gn[j], (float)sh[j]), 0.f), a.hi);
          if (!(act > 0.f && act < a.hi)) v = (bf16)0.f;
        }
        const float vf = (float)v;
        sum[j] += vf;
        if (ZK != NO_Z) mul[j] = fmaf(vf, zz, mul[j]);
        m[j] = v;
        o[j] = (bf16)(vf * (float)gn[j]);
      }
      if (a.dmid) *(bf16x8*)(a.dmid + at) = m;
      if (a.dout) *(bf16x8*)(a.dout + at) = o;
    }
  }
  if (!a.part_sum && !a.part_mul) return;
  // rows of the workgroup, then groups of rows, added in ascending order
  const int n = pl.cw * 8, groups = 256 / n, grp = threadIdx.x / n, o = threadIdx.x % n;
  if (p < pl.pw) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      *(float4*)&red[0][p * n + c * 8 + h * 4] = make_float4(sum[h * 4], sum[h * 4 + 1], sum[h * 4 + 2], sum[h * 4 + 3]);
      if (ZK != NO_Z) *(float4*)&red[1][p * n + c * 8 + h * 4] = make_float4(mul[h * 4], mul[h * 4 + 1], mul[h * 4 + 2], mul[h * 4 + 3]);
    }
  }
  __syncthreads();
  float s = 0.f, t = 0.f;
  if (grp < groups)
#pragma unroll 4
    for (int k = grp; k < pl.pw; k += groups) {
      s += red[0][k * n + o];
      if (ZK != NO_Z) t += red[1][k * n + o];
    }
  part[0][threadIdx.x] = s;
  if (ZK != NO_Z) part[1][threadIdx.x] = t;
  __syncthreads();
  const int col = tile * n + o;
  if (grp == 0 && col < a.cols) {
    for (int k = 1; k < groups; k++) {
      s += part[0][k * n + o];
      if (ZK != NO_Z) t += part[1][k * n + o];
    }
    if (a.part_sum) a.part_sum[(long long)chunk * a.cols + col] = s;
    if (ZK != NO_Z && a.part_mul) a.part_mul[(long long)chunk * a.cols + col] = t;
  }
}

}  // namespace

int affine_back_parts(int rows, int cols) { return plan_of(rows, cols).chunks; }

hipError_t affine_back_part(const AffineBack& a, hipStream_t s) {
  if (a.rows <= 0 || a.cols <= 0 || (a.cols & 7) || !a.d || (!a.part_sum && !a.part_mul && !a.dout && !a.dmid)) return hipErrorInvalidValue;
  const bool need_z = a.part_mul != nullptr || a.mask_from_z;
  if (need_z && !a.z && !a.z32) return hipErrorInvalidValue;
  if ((a.dout || a.mask_from_z) && (!a.gain || !al16(a.gain))) return hipErrorInvalidValue;
  if (a.mask_from_z && (!a.z || a.y || !a.shift || !al16(a.shift))) return hipErrorInvalidValue;
  if (a.z32 && (a.z || a.y || a.add)) return hipErrorInvalidValue;   // (the stem's affine: nothing joins there)
  for (const void* p : {(const void*)a.d, (const void*)a.add, (const void*)a.y, (const void*)a.z, (const void*)a.z32, (const void*)a.dmid,
                        (const void*)a.dout, (const void*)a.part_sum, (const void*)a.part_mul})
    if (!al16(p)) return hipErrorInvalidValue;
  const Plan pl = plan_of(a.rows, a.cols);
  const dim3 grid((unsigned)(pl.tiles * pl.chunks));
  const int mask = a.mask_from_z ? FROM_Z : a.y ? FROM_Y : OPEN, zk = !need_z ? NO_Z : a.z32 ? Z_F32 : Z_BF16;
#define ET_AB(M, K, ADD) \
  if (mask == M && zk == K && (a.add != nullptr) == ADD) hipLaunchKernelGGL((affine_back_kernel<M, K, ADD>), grid, dim3(256), 0, s, a, pl)
  ET_AB(OPEN, NO_Z, false);
  ET_AB(OPEN, NO_Z, true);
  ET_AB(OPEN, Z_BF16, false);
  ET_AB(OPEN, Z_BF16, true);
  ET_AB(OPEN, Z_F32, false);
  ET_AB(FROM_Y, NO_Z, false);
  ET_AB(FROM_Y, NO_Z, true);
  ET_AB(FROM_Y, Z_BF16, false);
  ET_AB(FROM_Y, Z_BF16, true);
  ET_AB(FROM_Z, Z_BF16, false);
  ET_AB(FROM_Z, Z_BF16, true);
#undef ET_AB
  return hipGetLastError();
}

}  // namespace et
