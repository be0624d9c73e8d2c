// 3x3 depthwise convolution (zero padding 1, stride 1 or 2) on NHWC bf16, weights [C][9]: no reduction over channels,
// nothing for a matrix unit, bound by HBM.
//   forward  z = sum over taps (fp32), stored rounded; y = clamp(z * gain + shift, 0, 6) from the rounded z;
//   dx       input gradient in gather form, then + add, times the ReLU6 mask of the activation in front of the convolution;
//   dw       partial sums of d * x, one row per workgroup, finished by the column sum of the rows.
// A workgroup is cw groups of 4 channels x pw strips; a strip is one column of `seg` output rows that a thread walks down with
// its 3 x 3 window and its 36 weights (or sums) in registers.  A step of stride 1 loads three new pixels instead of nine, one
// step ahead of their use; the window's rows change roles with period 3, so the loop is written for three steps and nothing is
// moved.  The weights come through LDS: read by every thread for itself they are 144-byte strides, 64 lines per
// instruction, more work for the memory pipe than all the pixels of a short strip.
// 32 images, before (one pixel per thread; weight gradient: 65 536 workers, each leaving its own 72 sums, 19 MB per
// layer) and now, in us: forward 112x112x32 32 -> 17.6, 56x56x144 35 -> 18, 14x14x576 13 -> 7.6; dx 112x112x96 stride 2
// 64 -> 31 (5.6 TB/s), 56x56x144 38 -> 18; dw with the column sum 85 -> 20, 100 -> 21, 35 -> 11.6.  Small maps stay bound by
// the few steps in flight.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace et {
namespace {

typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

struct DwGeom { int B, H, W, C, stride, Ho, Wo; };
struct DwPlan { int cw, pw, tiles, seg, nseg; long long strips; };
struct F4 { float v[4]; };

__device__ __forceinline__ F4 widen(const bf16x4& a) {
  F4 r;
#pragma unroll
  for (int j = 0; j < 4; j++) r.v[j] = (float)a[j];
  return r;
}
// pixels w0 .. w0 + N - 1 of row h, 4 channels; zeros outside the image
template <int N>
__device__ __forceinline__ void load_row(const bf16* __restrict__ base, int h, int w0, int H, int W, int C, bf16x4 (&r)[N]) {
  const bool in = (unsigned)h < (unsigned)H;
  const long long at = ((long long)h * W + w0) * C;
#pragma unroll
  for (int k = 0; k < N; k++) {
    r[k] = bf16x4{};
    if (in && (unsigned)(w0 + k) < (unsigned)W) r[k] = *(const bf16x4*)(base + at + k * C);
  }
}
template <int N>
__device__ __forceinline__ void widen_row(const bf16x4 (&a)[N], F4 (&r)[N]) {
#pragma unroll
  for (int k = 0; k < N; k++) r[k] = widen(a[k]);
}
template <int I> using Idx = std::integral_constant<int, I>;
// calls step(top, mid, bot, ho) for rows h0 .. h1 - 1, the arguments being the places of the window's three rows
template <int S, typename F>
__device__ __forceinline__ void walk(int h0, int h1, F step) {
  for (int ho = h0; ho < h1; ho += 3) {
    step(Idx<0>(), Idx<1>(), Idx<2>(), ho);
    if (S == 1) {
      if (ho + 1 < h1) step(Idx<1>(), Idx<2>(), Idx<0>(), ho + 1);
      if (ho + 2 < h1) step(Idx<2>(), Idx<0>(), Idx<1>(), ho + 2);
    } else {   // the bottom row of a step is the top row of the next
      if (ho + 1 < h1) step(Idx<2>(), Idx<0>(), Idx<1>(), ho + 1);
      if (ho + 2 < h1) step(Idx<1>(), Idx<2>(), Idx<0>(), ho + 2);
    }
  }
}
struct Strip { int w, h0, h1; long long b; };
__device__ __forceinline__ Strip strip_of(long long i, const DwGeom& g, const DwPlan& p) {
  Strip s;
  s.w = (int)(i % g.Wo);
  i /= g.Wo;
  s.h0 = (int)(i % p.nseg) * p.seg;
  s.h1 = min(g.Ho, s.h0 + p.seg);
  s.b = i / p.nseg;
  return s;
}
// 36 weights of the thread's 4 channels, through LDS; MIRROR: in reverse order of the taps
template <bool MIRROR>
__device__ __forceinline__ void load_weights(const bf16* __restrict__ w, int c0, int n, int c, F4 (&wt)[9]) {
  __shared__ __attribute__((aligned(16))) bf16 lw[48 * 36];
  for (int i = threadIdx.x; i < n * 9; i += 256) *(bf16x4*)(lw + i * 4) = *(const bf16x4*)(w + (long long)c0 * 9 + i * 4);
  __syncthreads();
  bf16x4 raw[9];
#pragma unroll
  for (int k = 0; k < 9; k++) raw[k] = *(const bf16x4*)(lw + c * 36 + k * 4);
#pragma unroll
  for (int t = 0; t < 9; t++)
#pragma unroll
    for (int j = 0; j < 4; j++) wt[MIRROR ? 8 - t : t].v[j] = (float)raw[(j * 9 + t) >> 2][(j * 9 + t) & 3];
}
// + addend (zeros if none), rounded, times the mask
__device__ __forceinline__ bf16x4 finish_dx(const F4& acc, const bf16x4& add4, bool masked, const bf16x4& mk) {
  bf16x4 r;
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const bf16 v = (bf16)(acc.v[j] + (float)add4[j]);
    r[j] = !masked || ((float)mk[j] > 0.f && (float)mk[j] < 6.f) ? v : (bf16)0.f;
  }
  return r;
}

// MODE 0: forward (a = x, p0 = gain, p1 = shift, out0 = z nullable, out1 = y); MODE 1: input gradient of stride 1, i.e. the same
// convolution of d with mirrored taps (a = d, p0 = addend nullable, p1 = ReLU6 output nullable, out1 = result)
template <int S, int MODE>
__global__ __launch_bounds__(256) void depthwise_strip_kernel(const bf16* __restrict__ a, const bf16* __restrict__ w, const bf16* __restrict__ p0,
                                                              const bf16* __restrict__ p1, bf16* __restrict__ out0, bf16* __restrict__ out1, DwGeom g,
                                                              DwPlan pl) {
  const int c = threadIdx.x % pl.cw, p = threadIdx.x / pl.cw, n = min(pl.cw, (g.C >> 2) - (int)(blockIdx.x % pl.tiles) * pl.cw);
  const int c0 = (int)(blockIdx.x % pl.tiles) * pl.cw * 4, c4 = c0 + c * 4;
  F4 wt[9];
  load_weights<MODE == 1>(w, c0, n, c, wt);
  const long long i = (long long)(blockIdx.x / pl.tiles) * pl.pw + p;
  if (p >= pl.pw || c >= n || i >= pl.strips) return;
  F4 gn, sh;
  if (MODE == 0) {
    gn = widen(*(const bf16x4*)(p0 + c4));
    sh = widen(*(const bf16x4*)(p1 + c4));
  }
  const Strip s = strip_of(i, g, pl);
  const bf16* base = a + s.b * g.H * (long long)g.W * g.C + c4;
  const int w0 = s.w * S - 1;
  const long long step_at = (long long)g.Wo * g.C;
  long long at = ((s.b * g.Ho + s.h0) * g.Wo + s.w) * (long long)g.C + c4;
  F4 win[3][3];
  bf16x4 nm[3], nb[3], na = {}, nk = {};     // one step ahead: (stride 2: middle and) bottom row, addend, mask
  {
    bf16x4 r0[3], r1[3];
    load_row(base, s.h0 * S - 1, w0, g.H, g.W, g.C, r0);
    load_row(base, s.h0 * S, w0, g.H, g.W, g.C, r1);
    load_row(base, s.h0 * S + 1, w0, g.H, g.W, g.C, nb);
    if (MODE == 1 && p0) na = *(const bf16x4*)(p0 + at);
    if (MODE == 1 && p1) nk = *(const bf16x4*)(p1 + at);
    widen_row(r0, win[0]);
    if (S == 1) widen_row(r1, win[1]);
    else
#pragma unroll
      for (int k = 0; k < 3; k++) nm[k] = r1[k];
  }
  walk<S>(s.h0, s.h1, [&](auto top_, auto mid_, auto bot_, int ho) {
    constexpr int top = decltype(top_)::value, mid = decltype(mid_)::value, bot = decltype(bot_)::value;
    if (S == 2) widen_row(nm, win[mid]);
    widen_row(nb, win[bot]);
    const bf16x4 add4 = na, mk4 = nk;
    if (ho + 1 < s.h1) {
      if (S == 2) load_row(base, ho * 2 + 2, w0, g.H, g.W, g.C, nm);
      load_row(base, (ho + 1) * S + 1, w0, g.H, g.W, g.C, nb);
      if (MODE == 1 && p0) na = *(const bf16x4*)(p0 + at + step_at);
      if (MODE == 1 && p1) nk = *(const bf16x4*)(p1 + at + step_at);
    }
    F4 acc = {};   // taps of w in ascending order in either direction
#pragma unroll
    for (int t = 0; t < 9; t++) {
      const int at_w = MODE == 1 ? 8 - t : t, ky = at_w / 3, k = at_w % 3;
      const F4& px = win[ky == 0 ? top : ky == 1 ? mid : bot][k];
#pragma unroll
      for (int j = 0; j < 4; j++) acc.v[j] = fmaf(px.v[j], wt[at_w].v[j], acc.v[j]);
    }
    if (MODE == 0) {
      bf16x4 z4, r;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        z4[j] = (bf16)acc.v[j];
        r[j] = (bf16)fminf(fmaxf((float)z4[j] * gn.v[j] + sh.v[j], 0.f), 6.f);
      }
      if (out0) *(bf16x4*)(out0 + at) = z4;
      *(bf16x4*)(out1 + at) = r;
    } else {
      *(bf16x4*)(out1 + at) = finish_dx(acc, add4, p1 != nullptr, mk4);
    }
    at += step_at;
  });
}

// input gradient of stride 2: output pixel (ho, wo) owns the four input pixels (2 ho, 2 ho + 1) x (2 wo, 2 wo + 1), which lie in
// one, two, two and four windows; a strip walks down ho with rows ho and ho + 1 of d in registers
__global__ __launch_bounds__(256) void depthwise_dx2_kernel(const bf16* __restrict__ d, const bf16* __restrict__ w, const bf16* __restrict__ add,
                                                            const bf16* __restrict__ mask, bf16* __restrict__ out, DwGeom g, DwPlan pl) {
  const int c = threadIdx.x % pl.cw, p = threadIdx.x / pl.cw, n = min(pl.cw, (g.C >> 2) - (int)(blockIdx.x % pl.tiles) * pl.cw);
  const int c0 = (int)(blockIdx.x % pl.tiles) * pl.cw * 4, c4 = c0 + c * 4;
  F4 wt[9];
  load_weights<false>(w, c0, n, c, wt);
  const long long i = (long long)(blockIdx.x / pl.tiles) * pl.pw + p;
  if (p >= pl.pw || c >= n || i >= pl.strips) return;
  const Strip s = strip_of(i, g, pl);
  const bf16* base = d + s.b * g.Ho * (long long)g.Wo * g.C + c4;
  const bool right = 2 * s.w + 1 < g.W;
  bf16x4 t[2], b[2];
  load_row(base, s.h0, s.w, g.Ho, g.Wo, g.C, t);
  for (int ho = s.h0; ho < s.h1; ho++) {
    const long long at = ((s.b * g.H + 2 * ho) * g.W + 2 * s.w) * (long long)g.C + c4, down = (long long)g.W * g.C;
    const bool low = 2 * ho + 1 < g.H, has[4] = {true, right, low, low && right};
    load_row(base, ho + 1, s.w, g.Ho, g.Wo, g.C, b);
    bf16x4 ad[4], mk[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      ad[q] = mk[q] = bf16x4{};
      const long long o = at + (q & 1) * g.C + (q >> 1) * down;
      if (add && has[q]) ad[q] = *(const bf16x4*)(add + o);
      if (mask && has[q]) mk[q] = *(const bf16x4*)(mask + o);
    }
    F4 t0 = widen(t[0]), t1 = widen(t[1]), b0 = widen(b[0]), b1 = widen(b[1]), acc[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      acc[0].v[j] = t0.v[j] * wt[4].v[j];
      acc[1].v[j] = fmaf(t0.v[j], wt[5].v[j], t1.v[j] * wt[3].v[j]);
      acc[2].v[j] = fmaf(t0.v[j], wt[7].v[j], b0.v[j] * wt[1].v[j]);
      acc[3].v[j] = fmaf(t0.v[j], wt[8].v[j], fmaf(t1.v[j], wt[6].v[j], fmaf(b0.v[j], wt[2].v[j], b1.v[j] * wt[0].v[j])));
    }
#pragma unroll
    for (int q = 0; q < 4; q++)
      if (has[q]) *(bf16x4*)(out + at + (q & 1) * g.C + (q >> 1) * down) = finish_dx(acc[q], ad[q], mask != nullptr, mk[q]);
    t[0] = b[0];
    t[1] = b[1];
  }
}

// Weight gradient: every thread adds d * x over its strips, the workgroup adds its threads' sums in LDS, three taps at a time
// and in a fixed order, and leaves one row [C * 9].
template <int S>
__global__ __launch_bounds__(256) void depthwise_dw_kernel(const bf16* __restrict__ d, const bf16* __restrict__ x, float* __restrict__ part, DwGeom g,
                                                           DwPlan pl) {
  __shared__ __attribute__((aligned(16))) float red[256 * 12];
  __shared__ float red2[256];
  const int c = threadIdx.x % pl.cw, p = threadIdx.x / pl.cw, c0 = (int)(blockIdx.x % pl.tiles) * pl.cw * 4, c4 = c0 + c * 4;
  F4 acc[9] = {};
  if (p < pl.pw && c4 < g.C) {
    for (long long i = (long long)(blockIdx.x / pl.tiles) * pl.pw + p; i < pl.strips; i += (long long)(gridDim.x / pl.tiles) * pl.pw) {
      const Strip s = strip_of(i, g, pl);
      const bf16* base = x + s.b * g.H * (long long)g.W * g.C + c4;
      const int w0 = s.w * S - 1;
      const long long step_at = (long long)g.Wo * g.C;
      const bf16* dp = d + ((s.b * g.Ho + s.h0) * g.Wo + s.w) * (long long)g.C + c4;
      F4 win[3][3];
      bf16x4 nm[3], nb[3], nd = *(const bf16x4*)dp;
      {
        bf16x4 r0[3], r1[3];
        load_row(base, s.h0 * S - 1, w0, g.H, g.W, g.C, r0);
        load_row(base, s.h0 * S, w0, g.H, g.W, g.C, r1);
        load_row(base, s.h0 * S + 1, w0, g.H, g.W, g.C, nb);
        widen_row(r0, win[0]);
        if (S == 1) widen_row(r1, win[1]);
        else
#pragma unroll
          for (int k = 0; k < 3; k++) nm[k] = r1[k];
      }
      walk<S>(s.h0, s.h1, [&](auto top_, auto mid_, auto bot_, int ho) {
        constexpr int top = decltype(top_)::value, mid = decltype(mid_)::value, bot = decltype(bot_)::value;
        if (S == 2) widen_row(nm, win[mid]);
        widen_row(nb, win[bot]);
        const F4 dv = widen(nd);
        dp += step_at;
        if (ho + 1 < s.h1) {
          if (S == 2) load_row(base, ho * 2 + 2, w0, g.H, g.W, g.C, nm);
          load_row(base, (ho + 1) * S + 1, w0, g.H, g.W, g.C, nb);
          nd = *(const bf16x4*)dp;
        }
#pragma unroll
        for (int k = 0; k < 3; k++)
#pragma unroll
          for (int j = 0; j < 4; j++) {
            acc[k].v[j] = fmaf(dv.v[j], win[top][k].v[j], acc[k].v[j]);
            acc[3 + k].v[j] = fmaf(dv.v[j], win[mid][k].v[j], acc[3 + k].v[j]);
            acc[6 + k].v[j] = fmaf(dv.v[j], win[bot][k].v[j], acc[6 + k].v[j]);
          }
      });
    }
  }
  const int n = pl.cw * 12, groups = max(1, 256 / n), grp = threadIdx.x / n;
  float* row = part + (long long)(blockIdx.x / pl.tiles) * g.C * 9;
#pragma unroll
  for (int t = 0; t < 3; t++) {
    if (p < pl.pw)
#pragma unroll
      for (int k = 0; k < 3; k++) {
        const F4& q = acc[3 * t + k];
        *(float4*)(red + p * n + (k * pl.cw + c) * 4) = make_float4(q.v[0], q.v[1], q.v[2], q.v[3]);
      }
    __syncthreads();
    if (groups > 1) {
      const int o = threadIdx.x % n;
      float s = 0.f;
      if (grp < groups)
        for (int k = grp; k < pl.pw; k += groups) s += red[k * n + o];
      red2[threadIdx.x] = s;
      __syncthreads();
    }
    const float* from = groups > 1 ? red2 : red;
    for (int o = threadIdx.x; o < n; o += 256) {
      float s = 0.f;
      for (int k = 0; k < (groups > 1 ? groups : pl.pw); k++) s += from[k * n + o];
      const int tap = 3 * t + o / (pl.cw * 4), ch = c0 + o % (pl.cw * 4);
      if (ch < g.C) row[ch * 9 + tap] = s;
    }
    __syncthreads();
  }
}

bool dw_geom(DwGeom& g, int B, int H, int W, int C, int stride) {
  if (B < 1 || H < 1 || W < 1 || C < 8 || (C & 7) || (stride != 1 && stride != 2)) return false;
  g.B = B; g.H = H; g.W = W; g.C = C; g.stride = stride;
  g.Ho = (H - 1) / stride + 1;
  g.Wo = (W - 1) / stride + 1;
  return true;
}
// Channel groups of a workgroup: 16 (a 128-byte line per pixel) where that divides C / 4, or else all up to 48, so that
// neighbouring pixels follow without a gap (56x56x144 forward: 24.6 us with 12 groups, 20.8 with 36); beyond, the largest divisor
// that is above 16, or 16 and a tail of idle threads.  Strips as long as there are `threads` in all, at most 16 rows (the two
// more rows that a strip reads are then an eighth).  Threads asked for, total of ten layers of 32 images: forward + dx 350 us at
// 60 000, 321 at 100 000, 316 at 150 000, 334 at 300 000; dw 226 at 50 000 with four workgroups per CU, 234 with three, 312 at
// 200 000 with six (more rows of sums to write and add).
DwPlan dw_plan(const DwGeom& g, long long threads) {
  DwPlan p;
  const int c4n = g.C >> 2;
  p.cw = c4n % 16 ? std::min(c4n, 48) : 16;
  while (p.cw > 16 && c4n % p.cw) p.cw--;
  p.pw = 256 / p.cw;
  p.tiles = (c4n + p.cw - 1) / p.cw;
  const long long per_row = (long long)g.B * g.Wo * c4n;
  const long long nseg = std::min<long long>(g.Ho, std::max<long long>(1, (threads + per_row - 1) / per_row));
  p.seg = (int)std::max<long long>(1, std::min<long long>(16, g.Ho / nseg));
  p.nseg = (g.Ho + p.seg - 1) / p.seg;
  p.strips = (long long)g.B * p.nseg * g.Wo;
  return p;
}
DwPlan dw_plan_sums(const DwGeom& g) { return dw_plan(g, 50000); }
// workgroups over the strips of a weight gradient: four per CU
int dw_chunks(const DwPlan& p) {
  return (int)std::max<long long>(1, std::min<long long>((p.strips + p.pw - 1) / p.pw, 1024 / p.tiles));
}

}  // namespace

hipError_t depthwise3x3_fwd(const bf16* x, const bf16* w, const bf16* gain, const bf16* shift, bf16* z, bf16* y, int B, int H,
                            int W, int C, int stride, hipStream_t s) {
  DwGeom g;
  if (!dw_geom(g, B, H, W, C, stride) || !al16(x) || !al16(w) || !al16(gain) || !al16(shift) || (z && !al16(z)) || !al16(y))
    return hipErrorInvalidValue;
  const DwPlan p = dw_plan(g, 150000);
  const long long wgs = (p.strips + p.pw - 1) / p.pw * p.tiles;
  if (wgs > 0xfffffe) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs);
  if (stride == 1)
    hipLaunchKernelGGL((depthwise_strip_kernel<1, 0>), grid, dim3(256), 0, s, x, w, gain, shift, z, y, g, p);
  else
    hipLaunchKernelGGL((depthwise_strip_kernel<2, 0>), grid, dim3(256), 0, s, x, w, gain, shift, z, y, g, p);
  return hipGetLastError();
}

hipError_t depthwise3x3_dx(const bf16* d, const bf16* w, const bf16* add, const bf16* relu6_y, bf16* out, int B, int H, int W,
                           int C, int stride, hipStream_t s) {
  DwGeom g;
  if (!dw_geom(g, B, H, W, C, stride) || !al16(d) || !al16(w) || (add && !al16(add)) || (relu6_y && !al16(relu6_y)) || !al16(out))
    return hipErrorInvalidValue;
  const DwPlan p = dw_plan(g, 150000);
  const long long wgs = (p.strips + p.pw - 1) / p.pw * p.tiles;
  if (wgs > 0xfffffe) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs);
  if (stride == 1)
    hipLaunchKernelGGL((depthwise_strip_kernel<1, 1>), grid, dim3(256), 0, s, d, w, add, relu6_y, nullptr, out, g, p);
  else
    hipLaunchKernelGGL(depthwise_dx2_kernel, grid, dim3(256), 0, s, d, w, add, relu6_y, out, g, p);
  return hipGetLastError();
}

int depthwise3x3_dw_rows(int B, int H, int W, int C, int stride) {
  DwGeom g;
  return dw_geom(g, B, H, W, C, stride) ? dw_chunks(dw_plan_sums(g)) : 0;
}

hipError_t depthwise3x3_dw(const bf16* d, const bf16* x, float* part, int B, int H, int W, int C, int stride, hipStream_t s) {
  DwGeom g;
  if (!dw_geom(g, B, H, W, C, stride) || !al16(d) || !al16(x) || !al16(part)) return hipErrorInvalidValue;
  const DwPlan p = dw_plan_sums(g);
  const dim3 grid((unsigned)(p.tiles * dw_chunks(p)));
  if (stride == 1)
    hipLaunchKernelGGL((depthwise_dw_kernel<1>), grid, dim3(256), 0, s, d, x, part, g, p);
  else
    hipLaunchKernelGGL((depthwise_dw_kernel<2>), grid, dim3(256), 0, s, d, x, part, g, p);
  return hipGetLastError();
}

}  // namespace et
