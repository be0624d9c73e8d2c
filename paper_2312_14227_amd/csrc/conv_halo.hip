// 3x3 / stride 1 / zero padding 1 convolution of 64 input channels (forward, or gradient passing with the mirrored weight): the input is read
// once per tile into LDS, with its border, instead of once per tap through the L2.
//
// What bounds the gathered products on these layers is the operand traffic: every pixel's 128 bytes travel nine times from the L2 ([224 x 224 x 64]
// -> 64 at 32 images: 1.85 GB of gathered rows, and as much again of weights that every tile reads anew, for 205 MB of input, 256 us), and the
// reduction is only nine slices long.  Here a workgroup owns 8 x 32 output pixels and 64 output channels at a time: 10 x 34 input
// pixels (43 KB) come straight to LDS, pixels outside the image from a
// block of zeros, while the tile before them is computed from the other buffer.  The 64 x 576 weights stay in registers for all the tiles of a
// resident workgroup: a wave owns 2 rows of 32 pixels and 32 channels, i.e. 36 fragments of 16 k values, 144 registers, so that LDS delivers
// two fragments of pixels for three matrix instructions and nothing else.  The sums run over taps, then channels, in the order of the gathered
// products that are not split: the same bits.
// Measured at 32 images, against the gathered products: [224 x 224 x 64] -> 64 channels 256 -> 119 us (410 MB in and out, 3.4 TB/s; the floor of the
// matrix cores is 45 us), [112 x 112 x 64] -> 128 124 -> 68 us, [56 x 56 x 64] -> 64 23.7 -> 15.2 us.  With all the waves storing and requesting at the
// same time, and the weights loaded straight into registers, 124, 74 and 21 us.
#include <algorithm>

#include "gemm_bf16_kernels.h"

namespace et {
namespace {

using namespace gemm;

constexpr int TH = 8, TW = 32, HW = TW + 2, HPIX = (TH + 2) * HW;          // tile, halo
constexpr int PIECES = (HPIX + 7) / 8, PER_WAVE = (PIECES + 3) / 4;        // wave-wide loads of 8 pixels, by the four waves of a group
constexpr int HALO_BYTES = PIECES * 1024, STAGE_BYTES = 2048, WEIGHT_BYTES = 64 * 9 * 128;
// two halos and the waves' staging areas; the weights pass through everything but the first halo before the first tile
constexpr int LDS_BYTES = HALO_BYTES + (HALO_BYTES + 8 * STAGE_BYTES > WEIGHT_BYTES ? HALO_BYTES + 8 * STAGE_BYTES : WEIGHT_BYTES);

struct HaloParams {
  const bf16* x;
  const bf16* w;       // [N][9][64]
  int H, W, N, images;
  int tiles_x, tiles_y, tiles;   // per image, in all
  bf16 *C, *C2;
  const bf16 *bias, *gain, *U;
  float lo, hi, mask_hi;
};

template <int EPI>
__global__ __launch_bounds__(512) void conv_halo_kernel(HaloParams g) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS_BYTES];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, khalf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pg = wave >> 1, og = wave & 1, group = wave >> 2;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  // workgroup b works on channel block b % blocks and every (gridDim.x / blocks)-th tile
  const int blocks = g.N >> 6, n0 = ((int)blockIdx.x % blocks) * 64 + og * 32, stride = (int)gridDim.x / blocks;
  int tile = (int)blockIdx.x / blocks;
  if (tile >= g.tiles) return;

  // the halo of a tile into buffer `buf`, by the second group's waves: position p of the halo at 128 p, its 16-byte chunk c at c ^ ((p >> 1) & 7)
  auto request = [&](int t, int buf) {
    const int per = g.tiles_x * g.tiles_y, img = t / per, in = t - img * per, ty = in / g.tiles_x, tx = in - ty * g.tiles_x;
    const int y0 = ty * TH - 1, x0 = tx * TW - 1;
    const bf16* base = g.x + (((long long)img * g.H + y0) * g.W + x0) * 64;   // of the halo's corner: only offset into, where the pixel exists
    int s_lane = lane;
    asm volatile("" : "+v"(s_lane));
#pragma unroll
    for (int i = 0; i < PER_WAVE; i++) {
      const int q = (wave & 3) + i * 4;
      if (q < PIECES) {   // uniform
        const int p = q * 8 + (s_lane >> 3), chunk = (s_lane & 7) ^ ((p >> 1) & 7);
        const int hy = (p * 241) >> 13, hx = p - hy * HW;   // p / 34 for p < 344
        const bool ok = p < HPIX && (unsigned)(y0 + hy) < (unsigned)g.H && (unsigned)(x0 + hx) < (unsigned)g.W;
        const bf16* src = ok ? base + (__mul24(hy, g.W) + hx) * 64 + chunk * 8 : (const bf16*)kZeroBlock;
        dma16(src, __builtin_amdgcn_readfirstlane(lds0 + buf * HALO_BYTES + q * 1024));
      }
    }
  };
  // weights of the 64 channels, as they lie in memory, through LDS behind the first halo: tap t of channel r at 128 (9 r + t), its 16-byte chunk
  // c at c ^ ((r >> 1) & 7); straight into registers a load would touch 32 rows of 1152 bytes
  {
    const bf16* w = g.w + (long long)(n0 - og * 32) * 576;
#pragma unroll
    for (int i = 0; i < 9; i++) {
      const int at = (wave * 9 + i) * 8 + (lane >> 3), chunk = (lane & 7) ^ (((at / 9) >> 1) & 7);
      dma16(w + at * 64 + chunk * 8, __builtin_amdgcn_readfirstlane(lds0 + HALO_BYTES + (wave * 9 + i) * 1024));
    }
  }
  if (group) request(tile, 0);
  wait_vmcnt<0>();
  block_barrier();
  // this wave's 32 channels: k-step s = tap * 4 + ks covers channels 16 ks .. 16 ks + 15 of a tap
  bf16x8 wf[36];
  {
    const int r = og * 32 + l32;
    const unsigned char* w = smem + HALO_BYTES + r * 1152;
#pragma unroll
    for (int s = 0; s < 36; s++) wf[s] = *(const bf16x8*)(w + (s >> 2) * 128 + ((((s & 3) * 2 + khalf) ^ ((r >> 1) & 7)) << 4));
  }
  // parameters of the channels a lane stores: 8 of them in row order (affine), 4 per register quadruple (bias)
  const int c8 = (lane & 3) * 8, r4 = lane >> 2;   // read-back: 16 pixels per instruction, 4 lanes of 16 bytes each
  bf16x8 gain = {}, shift = {};
  bf16x4 bias_q[4] = {};
  if (EPI == E_AFFINE) {
    gain = *(const bf16x8*)(g.gain + n0 + c8);
    shift = *(const bf16x8*)(g.bias + n0 + c8);
  }
  if (EPI == E_BIAS_RELU) {
#pragma unroll
    for (int q = 0; q < 4; q++) bias_q[q] = *(const bf16x4*)(g.bias + n0 + q * 8 + khalf * 4);
  }
  unsigned char* area = smem + 2 * HALO_BYTES + wave * STAGE_BYTES;
  f32x16 acc[2];
  auto store = [&](int t) {
    const int per = g.tiles_x * g.tiles_y, img = t / per, in = t - img * per, ty = in / g.tiles_x, tx = in - ty * g.tiles_x;
#pragma unroll
    for (int mi = 0; mi < 2; mi++) {
      const int y = ty * TH + pg * 2 + mi, xb = tx * TW;
      if (y >= g.H) continue;   // uniform
      // lane: pixel l32, channels q * 8 + khalf * 4 + 0..3; through LDS (rows of 64 bytes, chunk c at c ^ ((row >> 2) & 3)) to rows of channels
#pragma unroll
      for (int q = 0; q < 4; q++) {
        bf16x4 o;
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const float v = acc[mi][q * 4 + j];
          o[j] = (bf16)(EPI == E_BIAS_RELU ? fmaxf(v + (float)bias_q[q][j], 0.f) : v);
        }
        *(bf16x4*)(area + l32 * 64 + ((q ^ ((l32 >> 2) & 3)) << 4) + khalf * 8) = o;
      }
#pragma unroll
      for (int it = 0; it < 2; it++) {
        const int row = it * 16 + r4, xx = xb + row;
        bf16x8 v = *(const bf16x8*)(area + row * 64 + (((lane & 3) ^ ((row >> 2) & 3)) << 4));
        if (xx >= g.W) continue;
        const long long at = (((long long)img * g.H + y) * g.W + xx) * g.N + n0 + c8;
        if (EPI == E_AFFINE) {
          bf16x8 yv;
#pragma unroll
          for (int j = 0; j < 8; j++) yv[j] = (bf16)fminf(fmaxf((float)v[j] * (float)gain[j] + (float)shift[j], g.lo), g.hi);
          if (g.C) *(bf16x8*)(g.C + at) = v;
          *(bf16x8*)(g.C2 + at) = yv;
        } else {
          if (EPI == E_RELU_MASK) {
            const bf16x8 u = *(const bf16x8*)(g.U + at);
#pragma unroll
            for (int j = 0; j < 8; j++) v[j] = ((float)u[j] > 0.f && (float)u[j] < g.mask_hi) ? v[j] : (bf16)0.f;
          }
          *(bf16x8*)(g.C + at) = v;
        }
      }
    }
  };
  // The two waves of a SIMD (one of each group) take turns: the second group requests the next halo and stores the tile before while the first
  // one multiplies, and multiplies while the first one stores.
  int before = -1;
  for (int buf = 0; tile < g.tiles; tile += stride, buf ^= 1) {
    // everyone's share of this tile's halo has landed, and everyone is done with the other buffer
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    block_barrier();
    if (group) {
      if (tile + stride < g.tiles) request(tile + stride, buf ^ 1);
      if (before >= 0) store(before);
    }
    const unsigned char* halo = smem + buf * HALO_BYTES;
#pragma unroll
    for (int mi = 0; mi < 2; mi++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[mi][r] = 0.f;
    // Input row r of the wave's four feeds output row 0 as tap row r and output row 1 as tap row r - 1, from the same fragments; those of the next
    // (r, dx) are fetched under the current multiplications.  (Addresses from an opaque copy of the lane: recomputed per tile.)
    int t_l32 = l32;
    asm volatile("" : "+v"(t_l32));
    bf16x8 a[2][4];
    auto fetch = [&](int step, bf16x8 (&f)[4]) {
      const int p = (pg * 2 + step / 3) * HW + step % 3 + t_l32;
      const int at = p * 128 + ((khalf ^ ((p >> 1) & 7)) << 4);
#pragma unroll
      for (int ks = 0; ks < 4; ks++) f[ks] = *(const bf16x8*)(halo + (at ^ (ks << 5)));
    };
    fetch(0, a[0]);
#pragma unroll
    for (int step = 0; step < 12; step++) {
      const int r = step / 3, dx = step % 3;
      __builtin_amdgcn_sched_barrier(0);
      if (step < 11) fetch(step + 1, a[(step + 1) & 1]);
#pragma unroll
      for (int ks = 0; ks < 4; ks++) {
        if (r < 3) acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[(r * 3 + dx) * 4 + ks], a[step & 1][ks], acc[0], 0, 0, 0);
        if (r > 0) acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[((r - 1) * 3 + dx) * 4 + ks], a[step & 1][ks], acc[1], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (group) wait_vmcnt<0>();   // the next halo has landed
    else store(tile);
    before = tile;
  }
  if (group && before >= 0) store(before);
}

}  // namespace

// A layer that these tiles cover: the plan does not split its reduction, at least two thirds of the tiles' pixels lie in the image, and all
// accesses are aligned.
bool conv_halo_takes(const GemmDesc& d) {
  const auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (d.conv_c != 64 || d.conv_taps != 3 || d.conv_stride != 1 || d.a_t || d.b_t || d.split_k > 1 || (d.N & 63) || d.N < 64 || d.K != 576 || d.ldb != 576 ||
      d.ldc != d.N || d.c_f32 || d.residual || d.alpha != 1.f || d.z_outer != 1 || d.z_inner != 1 || d.colsum)
    return false;
  if (d.conv_h < 1 || d.conv_w < 1 || d.conv_h > 4095 || d.conv_w > 4095 || d.M < 1 || d.M % (d.conv_h * d.conv_w)) return false;
  if (!al(d.A) || !al(d.B) || !al(d.C) || !al(d.C2) || !al(d.bias) || !al(d.gain) || !al(d.U) || !d.A || !d.B) return false;
  if (d.mode == EPI_AFFINE_RELU) {
    if (!d.C2 || !d.gain || !d.bias) return false;
  } else if (!d.C || (d.mode == EPI_PLAIN && d.bias) || (d.mode == EPI_BIAS_RELU && !d.bias) || (d.mode == EPI_RELU_MASK && (!d.U || d.bias)) ||
             (d.mode != EPI_PLAIN && d.mode != EPI_BIAS_RELU && d.mode != EPI_RELU_MASK)) {
    return false;
  }
  const long long covered = (long long)((d.conv_h + TH - 1) / TH * TH) * ((d.conv_w + TW - 1) / TW * TW);
  return 3ll * d.conv_h * d.conv_w >= 2 * covered;
}

// Where these tiles are the faster ones: a workgroup's first tile waits for the weights and for a halo (8 us in all), and there is one workgroup per
// CU.  84 tiles ([6 x 50 x 50]) take 8.3 us here and 8 us as gathered products, 448 tiles ([32 x 56 x 56]) 15.2 and 23.7 us.  Over 597 shapes of 8 x 32 ..
// 224 x 224 pixels, 64 .. 512 channels and 1 .. 96 images that the rule takes, 0.68 of the gathered products' time in the mean; those of 128 .. 160 tiles
// 0.81, none slower.
bool conv_halo_pays(const GemmDesc& d) {
  if (!conv_halo_takes(d)) return false;
  const long long tiles = (long long)(d.M / (d.conv_h * d.conv_w)) * ((d.conv_h + TH - 1) / TH) * ((d.conv_w + TW - 1) / TW);
  return tiles * (d.N / 64) >= 128;
}

hipError_t conv_halo(const GemmDesc& d, hipStream_t s) {
  if (!conv_halo_takes(d)) return hipErrorInvalidValue;
  HaloParams p;
  p.x = d.A; p.w = d.B; p.H = d.conv_h; p.W = d.conv_w; p.N = d.N; p.images = d.M / (d.conv_h * d.conv_w);
  p.tiles_x = (p.W + TW - 1) / TW; p.tiles_y = (p.H + TH - 1) / TH;
  const long long tiles = (long long)p.images * p.tiles_x * p.tiles_y;
  if (tiles >= (1ll << 30)) return hipErrorInvalidValue;
  p.tiles = (int)tiles;
  p.C = (bf16*)d.C; p.C2 = d.C2; p.bias = d.bias; p.gain = d.gain; p.U = d.U;
  p.lo = d.act_lo; p.hi = d.act_hi; p.mask_hi = d.mask_hi;
  // one workgroup per CU, the same number of tiles for each
  const int blocks = p.N / 64, cus = compute_units();
  const int most = std::max(1, cus / blocks);
  const int rounds = (p.tiles + most - 1) / most, per_block = (p.tiles + rounds - 1) / rounds;
  const dim3 grid(per_block * blocks), block(512);
  switch (d.mode) {
    case EPI_AFFINE_RELU: hipLaunchKernelGGL((conv_halo_kernel<E_AFFINE>), grid, block, 0, s, p); break;
    case EPI_BIAS_RELU: hipLaunchKernelGGL((conv_halo_kernel<E_BIAS_RELU>), grid, block, 0, s, p); break;
    case EPI_RELU_MASK: hipLaunchKernelGGL((conv_halo_kernel<E_RELU_MASK>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((conv_halo_kernel<E_BF16>), grid, block, 0, s, p); break;
  }
  return hipGetLastError();
}

}  // namespace et
