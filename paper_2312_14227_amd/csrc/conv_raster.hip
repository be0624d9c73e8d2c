// 3x3 / stride 1 / zero padding 1 convolution of small images with many channels (forward, or gradient passing with the mirrored weight).
//
// What bounds the gathered products on these layers ([32 x 14 x 14 x 256] -> 256: 7.4 GFLOP in 21.5 us) is bringing operands to a CU: a 64 x 64
// tile takes 16 KB per slice of 64 k values, half of it pixels, of which the eight other taps bring 8/9 again, at 10 ns per KB.  Here the pixels of
// 64 input channels lie in LDS once for all nine taps.  The images are laid out as one raster with a column of zeros in front of every row and a
// row of zeros in front of every image, which also serve as the borders behind: position s = (image * (H + 1) + Y) * (W + 1) + X holds pixel
// (Y - 1, X - 1), and the output at raster position p reads p + dy (W + 1) + dx for tap (dy, dx), whatever the width.  A workgroup owns
// 128 positions (those in a zero row or column are not stored: 13 % of them at 14 x 14) and 64 output channels; its window of 128 + 2 (W + 1) + 2
// positions is double buffered over the chunks of 64 input channels, the weights of a (chunk, tap) slice come through a ring of 8 KB
// stages.  Per slice: 8 KB of weights and a ninth of 20 KB of pixels for 128 x 64 x 64 products, 0.10 us of loading for 0.107 us of matrix
// instructions.
// The fragments of 64 x 64 products with 16 k values each are the cheapest that LDS can deliver at that rate (32 KB per slice): eight waves share
// the tile as 2 halves of the positions x 4 quarters of every slice's k values.  The quarters are added through LDS at the end, in two
// exchanges (0.7 us): (q0 + q2) + (q1 + q3).
// Measured at 32 images against the gathered products: 14 x 14 x 256 20.1 -> 13.7 us, 7 x 7 x 512 24.2 -> 19.7, 28 x 28 x 128 19.0 -> 16.1 (256
// positions per workgroup), 14 x 14 x 512 42.8 -> 37.2.  A tap takes 0.186 us (256 positions: 0.306) for 0.107 (0.213) of matrix instructions, with a
// barrier for every tap instead of every third 0.24; the first window, the quarters and the epilogue 5.4 (8.5) us per workgroup.
#include <algorithm>

#include "gemm_bf16_kernels.h"

namespace et {
namespace {

using namespace gemm;

constexpr int BN = 64, TAP_BYTES = BN * 128, STAGE_BYTES = 3 * TAP_BYTES;

struct RasterParams {
  const bf16* x;
  const bf16* w;       // [N][9][C]
  int H, W, C, N, images;
  int tiles_n, units;
  bf16 *out, *out2;
  const bf16 *bias, *gain, *U;
  float lo, hi, mask_hi;
};

// PW: window pieces of 8 positions per wave (the window has at most 64 PW positions)
// MI: 64 MI positions per workgroup
template <int EPI, int MI, int PW>
__global__ __launch_bounds__(512) void conv_raster_kernel(RasterParams g) {
  constexpr int BM = 64 * MI, WINDOW = PW * 8 * 1024, B_AT = 2 * WINDOW, SMEM = B_AT + 3 * STAGE_BYTES;
  static_assert(SMEM >= 8 * MI * 4096 && SMEM <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, khalf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), mh = wave >> 2, kq = wave & 3;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  // the workgroups of one XCD (blockIdx % 8) own consecutive units, the channel blocks of a window next to each other
  const int xcd = (int)blockIdx.x % NUM_XCD, idx = (int)blockIdx.x / NUM_XCD;
  const int per = g.units / NUM_XCD, rem = g.units % NUM_XCD;
  const int unit = xcd * per + min(xcd, rem) + idx;
  const int p0 = unit / g.tiles_n * BM, n0 = unit % g.tiles_n * BN;
  const int W1 = g.W + 1, R = (g.H + 1) * W1;
  const int img0 = p0 / R, s0 = p0 - img0 * R;   // window position i is raster position s0 + i behind the start of image img0
  const float rcp_r = 1.f / (float)R, rcp_w = 1.f / (float)W1;
  // image (behind img0), row and column of a raster position
  auto locate = [&](int s, int& img, int& Y, int& X) {
    int in;
    divmod_small(s, R, rcp_r, img, in);
    divmod_small(in, W1, rcp_w, Y, X);
  };
  const char* xbase = (const char*)(g.x + (long long)img0 * g.H * g.W * g.C);
  const bf16* wbase = g.w + (long long)n0 * 9 * g.C;
  unsigned off_a[PW];   // bytes behind xbase; all ones: zeros
#pragma unroll
  for (int i = 0; i < PW; i++) {
    const int pos = (wave * PW + i) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((pos >> 1) & 7);
    int img, Y, X;
    locate(s0 + pos, img, Y, X);
    const bool ok = Y > 0 && X > 0 && img0 + img < g.images;
    off_a[i] = ok ? (unsigned)(((img * g.H + Y - 1) * g.W + X - 1) * g.C + chunk * 8) * 2u : 0xffffffffu;
  }
  unsigned off_b;
  {
    const int row = wave * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    off_b = (unsigned)(row * 9 * g.C + chunk * 8) * 2u;
  }
  auto request_a = [&](int i, int c) {   // piece i of this wave, channels 64 c ..
    const void* src = off_a[i] != 0xffffffffu ? (const void*)(xbase + off_a[i] + c * 128) : (const void*)kZeroBlock;
    dma16(src, __builtin_amdgcn_readfirstlane(lds0 + (c & 1) * WINDOW + (wave * PW + i) * 1024));
  };
  // the next stage of weights, three taps of a chunk, into the next slot of the ring
  int rc = 0, rt = 0, rs = 0;
  auto request_b = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 3; t++)
      dma16((const char*)(wbase + (rt + t) * g.C + rc * 64) + off_b,
            __builtin_amdgcn_readfirstlane(lds0 + B_AT + rs * STAGE_BYTES + t * TAP_BYTES + wave * 1024));
    rt += 3;
    if (rt == 9) { rt = 0; rc++; }
    rs = rs == 2 ? 0 : rs + 1;
  };
  const int chunks = g.C >> 6, total = chunks * 3;
  const bool more = chunks > 1;
#pragma unroll
  for (int i = 0; i < PW; i++) request_a(i, 0);
  request_b();
  request_b();
  if (more) {
#pragma unroll
    for (int i = 0; i < PW; i++) request_a(i, 1);
  }
  request_b();
  f32x16 acc[MI][2];
#pragma unroll
  for (int mi = 0; mi < MI; mi++)
#pragma unroll
    for (int ni = 0; ni < 2; ni++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[mi][ni][r] = 0.f;

  bf16x8 fa[2][MI], fb[2][2];
  const unsigned char* bfrag = smem + B_AT + l32 * 128 + (((kq * 2 + khalf) ^ ((l32 >> 1) & 7)) << 4);
  int slot = 0;   // of the stage being multiplied
  auto fetch = [&](auto set_tag, int c, int tap, int at) __attribute__((always_inline)) {
    constexpr int set = decltype(set_tag)::value;
    const int pos = mh * (BM / 2) + l32 + tap / 3 * W1 + tap % 3;
    const unsigned char* a = smem + (c & 1) * WINDOW + pos * 128 + (((kq * 2 + khalf) ^ ((pos >> 1) & 7)) << 4);
    const unsigned char* b = bfrag + at * STAGE_BYTES + tap % 3 * TAP_BYTES;
#pragma unroll
    for (int i = 0; i < MI; i++) fa[set][i] = *(const bf16x8*)(a + i * 4096);   // (32 positions or rows on, the chunk's place is the same)
#pragma unroll
    for (int i = 0; i < 2; i++) fb[set][i] = *(const bf16x8*)(b + i * 4096);
  };
  // One tap: its fragments have been fetched a tap ago, those of the next are fetched under its matrix instructions.  Before the last tap of
  // a stage everyone has read all of it: its slot is requested again, for the stage three further on, and after tap 8 the window of
  // the chunk as well, for the one two further on.  What has to have landed by then is the next stage and, for tap 8, the next window; the
  // stage after it (three requests a wave) and, before tap 2, the next window, requested in front of that stage, may still be under way.
  // (The same requests spread over the three taps of a stage: 0.21 instead of 0.186 us per tap.)
  auto tap_step = [&](auto set_tag, int c, auto tap_tag) __attribute__((always_inline)) {
    constexpr int set = decltype(set_tag)::value, TAP = decltype(tap_tag)::value;
    const int u = c * 3 + TAP / 3, after = slot == 2 ? 0 : slot + 1;
    if (TAP % 3 == 2) {
      __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
      if (u + 2 >= total) wait_vmcnt<0>();
      else if (TAP == 2 && c + 1 < chunks) wait_vmcnt<3 + PW>();
      else wait_vmcnt<3>();
      block_barrier();
      if (TAP == 8 && c + 2 < chunks) {
#pragma unroll
        for (int i = 0; i < PW; i++) request_a(i, c + 2);
      }
      if (u + 3 < total) request_b();
    }
    if (TAP < 8 || c + 1 < chunks)
      fetch(std::integral_constant<int, set ^ 1>{}, TAP == 8 ? c + 1 : c, TAP == 8 ? 0 : TAP + 1, TAP % 3 == 2 ? after : slot);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mi = 0; mi < MI; mi++)
#pragma unroll
      for (int ni = 0; ni < 2; ni++) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][ni], fa[set][mi], acc[mi][ni], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (TAP % 3 == 2) slot = after;
  };
  auto chunk = [&](auto set_tag, int c) __attribute__((always_inline)) {
    constexpr std::integral_constant<int, decltype(set_tag)::value ^ 1> other_tag;
    tap_step(set_tag, c, std::integral_constant<int, 0>{});
    tap_step(other_tag, c, std::integral_constant<int, 1>{});
    tap_step(set_tag, c, std::integral_constant<int, 2>{});
    tap_step(other_tag, c, std::integral_constant<int, 3>{});
    tap_step(set_tag, c, std::integral_constant<int, 4>{});
    tap_step(other_tag, c, std::integral_constant<int, 5>{});
    tap_step(set_tag, c, std::integral_constant<int, 6>{});
    tap_step(other_tag, c, std::integral_constant<int, 7>{});
    tap_step(set_tag, c, std::integral_constant<int, 8>{});
  };
  if (more) wait_vmcnt<6 + PW>();
  else wait_vmcnt<6>();
  block_barrier();
  constexpr std::integral_constant<int, 0> even;
  constexpr std::integral_constant<int, 1> odd;
  fetch(even, 0, 0, 0);
  int c = 0;
  for (; c + 1 < chunks; c += 2) {
    chunk(even, c);
    chunk(odd, c + 1);
  }
  if (c < chunks) chunk(even, c);

  // add the quarters: first with quarter kq ^ 2, halves of the positions exchanged, then with kq ^ 1, halves of the channels
  block_barrier();
  {
    constexpr int HALF = MI / 2;
    const int mq = kq >> 1, ni = kq & 1;   // this wave is left with the positions' half mq, the channels' half ni
    int e_tid = tid;   // (lane-dependent values below are not kept in registers through the loop)
    asm volatile("" : "+v"(e_tid));
    const int lane = e_tid & 63, l32 = lane & 31, khalf = lane >> 5;
    const auto put = [&](unsigned char* at, const f32x16& v) {
#pragma unroll
      for (int q = 0; q < 4; q++) *(float4*)(at + q * 1024 + lane * 16) = make_float4(v[q * 4], v[q * 4 + 1], v[q * 4 + 2], v[q * 4 + 3]);
    };
    const auto add = [&](const unsigned char* at, f32x16& v) {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const float4 t = *(const float4*)(at + q * 1024 + lane * 16);
        v[q * 4] += t.x; v[q * 4 + 1] += t.y; v[q * 4 + 2] += t.z; v[q * 4 + 3] += t.w;
      }
    };
    f32x16 keep[HALF][2], sum[HALF];
#pragma unroll
    for (int m = 0; m < HALF; m++)
#pragma unroll
      for (int n = 0; n < 2; n++) {
        put(smem + ((wave * HALF + m) * 2 + n) * 4096, mq ? acc[m][n] : acc[HALF + m][n]);
        keep[m][n] = mq ? acc[HALF + m][n] : acc[m][n];
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    block_barrier();
    unsigned char* mine = smem + (wave ^ 2) * HALF * 8192;   // read by this wave alone from here on
#pragma unroll
    for (int m = 0; m < HALF; m++) {
#pragma unroll
      for (int n = 0; n < 2; n++) add(mine + (m * 2 + n) * 4096, keep[m][n]);
      put(mine + m * 8192, ni ? keep[m][0] : keep[m][1]);
      sum[m] = ni ? keep[m][1] : keep[m][0];
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    block_barrier();
#pragma unroll
    for (int m = 0; m < HALF; m++) add(smem + ((wave ^ 1) ^ 2) * HALF * 8192 + m * 8192, sum[m]);

    // 32 positions x 32 channels at a time: lane l32 holds a position's channels q * 8 + khalf * 4 + 0..3; through LDS (rows of 64 bytes, chunk c at
    // c ^ ((row >> 2) & 3)) to rows of channels
    unsigned char* area = mine + 4096;
    const int col = n0 + ni * 32, c8 = (lane & 3) * 8;
#pragma unroll
    for (int m = 0; m < HALF; m++) {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        bf16x4 o, b = {};
        if (EPI == E_BIAS_RELU) b = *(const bf16x4*)(g.bias + col + q * 8 + khalf * 4);
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const float v = sum[m][q * 4 + j];
          o[j] = (bf16)(EPI == E_BIAS_RELU ? fmaxf(v + (float)b[j], 0.f) : v);
        }
        *(bf16x4*)(area + l32 * 64 + ((q ^ ((l32 >> 2) & 3)) << 4) + khalf * 8) = o;
      }
#pragma unroll
      for (int it = 0; it < 2; it++) {
        const int row = it * 16 + (lane >> 2);
        bf16x8 v = *(const bf16x8*)(area + row * 64 + (((lane & 3) ^ ((row >> 2) & 3)) << 4));
        int img, y, x;
        locate(s0 + mh * (BM / 2) + (mq * HALF + m) * 32 + row, img, y, x);
        if (y >= g.H || x >= g.W || img0 + img >= g.images) continue;
        const long long at = (((long long)(img0 + img) * g.H + y) * g.W + x) * g.N + col + c8;
        if (EPI == E_AFFINE) {
          const bf16x8 gain = *(const bf16x8*)(g.gain + col + c8), shift = *(const bf16x8*)(g.bias + col + c8);
          bf16x8 yv;
#pragma unroll
          for (int j = 0; j < 8; j++) yv[j] = (bf16)fminf(fmaxf((float)v[j] * (float)gain[j] + (float)shift[j], g.lo), g.hi);
          if (g.out) *(bf16x8*)(g.out + at) = v;
          *(bf16x8*)(g.out2 + at) = yv;
        } else {
          if (EPI == E_RELU_MASK) {
            const bf16x8 u = *(const bf16x8*)(g.U + at);
#pragma unroll
            for (int j = 0; j < 8; j++) v[j] = ((float)u[j] > 0.f && (float)u[j] < g.mask_hi) ? v[j] : (bf16)0.f;
          }
          *(bf16x8*)(g.out + at) = v;
        }
      }
    }
  }
}

// tiles of 64 mi positions x 64 channels
long long raster_units(const GemmDesc& d, int mi) {
  const long long positions = (long long)(d.M / (d.conv_h * d.conv_w)) * (d.conv_h + 1) * (d.conv_w + 1);
  return (positions + 64 * mi - 1) / (64 * mi) * (d.N / BN);
}
int raster_window(const GemmDesc& d, int mi) { return 64 * mi + 2 * (d.conv_w + 1) + 2; }

template <int EPI>
void launch(const RasterParams& p, int mi, int window, hipStream_t s) {
  const dim3 grid(p.units), block(512);
  if (mi == 4) hipLaunchKernelGGL((conv_raster_kernel<EPI, 4, 5>), grid, block, 0, s, p);
  else if (window > 192) hipLaunchKernelGGL((conv_raster_kernel<EPI, 2, 4>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((conv_raster_kernel<EPI, 2, 3>), grid, block, 0, s, p);
}

}  // namespace

// A layer that this kernel covers (d.tile says with how many positions per workgroup), the reduction not split
bool conv_raster_takes(const GemmDesc& d) {
  const auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (d.conv_c < 64 || (d.conv_c & 63) || d.conv_c > 8192 || d.conv_taps != 3 || d.conv_stride != 1 || d.a_t || d.b_t || d.split_k > 1 || (d.N & 63) ||
      d.N < 64 || d.K != 9 * d.conv_c || d.ldb != d.K || d.ldc != d.N || d.c_f32 || d.residual || d.alpha != 1.f || d.z_outer != 1 || d.z_inner != 1 ||
      d.colsum)
    return false;
  // the window fits; its raster positions and byte offsets behind its first image are small
  if (d.conv_h < 1 || d.conv_w < 1 || d.conv_h > 1023 || raster_window(d, 2) > 256 ||
      (d.tile == CONV_TILE_RASTER_256 && raster_window(d, 4) > 320) || d.M < 1 || d.M % (d.conv_h * d.conv_w)) return false;
  if ((long long)(d.conv_h * d.conv_w + 512) * d.conv_c * 2 >= (1ll << 31) || raster_units(d, 2) >= (1ll << 23)) return false;
  if (!al(d.A) || !al(d.B) || !al(d.C) || !al(d.C2) || !al(d.bias) || !al(d.gain) || !al(d.U) || !d.A || !d.B) return false;
  switch (d.mode) {
    case EPI_AFFINE_RELU: return d.C2 && d.gain && d.bias;
    case EPI_BIAS_RELU: return d.C && d.bias;
    case EPI_RELU_MASK: return d.C && d.U && !d.bias;
    case EPI_PLAIN: return d.C && !d.bias;
    default: return false;
  }
}

// Where this kernel is the faster one: its tiles fill the chip once.  Every further round costs the latency of its first window and the addition of the
// quarters again, and a single tile per CU has to make up for both: 128-position tiles, 52 tiles of [13 x 13 x 256] 12.2 us against 12.1 of the
// gathered products, 64 of [7 x 7 x 512] 19.6 / 17.0, but 128 of [7 x 7 x 512] 19.7 / 24.2, 228 of [14 x 14 x 256] 13.7 / 20.1, and 284 again
// 24.4 / 20.1; 256-position tiles: 211 of [28 x 28 x 128] 16.1 / 19.0, 228 of [14 x 14 x 512] 37.2 / 42.8, but 142 of [14 x 14 x 256] 20.5 / 20.1.
// At most 512 channels: the gathered products split longer reductions, and are then the faster ones up to 190 tiles (128 tiles of [7 x 7 x 1024] 32.9 /
// 29.7, [4 x 4 x 1024] 33.3 / 25.9) and the more precise ones (chains of 144 products of 16 against 96: a tenth more roundings to the wrong
// neighbour of a bf16 result; at 512 channels a fifth fewer).  Over 370 shapes of 4 x 4 .. 60 x 60 pixels, 64 .. 512 channels and 1 .. 128 images that
// this rule takes, time against the gathered products' by reduction and tiles: 1 chunk of 64 channels 0.83 - 0.93, 2 chunks 0.75 - 0.86, 4 and 8
// chunks 0.66 - 0.86 in the mean; the worst 1.03.
int conv_raster_tile(GemmDesc d) {
  d.split_k = 1;
  d.tile = CONV_TILE_RASTER;
  if (d.conv_c > 512 || !conv_raster_takes(d)) return 0;
  const long long small = raster_units(d, 2), large = raster_units(d, 4);
  if (small <= 256) return small >= 128 ? CONV_TILE_RASTER : 0;
  d.tile = CONV_TILE_RASTER_256;
  return large >= 160 && large <= 256 && conv_raster_takes(d) ? CONV_TILE_RASTER_256 : 0;
}

hipError_t conv_raster(const GemmDesc& d, hipStream_t s) {
  if (!conv_raster_takes(d)) return hipErrorInvalidValue;
  const int mi = d.tile == CONV_TILE_RASTER_256 ? 4 : 2;
  RasterParams p;
  p.x = d.A; p.w = d.B; p.H = d.conv_h; p.W = d.conv_w; p.C = d.conv_c; p.N = d.N; p.images = d.M / (d.conv_h * d.conv_w);
  p.tiles_n = d.N / BN; p.units = (int)raster_units(d, mi);
  p.out = (bf16*)d.C; p.out2 = d.C2; p.bias = d.bias; p.gain = d.gain; p.U = d.U;
  p.lo = d.act_lo; p.hi = d.act_hi; p.mask_hi = d.mask_hi;
  const int window = raster_window(d, mi);
  switch (d.mode) {
    case EPI_AFFINE_RELU: launch<E_AFFINE>(p, mi, window, s); break;
    case EPI_BIAS_RELU: launch<E_BIAS_RELU>(p, mi, window, s); break;
    case EPI_RELU_MASK: launch<E_RELU_MASK>(p, mi, window, s); break;
    default: launch<E_BF16>(p, mi, window, s); break;
  }
  return hipGetLastError();
}

}  // namespace et
