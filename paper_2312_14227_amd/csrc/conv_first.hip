// First 3x3 convolution of a chain, at most three input channels: all 9 C <= 27 products of an output are two matrix
// instructions, so no column matrix is written (for 32 images of 224x224, 1.6 million rows of 64 bytes: 93 us to write and 77 us for
// the product with 64 channels; 66 - 83 us here, 2.5 - 3.1 TB/s of output where a launch that only writes reaches 5.2.  It is not the gather that is in
// the way: with the window in four wide loads and the next tile's requested ahead of the stores it took 78.  48 and 24 us for 32 channels at stride 2).  A wave owns 32 output pixels at a time; a lane gathers the 8 + 8
// window values of its pixel that the fragments ask for, the weights stay in registers.  The instructions, their order and the
// epilogue are those of the product over the column matrix, and so are the results.
#include "gemm_bf16_kernels.h"

namespace et {
namespace {

using gemm::Params;
using gemm::bf16x8;
using gemm::f32x16;

constexpr int WAVES = 4;

template <int C, int NI, int EPI>
__global__ __launch_bounds__(WAVES * 64) void conv_first_kernel(Params g, int tiles) {
  constexpr int AREA = gemm::epi_wave_bytes<NI * 32>();
  __shared__ __attribute__((aligned(16))) unsigned char smem[WAVES * AREA];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, khalf = lane >> 5;
  const int n0 = blockIdx.y * (NI * 32);
  constexpr int K = 9 * C;
  // weights [N][K], zeros beyond; the window values of this lane as element offsets from its pixel
  bf16x8 wt[2][NI];
  int off[2][8];
#pragma unroll
  for (int ks = 0; ks < 2; ks++)
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const int k = ks * 16 + khalf * 8 + e, tap = k / C, ch = k % C;
      off[ks][e] = k < K ? ((tap / 3 - 1) * g.cW + tap % 3 - 1) * C + ch : 0;
#pragma unroll
      for (int ni = 0; ni < NI; ni++) {
        const int n = n0 + ni * 32 + l32;
        wt[ks][ni][e] = k < K && n < g.N ? g.B[(long long)n * K + k] : (bf16)0.f;
      }
    }
  for (int t = blockIdx.x * WAVES + wave; t < tiles; t += gridDim.x * WAVES) {
    const int m = min(t * 32 + l32, g.M - 1);
    const int wo = m % g.cWo, r = m / g.cWo, ho = r % g.cHo, img = r / g.cHo;
    const int h = ho * g.cS, w = wo * g.cS;
    const int at = ((img * g.cH + h) * g.cW + w) * C;   // (fewer than 2^31 elements in all)
    const auto value = [&](int o) { return *(const bf16*)((const char*)g.A + (size_t)((unsigned)(at + o) * 2u)); };
    bf16x8 a[2];
    if (__all(h > 0 && h + 1 < g.cH && w > 0 && w + 1 < g.cW)) {   // no pixel of the tile at the border: nothing to test
#pragma unroll
      for (int ks = 0; ks < 2; ks++)
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const bf16 v = value(off[ks][e]);
          a[ks][e] = ks * 16 + khalf * 8 + e < K ? v : (bf16)0.f;
        }
    } else {
#pragma unroll
      for (int ks = 0; ks < 2; ks++)
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const int k = ks * 16 + khalf * 8 + e, tap = k / C;
          bf16 v = (bf16)0.f;
          if (k < K && (unsigned)(h + tap / 3 - 1) < (unsigned)g.cH && (unsigned)(w + tap % 3 - 1) < (unsigned)g.cW) v = value(off[ks][e]);
          a[ks][e] = v;
        }
    }
    f32x16 acc[1][NI];
#pragma unroll
    for (int ni = 0; ni < NI; ni++)
#pragma unroll
      for (int i = 0; i < 16; i++) acc[0][ni][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
#pragma unroll
      for (int ni = 0; ni < NI; ni++) acc[0][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wt[ks][ni], a[ks], acc[0][ni], 0, 0, 0);
    gemm::wave_epilogue<EPI, 1, NI>(g, acc, smem + wave * AREA, t * 32, n0, 0, lane);
  }
}

}  // namespace

bool conv_first_supported(int k, int C) { return k == 3 && C >= 1 && 9 * C <= 32; }

hipError_t conv_first(const bf16* x, const bf16* w, const ConvGeom& g, int N, const bf16* gain, const bf16* shift, bf16* z, bf16* y, float lo,
                      float hi, hipStream_t s) {
  const auto al = [](const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; };
  if (!conv_first_supported(g.k, g.C) || g.pad != 1 || (g.stride != 1 && g.stride != 2) || g.B < 1 || g.H < 1 || g.W < 1 || N < 8 || (N & 7) ||
      g.Ho != (g.H - 1) / g.stride + 1 || g.Wo != (g.W - 1) / g.stride + 1 || !x || !w || !shift || !y)
    return hipErrorInvalidValue;
  if (!al(x, 16) || !al(gain, 8) || !al(shift, 8) || !al(z, 16) || !al(y, 16) || (z && !gain)) return hipErrorInvalidValue;
  const long long M = (long long)g.B * g.Ho * g.Wo;
  if (M > 0x7fffffc0ll || (long long)g.B * g.H * g.W * g.C > 0x7fffffffll) return hipErrorInvalidValue;
  Params p{};
  p.A = x; p.B = w; p.M = (int)M; p.N = N; p.K = 9 * g.C; p.ldb = 9 * g.C; p.alpha = 1.f; p.bias = shift; p.gain = gain; p.ldc = N;
  p.C = gain ? z : y; p.C2 = gain ? y : nullptr; p.act_lo = lo; p.act_hi = hi;
  p.cH = g.H; p.cW = g.W; p.cC = g.C; p.cS = g.stride; p.cHo = g.Ho; p.cWo = g.Wo;
  const int tiles = (int)((M + 31) / 32);
  const bool narrow = N <= 32;
  const unsigned wgs = (unsigned)((tiles + WAVES - 1) / WAVES);
  const dim3 grid(wgs < 2048u ? wgs : 2048u, narrow ? 1 : (N + 63) / 64), block(WAVES * 64);
#define ET_CF(C, NI, E) hipLaunchKernelGGL((conv_first_kernel<C, NI, gemm::E>), grid, block, 0, s, p, tiles)
#define ET_CFC(NI, E)                 \
  do {                                \
    if (g.C == 1) ET_CF(1, NI, E);    \
    else if (g.C == 2) ET_CF(2, NI, E); \
    else ET_CF(3, NI, E);             \
  } while (0)
  if (gain && narrow) ET_CFC(1, E_AFFINE);
  else if (gain) ET_CFC(2, E_AFFINE);
  else if (narrow) ET_CFC(1, E_BIAS_RELU);
  else ET_CFC(2, E_BIAS_RELU);
#undef ET_CFC
#undef ET_CF
  return hipGetLastError();
}

}  // namespace et
