// Instantiations of the ring bf16 GEMM kernel's implicit convolutions with eight waves (see gemm_bf16_ring.h).
#include "gemm_bf16_ring.h"

namespace et {
namespace gemm {
namespace {

template <int BM, int BN, int WGM, int WGN, int E, int CONV>
hipError_t launch(const Params& p, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WGM, WGN, 3, CONV == 2, CONV == 2, E, CONV>), grid, dim3(512), 0, s, p);
  return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN>
LaunchFn pick_conv(int epi) {
  switch (epi) {
    case E_F32: return launch<BM, BN, WGM, WGN, E_F32, 1>;
    case E_BF16: return launch<BM, BN, WGM, WGN, E_BF16, 1>;
    case E_BIAS_RELU: return launch<BM, BN, WGM, WGN, E_BIAS_RELU, 1>;
    case E_AFFINE: return launch<BM, BN, WGM, WGN, E_AFFINE, 1>;
    case E_RELU_MASK: return launch<BM, BN, WGM, WGN, E_RELU_MASK, 1>;
    case E_PARTIAL: return launch<BM, BN, WGM, WGN, E_PARTIAL, 1>;
    default: return nullptr;
  }
}

template <int BM, int BN, int WGM, int WGN>
LaunchFn pick_convdw(int epi) {
  if (epi == E_F32) return launch<BM, BN, WGM, WGN, E_F32, 2>;
  if (epi == E_PARTIAL) return launch<BM, BN, WGM, WGN, E_PARTIAL, 2>;
  return nullptr;
}

}  // namespace

LaunchFn ring_conv_64x128(int epi) { return pick_conv<64, 128, 2, 4>(epi); }
LaunchFn ring_conv_128x64(int epi) { return pick_conv<128, 64, 4, 2>(epi); }
LaunchFn ring_conv_128x128(int epi) { return pick_conv<128, 128, 4, 2>(epi); }
LaunchFn ring_convdw_64x128(int epi) { return pick_convdw<64, 128, 2, 4>(epi); }
LaunchFn ring_convdw_128x64(int epi) { return pick_convdw<128, 64, 4, 2>(epi); }

}  // namespace gemm
}  // namespace et
