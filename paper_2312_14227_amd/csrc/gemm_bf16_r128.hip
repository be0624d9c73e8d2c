// Instantiations of the ring bf16 GEMM kernel with eight waves: 64x128 and 128x128 tiles (see gemm_bf16_ring.h).
#include "gemm_bf16_ring.h"

namespace et {
namespace gemm {
namespace {

template <int BM, int BN, int WGM, int WGN, bool AT, bool BT, int E>
hipError_t launch(const Params& p, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WGM, WGN, 3, AT, BT, E>), grid, dim3(512), 0, s, p);
  return hipGetLastError();
}

}  // namespace

#define ET_PICK(AT, BT, E) \
  if (a_t == AT && b_t == BT && epi == E) return launch<BM, BN, WGM, WGN, AT, BT, E>;
#define ET_PICK_ROWS                \
  ET_PICK(false, false, E_F32)      \
  ET_PICK(false, false, E_F32_RES)  \
  ET_PICK(false, false, E_PARTIAL)  \
  ET_PICK(false, false, E_BF16)     \
  ET_PICK(false, false, E_GELU_FWD) \
  ET_PICK(false, false, E_GELU_ONLY)\
  ET_PICK(false, false, E_BIAS_RELU)\
  ET_PICK(false, false, E_AFFINE)   \
  ET_PICK(false, false, E_AFFINE_ADD)\
  ET_PICK(false, true, E_F32)       \
  ET_PICK(false, true, E_BF16)      \
  ET_PICK(false, true, E_GELU_BWD)  \
  ET_PICK(true, true, E_F32)        \
  ET_PICK(true, true, E_BF16)       \
  ET_PICK(true, true, E_PARTIAL)

LaunchFn ring_64x128(bool a_t, bool b_t, int epi) {
  constexpr int BM = 64, BN = 128, WGM = 2, WGN = 4;
  ET_PICK_ROWS
  return nullptr;
}

LaunchFn ring_128x128(bool a_t, bool b_t, int epi) {
  constexpr int BM = 128, BN = 128, WGM = 4, WGN = 2;
  ET_PICK_ROWS
  return nullptr;
}
#undef ET_PICK_ROWS
#undef ET_PICK

}  // namespace gemm
}  // namespace et
