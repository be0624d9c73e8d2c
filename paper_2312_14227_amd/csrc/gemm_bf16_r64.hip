// Instantiations of the ring bf16 GEMM kernel for one tile shape (see gemm_bf16_ring.h).
#include "gemm_bf16_ring.h"

namespace et {
namespace gemm {
namespace {

template <bool AT, bool BT, int E, int CONV = 0, int RING = 3>
hipError_t launch(const Params& p, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((gemm_ring_kernel<64, 64, 2, 2, RING, AT, BT, E, CONV>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

}  // namespace

LaunchFn ring_64x64(bool a_t, bool b_t, int epi) {
#define ET_PICK(AT, BT, E) \
  if (a_t == AT && b_t == BT && epi == E) return launch<AT, BT, E>;
  ET_PICK(false, false, E_F32)
  ET_PICK(false, false, E_F32_RES)
  ET_PICK(false, false, E_PARTIAL)
  ET_PICK(false, false, E_BF16)
  ET_PICK(false, false, E_GELU_FWD)
  ET_PICK(false, false, E_GELU_ONLY)
  ET_PICK(false, false, E_BIAS_RELU)
  ET_PICK(false, false, E_AFFINE)
  ET_PICK(false, false, E_AFFINE_ADD)
  ET_PICK(false, true, E_F32)
  ET_PICK(false, true, E_BF16)
  ET_PICK(false, true, E_GELU_BWD)
  ET_PICK(true, true, E_F32)
  ET_PICK(true, true, E_BF16)
  ET_PICK(true, true, E_PARTIAL)
#undef ET_PICK
  return nullptr;
}

LaunchFn ring_64x64_deep(bool a_t, bool b_t, int epi) {
#define ET_PICK(AT, BT, E) \
  if (a_t == AT && b_t == BT && epi == E) return launch<AT, BT, E, 0, 5>;
  ET_PICK(false, false, E_F32)
  ET_PICK(false, false, E_F32_RES)
  ET_PICK(false, false, E_BF16)
  ET_PICK(false, false, E_AFFINE)
  ET_PICK(false, false, E_AFFINE_ADD)
  ET_PICK(false, true, E_BF16)
#undef ET_PICK
  return nullptr;
}

LaunchFn ring_conv_64x64(int epi) {
#define ET_PICK(E) \
  if (epi == E) return launch<false, false, E, 1>;
  ET_PICK(E_F32)
  ET_PICK(E_BF16)
  ET_PICK(E_BIAS_RELU)
  ET_PICK(E_AFFINE)
  ET_PICK(E_RELU_MASK)
  ET_PICK(E_PARTIAL)
#undef ET_PICK
  return nullptr;
}

LaunchFn ring_convdw_64x64(int epi) {
  if (epi == E_F32) return launch<true, true, E_F32, 2>;
  if (epi == E_PARTIAL) return launch<true, true, E_PARTIAL, 2>;
  return nullptr;
}

}  // namespace gemm
}  // namespace et
