// Instantiations of the direct-to-LDS two-group GEMM kernel (see gemm_bf16_direct.h).
#include "gemm_bf16_direct.h"

namespace et {
namespace gemm {
namespace {

template <bool AT, bool BT, int E>
hipError_t launch(const Params& p, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((gemm_direct_kernel<4, AT, BT, E>), grid, dim3(512), 0, s, p);
  return hipGetLastError();
}

}  // namespace

LaunchFn direct_256x256(bool a_t, bool b_t, int epi) {
#define ET_PICK(AT, BT, E) \
  if (a_t == AT && b_t == BT && epi == E) return launch<AT, BT, E>;
  ET_PICK(false, false, E_F32)
  ET_PICK(false, false, E_F32_RES)
  ET_PICK(false, false, E_BF16)
  ET_PICK(false, false, E_GELU_FWD)
  ET_PICK(false, false, E_GELU_ONLY)
  ET_PICK(false, false, E_BIAS_RELU)
  ET_PICK(false, true, E_F32)
  ET_PICK(false, true, E_BF16)
  ET_PICK(false, true, E_GELU_BWD)
  ET_PICK(true, true, E_F32)
  ET_PICK(true, true, E_BF16)
  ET_PICK(true, true, E_PARTIAL)
#undef ET_PICK
  return nullptr;
}

}  // namespace gemm
}  // namespace et
