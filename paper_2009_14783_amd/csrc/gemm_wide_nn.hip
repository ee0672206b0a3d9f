// the wide, direct-to-LDS and split-contraction kernels for A m-major, B n-major
#include "gemm_ksplit.h"

hipError_t gemm_wide_launch_nn(int cfg, const GemmDev& p, int splits, hipStream_t s) {
  return launch_layout<false, false>(cfg, p, splits, s);
}

// weight-gradient products in one launch
hipError_t gemm_group_launch_nn(int cfg, const GemmGroupDev& g, hipStream_t s) {
  switch (cfg) {
    case 9: return launch_dma_group<Dma128x128>(g, s);
    case 11: return launch_dma_group<Dma64x64>(g, s);
    default: return hipErrorInvalidValue;
  }
}
