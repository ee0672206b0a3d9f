// the wide, direct-to-LDS and split-contraction kernels for A m-major, B n-major
#include "gemm_ksplit.h"

hipError_t gemm_wide_launch_nn(int cfg, const GemmDev& p, int splits, hipStream_t s) {
  return launch_layout<false, false>(cfg, p, splits, s);
}

// weight-gradient products in one launch
hipError_t gemm_group_launch_nn(int cfg, const GemmGroupDev& g, hipStream_t s) {
  switch (cfg) {
    case 1: return launch_dma_group<Dma256x256>(g, s);
    case 9: return launch_dma_group<Dma128x128>(g, s);
    case 10: return launch_dma_group<Dma256x128>(g, s);
    case 11: return launch_dma_group<Dma64x64Group>(g, s);
    default: return hipErrorInvalidValue;
  }
}
