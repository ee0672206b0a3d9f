// the wide, direct-to-LDS and split-contraction kernels for A k-major, B k-major
#include "gemm_ksplit.h"

hipError_t gemm_wide_launch_kk(int cfg, const GemmDev& p, int splits, hipStream_t s) {
  return launch_layout<true, true>(cfg, p, splits, s);
}
