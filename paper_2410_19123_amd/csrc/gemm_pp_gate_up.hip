// Grouped GEMM kernels on 16x16x32 MFMA (gemm_pp.hpp).  One translation unit
// per epilogue so that the kernels compile in parallel.
#include "gemm_pp.hpp"

namespace readme {

hipError_t launch_pp_bf16_gate_up(int tile, GemmArgs g, hipStream_t s) {
    return launch_pp_tile<EPI_GATE_UP_SILU>(tile, g, s);
}

}  // namespace readme
