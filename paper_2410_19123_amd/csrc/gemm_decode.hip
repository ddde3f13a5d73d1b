// Decode GEMM kernels (gemm_decode.hpp).
#include "gemm_decode.hpp"

namespace readme {

hipError_t launch_decode_bf16(int tile, int epi, GemmArgs g, hipStream_t s) {
    if (tile == TILE_DECODE_128) {
        if (epi == EPI_GATE_UP_SILU) return launch_decode<EPI_GATE_UP_SILU>(g, s);
        if (epi == EPI_RESID_ADD) return launch_decode<EPI_RESID_ADD>(g, s);
        return launch_decode<EPI_STORE>(g, s);
    }
    if (g.rms_in)
        return tile == TILE_SKINNY_16 ? launch_skinny<1, EPI_GATE_UP_SILU, true>(g, s)
                                      : launch_skinny<2, EPI_GATE_UP_SILU, true>(g, s);
    if (tile == TILE_SKINNY_16) {
        if (epi == EPI_GATE_UP_SILU) return launch_skinny<1, EPI_GATE_UP_SILU, false>(g, s);
        if (epi == EPI_RESID_ADD) return launch_skinny<1, EPI_RESID_ADD, false>(g, s);
        return launch_skinny<1, EPI_STORE, false>(g, s);
    }
    if (tile == TILE_SKINNY_64) {
        if (epi == EPI_GATE_UP_SILU) return launch_skinny<4, EPI_GATE_UP_SILU, false>(g, s);
        if (epi == EPI_RESID_ADD) return launch_skinny<4, EPI_RESID_ADD, false>(g, s);
        return launch_skinny<4, EPI_STORE, false>(g, s);
    }
    if (epi == EPI_GATE_UP_SILU) return launch_skinny<2, EPI_GATE_UP_SILU, false>(g, s);
    if (epi == EPI_RESID_ADD) return launch_skinny<2, EPI_RESID_ADD, false>(g, s);
    return launch_skinny<2, EPI_STORE, false>(g, s);
}

}  // namespace readme
