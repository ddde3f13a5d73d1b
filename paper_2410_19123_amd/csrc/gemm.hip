// Host side of the grouped GEMM: tile choice and dispatch.  The kernels are
// in gemm_kernels.hpp, instantiated in gemm_f32.hip and gemm_bf16_*.hip.
#include <limits.h>

#include "gemm_pp.hpp"

namespace readme {

// Tile override of the calling host thread (0 = automatic): a tuning and
// test knob that affects only launches made from the thread that set it.
static thread_local int t_forced_tile = TILE_AUTO;
static int forced_tile() { return t_forced_tile; }

bool set_gemm_tile(int tile) {
    if (tile < TILE_AUTO || tile > TILE_LAST) return false;
    t_forced_tile = tile;
    return true;
}

int get_gemm_tile() { return t_forced_tile; }

// Estimated time (us, up to a common offset) of one launch on tiles of
// `height` rows, from the token count, the expert count and the GEMM's size:
// the host does not know the split over experts, so each row group is taken
// to end in half a tile of padding.  A tile costs a fixed start and end plus
// a time per 64-element K-step; up to 256 tiles run at once (one per CU), and
// past that a round costs more than its share because rounds end ragged.  The
// constants fit a sweep of all tiles on MI355X (E = 8, 16, 32; d = 1024 ..
// 8192; 8 .. 768 tokens per expert, uniform and Zipf loads; us of gate/up):
//   d 4096, I 1376, 64 / 128 / 256 / 768 per expert:
//     32x128 53/78/120/276, 64x256 57/56/90/185, 128 rows 61/66/66/166,
//     256 rows 61/75/82/167
//   d 8192, I 3584, 32 / 64 / 128 / 384 / 768 per expert:
//     32x128 178/243/340/901/1690, 64x256 152/212/285/496/930,
//     128 rows 153/156/253/470/739, 256 rows 152/157/186/373/570
static float tile_cost(int height, const GemmArgs& g) {
    const float nk = (float)g.K / 64.0f;
    const int64_t groups = g.E + g.shared_groups;
    const int64_t rows = g.T * (1 + g.shared_groups);
    const int64_t n_n = ceil_div(g.N, height == 32 ? 128 : 256);
    const float tiles =
        (height == 32 && g.m_tiles32 > 0 ? (float)g.m_tiles32
                                         : (float)rows / height + 0.5f * groups) * n_n / 256.0f;
    if (height == 32) {  // several workgroups per CU: no rounds
        const float t = 0.42f * tiles;
        return 3.0f + nk * (t > 0.5f ? t : 0.5f);
    }
    const float rounds = tiles <= 1.0f ? 1.0f : tiles + 0.4f;
    if (height == 64) return rounds * (5.0f + 0.75f * nk);
    if (height == 128) return rounds * (5.6f + 0.92f * nk);
    return rounds * (6.4f + 1.22f * nk);
}

// Tile of a launch.  bf16: the cheapest by tile_cost of 32 x 128 (four waves
// each streaming one weight group), 64 x 256 (four waves), and the two
// mixed-height launches of gemm_pp.hpp, whose tall tiles are the fastest per
// flop.
static int tile_by_shape(bool f32, bool gate_up, const GemmArgs& g) {
    const int f = forced_tile();
    if (f > 0) return f;
    if (g.tile > TILE_AUTO && g.tile <= TILE_LAST) return g.tile;
    if (f32) {  // both operands through LDS (the other kernels are bf16 only)
        const int64_t per_expert = g.T / (g.E > 0 ? g.E : 1);
        if (per_expert >= (gate_up ? 768 : 192)) return TILE_256x256;
        return per_expert >= 96 && !gate_up ? TILE_128x256 : TILE_32x128;
    }
    constexpr int kHeights = 4;
    const int height[kHeights] = {32, 64, 128, 256};
    const int tile[kHeights] = {TILE_BD_32x128_W4, TILE_BD_64x256, TILE_PP_128, TILE_PP_256};
    int best = 0;
    float cost = tile_cost(height[0], g);
    for (int i = 1; i < kHeights; ++i) {
        const float c = tile_cost(height[i], g);
        if (c < cost) {
            cost = c;
            best = i;
        }
    }
    // Few 32-row tiles, known from the caller's counts (tokens concentrated
    // on few experts): 64 columns, so that twice as many workgroups stream.
    if (best == 0 && g.m_tiles32 > 0 && (int64_t)g.m_tiles32 * ceil_div(g.N, 128) < 128)
        return TILE_BD_32x64;
    return tile[best];
}

hipError_t launch_grouped_gemm(bool f32, int epi, GemmArgs g, hipStream_t s) {
    // The kernels address one weight index with 32-bit per-lane offsets and
    // find a K-step's segment by a multiply-high that is exact below 2^16
    // K-steps (K-steps are at least 32 elements).
    if (g.b_expert_stride * (f32 ? 4 : 2) > INT32_MAX) return hipErrorInvalidValue;
    if (g.K >= (int64_t)32 << 16) return hipErrorInvalidValue;
    if (g.k_segs > 1 && epi != EPI_STORE) return hipErrorInvalidValue;  // segments: down only
    int tile = tile_by_shape(f32, epi == EPI_GATE_UP_SILU, g);
    // gemm_pp.hpp keeps activation offsets in 32 bits of 16 bytes each.
    if (is_pp_tile(tile) && g.T * (g.lda >> 3) > INT32_MAX) tile = TILE_MIX_256;
    if (!f32 && is_pp_tile(tile)) {
        if (epi == EPI_GATE_UP_SILU) return launch_pp_bf16_gate_up(tile, g, s);
        if (epi == EPI_RESID_ADD) return launch_pp_bf16_resid(tile, g, s);
        return launch_pp_bf16_store(tile, g, s);
    }
    if (!f32 && is_mix_tile(tile)) {
        if (epi == EPI_GATE_UP_SILU) return launch_mix_bf16_gate_up(tile, g, s);
        if (epi == EPI_RESID_ADD) return launch_mix_bf16_resid(tile, g, s);
        return launch_mix_bf16_store(tile, g, s);
    }
    if (f32) {
        if (epi == EPI_GATE_UP_SILU) return launch_tile_f32_gate_up(tile, g, s);
        return launch_tile_f32_store(tile, g, s);
    }
    if (epi == EPI_GATE_UP_SILU) return launch_tile_bf16_gate_up(tile, g, s);
    if (epi == EPI_RESID_ADD) return launch_tile_bf16_resid(tile, g, s);
    return launch_tile_bf16_store(tile, g, s);
}

}  // namespace readme
