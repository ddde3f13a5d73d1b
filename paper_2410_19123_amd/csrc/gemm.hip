// Host side of the grouped GEMM: tile choice and dispatch.  The kernels are
// in gemm_kernels.hpp, instantiated in gemm_f32.hip and gemm_bf16_*.hip.
#include <limits.h>
#include <math.h>

#include "gemm_pp.hpp"
#include "gemm_decode.hpp"

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

// Row groups of the launch (experts, then permanent groups) and their rows.
static int64_t row_groups(const GemmArgs& g) { return g.E + g.shared_groups; }
static int64_t group_rows(const GemmArgs& g) { return g.T * (1 + (int64_t)g.shared_groups); }

// Experts that T tokens of a uniform load reach.
static float active_experts(const GemmArgs& g) {
    const float E = (float)g.E;
    return E * (1.0f - powf(1.0f - 1.0f / E, (float)g.T));
}

// Estimated row tiles of `height` rows: the host does not know the split over
// experts, so each row group is taken to end in about half a tile of padding
// and to have at least one tile.
static float row_tiles(int height, const GemmArgs& g) {
    const float groups = active_experts(g) + (float)g.shared_groups;
    const float full = (float)group_rows(g) / height + (height == 32 ? 0.52f : 0.47f) * groups;
    return full > groups ? full : groups;
}

// Estimated time of one launch on tiles of `height` rows x 256 columns, to
// compare heights (not in us).  A tile costs a start and end that grow with its
// rows and a time per 64-element K-step that hardly does (the CU's load path);
// 256 tiles run at once (one per CU), a launch of just 256 no longer does (the
// tiles are dealt to the XCDs in whole numbers), and past that a round costs
// more than its share because rounds end ragged.  The constants fit a sweep of
// all tiles on MI355X over 4837 layers (d 512 .. 8192, I 64 .. 4096, 1 .. 128
// experts, 1 .. 4096 tokens per expert; uniform, Zipf and one-expert loads), for
// the time and against launches longer than on the tiles chosen before.  Over
// 11254 GEMMs of such layers, geometric mean: 28.1 us on the register-streamed
// tiles by tokens per expert alone, 22.2 by an estimate without a tile per row
// group and a start and end per decode tile, 22.0 by this one; 7.0% and 1.9% of
// the launches take over 4% longer than on the first, 0.7% than by the second.
// us of gate/up, uniform load, 32x128 / 64x256 / 128 rows / 256 rows:
//   d 6400, I 955, 32 experts of 48 tokens      163 / 198 / 195 / 196
//   d 1024, I 512, 128 experts of 64             73 /  59 /  76 /  78
//   d 4096, I 1376, 8 experts of 128             78 /  56 /  66 /  75
//   d 8192, I 3584, 4 experts of 192            236 / 179 / 128 / 151
static float tile_cost(int height, const GemmArgs& g) {
    const float nk = (float)g.K / 64.0f;
    const float tiles = row_tiles(height, g) * ceil_div(g.N, 256) / 256.0f;
    const float rounds = tiles <= 0.985f ? 1.0f : (tiles > 1.0f ? tiles : 1.0f) + 0.29f;
    if (height == 64) return rounds * (4.2f + 0.86f * nk);
    if (height == 128) return rounds * (5.6f + 0.905f * nk);
    return rounds * (7.2f + 0.895f * nk);
}

// Whether the launch is a decode launch: by its sizes alone, never by the
// counts, since the summation order follows from it.  Under 8 rows per group
// always: a taller tile is then mostly padding, and the weights it streams come
// in with fewer workgroups (64 x 256 against 32 x 128, 16 to 64 experts: 1.02
// to 1.10 times as long at 8 rows, 0.89 to 0.97 at 32).  Else where the time of
// its 32 x 128 tiles, many of them on the chip at once, is the least.
static bool decode_launch(const GemmArgs& g) {
    if (group_rows(g) < 8 * row_groups(g)) return true;
    const float cost = row_tiles(32, g) * ceil_div(g.N, 128) / 256.0f *
                       (0.94f + 0.475f * (float)g.K / 64.0f);
    return cost <= tile_cost(64, g) && cost <= tile_cost(128, g) && cost <= tile_cost(256, g);
}

// Decode: the estimated 32-row tiles of the launch.  Without the caller's
// counts, the experts that T tokens of a uniform load reach, and half a tile
// of padding for each expert when they fill tiles.
static float decode_m_tiles(const GemmArgs& g) {
    if (g.m_tiles32 > 0) return (float)g.m_tiles32;
    const float active = active_experts(g);
    const float full = (float)g.T / 32.0f + 0.5f * active;
    const float m = (active > full ? active : full) + g.shared_groups * ceilf((float)g.T / 32.0f);
    const float bound = (float)m_tiles_bound(g, 32);
    return m < bound ? m : bound;
}

// Time (us) of a decode launch with m 32-row tiles on the workgroup of `cols`
// columns: 256 at a time, each CU moving about 46 bytes per ns of weights and
// activation rows (16 rows per 16-token tile, all of them by every
// workgroup).  128 columns: the tile whose waves share the rows through LDS;
// more than one fits a CU, so a second round costs less than a whole one.
// This ranks the widths, no more: 46 bytes per ns and CU is past what HBM
// delivers to all 256 (23).  Holding each width to the stream's time as well (5.0
// or 5.6 TB/s) made the choice no better over 2052 launches of under 28 rows per
// expert (I 256 .. 3584; geometric mean 23.10 us, held 23.17 and 23.11;
// the best width of each 22.3).
static float decode_cost(int cols, const GemmArgs& g, float m) {
    const float n = m * (float)ceil_div(g.N, (int64_t)cols) / 256.0f;
    const float rows = cols == 128 || (float)g.T > 16.0f * m ? 32.0f : 16.0f;
    const float bytes = 2.0f * (float)g.K * ((float)cols + rows);
    const float rounds = n <= 1.0f ? 1.0f : cols == 128 ? n + 0.3f : ceilf(n);
    return rounds * ((cols == 128 ? 1.5f : 2.5f) + bytes / 46000.0f);
}

// fp32: waves of 32 x 32 outputs.  A wave's chain of 32x32x2 MFMAs (64 clocks
// each) is then half a 32 x 64 wave's, and with two to four small workgroups
// per CU one wave's LDS waits are covered by another's MFMAs, which the tall
// tiles (one workgroup per CU, two waves per SIMD) do not reach at any size.
// Past 64 tokens per expert 64 x 64 tiles; below, 32 x 64 with six K-steps in
// flight while all tiles (half a tile of padding per row group) are on the
// chip at once, with three, and so four per CU, past that.  Whole layers, us:
// tall tiles and 32 x 128 / 32 x 64 six / 32 x 64 three / 64 x 64:
//   256 tokens, d 512, 4 experts of 512        57 /   40 /   41 /   43
//   600 tokens, d 512, 64 experts of 256       79 /   68 /   73 /   78
//   1500 tokens, d 1024, 64 experts of 512    304 /  231 /  199 /  231
//   300 tokens, d 2048, 4 experts of 1536     261 /  177 /  155 /  145
//   2048 tokens, d 2048, 4 experts of 1500   1026 /  668 /  489 /  431
//   8192 tokens, d 4096, 4 experts of 1376   3153 / 4441 / 2988 / 2618
// A grid holds fewer than 2^32 threads: past 2^24 tiles of 64 x 64 (256 threads,
// so 2^36 outputs) the launch takes 256 x 256 tiles, a sixteenth as many.
static int f32_tile(const GemmArgs& g) {
    if (g.T / (g.E > 0 ? g.E : 1) > 64) {
        const int64_t tiles = m_tiles_bound(g, 64) * ceil_div(g.N, 64);
        return tiles < (1 << 24) - 8 ? TILE_F32_64x64_W4 : TILE_256x256;
    }
    const int64_t groups = g.E + g.shared_groups;
    const int64_t rows = g.T * (1 + g.shared_groups);
    const int64_t tiles = (rows / 32 + groups / 2) * ceil_div(g.N, 64);
    return tiles <= 512 ? TILE_F32_32x64_W2 : TILE_F32_32x64_W2_S3;
}

// Tile of a launch.  bf16, by the estimates above.  Decode (the 32 x 128 tile
// would be the cheapest of the fixed heights, whatever the split over
// experts): the kernels of gemm_decode.hpp, whose one summation order lets the
// caller's counts choose among them.  Where no caller can give counts (a layer
// outside a stack), the 32 x 128 tile is the register-streamed one instead: it
// keeps six K-steps in flight where the other has registers for five, and was
// the faster one of 4314 GEMMs by 1 to 2% at the median, by 7 to 16% (1 to 3 us)
// where fewer than 64 tiles have rows, so that a CU has one workgroup that waits
// for its own loads, and K is 1024 or more; with K below that it is 3% (0.2 us)
// slower there and not taken.  Else 64 x 256 (four waves) or one of the
// mixed-height launches of gemm_pp.hpp, whose tall tiles are the fastest per
// flop.
static int tile_by_shape(bool f32, const GemmArgs& g) {
    const int f = forced_tile();
    if (f > 0) return f;
    if (g.tile > TILE_AUTO) return g.tile;
    if (f32) return f32_tile(g);  // both operands through LDS (the other kernels are bf16 only)
    const float c64 = tile_cost(64, g), c128 = tile_cost(128, g), c256 = tile_cost(256, g);
    if (decode_launch(g)) {
        const float m = decode_m_tiles(g);
        const int tile[4] = {TILE_DECODE_128, TILE_SKINNY_64, TILE_SKINNY_32, TILE_SKINNY_16};
        int best = 0;
        float cost = decode_cost(128, g, m);
        for (int i = 1; i < 4; ++i) {
            const float c = decode_cost(128 >> i, g, m);
            if (c < 0.97f * cost) {
                cost = c;
                best = i;
            }
        }
        if (best == 0 && !g.counts_order && g.K >= 1024) return TILE_BD_32x128_W4;
        return tile[best];
    }
    if (c64 <= c128 && c64 <= c256) return TILE_BD_64x256;
    return c128 <= c256 ? TILE_PP_128 : TILE_PP_256;
}

static bool is_decode_tile(int tile) { return tile >= TILE_SKINNY_16 && tile <= TILE_DECODE_128; }

// The tile a launch runs: tile_by_shape, or the tile that takes its place where
// activation offsets do not fit the 32 bits (of 16 bytes each) that
// gemm_pp.hpp and the weight streams of gemm_decode.hpp keep them in.  The
// fp32 tiles address in 64 bits.
static int launch_tile_number(bool f32, const GemmArgs& g) {
    int tile = tile_by_shape(f32, g);
    if (f32) return tile;
    if (tile == TILE_192_128_64) tile = TILE_PP_256;
    if (g.T * (g.lda >> 3) <= INT32_MAX) return tile;
    if (is_pp_tile(tile)) return TILE_MIX_256;
    return is_decode_tile(tile) ? TILE_DECODE_128 : tile;
}

bool gate_up_takes_norm(GemmArgs g) {
    if (forced_tile() > 0 || g.T > kNormRows || g.K > kNormWidth) return false;
    return decode_launch(g);
}

hipError_t launch_grouped_gemm(bool f32, int epi, GemmArgs g, hipStream_t s) {
    // The kernels address one weight index with 32-bit per-lane offsets and
    // find a K-step's segment by a multiply-high that is exact below 2^16
    // K-steps (K-steps are at least 32 elements).
    if (g.b_expert_stride * (f32 ? 4 : 2) > INT32_MAX) return hipErrorInvalidValue;
    if (g.K >= (int64_t)32 << 16) return hipErrorInvalidValue;
    if (g.k_segs > 1 && epi != EPI_STORE) return hipErrorInvalidValue;  // segments: down only
    int tile = launch_tile_number(f32, g);
    if (g.rms_in) {  // gate_up_takes_norm: a weight stream, of at most 32 columns
        if (tile != TILE_SKINNY_16) tile = TILE_SKINNY_32;
        return launch_decode_bf16(tile, epi, g, s);
    }
    if (!f32 && is_decode_tile(tile)) return launch_decode_bf16(tile, epi, g, s);
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

// Outside readme.h, for tests: readme_set_gemm_tile for the kernels only the
// automatic choice takes too, and the tile number (TileCfg) of a GEMM launch
// with these sizes and the calling thread's override.
extern "C" int32_t readme_internal_set_gemm_tile(int32_t tile) {
    if (tile < readme::TILE_AUTO || tile > readme::TILE_PP_128) return README_ERR_ARG;
    readme::t_forced_tile = tile;
    return README_OK;
}

extern "C" int32_t readme_internal_gemm_tile(int32_t f32, int64_t T, int64_t N, int64_t K,
                                             int32_t E, int32_t shared_groups,
                                             int32_t m_tiles32, int32_t counts_order) {
    readme::GemmArgs g{};
    g.T = T;
    g.N = N;
    g.K = g.lda = K;
    g.E = E;
    g.shared_groups = shared_groups;
    g.m_tiles32 = m_tiles32;
    g.counts_order = counts_order != 0;
    return readme::launch_tile_number(f32 != 0, g);
}
