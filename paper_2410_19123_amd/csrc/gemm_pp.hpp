// Grouped GEMM on 16x16x32 MFMA with both operands staged in LDS and two
// wave groups in opposite phase (bf16), tiles of 256, 128 and 64 rows.
//
// A workgroup of eight waves (two per SIMD) owns a BM x 256 tile: two rows of
// waves (tokens) by four (weight columns), so a wave owns BM/2 tokens and 64
// columns, i.e. two 32-row packed weight groups (for gate/up: the gate and
// the up group of the same 32 neurons, which therefore meet in one lane).
//
// What bounds it.  On real values the card holds its power, not its clock: a
// loop of nothing but MFMAs on N(0,1) bf16 runs at 1775 TFLOP/s with 32x32x16
// and 2031 with 16x16x32 (half the accumulator traffic per flop; on zeros
// both reach 2472), and 1564 / 1664 with this tile's LDS reads added.  Per
// 64-element K-step a 256-row tile needs 2048 clocks of MFMA and 64 KB through
// the CU's load path, which delivers 20 to 36 bytes a clock: without the
// MFMAs the request batch's gate/up takes 599 us, without the loads 678 us,
// with both 753 to 830 us (1160 to 1280 TFLOP/s).  The tiles it replaced
// (weights in registers, eight waves reading all token rows: 4/3 of the LDS
// reads per flop, one barrier per K-step for all) took 905 to 1010 us.  Other
// shapes, before and after, gate/up and down in us: skewed prefill 246, 149 ->
// 191, 135; top-2 layer 117, 81 -> 92, 68; Llama-7B-shaped layer 74, 43 -> 68,
// 38.  Weights straight to registers here (every fragment then fetched by both
// token halves, 96 KB per K-step) took 951 us.
//
// Loads.  Both operands go global -> LDS (global_load_lds_dwordx4) in parts
// that are refilled as soon as both wave groups have read them: a 256-row
// K-step has token halves A0, A1 and weight halves B0, B1 of 16 KB in two
// buffers, the smaller tiles three buffers.  The token rows are XOR-swizzled
// on the global side and the weights lie as packed; both kinds of fragment
// read are free of bank conflicts (counter 0).  The compiler would wait for
// all transfers before an LDS read that may alias one, so every part is an
// array of its own, the waits are the builtin's (inline asm is invisible to
// the wait insertion) and the steady loop has no branch.
//
// Phases.  A K-step of a 256-row tile is two phases of 32 MFMAs per wave: A0
// with both weight halves, then A1.  A phase has a load half (12 fragment
// reads, the next transfers) and an MFMA half, each ended by a barrier, and
// the two wave groups (one wave of each per SIMD) run half a phase apart, so
// on every SIMD one wave computes while the other loads.  Reads are spread
// evenly: phase A reads B and half of A1, phase B the other half and the next
// K-step's A0.  (Four phases of 16 MFMAs with 12, 4, 8 and 0 reads: 822 to
// 872 us.)
//
// Output.  The weights are the MFMA's first operand and the tokens the
// second, so a lane's four accumulator values are four consecutive output
// columns of one token; one lane exchange (v_permlane16_swap) makes that
// eight bf16 columns and the epilogue stores 16 bytes per lane straight from
// registers, with no LDS and no barrier.  The sums equal those of the other
// tiles that run straight through K (the LDS and the register-streamed ones, the
// residual first where it is added) bit for bit; the decode tiles add K in four
// ranges (gemm_decode.hpp).
#pragma once

#include "gemm_mix.hpp"

namespace readme {

constexpr int PP_SLOTS = 1024;  // 16-byte slots of one LDS part (16 KB)
constexpr int PP_PARTS = 9;

// s_waitcnt with the given outstanding counts.  The builtin (unlike inline
// asm) is understood by the compiler's own wait insertion, which then knows
// that the LDS transfers it waited for are done and adds no wait of its own.
template <int VM, int LGKM>
__device__ __forceinline__ void pp_wait() {
    static_assert(VM >= 0 && VM < 64 && LGKM >= 0 && LGKM < 16, "counter range");
    __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (LGKM << 8) | ((VM >> 4) << 14));
}

__device__ __forceinline__ void pp_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// The LDS parts, one __shared__ array each: the compiler tells distinct
// arrays apart, so a read of one does not wait for transfers into another.
struct PpLds {
    u32x4* p[PP_PARTS];
};

template <int BM, int NB, int EPI>
struct PpTile {
    static constexpr int PA = BM == 256 ? 2 : 1;    // parts of a K-step's token rows
    static constexpr int TMW = BM / 32;             // 16-token tiles per wave
    static constexpr int TP = TMW / PA;             // of them per part
    static constexpr int PROWS = BM / PA;           // token rows per part
    static constexpr int AI = PROWS / 64;           // DMA instructions per wave and part
    static constexpr int BI = 2;
    static constexpr int PPS = PA + 2;              // parts per K-step
    static_assert(NB * PPS <= PP_PARTS && AI >= 1, "parts");

    // LDS part of buffer b's token part p / weight half h: token parts first,
    // so that one address register and the instructions' 64 KB offsets reach
    // all of them.
    static constexpr int a_part(int b, int p) { return b * PA + p; }
    static constexpr int b_part(int b, int h) { return NB * PA + b * 2 + h; }

    __device__ __forceinline__ static void run(const GemmArgs& g, const TileLoc& t, const PpLds& L,
                                               int32_t* crow) {
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wm = wave >> 2, wn = wave & 3;
        const int64_t m0 = t.m0, m_end = t.m_end;
        const int64_t n0 = (int64_t)t.n_tile * 256;
        const int nk = (int)(g.K >> 6);

        // Weight sources: KB q of a half's 16 KB is KB q%4 of the half's
        // q/4-th row group; groups past N reuse the last one (never stored).
        const WeightSteps wst = weight_steps<EPI == EPI_STORE>(g, t.e, 2);
        uint32_t b_off[2][BI];  // wave-uniform; each lane adds 16 * lane
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < BI; ++i) {
                const int q = wave + 8 * i;
                int64_t grp = (n0 >> 5) + (q >> 2) * 2 + h;
                const int64_t last = (g.N >> 5) - 1;
                grp = grp < last ? grp : last;
                b_off[h][i] = (uint32_t)(grp * 4096 + (q & 3) * 1024);
            }
        const uint32_t b_lane = lane * 16;
        // Token sources, as in the other tiles: clamped to the block's last
        // row, through the row map where there is one.
        uint32_t a_src[PA][AI];  // in units of 16 bytes
#pragma unroll
        for (int p = 0; p < PA; ++p)
#pragma unroll
            for (int i = 0; i < AI; ++i) {
                const int pr = 8 * (wave + 8 * i) + (lane >> 3);
                const int r = (pr / (PROWS / 2)) * (BM / 2) + p * (PROWS / 2) + pr % (PROWS / 2);
                int64_t row = m0 + r;
                row = row < m_end ? row : m_end - 1;
                if (g.a_rows) {
                    row = g.a_rows[row];
                    row = (row >= 0 && row < g.T) ? row : 0;  // a corrupt map stays in bounds
                    if (g.a_rows_div > 1) row /= g.a_rows_div;  // pair -> token
                }
                a_src[p][i] = (uint32_t)(row * (g.lda >> 3)) + swz(lane & 7, pr);
            }
        if (g.c_rows && tid < BM) {
            int64_t row = m0 + tid;
            row = row < m_end ? row : m_end - 1;
            crow[tid] = g.c_rows[row];
        }

        f32x4 acc[TMW][2][2];
        // Wave-tile token row and output column of accumulator (i, h, tt).
        const int trow = wm * (BM / 2) + (lane & 15);
        const int64_t col0 = n0 + wn * 64;
#pragma unroll
        for (int i = 0; i < TMW; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    acc[i][h][tt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    if constexpr (EPI == EPI_RESID_ADD) {
                        const int rt = trow + i * 16;
                        const int64_t row = m0 + (rt < t.rows ? rt : 0);
                        int64_t c = col0 + h * 32;
                        c = c < g.N ? c : 0;
                        acc[i][h][tt] = *reinterpret_cast<const f32x4*>(
                            reinterpret_cast<const float*>(g.C) + row * g.ldc + c + tt * 16 +
                            (lane >> 4) * 4);
                    }
                }

        auto dma_a = [&](auto bc, auto pc, int kt) {
            constexpr int b = decltype(bc)::value, p = decltype(pc)::value;
#pragma unroll
            for (int i = 0; i < AI; ++i)
                dma16(reinterpret_cast<const char*>(g.A) + (int64_t)kt * 128 +
                          (uint64_t)keep32(a_src[p][i]) * 16,
                      L.p[a_part(b, p)] + (wave + 8 * i) * 64);
        };
        auto dma_b = [&](auto bc, auto hc, const char* bs) {
            constexpr int b = decltype(bc)::value, h = decltype(hc)::value;
#pragma unroll
            for (int i = 0; i < BI; ++i)
                dma16(bs + b_off[h][i] + keep32(b_lane), L.p[b_part(b, h)] + (wave + 8 * i) * 64);
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;

        const int a_slot = (wm * (PROWS / 2) + (lane & 15)) * CPR;
        const int a_ch = (lane >> 4) ^ ((lane >> 1) & 7);
        const int b_slot = wn * 256 + (lane >> 4) * 32 + (lane & 15);
        u32x4 af[PA][TP][2], bf[2][2][2];  // [part][token tile][kk], [half][column tile][kk]
        // Fragments [k0, k1) of part p: fragment f is token tile f % TP, kk f / TP.
        auto read_a = [&](auto bc, auto pc, auto k0, auto k1) {
            constexpr int b = decltype(bc)::value, p = decltype(pc)::value;
            static_for<decltype(k0)::value, decltype(k1)::value>([&](auto fc) {
                constexpr int f = decltype(fc)::value, i = f % TP, kk = f / TP;
                af[p][i][kk] = L.p[a_part(b, p)][a_slot + i * 16 * CPR + (a_ch ^ (kk * 4))];
            });
        };
        auto read_b = [&](auto bc, auto hc) {
            constexpr int b = decltype(bc)::value, h = decltype(hc)::value;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
                    bf[h][tt][kk] = L.p[b_part(b, h)][b_slot + kk * 128 + tt * 16];
        };
        // MFMAs of token part p with weight halves [h0, h1).
        auto mfmas = [&](auto pc, auto h0, auto h1) {
            constexpr int p = decltype(pc)::value;
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int h = decltype(h0)::value; h < decltype(h1)::value; ++h)
#pragma unroll
                    for (int i = 0; i < TP; ++i)
#pragma unroll
                        for (int tt = 0; tt < 2; ++tt)
                            acc[p * TP + i][h][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, bf[h][tt][kk]),
                                __builtin_bit_cast(bf16x8, af[p][i][kk]), acc[p * TP + i][h][tt],
                                0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
        };
        // End of a phase's load half: its own reads are complete and the next
        // phase's parts have arrived (all of them near the end of K, where
        // fewer transfers are outstanding).
        auto settle = [&](auto ahead, bool steady) {
            if (steady)
                pp_wait<decltype(ahead)::value, 0>();
            else
                pp_wait<0, 0>();
            pp_barrier();
        };
        using I2 = std::integral_constant<int, 2>;
        using IF = std::integral_constant<int, 2 * TP>;  // all fragments of a part
        using IH = std::integral_constant<int, TP>;      // half of them

        if constexpr (PA == 2) {
            // Transfers in program order: phase A of K-step k issues A1(k+1)
            // and A0(k+2), phase B issues B(k+2).
            static_assert(NB == 2, "two buffers");
            using AheadA = std::integral_constant<int, AI + 2 * BI>;      // before a phase A
            using AheadB = std::integral_constant<int, 2 * AI + 2 * BI>;  // before a phase B
            const int k1 = nk > 1 ? 1 : 0;
            dma_a(I0{}, I0{}, 0);
            dma_b(I0{}, I0{}, wst.at(0));
            dma_b(I0{}, I1{}, wst.at(0));
            dma_a(I0{}, I1{}, 0);
            dma_a(I1{}, I0{}, k1);
            dma_b(I1{}, I0{}, wst.at(k1));
            dma_b(I1{}, I1{}, wst.at(k1));
            pp_wait<AheadA::value, 0>();
            pp_barrier();
            read_a(I0{}, I0{}, I0{}, IF{});
            pp_wait<AheadA::value, 0>();
            pp_barrier();
            if (wm == 1) pp_barrier();  // the second group runs half a phase behind
            auto step = [&](auto bc, auto steady, int kt) {
                constexpr int b = decltype(bc)::value;
                using BC = std::integral_constant<int, b>;
                using BN = std::integral_constant<int, 1 - b>;
                const bool next = decltype(steady)::value || kt + 1 < nk;
                const bool more = decltype(steady)::value || kt + 2 < nk;
                read_b(BC{}, I0{});
                read_b(BC{}, I1{});
                read_a(BC{}, I1{}, I0{}, IH{});
                if (next) dma_a(BN{}, I1{}, kt + 1);
                if (more) dma_a(BC{}, I0{}, kt + 2);
                settle(AheadB{}, more);
                mfmas(I0{}, I0{}, I2{});
                pp_barrier();
                read_a(BC{}, I1{}, IH{}, IF{});
                if (next) read_a(BN{}, I0{}, I0{}, IF{});
                if (more) {
                    const char* bs = wst.at(kt + 2);
                    dma_b(BC{}, I0{}, bs);
                    dma_b(BC{}, I1{}, bs);
                }
                settle(AheadA{}, more);
                mfmas(I1{}, I0{}, I2{});
                pp_barrier();
            };
            int kt = 0;
            // The steady loop has no branch: where paths meet, the compiler
            // would wait for every transfer before the next LDS read.
            for (; kt + 4 <= nk; kt += 2) {
                step(I0{}, std::true_type{}, kt);
                step(I1{}, std::true_type{}, kt + 1);
            }
            for (; kt < nk; kt += 2) {
                step(I0{}, std::false_type{}, kt);
                if (kt + 1 < nk) step(I1{}, std::false_type{}, kt + 1);
            }
        } else {
            using Ahead = std::integral_constant<int, (NB - 1) * (AI + 2 * BI)>;
            // Prologue: K-steps 0 .. NB-1, but for the second weight half of
            // step NB-1, which the first phase issues.
            static_for<0, NB>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                const int kt = b < nk ? b : nk - 1;
                dma_a(bc, I0{}, kt);
                dma_b(bc, I0{}, wst.at(kt));
                if constexpr (b < NB - 1) dma_b(bc, I1{}, wst.at(kt));
            });
            pp_wait<Ahead::value, 0>();
            pp_barrier();
            if (wm == 1) pp_barrier();
            auto step = [&](auto bc, auto steady, int kt) {
                constexpr int b = decltype(bc)::value;
                using BC = std::integral_constant<int, b>;
                using BL = std::integral_constant<int, (b + NB - 1) % NB>;
                const bool last = decltype(steady)::value || kt + NB - 1 < nk;
                const bool more = decltype(steady)::value || kt + NB < nk;
                read_a(BC{}, I0{}, I0{}, IF{});
                read_b(BC{}, I0{});
                if (last) dma_b(BL{}, I1{}, wst.at(kt + NB - 1));
                settle(Ahead{}, last);
                mfmas(I0{}, I0{}, I1{});
                pp_barrier();
                read_b(BC{}, I1{});
                if (more) {
                    dma_a(BC{}, I0{}, kt + NB);
                    dma_b(BC{}, I0{}, wst.at(kt + NB));
                }
                settle(Ahead{}, more);
                mfmas(I0{}, I1{}, I2{});
                pp_barrier();
            };
            int kt0 = 0;
            for (; kt0 + 2 * NB <= nk; kt0 += NB)
                static_for<0, NB>([&](auto bc) {
                    step(bc, std::true_type{}, kt0 + decltype(bc)::value);
                });
            for (; kt0 < nk; kt0 += NB)
                static_for<0, NB>([&](auto bc) {
                    if (kt0 + decltype(bc)::value < nk)
                        step(bc, std::false_type{}, kt0 + decltype(bc)::value);
                });
        }
        if (wm == 0) pp_barrier();
        pp_wait<0, 0>();

        epilogue(g, t, acc, crow, lane, wm, wn, n0);
    }

    __device__ __forceinline__ static uint32_t pack2(float lo, float hi) {
        return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
    }

    // Eight columns of one token per lane from the four of each of two 16
    // column tiles a, b: lane group q (of four) then holds columns
    // (q&1)*16 + (q>>1)*8 .. +7 of the 32.
    __device__ __forceinline__ static u32x4 join(const float (&a)[4], const float (&b)[4]) {
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const auto s = __builtin_amdgcn_permlane16_swap(pack2(a[2 * w], a[2 * w + 1]),
                                                            pack2(b[2 * w], b[2 * w + 1]), false,
                                                            false);
            o[w] = s[0];
            o[2 + w] = s[1];
        }
        return o;
    }

    __device__ __forceinline__ static void epilogue(const GemmArgs& g, const TileLoc& t,
                                                    const f32x4 (&acc)[TMW][2][2],
                                                    const int32_t* crow, int lane, int wm, int wn,
                                                    int64_t n0) {
        const int q = lane >> 4;
        const int sub = (q & 1) * 16 + (q >> 1) * 8;
#pragma unroll
        for (int i = 0; i < TMW; ++i) {
            const int rt = wm * (BM / 2) + i * 16 + (lane & 15);
            const bool in = rt < t.rows;
            const int64_t row = g.c_rows ? (int64_t)crow[in ? rt : 0] : t.m0 + rt;
            const bool ok = in && row >= 0 && row < g.T;  // a corrupt map writes nothing
            if constexpr (EPI == EPI_GATE_UP_SILU) {
                float v[2][4];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        v[tt][r] = silu_f32(acc[i][0][tt][r]) * acc[i][1][tt][r];
                const u32x4 o = join(v[0], v[1]);
                const int64_t c = n0 / 2 + wn * 32;
                if (ok && c < g.N / 2)
                    *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C) + row * g.ldc + c +
                                              sub) = o;
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int64_t c = n0 + wn * 64 + h * 32;
                    if constexpr (EPI == EPI_RESID_ADD) {
                        if (ok && c < g.N) {
                            f32x4* y = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) +
                                                                row * g.ldc + c + q * 4);
                            y[0] = acc[i][h][0];
                            y[4] = acc[i][h][1];
                        }
                    } else {
                        float v[2][4];
#pragma unroll
                        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                            for (int r = 0; r < 4; ++r) v[tt][r] = acc[i][h][tt][r];
                        const u32x4 o = join(v[0], v[1]);
                        if (ok && c < g.N)
                            *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C) +
                                                      row * g.ldc + c + sub) = o;
                    }
                }
            }
        }
    }
};

// Tiles of 256, 128 and 64 rows in one launch (classes as in gemm_mix.hpp).
template <int B0, int B1, int B2, int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void k_grouped_gemm_pp(GemmArgs g) {
    __shared__ u32x4 p0[PP_SLOTS], p1[PP_SLOTS], p2[PP_SLOTS], p3[PP_SLOTS], p4[PP_SLOTS],
        p5[PP_SLOTS], p6[PP_SLOTS], p7[PP_SLOTS], p8[PP_SLOTS];
    __shared__ int32_t crow[B0];
    const PpLds L = {{p0, p1, p2, p3, p4, p5, p6, p7, p8}};
    using Mix = MixRows<B0, B1, B2, 0>;
    const int bid = blockIdx.x;
    int c = 0;
    while (c + 1 < Mix::NC && bid >= g.mix_start[c + 1]) ++c;
    const int local = bid - g.mix_start[c];
    const int total = mix_count<Mix>(g, c);
    const int per_xcd = (total + 7) >> 3;
    const int j = local >> 3;
    if (j >= per_xcd) return;
    const int n = (local & 7) * per_xcd + j;
    if (n >= total) return;
    TileLoc t;
    if (!mix_locate<Mix>(g, c, n, t)) return;
    using OT = std::conditional_t<EPI == EPI_RESID_ADD, float, uint16_t>;
    const GemmArgs a = tile_args<OT>(g, t.e);
    if (c == 0)
        PpTile<B0, B0 == 256 ? 2 : 3, EPI>::run(a, t, L, crow);
    else if (c == 1) {
        if constexpr (B1 > 0) PpTile<B1, 3, EPI>::run(a, t, L, crow);
    } else {
        if constexpr (B2 > 0) PpTile<B2, 3, EPI>::run(a, t, L, crow);
    }
}

template <int B0, int B1, int B2, int EPI>
inline hipError_t launch_pp(GemmArgs g, hipStream_t s) {
    const hipError_t err = mix_ranges<MixRows<B0, B1, B2, 0>>(g, 256);
    if (err != hipSuccess || g.mix_start[4] == 0) return err;
    k_grouped_gemm_pp<B0, B1, B2, EPI><<<dim3((unsigned)g.mix_start[4]), dim3(512), 0, s>>>(g);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_pp_tile(int tile, GemmArgs g, hipStream_t s) {
    switch (tile) {
        case TILE_PP_256: return launch_pp<256, 128, 64, EPI>(g, s);
        case TILE_PP_128: return launch_pp<128, 64, 0, EPI>(g, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace readme
