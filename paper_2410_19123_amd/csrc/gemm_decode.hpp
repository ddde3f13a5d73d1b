// Grouped GEMM for few tokens per expert (decode, bf16): weight streams.
//
// What bounds it: bytes.  One Llama-7B-shaped expert's gate/up is 23 MB, 4 us
// at the card's read rate of 5.8 TB/s (23 bytes per ns and CU with all 256
// pulling; one of few pulls up to about 46, activation rows from L2 included,
// however its waves are arranged), so what matters is how many workgroups a
// launch has and how evenly the CUs are loaded.  A 32 x 128 tile gives one
// expert 22 workgroups (gate/up) and 32 (down): 24.5 and 11.8 us for one
// token, five times the stream's time.
//
// k_skinny: 16, 32 or 64 columns per workgroup, so that one to five experts
// fill the chip.  With so few columns the waves cannot share activation rows,
// so they split K instead: four waves, a quarter of K each, weights and
// activation fragments straight from global memory into registers, no LDS and
// no barrier in the loop, the quarters' sums added in LDS at the end in
// order.  Token rows past 16 are a second MFMA tile.  Every workgroup reads
// all its rows, so narrow tiles lose to wide ones once the rows outweigh the
// weights or the workgroups outnumber what the CUs hold: decode_cost in
// gemm.hip draws that line.  Measured, us per Llama-7B-shaped layer (norm,
// gate/up, down), 32 x 128 tile and the choice made here: 1 token 39.6 -> 16.0,
// 64 tokens on one expert (counts known) 34.6 -> 27.0, 4 tokens on 4 experts
// 43.4 -> 34.4, 16 on 5 (counts known) 46.2 -> 41.2.
//
// k_decode: 32 x 128, token rows shared through LDS, for more experts than
// that in a stack (gemm.hip says which tile a layer takes instead): 64 tokens on 7 experts move 5.3 TB/s in gate/up (32.6 us with its
// launch, 28.2 at 5.6 TB/s).
//
// Both add K in the same order -- DECODE_SPLITS ranges, each from zero, then
// the ranges in order, then the residual -- so the choice between them may
// use the caller's token counts without a change in the results.
#pragma once

#include "gemm_kernels.hpp"

namespace readme {

// Ranges that the decode kernels split K into; range r of nk K-steps starts
// at K-step decode_range(r, nk).
constexpr int DECODE_SPLITS = 4;
__device__ __forceinline__ int decode_range(int r, int nk) { return r * nk / DECODE_SPLITS; }

// Four consecutive output columns of one row.
__device__ __forceinline__ void decode_store4(const GemmArgs& g, int64_t row, int64_t col,
                                              const float (&v)[4]) {
    uint2 o;
    o.x = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
    o.y = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(g.C) + row * g.ldc + col) = o;
}

// Activation row of grouped row `row` (clamped where a map is corrupt).
__device__ __forceinline__ int64_t decode_a_row(const GemmArgs& g, int64_t row) {
    if (g.a_rows) {
        row = g.a_rows[row];
        row = (row >= 0 && row < g.T) ? row : 0;
        if (g.a_rows_div > 1) row /= g.a_rows_div;  // pair -> token
    }
    return row;
}

constexpr int kNormRows = 1;      // gate/up normalises its rows itself up to here
constexpr int kNormWidth = 8192;  // and up to this row length

// The tile's one row normalised, in LDS: xn[k] = bf16(x[m0][k] * r), the
// arithmetic and summation order of k_rms_to_bf16 (256 threads), so the same
// bits.  The row is requested before the weights and reduced while they
// arrive (loads return in order).  Decode of one token, us per layer: norm in
// a launch of its own 17.6, here 16.0 (with the row requested after the
// weights 17.0).
struct SkinnyNorm {
    static constexpr int NV = kNormWidth / 1024;
    float4 v[NV];

    __device__ __forceinline__ void request(const GemmArgs& g, const TileLoc& t) {
        const int tt = threadIdx.x, n4 = (int)(g.K / 4);
        const float4* row = reinterpret_cast<const float4*>(
            reinterpret_cast<const float*>(g.A) + t.m0 * g.lda);
#pragma unroll
        for (int i = 0; i < NV; ++i)
            v[i] = tt + 256 * i < n4 ? row[tt + 256 * i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }

    __device__ __forceinline__ void finish(const GemmArgs& g, uint16_t* xn, float* sums);
};

__device__ __forceinline__ void SkinnyNorm::finish(const GemmArgs& g, uint16_t* xn,
                                                   float* sums) {
    const int tt = threadIdx.x, n4 = (int)(g.K / 4);
    float ss = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (tt + 256 * i < n4) {
            ss += v[i].x * v[i].x;
            ss += v[i].y * v[i].y;
            ss += v[i].z * v[i].z;
            ss += v[i].w * v[i].w;
        }
    }
    for (int off = 32; off >= 1; off >>= 1) ss += __shfl_down(ss, off, 64);
    if ((tt & 63) == 0) sums[tt >> 6] = ss;
    __syncthreads();
    const float tot = (sums[0] + sums[1]) + (sums[2] + sums[3]);
    const float rs = 1.0f / sqrtf(tot / (float)g.K + g.rms_eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (tt + 256 * i < n4) {
            uint2 o;
            o.x = (uint32_t)f32_to_bf16(v[i].x * rs) | ((uint32_t)f32_to_bf16(v[i].y * rs) << 16);
            o.y = (uint32_t)f32_to_bf16(v[i].z * rs) | ((uint32_t)f32_to_bf16(v[i].w * rs) << 16);
            reinterpret_cast<uint2*>(xn)[tt + 256 * i] = o;
        }
    }
    __syncthreads();
}

// NC 16-column tiles of TT 16-token tiles per workgroup.  Column tile layout:
//   store / residual: NC * 16 consecutive columns;
//   gate/up, NC = 1: 8 gate rows, then the 8 up rows of the same neurons;
//   gate/up, NC = 2, 4: NC/2 tiles of 16 gate rows, then their up rows.
template <int TT, int NC, int EPI, bool NORM>
struct SkinnyTile {
    // K-steps in flight per wave: what the registers hold.
    static constexpr int S = NORM ? 8 : 12 / (NC + TT) + (NC + TT == 5);

    __device__ __forceinline__ static void run(const GemmArgs& g, const TileLoc& t, f32x4* part,
                                               uint16_t* xn, float* sums) {
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int q = lane >> 4, l16 = lane & 15;
        const int nk = (int)(g.K >> 6);
        const int k0 = decode_range(wave, nk), k1 = decode_range(wave + 1, nk);  // this wave's K

        const WeightSteps wst = weight_steps<EPI == EPI_STORE>(g, t.e, 2);
        uint32_t w_off[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            int grp, row;
            if constexpr (EPI == EPI_GATE_UP_SILU && NC == 1) {
                grp = 2 * (t.n_tile >> 2) + (l16 >> 3);
                row = (t.n_tile & 3) * 8 + (l16 & 7);
            } else {  // 16-row units; past N the last one (never stored)
                const bool gu = EPI == EPI_GATE_UP_SILU;
                int unit = gu ? t.n_tile * (NC / 2) + c % ((NC + 1) / 2) : t.n_tile * NC + c;
                unit = min(unit, (int)(g.N >> (gu ? 5 : 4)) - 1);
                grp = gu ? 2 * (unit >> 1) + c / ((NC + 1) / 2) : unit >> 1;
                row = (unit & 1) * 16 + l16;
            }
            w_off[c] = (uint32_t)(grp * 4096 + q * 512 + row * 16);
        }
        uint32_t a_src[TT];  // in units of 16 bytes
        const uint16_t* x_src[TT];
#pragma unroll
        for (int i = 0; i < TT; ++i) {
            int r = i * 16 + l16;
            r = r < t.rows ? r : t.rows - 1;
            if constexpr (NORM) {
                x_src[i] = xn + q * 8;
            } else {
                a_src[i] = (uint32_t)(decode_a_row(g, t.m0 + r) * (g.lda >> 3)) + q;
            }
        }

        f32x4 acc[TT][NC];
#pragma unroll
        for (int i = 0; i < TT; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[i][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

        u32x4 wq[S][NC][2], aq[S][TT][2];
        auto load_w = [&](auto sc, int kt) {
            constexpr int s = decltype(sc)::value;
            const char* bs = wst.at(kt);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const uint32_t o = keep32(w_off[c]);
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
                    wq[s][c][kk] = *reinterpret_cast<const u32x4*>(bs + o + kk * 2048);
            }
        };
        auto load_a = [&](auto sc, int kt) {
            constexpr int s = decltype(sc)::value;
#pragma unroll
            for (int i = 0; i < TT; ++i) {
                const char* as = reinterpret_cast<const char*>(g.A) + (int64_t)kt * 128 +
                                 (NORM ? 0 : (uint64_t)keep32(a_src[i]) * 16);
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    if constexpr (NORM)
                        aq[s][i][kk] =
                            *reinterpret_cast<const u32x4*>(x_src[i] + kt * 64 + kk * 32);
                    else
                        aq[s][i][kk] = *reinterpret_cast<const u32x4*>(as + kk * 64);
                }
            }
        };
        auto mfmas = [&](auto sc) {
            constexpr int s = decltype(sc)::value;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int i = 0; i < TT; ++i)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, wq[s][c][kk]),
                            __builtin_bit_cast(bf16x8, aq[s][i][kk]), acc[i][c], 0, 0, 0);
        };
        auto load = [&](auto sc, int kt) {
            load_w(sc, kt);
            if constexpr (!NORM) load_a(sc, kt);
        };
        auto use = [&](auto sc, int kt) {
            if constexpr (NORM) load_a(sc, kt);
            mfmas(sc);
        };
        SkinnyNorm norm;
        if constexpr (NORM) norm.request(g, t);
        if (k1 - k0 >= S) {
            static_for<0, S>([&](auto sc) { load(sc, k0 + decltype(sc)::value); });
            if constexpr (NORM) norm.finish(g, xn, sums);
            int kt = k0;
            for (; kt + 2 * S <= k1; kt += S)
                static_for<0, S>([&](auto sc) {
                    use(sc, kt + decltype(sc)::value);
                    load(sc, kt + decltype(sc)::value + S);
                });
            // The last S full steps, and up to S - 1 more loaded as their
            // registers come free.
            static_for<0, S>([&](auto sc) {
                const int k = kt + decltype(sc)::value;
                use(sc, k);
                if (k + S < k1) load(sc, k + S);
            });
            kt += S;
            static_for<0, S - 1>([&](auto sc) {
                const int k = kt + decltype(sc)::value;
                if (k < k1) use(sc, k);
            });
        } else {
            static_for<0, S - 1>([&](auto sc) {
                const int k = k0 + decltype(sc)::value;
                if (k < k1) load(sc, k);
            });
            if constexpr (NORM) norm.finish(g, xn, sums);
            static_for<0, S - 1>([&](auto sc) {
                const int k = k0 + decltype(sc)::value;
                if (k < k1) use(sc, k);
            });
        }

        // The ranges' sums meet in LDS and are added in order.
#pragma unroll
        for (int i = 0; i < TT; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c) part[((wave * TT + i) * NC + c) * 64 + lane] = acc[i][c];
        __syncthreads();
        if (tid >= TT * 64) return;
        const int i = tid >> 6;
        auto total = [&](int c, int ln) {
            f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < DECODE_SPLITS; ++w) s += part[((w * TT + i) * NC + c) * 64 + ln];
            return s;
        };
        const int rt = i * 16 + l16;
        if (rt >= t.rows) return;
        const int64_t row = g.c_rows ? (int64_t)g.c_rows[t.m0 + rt] : t.m0 + rt;
        if (row < 0 || row >= g.T) return;  // a corrupt map writes nothing
        if constexpr (EPI == EPI_GATE_UP_SILU) {
            if (NC == 1 && q >= 2) return;
#pragma unroll
            for (int c = 0; c < (NC + 1) / 2; ++c) {
                const f32x4 gt = total(c, lane);
                const f32x4 up = NC == 1 ? total(0, lane + 32) : total(c + NC / 2, lane);
                float h[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) h[r] = silu_f32(gt[r]) * up[r];
                const int64_t col = (int64_t)t.n_tile * (8 * NC) + c * 16 + q * 4;
                if (col < g.N / 2) decode_store4(g, row, col, h);
            }
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const f32x4 s = total(c, lane);
                const int64_t col = ((int64_t)t.n_tile * NC + c) * 16 + q * 4;
                if (col >= g.N) continue;
                if constexpr (EPI == EPI_RESID_ADD) {
                    f32x4* y = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) +
                                                        row * g.ldc + col);
                    *y = *y + s;
                } else {
                    const float v[4] = {s[0], s[1], s[2], s[3]};
                    decode_store4(g, row, col, v);
                }
            }
        }
    }
};

template <int NC, int EPI, bool NORM>
__global__ __launch_bounds__(DECODE_SPLITS * 64) __attribute__((amdgpu_waves_per_eu(2)))
void k_skinny(GemmArgs args) {
    constexpr int TTMAX = NORM ? 1 : 2;
    __shared__ f32x4 part[DECODE_SPLITS * TTMAX * NC * 64];
    TileLoc t;
    if (!find_tile<TTMAX * 16>(args, t)) return;
    using OT = std::conditional_t<EPI == EPI_RESID_ADD, float, uint16_t>;
    const GemmArgs g = tile_args<OT>(args, t.e);
    if constexpr (NORM) {
        __shared__ __attribute__((aligned(16))) uint16_t xn[kNormRows * kNormWidth];
        __shared__ float sums[4];
        SkinnyTile<1, NC, EPI, true>::run(g, t, part, xn, sums);
    } else {
        if (t.rows <= 16)
            SkinnyTile<1, NC, EPI, false>::run(g, t, part, nullptr, nullptr);
        else
            SkinnyTile<2, NC, EPI, false>::run(g, t, part, nullptr, nullptr);
    }
}

template <int NC, int EPI, bool NORM>
inline hipError_t launch_skinny(GemmArgs g, hipStream_t s) {
    g.n_tiles = (int)ceil_div(g.N, 16 * NC);
    g.m_tiles_max = (int)m_tiles_bound(g, NORM ? 16 : 32);
    const int64_t blocks = round_up((int64_t)g.n_tiles * g.m_tiles_max, 8);
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    k_skinny<NC, EPI, NORM><<<dim3((unsigned)blocks), dim3(DECODE_SPLITS * 64), 0, s>>>(g);
    return hipGetLastError();
}

// 32 rows x 128 columns: four waves of 32 weight rows each (gate/up: 16 gate
// rows and the 16 up rows of the same neurons, which meet in one lane), the
// token rows shared through LDS.
template <int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void k_decode(GemmArgs args) {
    constexpr int S = 5;  // K-steps in flight: what three waves per SIMD hold
    constexpr bool GU = EPI == EPI_GATE_UP_SILU;
    __shared__ u32x4 lds[2][32 * CPR];
    TileLoc t;
    if (!find_tile<32>(args, t)) return;
    using OT = std::conditional_t<EPI == EPI_RESID_ADD, float, uint16_t>;
    const GemmArgs g = tile_args<OT>(args, t.e);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int nk = (int)(g.K >> 6);

    const WeightSteps wst = weight_steps<EPI == EPI_STORE>(g, t.e, 2);
    const int unit = t.n_tile * 4 + wave;  // 16 neurons or 32 columns
    const int u = min(unit, (int)(g.N >> 5) - 1);
    const int grp = GU ? 2 * (u >> 1) + (l32 >> 4) : u;
    const int wrow = GU ? (u & 1) * 16 + (l32 & 15) : l32;
    const uint32_t w_off = (uint32_t)(grp * 4096 + half * 512 + wrow * 16);
    u32x4 wq[S][4];
    auto load_w = [&](auto sc, const char* bs) {
        constexpr int s = decltype(sc)::value;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            wq[s][q] = *reinterpret_cast<const u32x4*>(bs + w_off + q * 1024);
    };
    // The weight stream does not depend on the row map: its first K-steps are
    // requested before the row map is read.
    static_for<0, S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        load_w(sc, wst.at(s < nk ? s : nk - 1));
    });

    const int ar = tid >> 3;
    const char* a_src = reinterpret_cast<const char*>(g.A) +
                        decode_a_row(g, t.m0 + min(ar, t.rows - 1)) * g.lda * 2 +
                        swz(tid & 7, ar) * 16;
    const bool in = l32 < t.rows;
    int64_t crow = t.m0 + (in ? l32 : 0);
    if (g.c_rows) crow = g.c_rows[crow];
    u32x4 aq[S];
    static_for<0, S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        aq[s] = *reinterpret_cast<const u32x4*>(a_src + (int64_t)(s < nk ? s : nk - 1) * 128);
    });
    lds[0][tid] = aq[0];

    f32x16 acc, tot;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = tot[r] = 0.0f;
    auto fold = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            tot[r] += acc[r];
            acc[r] = 0.0f;
        }
    };
    int range = 1, next = decode_range(1, nk);
    __syncthreads();
    auto step = [&](auto sc, int kt) {
        constexpr int s = decltype(sc)::value;
        if (kt == next) {  // a range of K starts: close the one before
            fold();
            do next = decode_range(++range, nk);  // skip empty ranges
            while (next == kt && range < DECODE_SPLITS);
        }
        const u32x4* L = lds[kt & 1];
        const int ktn = kt + S < nk ? kt + S : nk - 1;  // K-step the refills fetch
        const char* bs = wst.at(ktn);
        u32x4 af[2];
        af[0] = L[l32 * CPR + swz(half, l32)];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            if (kk + 1 < 4) af[(kk + 1) & 1] = L[l32 * CPR + swz(2 * kk + 2 + half, l32)];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, wq[s][kk]), __builtin_bit_cast(bf16x8, af[kk & 1]), acc,
                0, 0, 0);
            wq[s][kk] = *reinterpret_cast<const u32x4*>(bs + w_off + kk * 1024);
        }
        aq[s] = *reinterpret_cast<const u32x4*>(a_src + (int64_t)ktn * 128);
        lds[(kt + 1) & 1][tid] = aq[(s + 1) % S];
        __syncthreads();
    };
    int kt0 = 0;
    for (; kt0 + S <= nk; kt0 += S)
        static_for<0, S>([&](auto sc) { step(sc, kt0 + decltype(sc)::value); });
    f32x4 res[4];
    if constexpr (EPI == EPI_RESID_ADD) {  // arrives during the last K-steps
#pragma unroll
        for (int i = 0; i < 4; ++i)
            res[i] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.C) +
                                                     crow * g.ldc + u * 32 + i * 8 + half * 4);
    }
    static_for<0, S - 1>([&](auto sc) {
        if (kt0 + decltype(sc)::value < nk) step(sc, kt0 + decltype(sc)::value);
    });
    fold();

    const bool ok = in && crow >= 0 && crow < g.T && unit * 32 < g.N;
    if (EPI == EPI_RESID_ADD && !ok) return;
    if constexpr (EPI == EPI_RESID_ADD) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 o = {res[i][0] + tot[4 * i], res[i][1] + tot[4 * i + 1],
                             res[i][2] + tot[4 * i + 2], res[i][3] + tot[4 * i + 3]};
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + crow * g.ldc + unit * 32 +
                                      i * 8 + half * 4) = o;
        }
    } else {
#pragma unroll
        for (int i = 0; i < (GU ? 2 : 4); i += 2) {
            // Columns 8i + 4*half .. +3 and 8(i+1) + 4*half .. +3; the other
            // half's lane of the row holds their neighbours.
            uint32_t w[2][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = 4 * (i + j) + r;
                    v[r] = GU ? silu_f32(tot[k]) * tot[(8 + k) & 15] : tot[k];
                }
                w[j][0] = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
                w[j][1] = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
            }
            const auto a = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
            const auto b = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
            const u32x4 o = {a[0], b[0], a[1], b[1]};
            const int64_t col = (int64_t)unit * (GU ? 16 : 32) + (i + half) * 8;
            if (ok)
                *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C) + crow * g.ldc + col) =
                    o;
        }
    }
}

template <int EPI>
inline hipError_t launch_decode(GemmArgs g, hipStream_t s) {
    g.n_tiles = (int)ceil_div(g.N, 128);
    g.m_tiles_max = (int)m_tiles_bound(g, 32);
    const int64_t blocks = round_up((int64_t)g.n_tiles * g.m_tiles_max, 8);
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    k_decode<EPI><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(g);
    return hipGetLastError();
}

}  // namespace readme
