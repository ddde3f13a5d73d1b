// The router block G at D = 512 in three launches: everything before the
// attention (embedding, norm, q|k|v, RoPE) and everything after it (Wo,
// residual, norm, MLP, residual, norm, gate) in one kernel each.
//
// A workgroup of eight waves owns 32 tokens and keeps their rows on chip (a
// norm or the MLP's hidden row in LDS, the fp32 residual in registers), so
// between the products there is neither a launch nor a pass over memory; the
// intermediates are still written to the workspace for the caller, and never
// read back.  What is left is the weights: 1.5 MB (q|k|v) and 2 MB (F = 512)
// stream from L2 through every workgroup, each wave taking its own 32-row
// weight groups straight into registers, four K-steps (32 KB) ahead, across
// the ends of the products too, since the weights do not depend on the data.
//
// Products: 32x32x16 MFMA with the weights as the first operand, so a lane
// holds one token and, four at a time, consecutive columns: norms need one
// lane exchange and a sum over waves in LDS, SiLU*mul and RoPE pairs meet in
// one lane, and rows are stored 16 bytes a lane.  K is summed in the order of
// the grouped GEMMs (the residual first where it is added).
//
// What bounds it: the 50 to 58 bytes per ns a CU takes from L2 (the same with
// 2 workgroups on the card as with 256), 36 us before and 45 us after the
// attention at F = 512 whatever the tokens up to 8192.  The nine launches take
// longer from about 1800 + 1.4 F tokens on: 4096 tokens 90 -> 78 us, 8192 123
// -> 90 (six launches and their passes over 8 to 34 MB gone),
// 16384 195 -> 165; at F = 1536, 4096 tokens 107 -> 104, 8192 157 -> 123; below
// that they are the faster form (2048 tokens: 68 against 74).  Starting each
// workgroup on another of q, k and v made no difference.
//
// D = 512, the width the block is specified with, is compiled in: a wave's two
// groups of 32 columns, the row of 64 16-byte chunks (one per lane) and the fp32
// residual in registers are sized for it.  Other widths keep the nine launches;
// what two kernels would give them has not been measured.
#include "gemm_kernels.hpp"
#include "router_common.hpp"

namespace readme {

namespace {

constexpr int D = kFusedRouterWidth;
constexpr int NKD = D / 64;       // K-steps of a product over D
constexpr int TOK = 32;           // tokens per workgroup
constexpr int NW = 8;             // waves
constexpr int S = 4;              // K-steps of weights in flight
constexpr int KSLOTS = TOK * CPR; // 16-byte LDS slots per K-step of a row block

typedef u32x4 WeightRing[S][2][4];  // [K-step][weight group][16-byte chunk pair]

// Weight address of a K-step: the wave's first group; the second is
// `second` bytes on.
template <int SL>
__device__ __forceinline__ void load_step(WeightRing& w, const char* p, int second, uint32_t lane16) {
    const uint32_t o = keep32(lane16);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        w[SL][0][q] = *reinterpret_cast<const u32x4*>(p + o + q * 1024);
        w[SL][1][q] = *reinterpret_cast<const u32x4*>(p + second + o + q * 1024);
    }
}

// LDS slot of 16-byte chunk c (of the whole row) of row r.
__device__ __forceinline__ int row_slot(int c, int r) {
    return (c >> 3) * KSLOTS + r * CPR + swz(c & 7, r);
}

template <int SL>
__device__ __forceinline__ void mfma_step(const WeightRing& w, const u32x4* rows, int kt, int l32,
                                          int half, f32x16 (&acc)[2]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const u32x4 a = rows[kt * KSLOTS + l32 * CPR + swz(2 * kk + half, l32)];
#pragma unroll
        for (int g = 0; g < 2; ++g)
            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[SL][g][kk]),
                                                             __builtin_bit_cast(bf16x8, a), acc[g],
                                                             0, 0, 0);
    }
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

// Sixteen columns (of a 32-column group) held four at a time -- v[4i + r] is
// column 8i + 4*half + r -- as two pieces of eight: piece j of this lane is
// columns 16j + 8*half .. +7.
__device__ __forceinline__ void pieces(const float (&v)[16], u32x4 (&out)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const auto a = __builtin_amdgcn_permlane32_swap(pack2(v[8 * j], v[8 * j + 1]),
                                                        pack2(v[8 * j + 4], v[8 * j + 5]), false,
                                                        false);
        const auto b = __builtin_amdgcn_permlane32_swap(pack2(v[8 * j + 2], v[8 * j + 3]),
                                                        pack2(v[8 * j + 6], v[8 * j + 7]), false,
                                                        false);
        out[j] = u32x4{a[0], b[0], a[1], b[1]};
    }
}

// A 32-column group of bf16 values to row t of a global array and, if lds, to
// the LDS rows.
__device__ __forceinline__ void put_group(const float (&v)[16], int grp, int l32, int half, bool ok,
                                          uint16_t* row, u32x4* lds) {
    u32x4 p[2];
    pieces(v, p);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = grp * 4 + 2 * j + half;  // 16-byte chunk of the row
        if (lds) lds[row_slot(c, l32)] = p[j];
        if (ok) *reinterpret_cast<u32x4*>(row + c * 8) = p[j];
    }
}

// Embedding, norm, q|k|v, RoPE.
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
void k_router_head(int64_t T, int32_t R, int64_t V, float eps, const int32_t* __restrict__ tokens,
                   const int32_t* __restrict__ ro, const uint16_t* __restrict__ emb,
                   float* __restrict__ x, uint16_t* __restrict__ a, int32_t* __restrict__ pos,
                   int32_t* __restrict__ offs, const char* __restrict__ wqkv,
                   uint16_t* __restrict__ qkv) {
#pragma clang fp contract(off)
    __shared__ u32x4 rows[NKD * KSLOTS];
    __shared__ double2 cs[64 * TOK];  // cosine and sine of (pair, token)
    __shared__ double inv[64];
    __shared__ int32_t pos_lds[TOK];
    __shared__ int32_t ro_lds[kRoLds];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * TOK;

    // Rows 4 * wave .. +3: one 16-byte chunk per lane.
    u32x4 e[4];
    int64_t tok[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t t = t0 + wave * 4 + j;
        tok[j] = t < T ? (int64_t)tokens[t] : -1;
    }
    const bool staged = R + 1 <= kRoLds;
    if (staged)
        for (int i = tid; i <= R; i += NW * 64) ro_lds[i] = ro[i];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool ok = tok[j] >= 0 && tok[j] < V;
        e[j] = u32x4{0u, 0u, 0u, 0u};
        if (ok) e[j] = *reinterpret_cast<const u32x4*>(emb + tok[j] * D + lane * 8);
    }
    // Pass p (q, k, v): wave w takes head w / 2, its 32-column groups w % 2
    // and w % 2 + 2, so that RoPE's pairs (i, i + 64) meet in a lane.
    constexpr int64_t STEP = (int64_t)(3 * D / 32) * 4096;
    const char* wbase = wqkv + ((wave >> 1) * 4 + (wave & 1)) * 4096;
    const uint32_t lane16 = lane * 16;
    WeightRing w;
    static_for<0, S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        load_step<s>(w, wbase + s * STEP, 2 * 4096, lane16);
    });

    __syncthreads();
    if (lane < 4) {
        const int64_t t = t0 + wave * 4 + lane;
        const int32_t p = t < T ? position_of(t, R, staged ? ro_lds : ro) : 0;
        if (t < T) pos[t] = p;
        pos_lds[wave * 4 + lane] = p;
    }
    if (tid < 64) inv[tid] = pow(10000.0, -2.0 * (double)tid / 128.0);
    if (blockIdx.x == 0 && tid == 0) {
        offs[0] = 0;
        offs[1] = (int32_t)T;
    }
    __syncthreads();
    // The angles while the rows are on their way.
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int i = (tid >> 5) + 16 * j;
        double sn, c;
        sincos((double)pos_lds[l32] * inv[i], &sn, &c);
        cs[i * TOK + l32] = make_double2(c, sn);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t t = t0 + wave * 4 + j;
        const float v[8] = {bf16_lo(e[j][0]), bf16_hi(e[j][0]), bf16_lo(e[j][1]), bf16_hi(e[j][1]),
                            bf16_lo(e[j][2]), bf16_hi(e[j][2]), bf16_lo(e[j][3]), bf16_hi(e[j][3])};
        float ss = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) ss = fmaf(v[k], v[k], ss);
        const float r = 1.0f / sqrtf(wave_sum_bcast(ss) / (float)D + eps);
        const u32x4 o = {pack2(v[0] * r, v[1] * r), pack2(v[2] * r, v[3] * r),
                         pack2(v[4] * r, v[5] * r), pack2(v[6] * r, v[7] * r)};
        rows[row_slot(lane, wave * 4 + j)] = o;
        if (t < T) {
            f32x4* xd = reinterpret_cast<f32x4*>(x + t * D + lane * 8);
            xd[0] = f32x4{v[0], v[1], v[2], v[3]};
            xd[1] = f32x4{v[4], v[5], v[6], v[7]};
            *reinterpret_cast<u32x4*>(a + t * D + lane * 8) = o;
        }
    }
    __syncthreads();
    const int64_t t = t0 + l32;
    const bool ok = t < T;
    uint16_t* qrow = qkv + (ok ? t : 0) * (3 * D);
    for (int p = 0; p < 3; ++p) {
        f32x16 acc[2];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][r] = 0.0f;
        const char* here = wbase + p * (D / 32) * 4096;
        const char* then = p < 2 ? here + (D / 32) * 4096 : here;  // the last pass re-reads
        static_for<0, NKD>([&](auto kc) {
            constexpr int kt = decltype(kc)::value, s = kt % S;
            mfma_step<s>(w, rows, kt, l32, half, acc);
            load_step<s>(w, kt + S < NKD ? here + (kt + S) * STEP : then + (kt + S - NKD) * STEP,
                         2 * 4096, lane16);
        });
        float lo[16], hi[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            lo[r] = acc[0][r];
            hi[r] = acc[1][r];
            if (p < 2) {  // rotate the rounded projections in fp64
                const int i = (wave & 1) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                const double2 z = cs[i * TOK + l32];
                const double av = (double)bf16_lo(f32_to_bf16(lo[r]));
                const double bv = (double)bf16_lo(f32_to_bf16(hi[r]));
                lo[r] = (float)(av * z.x - bv * z.y);
                hi[r] = (float)(bv * z.x + av * z.y);
            }
        }
        const int grp = p * (D / 32) + (wave >> 1) * 4 + (wave & 1);
        put_group(lo, grp, l32, half, ok, qrow, nullptr);
        put_group(hi, grp + 2, l32, half, ok, qrow, nullptr);
    }
}

// 1 / rms of each token's row held as two 32-column groups per wave: each lane
// sums its 32 values, then its other half, then the waves in order.  Ends
// after a barrier (and reads of LDS rows before the call are complete).
__device__ __forceinline__ float row_rms(const f32x16 (&v)[2], float eps, float (&part)[NW][TOK],
                                         int wave, int l32, int half) {
    float ss = 0.0f;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r) ss = fmaf(v[g][r], v[g][r], ss);
    ss += __shfl_xor(ss, 32, 64);
    if (half == 0) part[wave][l32] = ss;
    __syncthreads();
    float tot = 0.0f;
#pragma unroll
    for (int i = 0; i < NW; ++i) tot += part[i][l32];
    return 1.0f / sqrtf(tot / (float)D + eps);
}

// Wo + residual, norm, SwiGLU MLP + residual, norm, gate.
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
void k_router_tail(int64_t T, int Fp, int E, float eps, const uint16_t* __restrict__ o,
                   const char* __restrict__ wo, const char* __restrict__ mlp,
                   const uint16_t* __restrict__ gate, const float* __restrict__ bias,
                   float* __restrict__ x, uint16_t* __restrict__ m, uint16_t* __restrict__ h,
                   uint16_t* __restrict__ f, int32_t* __restrict__ ids,
                   float* __restrict__ logits) {
    __shared__ u32x4 rows[NKD * KSLOTS];                       // o, then m, then f
    __shared__ u32x4 hrows[kFusedRouterMlp / 64 * KSLOTS];     // the hidden rows
    __shared__ float part[2][NW][TOK];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * TOK;
    const int64_t t = t0 + l32;
    const bool ok = t < T;

    u32x4 orow[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int64_t r = t0 + wave * 4 + j;
        r = r < T ? r : T - 1;
        orow[j] = *reinterpret_cast<const u32x4*>(o + r * D + lane * 8);
    }
    f32x16 acc[2];
    float* xrow = x + (ok ? t : T - 1) * D;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 v =
                *reinterpret_cast<const f32x4*>(xrow + (wave * 2 + g) * 32 + 8 * i + 4 * half);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[g][4 * i + r] = v[r];
        }

    // The weight stream, one K-step of two groups at a time: Wo, then the
    // gate/up passes of 256 neurons (group pair 2n, 2n + 1 of neuron group n =
    // pass * 8 + wave, clamped), then W2.
    const int passes = (Fp + 255) / 256, nf = Fp / 64;
    const int first_mlp = NKD, first_w2 = NKD * (1 + passes), total = first_w2 + nf;
    const char* w2 = mlp + (int64_t)2 * Fp * D * 2;
    const uint32_t lane16 = lane * 16;
    auto address = [&](int n) {
        n = n < total ? n : total - 1;
        if (n < first_mlp) return wo + (int64_t)n * (D / 32) * 4096 + wave * 2 * 4096;
        if (n < first_w2) {
            const int q = n - first_mlp, ng = min((q / NKD) * NW + wave, Fp / 32 - 1);
            return mlp + ((int64_t)(q % NKD) * (2 * Fp / 32) + ng * 2) * 4096;
        }
        return w2 + ((int64_t)(n - first_w2) * (D / 32) + wave * 2) * 4096;
    };
    WeightRing w;
    static_for<0, S>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        load_step<s>(w, address(s), 4096, lane16);
    });
#pragma unroll
    for (int j = 0; j < 4; ++j) rows[row_slot(lane, wave * 4 + j)] = orow[j];
    __syncthreads();

    int n = 0;  // K-step of the stream
    auto product = [&](const u32x4* src) {  // one product over D
        static_for<0, NKD>([&](auto kc) {
            constexpr int kt = decltype(kc)::value, s = kt % S;
            mfma_step<s>(w, src, kt, l32, half, acc);
            load_step<s>(w, address(n + kt + S), 4096, lane16);
        });
        n += NKD;
    };
    product(rows);  // x1 = x + o Wo^T
    f32x16 x1[2] = {acc[0], acc[1]};
    const float r1 = row_rms(x1, eps, part[0], wave, l32, half);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = x1[g][r] * r1;
        put_group(v, wave * 2 + g, l32, half, ok, m + (ok ? t : 0) * D, rows);
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[g][r] = 0.0f;
        product(rows);
        const int ng = p * NW + wave;
        if (ng < Fp / 32) {
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = silu_f32(acc[0][r]) * acc[1][r];
            put_group(v, ng, l32, half, ok, h + (ok ? t : 0) * Fp, hrows);
        }
    }
    __syncthreads();
    acc[0] = x1[0];
    acc[1] = x1[1];
    for (int kt = 0; kt < nf; kt += S)
        static_for<0, S>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if (kt + s < nf) {
                mfma_step<s>(w, hrows, kt + s, l32, half, acc);
                load_step<s>(w, address(n + kt + s + S), 4096, lane16);
            }
        });
    if (ok) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<f32x4*>(xrow + (wave * 2 + g) * 32 + 8 * i + 4 * half) =
                    f32x4{acc[g][4 * i], acc[g][4 * i + 1], acc[g][4 * i + 2], acc[g][4 * i + 3]};
    }
    const float r2 = row_rms(acc, eps, part[1], wave, l32, half);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = acc[g][r] * r2;
        put_group(v, wave * 2 + g, l32, half, ok, f + (ok ? t : 0) * D, rows);
    }
    __syncthreads();

    // The gate, readme_route's canonical order: lane l holds 16-byte chunk l
    // of the row (D / 8 = 64 chunks), fused multiply-adds in ascending k from
    // +0, the pairwise fold 32 .. 1, then the bias; the first largest wins.
    float fv[4][8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const u32x4 c = rows[row_slot(lane, wave * 4 + j)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            fv[j][2 * k] = bf16_lo(c[k]);
            fv[j][2 * k + 1] = bf16_hi(c[k]);
        }
    }
    float best[4];
    int best_e[4];
    for (int e = 0; e < E; ++e) {
        const u32x4 c = *reinterpret_cast<const u32x4*>(gate + (int64_t)e * D + lane * 8);
        float p[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[j] = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                p[j] = fmaf(fv[j][2 * k], bf16_lo(c[k]), p[j]);
                p[j] = fmaf(fv[j][2 * k + 1], bf16_hi(c[k]), p[j]);
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int j = 0; j < 4; ++j) p[j] = p[j] + __shfl_down(p[j], off, 64);
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t tt = t0 + wave * 4 + j;
                const float lg = bias ? p[j] + bias[e] : p[j];
                if (logits && tt < T) logits[tt * E + e] = lg;
                if (e == 0 || lg > best[j]) {
                    best[j] = lg;
                    best_e[j] = e;
                }
            }
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t0 + wave * 4 + j < T) ids[t0 + wave * 4 + j] = best_e[j];
    }
}

}  // namespace

hipError_t launch_router_head(int64_t T, int32_t R, int64_t V, float eps, const int32_t* tokens,
                              const int32_t* ro, const void* emb, float* x, uint16_t* a,
                              int32_t* pos, int32_t* offs, const void* wqkv, uint16_t* qkv,
                              hipStream_t s) {
    k_router_head<<<(unsigned)ceil_div(T, TOK), NW * 64, 0, s>>>(
        T, R, V, eps, tokens, ro, reinterpret_cast<const uint16_t*>(emb), x, a, pos, offs,
        reinterpret_cast<const char*>(wqkv), qkv);
    return hipGetLastError();
}

hipError_t launch_router_tail(int64_t T, int64_t F, int E, float eps, const uint16_t* o,
                              const void* wo, const void* mlp, const void* gate, const float* bias,
                              float* x, uint16_t* m, uint16_t* h, uint16_t* f, int32_t* ids,
                              float* logits, hipStream_t s) {
    k_router_tail<<<(unsigned)ceil_div(T, TOK), NW * 64, 0, s>>>(
        T, (int)padded_I(F), E, eps, o, reinterpret_cast<const char*>(wo),
        reinterpret_cast<const char*>(mlp), reinterpret_cast<const uint16_t*>(gate), bias, x, m, h,
        f, ids, logits);
    return hipGetLastError();
}

}  // namespace readme
