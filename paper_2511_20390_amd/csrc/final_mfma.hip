// Final layer of the DiT (LayerNorm without affine, per-sample modulate, linear D -> p*p*C_out,
// unpatchify to [B, C_out, H, W]) on the matrix cores, bf16 or fp32 weights.
//
// One workgroup per 16 token rows, four wavefronts that split the hidden dimension in four
// contiguous quarters: a lane holds its 8-float pieces of the quarter in registers (72 floats at
// D = 1152), so the rows are read from memory exactly once, all workgroups' loads are in flight
// together, and the two-pass statistics (mean, then centred variance) run on registers with one
// small LDS exchange between the wavefronts each.  The normalised, modulated values are split into
// a bf16 high part and a bf16 remainder (two v_mfma_f32_16x16x32_bf16 per k-step), so the fp32
// activations lose nothing that matters against the fp32 accumulation; weight rows are the A
// operand, read from global memory (L2) in operand layout.  The four partial 32 x 16 products are
// added through LDS and scattered to the image layout.
// With fp32 weights the same pieces feed v_mfma_f32_16x16x4_f32, eight per k-step and output tile (2 x 256 rows of 1152 35 -> 11.6 us
// against the kernel of one wavefront per row, 12 x 1024 rows 122 -> 30).  The instruction adds its products one after the other, so that
// all of a wavefront's in one accumulator are a chain of 288 roundings; two instructions at a time and their sums pair by pair are
// as short a chain as the other kernel's: 2-norm error against 64 bits at width 384 / 768 / 1024 / 1152 one wavefront per row 1.30e-7 /
// 1.29e-7 / 1.19e-7 / 1.40e-7, one accumulator 2.2e-7 / 2.9e-7 / 3.1e-7 / 3.5e-7 (10.6 us), here 1.29e-7 / 1.28e-7 / 1.15e-7 / 1.33e-7.
//
// The per-row kernel this replaces re-read the whole weight matrix (74 KB) from cache for every
// token row and reduced each of the 32 outputs across the wavefront separately: 120 us at 12288
// rows against 10 us for reading the rows once.
#include "free_internal.h"
#include "lanes.h"

#include <type_traits>

namespace freemi {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float float8_t __attribute__((ext_vector_type(8), aligned(16)));

// Sum of N values added pair by pair, pairs pair by pair, ...: a value passes log2 N roundings instead of up to N.  add() in order, i known
// at compile time.
template <int N, typename T>
struct PairSum {
    T level[32 - __builtin_clz(N)] = {};           // level l: 2^l values, where bit l of the number of values is set
    __device__ __forceinline__ void add(int i, T v) {
        int l = 0;
        for (; (i >> l) & 1; ++l) v = level[l] + v;
        level[l] = v;
    }
    __device__ __forceinline__ T result() const {
        T v = {};
        bool first = true;
#pragma unroll
        for (int l = 0; l < 32 - __builtin_clz(N); ++l) {
            if (!((N >> l) & 1)) continue;
            v = first ? level[l] : level[l] + v;
            first = false;
        }
        return v;
    }
};

constexpr int kThreads = 256;
constexpr int kRows = 16;                 // token rows per workgroup (the N dimension of the MFMA)

// kMean: what a drafting step computes from the noise estimates (FinalMean) in their place.  The rows of a workgroup are then 16 / dup
// tokens of each state, so that both estimates of a pixel are in one wavefront, eight lanes apart.  A launch less per step, of 2.9 us
// at 256 tokens and 4.7 at 2 x 1024.
template <typename WT, int NS, bool kMean>            // NS: k-steps of 32 per wavefront, D = 128 NS
__global__ __launch_bounds__(kThreads) void final_layer_mfma_kernel(
    const float* __restrict__ x, RowVec shift, RowVec scale, int32_t M, int32_t gh, int32_t gw, int32_t p,
    int32_t c_out, const WT* __restrict__ w, const float* __restrict__ bias, float* __restrict__ out,
    FinalMean step) {
    constexpr int D = 128 * NS;
    constexpr bool kF32 = std::is_same<WT, float>::value;
    __shared__ float red[2][4][kRows];
    __shared__ __attribute__((aligned(16))) float part[4][2][64][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lq = lane >> 4;
    const int ntok = gh * gw;
    int row = blockIdx.x * kRows + l16;
    bool stored = row < M;
    row = stored ? row : M - 1;                                    // rows past M repeat the last one, never stored
    if constexpr (kMean) {
        const int per = kRows / step.dup, state = l16 / per, n = blockIdx.x * per + l16 - state * per;
        stored = state == 0 && n < ntok;
        row = state * ntok + (n < ntok ? n : ntok - 1);
    }
    const int k0 = wave * NS * 32 + lq * 8;                        // + 32 s: this lane's 8 columns of k-step s
    const float* xr = x + static_cast<int64_t>(row) * D + k0;
    f32x4_t xa[NS][2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        xa[s][0] = *reinterpret_cast<const f32x4_t*>(xr + 32 * s);
        xa[s][1] = *reinterpret_cast<const f32x4_t*>(xr + 32 * s + 4);
    }
    // Where this thread's sums go (the first two wavefronts: outputs 16 t + 4 (lane / 16) + i of token row lane % 16) and their bias:
    // some twenty divisions, done while the loads above are under way.
    const int P = p * p * c_out;
    int64_t dst[4];
    float bias_out[4];
    [[maybe_unused]] float x_in[4], xi_in[4], cx, ce, sg;
    if (wave < 2) {
        if constexpr (kMean) {
            cx = *step.coef_x;
            ce = *step.coef_eps;
            sg = *step.sigma;
        }
        const int b = row / ntok, n = row - b * ntok, gi = n / gw, gj = n - gi * gw;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = 16 * wave + 4 * lq + i, oc = o < P ? o : 0;
            const int pp = oc / c_out, c = oc - pp * c_out, ph = pp / p, pq = pp - ph * p;
            const bool on = o < P && stored && (!kMean || c < step.C);
            dst[i] = on ? ((static_cast<int64_t>(b) * c_out + c) * gh * p + gi * p + ph) * gw * p + gj * p + pq : -1;
            bias_out[i] = bias[oc];
            if constexpr (kMean) {
                x_in[i] = step.x[on ? dst[i] : 0];
                xi_in[i] = step.xi[on ? dst[i] : 0];
            }
        }
    }
    // a row lives in the four lanes l16 + 16 lq of each of the four wavefronts
    auto row_total = [&](float v, int slot) {
        v = add_lane_xor<32>(add_lane_xor<16>(v));
        if (lq == 0) red[slot][wave][l16] = v;
        __syncthreads();
        return (red[slot][0][l16] + red[slot][1][l16]) + (red[slot][2][l16] + red[slot][3][l16]);
    };
    // this lane's pieces of a sum: one after the other, in fp32 pair by pair (PairSum)
    auto lane_total = [&](auto&& piece) {
        std::conditional_t<kF32, PairSum<2 * NS, float>, float> total{};
#pragma unroll
        for (int j = 0; j < 2 * NS; ++j) {
            if constexpr (kF32) total.add(j, piece(xa[j >> 1][j & 1]));
            else total += piece(xa[j >> 1][j & 1]);
        }
        if constexpr (kF32) return total.result();
        else return total;
    };
    const float mean = row_total(lane_total([](const f32x4_t& v) { return (v[0] + v[1]) + (v[2] + v[3]); }), 0) / static_cast<float>(D);
    const float q = lane_total([&](const f32x4_t& v) {
        const float a = v[0] - mean, b = v[1] - mean, c = v[2] - mean, d = v[3] - mean;
        return (a * a + b * b) + (c * c + d * d);
    });
    const float rstd = rsqrtf(row_total(q, 1) / static_cast<float>(D) + kLnEps);

    const float* shr = shift.base + static_cast<int64_t>(row / shift.rows_per_sample) * shift.stride + k0;
    const float* scr = scale.base + static_cast<int64_t>(row / scale.rows_per_sample) * scale.stride + k0;
    f32x4_t acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    [[maybe_unused]] PairSum<4 * NS, f32x4_t> sums[2];       // fp32: of eight products each, see below
    // k-steps in groups of kG: the shift, scale and weight pieces of a whole group are requested together and
    // only then used - one memory round trip per group on the critical path of the workgroup instead of two per
    // k-step (left to itself the compiler keeps 72 registers and waits for every piece where it is used)
    // (groups of two: 152 registers at NS = 9, three wavefronts per SIMD - every workgroup of a 12288-row launch
    // resident at once; groups of three need 176 and were slower there)
    constexpr int kG = 2;
#pragma unroll
    for (int g0 = 0; g0 < NS; g0 += kG) {
        f32x4_t shv[kG][2], scv[kG][2];
        std::conditional_t<kF32, float8_t, u32x4_t> wv[kG][2];          // eight weights
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            const int s = g0 + u;
            if (s >= NS) continue;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                shv[u][h] = *reinterpret_cast<const f32x4_t*>(shr + 32 * s + 4 * h);
                scv[u][h] = *reinterpret_cast<const f32x4_t*>(scr + 32 * s + 4 * h);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int o = 16 * t + l16;
                // (outputs past P re-read row 0 and are multiplied into columns that are never stored)
                wv[u][t] = *reinterpret_cast<decltype(&wv[0][0])>(const_cast<WT*>(w + static_cast<int64_t>(o < P ? o : 0) * D + k0 + 32 * s));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kG; ++u) {
            const int s = g0 + u;
            if (s >= NS) continue;
            float v[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = fmaf((xa[s][c >> 2][c & 3] - mean) * rstd, 1.0f + scv[u][c >> 2][c & 3], shv[u][c >> 2][c & 3]);
            if constexpr (kF32) {
                // element e: the four lane groups hold four k of one product
#pragma unroll
                for (int e = 0; e < 8; e += 2)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const float a0 = wv[u][t][e], a1 = wv[u][t][e + 1];
                        const bool on = 16 * t + l16 < P;
                        f32x4_t r = __builtin_amdgcn_mfma_f32_16x16x4f32(on ? a0 : 0.f, v[e], f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                        r = __builtin_amdgcn_mfma_f32_16x16x4f32(on ? a1 : 0.f, v[e + 1], r, 0, 0, 0);
                        sums[t].add(4 * s + e / 2, r);
                    }
            } else {
                uint32_t hi[4], lo[4];
#pragma unroll
                for (int c2 = 0; c2 < 4; ++c2) {
                    const uint32_t hp = pack_bf16_pair(v[2 * c2], v[2 * c2 + 1]);
                    hi[c2] = hp;
                    lo[c2] = pack_bf16_pair(v[2 * c2] - __uint_as_float(hp << 16), v[2 * c2 + 1] - __uint_as_float(hp & 0xffff0000u));
                }
                const bf16x8_t bh = __builtin_bit_cast(bf16x8_t, u32x4_t{hi[0], hi[1], hi[2], hi[3]});
                const bf16x8_t bl = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], lo[2], lo[3]});
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const bf16x8_t a = __builtin_bit_cast(bf16x8_t, 16 * t + l16 < P ? wv[u][t] : u32x4_t{0, 0, 0, 0});
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bh, acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc[t], 0, 0, 0);
                }
            }
        }
    }
    if constexpr (kF32) {
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = sums[t].result();
    }
    // accumulator register i of lane l: output 16 t + 4 (l / 16) + i, token row l % 16
#pragma unroll
    for (int t = 0; t < 2; ++t) *reinterpret_cast<f32x4_t*>(part[wave][t][lane]) = acc[t];
    __syncthreads();
    if (wave < 2) {
        f32x4_t from[4], v;
#pragma unroll
        for (int wv = 0; wv < 4; ++wv) from[wv] = *reinterpret_cast<const f32x4_t*>(part[wv][wave][lane]);
        v = kF32 ? (from[0] + from[1]) + (from[2] + from[3]) : ((from[0] + from[1]) + from[2]) + from[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float e = v[i] + bias_out[i];
            if constexpr (!kMean) {
                if (dst[i] >= 0) out[dst[i]] = e;
            } else {
                const float null = lane_xor<8>(e);
                if (step.dup == 2) e = fmaf(step.cfg_scale, e - null, null);
                const float m = fmaf(cx, x_in[i], ce * e);
                if (dst[i] < 0) continue;
                step.m[dst[i]] = m;
                step.x_next[dst[i]] = fmaf(sg, xi_in[i], m);
                if (step.x_copy) step.x_copy[dst[i]] = x_in[i];
            }
        }
    }
}

}  // namespace

// bf16 or fp32 weights, D one of 384 / 768 / 1024 / 1152 (the DiT-S/B/L/XL widths), at most 32 outputs per
// token, 16-byte aligned rows of x, the weights and the modulation vectors.
bool final_mfma_supported(int32_t D, int32_t P) {
    return (D == 384 || D == 768 || D == 1024 || D == 1152) && P >= 1 && P <= 32;
}

int32_t launch_final_layer_mfma(const float* x, RowVec shift, RowVec scale, int32_t M, int32_t gh, int32_t gw,
                                int32_t p, int32_t c_out, int32_t D, const void* w, int32_t dtype, const float* bias,
                                float* out, hipStream_t s, const FinalMean* mean) {
    const int per = mean ? kRows / mean->dup : kRows, rows = mean ? gh * gw : M;
    const dim3 grid((rows + per - 1) / per), block(kThreads);
    const FinalMean fm = mean ? *mean : FinalMean{};
#define FREE_FIN_MFMA(WT, NS, MEAN)                                                                                            \
    hipLaunchKernelGGL((final_layer_mfma_kernel<WT, NS, MEAN>), grid, block, 0, s, x, shift, scale, M, gh, gw, p, c_out,       \
                       static_cast<const WT*>(w), bias, out, fm)
#define FREE_FIN_CASE(NS)                                                   \
    do {                                                                    \
        if (dtype == FREE_BF16 && mean) FREE_FIN_MFMA(bf16_t, NS, true);    \
        else if (dtype == FREE_BF16) FREE_FIN_MFMA(bf16_t, NS, false);      \
        else if (mean) FREE_FIN_MFMA(float, NS, true);                      \
        else FREE_FIN_MFMA(float, NS, false);                               \
    } while (0)
    switch (D) {
        case 384: FREE_FIN_CASE(3); break;
        case 768: FREE_FIN_CASE(6); break;
        case 1024: FREE_FIN_CASE(8); break;
        case 1152: FREE_FIN_CASE(9); break;
        default: return FREE_ERR_SHAPE;
    }
#undef FREE_FIN_CASE
#undef FREE_FIN_MFMA
    return launch_ok() ? FREE_OK : FREE_ERR_HIP;
}

}  // namespace freemi
