// Device code shared by the matrix-core GEMM kernels: operand types, the order in which the tiles of an output are
// walked, and the epilogue that turns accumulators into output (bias / GELU / gated residual update / folded LayerNorm).
#pragma once

#include <type_traits>

#include "free_internal.h"
#include "lanes.h"

namespace freemi {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int BK = 64;                    // bf16 elements per K slice (128 bytes per row)
constexpr int kRowBytes = BK * 2;
constexpr int kNumXcd = 8;

__device__ inline float gelu_fast(float v) {
    // tanh-form GELU: 0.5 v (1 + tanh(u)) = v / (1 + exp(-2u)), u = sqrt(2/pi)(v + 0.044715 v^3)
    // exp(-2u) = 2^(v (a + b v^2)) with the constants folded; v_exp_f32 and v_rcp_f32 directly (1 ulp each,
    // far below the bf16 rounding of the result).  The correctly rounded reciprocal is a ten-instruction
    // division sequence per element, and this runs on every element of the MLP's hidden layer while the
    // matrix cores wait.  2^t overflows to +inf for very negative v: 1 / inf = 0, the right limit.
    constexpr float a = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
    constexpr float b = a * 0.044715f;
    const float t = v * fmaf(v * v, b, a);
    return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

__device__ inline uint32_t pack2(float lo, float hi) {
    const f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));   // v_cvt_pk_bf16_f32 (RNE)
}

// Issue-order hints for one k-step of MF MFMAs: every MFMA is followed by at most one
// fragment read (NR of them), one LDS write (NW) and one global load (NL), so the matrix
// pipe never waits behind a burst of memory instructions.
constexpr int kMfma = 0x008, kVmemRd = 0x020, kDsRd = 0x100, kDsWr = 0x200;
template <int Q, int MF, int NR, int NW, int NL>
__device__ __forceinline__ void sched_hints() {
    if constexpr (Q < MF) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
        if constexpr (Q < NR) __builtin_amdgcn_sched_group_barrier(kDsRd, 1, 0);
        if constexpr (Q < NW) __builtin_amdgcn_sched_group_barrier(kDsWr, 1, 0);
        if constexpr (Q < NL) __builtin_amdgcn_sched_group_barrier(kVmemRd, 1, 0);
        sched_hints<Q + 1, MF, NR, NW, NL>();
    } else {
        __builtin_amdgcn_sched_barrier(0);
    }
}

// XCD-aware tile order: workgroup ids are dealt round-robin to the 8 XCDs, so the
// ids of one XCD are made contiguous first, then walked in groups of kGroupM row
// tiles (column-major inside a group) so concurrent workgroups share X and W panels.
__device__ inline int xcd_tile(int pid, int total) {
    const int q = total / kNumXcd, r = total % kNumXcd;
    const int x = pid % kNumXcd, j = pid / kNumXcd;
    return x * q + (x < r ? x : r) + j;
}

__device__ inline void tile_coords(int kGroupM, int pid, int tiles_m, int tiles_n, int* tm, int* tn) {
    const int npid = xcd_tile(pid, tiles_m * tiles_n);
    const int per_group = kGroupM * tiles_n;
    const int group = npid / per_group;
    const int first_m = group * kGroupM;
    const int gsize = (tiles_m - first_m < kGroupM) ? tiles_m - first_m : kGroupM;
    const int in_group = npid % per_group;
    *tm = first_m + in_group % gsize;
    *tn = in_group / gsize;
}

// Epilogue shared by the GEMM kernels.  Register e of acc[i][j] in lane l is output row
// m = gm_lane + 32 i (gm_lane already includes l % 32), column n = gn_wave + 32 j + 8 (e/4) + 4 lhi + e%4.
// QB: for the residual update, chunks per lane whose loads are in flight together in the LDS-staged form; 0
// selects the direct form.
// Folded LayerNorm (see LnFold): kPrep - the residual update also writes z, and the sums of x and x^2 over this
// wavefront's 64 columns to row_sums[row in the wavefront's part * row_sums_stride + 0 / 1] (LDS; the caller adds the two
// halves of a 128-column slot);
// kLn - the accumulators hold z W^T - mu c1 + c0 / r (the kernel adds the rank-2 term as an extra k-step before
// its K loop), so the output is r acc with the per-row factor ln_a = r of this lane's rows: no bias, one
// multiplication per element.
template <typename OT, int TM, int TN, int EPI, int QB>
__device__ __forceinline__ void write_tile(const f32x16_t (&acc)[TM][TN], int gm_lane, int gn_wave, int lane, int32_t M,
                                           int32_t N, int32_t vec_ok, const float* __restrict__ bias,
                                           OT* __restrict__ out, float* __restrict__ resid, const RowVec& gate,
                                           char* wave_lds, const LnFold& ln, const float (&ln_a)[TM],
                                           float* row_sums = nullptr, int row_sums_stride = 0) {
    constexpr bool kF32Out = std::is_same<OT, float>::value;   // fp32 mode: the output of the bias / GELU epilogues is fp32
    constexpr bool kPrep = EPI == FREE_EPI_GATE_RESID_PREP;
    constexpr bool kResid = EPI == FREE_EPI_GATE_RESID || kPrep;
    constexpr bool kLn = EPI == FREE_EPI_LN_BIAS || EPI == FREE_EPI_LN_BIAS_GELU;
    constexpr bool kGelu = EPI == FREE_EPI_BIAS_GELU || EPI == FREE_EPI_LN_BIAS_GELU;
    static_assert(!kPrep || (QB > 0 && TN == 2), "z and the row sums come out of the staged residual update of a 64-column wavefront");
    static_assert(!kLn || !kF32Out, "folded LayerNorm: bf16 path only");
    const int lhi = lane >> 5;
    if (vec_ok) {
        // N % 8 == 0 and 16-byte aligned rows: runs of 4 / 8 columns are all inside or all outside.
        // Rows past M and runs past N (ragged edge tiles) are masked per lane.
        if constexpr (kF32Out && !kResid && QB == 0) {
            // fp32 output straight from the accumulator layout (four-wavefront configurations)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int gn0 = gn_wave + j * 32 + 4 * lhi;
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    if (gn0 + 8 * e4 >= N) continue;
                    const f32x4_t bv = *reinterpret_cast<const f32x4_t*>(bias + gn0 + 8 * e4);
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int gm = gm_lane + i * 32;
                        if (gm >= M) continue;
                        f32x4_t o;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            o[c] = acc[i][j][4 * e4 + c] + bv[c];
                            if (kGelu) o[c] = gelu_fast(o[c]);
                        }
                        *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(out) + static_cast<int64_t>(gm) * N + gn0 + 8 * e4) = o;
                    }
                }
            }
        } else if constexpr (EPI == FREE_EPI_GATE_RESID && QB == 0) {
            // read-modify-write of the fp32 residual stream straight from the accumulator layout (32 rows x
            // 32 bytes per instruction).  All loads of a column tile j are issued before its first store (a
            // store would otherwise fence the following loads).  Faster than the staged form below for the
            // four-wavefront configurations: with one wavefront per SIMD the LDS round trip is not hidden.
            const float* __restrict__ gbase = gate.base;
            int64_t g_off[TM], r_off[TM];
            bool row_ok[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int gm = gm_lane + i * 32;
                row_ok[i] = gm < M;
                g_off[i] = static_cast<int64_t>(gm / gate.rows_per_sample) * gate.stride;
                r_off[i] = static_cast<int64_t>(gm) * N;
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int gn0 = gn_wave + j * 32 + 4 * lhi;
                f32x4_t bv[4], g[TM][4], r[TM][4];
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4)
                    if (gn0 + 8 * e4 < N) bv[e4] = *reinterpret_cast<const f32x4_t*>(bias + gn0 + 8 * e4);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4)
                        if (row_ok[i] && gn0 + 8 * e4 < N) {
                            g[i][e4] = *reinterpret_cast<const f32x4_t*>(gbase + g_off[i] + gn0 + 8 * e4);
                            r[i][e4] = *reinterpret_cast<const f32x4_t*>(resid + r_off[i] + gn0 + 8 * e4);
                        }
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int e4 = 0; e4 < 4; ++e4)
                        if (row_ok[i] && gn0 + 8 * e4 < N) {
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                r[i][e4][c] = fmaf(g[i][e4][c], acc[i][j][4 * e4 + c] + bv[e4][c], r[i][e4][c]);
                            *reinterpret_cast<f32x4_t*>(resid + r_off[i] + gn0 + 8 * e4) = r[i][e4];
                        }
            }
        } else if constexpr (kResid || kF32Out) {
            // read-modify-write of the fp32 residual stream (or, in fp32 mode, the plain fp32 output of the
            // bias / GELU epilogues: same staging, no read).  As for the bf16 output below, the accumulator
            // layout would touch 32 rows x 32 bytes per instruction; each 32-row block is staged in the
            // wave-private LDS region CG column tiles at a time (rows padded by 16 bytes) and read back
            // row-major, so that the loads and stores of the residual cover whole 128-byte lines.
            constexpr int CG = (TN % 2 == 0) ? 2 : 1;          // column tiles per staged group (rows of 256 / 128 bytes)
            constexpr int CH = CG * 8;                         // 16-byte chunks (4 floats) per staged row
            constexpr int kStageRow = (CH + 1) * 16;
            constexpr int NQ = 32 * CH / 64;                   // chunks per lane per group
            const int l32 = lane & 31;
            const float* __restrict__ gbase = gate.base;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int gm_blk = gm_lane - l32 + i * 32;     // first row of the block (wave-uniform)
                // one sample for the whole block (the usual case: rows per sample a multiple of 32)?
                const int s_first = gm_blk / gate.rows_per_sample;
                const bool one_sample = (gm_blk + 31) / gate.rows_per_sample == s_first;
                // kPrep: sums of x and x^2 over this wavefront's 64 columns, for the rows 4 q + lane / 16 of the block
                // (ps[2 q], ps[2 q + 1]); this lane adds the four columns of its chunk in each staged group
                [[maybe_unused]] float ps[2 * NQ];
                if constexpr (kPrep) {
#pragma unroll
                    for (int k = 0; k < 2 * NQ; ++k) ps[k] = 0.f;
                }
#pragma unroll
                for (int jg = 0; jg < TN; jg += CG) {
#pragma unroll
                    for (int jj = 0; jj < CG; ++jj)
#pragma unroll
                        for (int e4 = 0; e4 < 4; ++e4) {
                            const f32x4_t v = {acc[i][jg + jj][4 * e4], acc[i][jg + jj][4 * e4 + 1],
                                               acc[i][jg + jj][4 * e4 + 2], acc[i][jg + jj][4 * e4 + 3]};
                            // columns jj*32 + 8 e4 + 4 lhi .. +3 -> chunk 8 jj + 2 e4 + lhi
                            *reinterpret_cast<f32x4_t*>(wave_lds + l32 * kStageRow + ((8 * jj + 2 * e4 + lhi) << 4)) = v;
                        }
                    // batches of 4 chunks per lane: all loads of a batch before its first store, and few
                    // enough registers beside the accumulators.  A lane's chunks of a group are the same four
                    // columns of different rows (64 % CH == 0), so the bias and - when the block lies in one sample -
                    // the gate and the next scale are loaded once per group, not once per chunk: per chunk they
                    // would quadruple what the epilogue pulls through the L1.
                    constexpr int QN = (QB > 0 && QB < NQ) ? QB : NQ;
                    static_assert(NQ % QN == 0 && 64 % CH == 0, "whole batches; one chunk column per lane");
                    const int gn = gn_wave + jg * 32 + (lane % CH) * 4;
                    f32x4_t bvc = {0.f, 0.f, 0.f, 0.f}, gc = {0.f, 0.f, 0.f, 0.f};
                    [[maybe_unused]] f32x4_t snc = {0.f, 0.f, 0.f, 0.f};
                    if (gn < N) {
                        bvc = *reinterpret_cast<const f32x4_t*>(bias + gn);
                        if constexpr (kResid) {
                            if (one_sample) {
                                gc = *reinterpret_cast<const f32x4_t*>(gbase + static_cast<int64_t>(s_first) * gate.stride + gn);
                                if constexpr (kPrep)
                                    snc = *reinterpret_cast<const f32x4_t*>(ln.scale_next + static_cast<int64_t>(s_first) * gate.stride + gn);
                            }
                        }
                    }
#pragma unroll
                    for (int q0 = 0; q0 < NQ; q0 += QN) {
                        f32x4_t r[QN], g[QN];
                        [[maybe_unused]] f32x4_t sn[QN];
                        int64_t off[QN];
                        bool ok[QN];
#pragma unroll
                        for (int q = 0; q < QN; ++q) {
                            const int f = (q0 + q) * 64 + lane;
                            const int gm = gm_blk + f / CH;
                            ok[q] = gm < M && gn < N;
                            off[q] = static_cast<int64_t>(gm) * N + gn;
                            g[q] = gc;
                            if constexpr (kPrep) sn[q] = snc;
                            if (ok[q]) {
                                if constexpr (kResid) {
                                    r[q] = *reinterpret_cast<const f32x4_t*>(resid + off[q]);
                                    if (!one_sample) {
                                        const int64_t so = static_cast<int64_t>(gm / gate.rows_per_sample) * gate.stride + gn;
                                        g[q] = *reinterpret_cast<const f32x4_t*>(gbase + so);
                                        if constexpr (kPrep) sn[q] = *reinterpret_cast<const f32x4_t*>(ln.scale_next + so);
                                    }
                                }
                            }
                        }
#pragma unroll
                        for (int q = 0; q < QN; ++q)
                            if (ok[q]) {
                                const int f = (q0 + q) * 64 + lane;
                                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(wave_lds + (f / CH) * kStageRow + ((f % CH) << 4));
                                if constexpr (kResid) {
#pragma unroll
                                    for (int c = 0; c < 4; ++c) r[q][c] = fmaf(g[q][c], v[c] + bvc[c], r[q][c]);
                                    *reinterpret_cast<f32x4_t*>(resid + off[q]) = r[q];
                                    if constexpr (kPrep) {
                                        const u32x2_t zz = {pack2(r[q][0] * (1.0f + sn[q][0]), r[q][1] * (1.0f + sn[q][1])),
                                                            pack2(r[q][2] * (1.0f + sn[q][2]), r[q][3] * (1.0f + sn[q][3]))};
                                        *reinterpret_cast<u32x2_t*>(static_cast<bf16_t*>(ln.z) + off[q]) = zz;
                                        ps[2 * (q0 + q)] += (r[q][0] + r[q][1]) + (r[q][2] + r[q][3]);
                                        ps[2 * (q0 + q) + 1] += (r[q][0] * r[q][0] + r[q][1] * r[q][1]) +
                                                                (r[q][2] * r[q][2] + r[q][3] * r[q][3]);
                                    }
                                } else {
#pragma unroll
                                    for (int c = 0; c < 4; ++c) {
                                        r[q][c] = v[c] + bvc[c];
                                        if (kGelu) r[q][c] = gelu_fast(r[q][c]);
                                    }
                                    *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(out) + off[q]) = r[q];
                                }
                            }
                    }
                }
                if constexpr (kPrep) {
                    // The 16 lanes that share lane / 16 hold partial sums ps[k] of the same rows 4 q + lane / 16
                    // (k = 2 q + 0 / 1): a halving exchange (each step a lane keeps the half of its
                    // values whose index bit matches its lane bit and adds the partner's) leaves sum k in the
                    // lane with lane % 16 == k.  Fixed order: the result does not depend on timing.
                    float w8[8], w4[4], w2[2];
                    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const float keep = b3 ? ps[8 + k] : ps[k], give = b3 ? ps[k] : ps[8 + k];
                        w8[k] = keep + lane_xor<8>(give);
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float keep = b2 ? w8[4 + k] : w8[k], give = b2 ? w8[k] : w8[4 + k];
                        w4[k] = keep + lane_xor<4>(give);
                    }
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const float keep = b1 ? w4[2 + k] : w4[k], give = b1 ? w4[k] : w4[2 + k];
                        w2[k] = keep + lane_xor<2>(give);
                    }
                    const float keep = b0 ? w2[1] : w2[0], give = b0 ? w2[0] : w2[1];
                    const float total = keep + lane_xor<1>(give);
                    const int k = lane & 15;                       // = 2 q + (0: sum, 1: sum of squares)
                    row_sums[(i * 32 + 4 * (k >> 1) + (lane >> 4)) * row_sums_stride + (k & 1)] = total;
                }
            }
        } else {
            // bf16 output.  In the accumulator layout a row lives in two lanes only, so a direct store
            // touches 32 rows x 32 bytes per instruction (partial cache lines).  Each 32-row block is
            // instead packed to bf16, staged in a wave-private LDS region (rows padded by 16 bytes: the
            // 16 lanes of a ds_write_b128 pass hit 16 distinct bank groups) and read back row-major, so
            // that consecutive lanes store consecutive 16-byte chunks of whole output rows.
            constexpr int CH = TN * 4;                         // 16-byte chunks per staged row
            constexpr int kStageRow = (CH + 1) * 16;           // bytes per staged row
            const int l32 = lane & 31;
            [[maybe_unused]] f32x4_t blo[kLn ? 1 : TN][2], bhi[kLn ? 1 : TN][2];
            if constexpr (!kLn) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e8 = 0; e8 < 2; ++e8) {
                        // this lane's two runs: n = nb + 4 lhi + {0..3} (lo) and nb + 8 + 4 lhi + {0..3} (hi);
                        // nb is a multiple of 16 and N of 8, so nb < N covers the lo run and nb + 8 < N the hi run
                        const int nb = gn_wave + j * 32 + 16 * e8;
                        blo[j][e8] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                        bhi[j][e8] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                        if (nb < N) blo[j][e8] = *reinterpret_cast<const f32x4_t*>(bias + nb + 4 * lhi);
                        if (nb + 8 < N) bhi[j][e8] = *reinterpret_cast<const f32x4_t*>(bias + nb + 8 + 4 * lhi);
                    }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e8 = 0; e8 < 2; ++e8) {
                        float v[8];
                        if constexpr (kLn) {
#pragma unroll
                            for (int c = 0; c < 8; ++c) v[c] = ln_a[i] * acc[i][j][8 * e8 + c];
                        } else {
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                v[c] = acc[i][j][8 * e8 + c] + blo[j][e8][c];
                                v[4 + c] = acc[i][j][8 * e8 + 4 + c] + bhi[j][e8][c];
                            }
                        }
                        if (kGelu) {
#pragma unroll
                            for (int c = 0; c < 8; ++c) v[c] = gelu_fast(v[c]);
                        }
                        uint32_t lo0 = pack2(v[0], v[1]), lo1 = pack2(v[2], v[3]);
                        uint32_t hi0 = pack2(v[4], v[5]), hi1 = pack2(v[6], v[7]);
                        // lower half-wave keeps its lo run and receives the partner's lo run (n+4..7);
                        // upper half-wave receives the partner's hi run (n+8..11) and keeps its own hi run
                        const u32x2_t s0 = __builtin_amdgcn_permlane32_swap(lo0, hi0, false, false);
                        const u32x2_t s1 = __builtin_amdgcn_permlane32_swap(lo1, hi1, false, false);
                        const u32x4_t o = {s0[0], s1[0], s0[1], s1[1]};
                        // row l32 of the block, columns j*32 + 16*e8 + 8*lhi .. +7 -> chunk 4j + 2 e8 + lhi
                        *reinterpret_cast<u32x4_t*>(wave_lds + l32 * kStageRow + ((4 * j + 2 * e8 + lhi) << 4)) = o;
                    }
                // read back: flat chunk f = q*64 + lane over 32 rows x CH chunks
#pragma unroll
                for (int q = 0; q < (32 * CH + 63) / 64; ++q) {
                    const int f = q * 64 + lane;
                    const int row = f / CH, ch = f % CH;
                    if ((32 * CH) % 64 != 0 && f >= 32 * CH) continue;
                    const u32x4_t o = *reinterpret_cast<const u32x4_t*>(wave_lds + row * kStageRow + (ch << 4));
                    const int gm = gm_lane - l32 + i * 32 + row, gn = gn_wave + ch * 8;
                    if (gm < M && gn < N)
                        *reinterpret_cast<u32x4_t*>(reinterpret_cast<bf16_t*>(out) + static_cast<int64_t>(gm) * N + gn) = o;
                }
            }
        }
        return;
    }
    // unaligned output: element-wise with bounds checks (the folded-LayerNorm epilogues are launched on
    // aligned shapes only)
    if constexpr (kLn || kPrep) return;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int gm = gm_lane + i * 32;
            if (gm >= M) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int gn = gn_wave + j * 32 + 8 * (e >> 2) + 4 * lhi + (e & 3);
                if (gn >= N) continue;
                const float v = acc[i][j][e] + bias[gn];
                const int64_t o = static_cast<int64_t>(gm) * N + gn;
                if (EPI == FREE_EPI_BIAS) {
                    store_f(out + o, v);
                } else if (EPI == FREE_EPI_BIAS_GELU) {
                    store_f(out + o, gelu_fast(v));
                } else {
                    const float g = gate.base[static_cast<int64_t>(gm / gate.rows_per_sample) * gate.stride + gn];
                    resid[o] = fmaf(g, v, resid[o]);
                }
            }
        }
}

}  // namespace
}  // namespace freemi
