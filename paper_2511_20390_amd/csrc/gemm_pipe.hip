// bf16 GEMM of the dense projections for problems of many token rows (the packed target forward, Alg. 1):
//   C[M,N] = X[M,K] . W[N,K]^T  (+bias, fused epilogue), fp32 accumulation, K a multiple of 64.
// Operand layout, accumulation order (k ascending, 16 per v_mfma_f32_32x32x16_bf16), LDS swizzle and epilogues are those of
// gemm_mfma.hip, so the two kernels give the same bits; what differs is how a K slice reaches the matrix cores.
//
// Two facts of the machine shape the loop (measured with kernels that do nothing else):
//  * a CU keeps about 32 KB of vector loads in flight, whatever is asked of it: 120 KB/us from its L2, 85 from the Infinity
//    Cache, 46 from HBM.  A 256 x 256 tile needs 64 KB per slice of 64, so the requests have to be spread over the slice;
//    a burst only blocks the wavefront that issues it - and the products behind it in its instruction stream.
//  * 64 KB of loads and the 64 products per SIMD of a slice overlap completely (1.28 us against 1.25 us for the products
//    alone) when the loads go to LDS directly and nothing waits for a load younger than half a slice.
// Hence, per slice of 64 with two LDS stages A (this slice) and B (the next):
//   quarter 0: products of k-step 0 | fragments of k-steps 1 and 2 (LDS -> registers)
//   quarter 1: products of k-step 1 | fragments of k-step 3;  barrier: every wavefront is done reading A
//   quarter 2: products of k-step 2 | first half of slice + 2, global -> A
//              wait for slice + 1 (requested a whole slice ago, all but the loads just issued), barrier
//   quarter 3: products of k-step 3 | fragments of k-step 0 from B | second half of slice + 2, global -> A
// Reading a stage in its first half is what leaves the other half, plus half of the next slice, for the loads; it costs
// the registers of three k-steps of fragments, as many as the staging registers of the register-staged loop take.
// Measured in one process, launches back to back, against the register-staged loop of gemm_mfma.hip (us, weights from HBM):
//   12288 rows: QKV 106 -> 98, out-projection 46.6 -> 45.5, MLP-1 (384 x 192) 141 -> 134, MLP-2 134 -> 123
//   8192 rows:  QKV 75 -> 69, out-projection 41 -> 34, MLP-1 114 -> 100, MLP-2 113 -> 90 (192 x 256 tiles)
// The bound of 1.25 us per slice is reached while part of the chip is idle.  Counters of MLP-2 on 256 x 256 tiles inside
// verification rounds: 80 workgroups 96 us at 2.4 GHz, 120 workgroups 101 us at 2.4 GHz, 240 workgroups 130 us at 2.0 GHz - with
// every CU at work the same launch takes 8 % more cycles and the chip, at its power limit, a quarter longer cycles.  Whole rounds
// (12 x 1024 tokens: 14.01 -> 13.74 ms, 32 x 256 tokens: 10.20 -> 9.31 ms) gain accordingly less than single launches.
#include <algorithm>

#include "free_internal.h"
#include "gemm_dma.h"

namespace freemi {

namespace {

template <int BM, int BN, int WGM, int WGN, int EPI>
__global__ __launch_bounds__(WGM * WGN * 64) void gemm_pipe_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, const float* __restrict__ bias, int32_t M, int32_t N, int32_t K,
    int32_t tiles_m, int32_t tiles_n, int32_t group_m, int32_t vec_ok, bf16_t* __restrict__ out, float* __restrict__ resid,
    RowVec gate, LnFold ln) {
    constexpr int ES = 2, NW = WGM * WGN;
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32, FR = TM + TN, MF = TM * TN;
    constexpr int LA = BM / 8 / NW, NL = (BM + BN) / 8 / NW;      // 1 KB blocks per wavefront and slice: of X, of both
    constexpr int D2 = NL / 2, D3 = NL - D2;                      // requested in quarters 2 and 3
    constexpr int kStageBytes = (BM + BN) * kRowBytes;
    static_assert((BM / 8) % NW == 0 && (BN / 8) % NW == 0 && (NW == 8 || WGM == 1), "whole blocks per wavefront");
    constexpr bool kLnEpi = EPI == FREE_EPI_LN_BIAS || EPI == FREE_EPI_LN_BIAS_GELU;
    constexpr bool kPrep = EPI == FREE_EPI_GATE_RESID_PREP;
    constexpr bool kSeg = EPI == FREE_EPI_GATE_RESID_SEG;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    int tile_m, tile_n;
    tile_coords(group_m, blockIdx.x, tiles_m, tiles_n, &tile_m, &tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Wavefronts w and w + 4 share a SIMD.  They get different column halves of the tile, so that in a tile whose right half
    // is padding (N = 1152 is 4.5 tiles of 256) every SIMD keeps one working wavefront.
    constexpr int kHalfN = NW == 8 ? WGN / 2 : WGN;
    const int wm = (wave & 3) / kHalfN, wn = (wave >> 2) * kHalfN + (wave & 3) % kHalfN;
    const int nk = K / BK;

    // ---- loads: block u holds tile rows 8 u .. 8 u + 7; lane -> row 8 u + lane / 8, LDS chunk lane % 8, which receives the
    // global 16-byte chunk (lane % 8) ^ ((row / 2) % 8); a wavefront's blocks w, w + NW, ... have the parity of w
    const u32x4_t xsrd = make_rsrc(X + static_cast<int64_t>(m0) * K, static_cast<int64_t>(M - m0) * K * ES);
    const u32x4_t wsrd = make_rsrc(W + static_cast<int64_t>(n0) * K, static_cast<int64_t>(N - n0) * K * ES);
    const int voff = (lane >> 3) * K * ES + (((lane & 7) ^ (((wave & 1) << 2) | (lane >> 4))) << 4);
    const uint32_t lds_base = lds_address(lds);
    auto dma = [&](int kt, int stage, int i) {
        const uint32_t dst = lds_base + stage * kStageBytes + wave * 1024;
        const int soff = wave * 8 * K * ES + kt * kRowBytes;
        if (i < LA) dma_1k(dst + i * NW * 1024, voff, xsrd, soff + i * NW * 8 * K * ES);
        else dma_1k(dst + BM * kRowBytes + (i - LA) * NW * 1024, voff, wsrd, soff + (i - LA) * NW * 8 * K * ES);
    };

    // ---- fragments of k-step ks: r in [0, TM) rows of X, [TM, FR) rows of W
    const int l32 = lane & 31, lhi = lane >> 5;
    const int sw = (l32 >> 1) & 7;
    const int x_row0 = (wm * TM * 32 + l32) * kRowBytes, w_row0 = (BM + wn * TN * 32 + l32) * kRowBytes;
    u32x4_t f[4][FR];
    auto read = [&](int stage, int ks, int r) {
        const int row = r < TM ? x_row0 + r * 32 * kRowBytes : w_row0 + (r - TM) * 32 * kRowBytes;
        f[ks][r] = *reinterpret_cast<const u32x4_t*>(lds + stage * kStageBytes + row + ((((ks << 1) | lhi) ^ sw) << 4));
    };
    f32x16_t acc[TM][TN];                                         // acc[i][j]: rows n (tile j), columns m (tile i)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // kSeg: the sums over the first parts of K (ResidJoin's order); the last part is added to them at the end
    [[maybe_unused]] f32x16_t sum[kSeg ? TM : 1][kSeg ? TN : 1];
    [[maybe_unused]] const int seg = nk / kSplitParts;
    [[maybe_unused]] int seg_end = seg;
    auto add_part = [&](bool last) {
        if constexpr (kSeg) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        if (last) {
                            acc[i][j][e] = sum[i][j][e] + acc[i][j][e];
                        } else {
                            sum[i][j][e] += acc[i][j][e];
                            acc[i][j][e] = 0.f;
                        }
                    }
        }
    };
    if constexpr (kSeg) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[i][j][e] = 0.f;
    }
    auto mma = [&](int ks, int t) {
        const int i = t / TN, j = t % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, f[ks][TM + j]),
                                                            __builtin_bit_cast(bf16x8_t, f[ks][i]), acc[i][j], 0, 0, 0);
    };
    // a quarter: the products of k-step ks with nd loads and nr fragment reads spread between them
    auto quarter = [&](auto ks_c, auto nd_c, auto nr_c, auto&& load, auto&& frag) {
        constexpr int ks = decltype(ks_c)::value, nd = decltype(nd_c)::value, nr = decltype(nr_c)::value;
#pragma unroll
        for (int t = 0; t < MF; ++t) {
#pragma unroll
            for (int d = t * nd / MF; d < (t + 1) * nd / MF; ++d) load(d);
#pragma unroll
            for (int r = t * nr / MF; r < (t + 1) * nr / MF; ++r) frag(r);
            mma(ks, t);
            if constexpr (nd > 0) {
                if ((t + 1) * nd / MF != t * nd / MF) __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (nd == 0) {
#pragma unroll
            for (int t = 0; t < MF; ++t) {
                __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
                if ((t + 1) * nr / MF != t * nr / MF) __builtin_amdgcn_sched_group_barrier(kDsRd, (nr + MF - 1) / MF, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // A wavefront whose part of the tile is all padding takes part in the loads and barriers only (kOn false): on a chip that
    // runs at its power limit products that are thrown away are not free for the others.
    auto slice = [&](int kt, auto on, auto more1, auto more2) {   // slices kt + 1, kt + 2 exist
        constexpr bool kOn = decltype(on)::value, m1 = decltype(more1)::value, m2 = decltype(more2)::value;
        constexpr int nd2 = m2 ? D2 : 0, nd3 = m2 ? D3 : 0;
        const int a = kt & 1, b = a ^ 1;
        auto load2 = [&](int d) { dma(kt + 2, a, d); };
        auto load3 = [&](int d) { dma(kt + 2, a, D2 + d); };
        if constexpr (kOn) {
            auto none = [](int) {};
            using std::integral_constant;
            quarter(integral_constant<int, 0>{}, integral_constant<int, 0>{}, integral_constant<int, 2 * FR>{}, none,
                    [&](int r) { read(a, 1 + r / FR, r % FR); });
            quarter(integral_constant<int, 1>{}, integral_constant<int, 0>{}, integral_constant<int, FR>{}, none,
                    [&](int r) { read(a, 3, r); });
            if constexpr (m2) wait_lds_barrier();
            quarter(integral_constant<int, 2>{}, integral_constant<int, nd2>{}, integral_constant<int, 0>{}, load2, none);
            if constexpr (m1) wait_vm_barrier<nd2>();
            quarter(integral_constant<int, 3>{}, integral_constant<int, nd3>{}, integral_constant<int, m1 ? FR : 0>{}, load3,
                    [&](int r) { read(b, 0, r); });
        } else {
            if constexpr (m2) wait_lds_barrier();
#pragma unroll
            for (int d = 0; d < nd2; ++d) load2(d);
            if constexpr (m1) wait_vm_barrier<nd2>();
#pragma unroll
            for (int d = 0; d < nd3; ++d) load3(d);
        }
    };
    const std::true_type yes{};
    const std::false_type no{};

    // ---- prologue
    // Folded LayerNorm: with mu and rho = sqrt(var + eps) of a row, the output is (z W^T - mu c1 + rho c0) / rho.
    // The rank-2 term -mu c1 + rho c0 is one extra k-step of the matrix product, issued in this prologue: row m
    // contributes the k-vector (-mu_h, -mu_l, -mu_h, rho_h, rho_l, rho_h, 0 ...), column n the k-vector
    // (c1_h, c1_h, c1_l, c0_h, c0_h, c0_l, 0 ...), with _h the bf16 value and _l the bf16 value of the remainder
    // (the product of two remainders, 2^-18 relative, is dropped).  Its loads - the partial sums of this lane's
    // rows, c1 / c0 of its columns - are requested with the first slices; nothing of it stays in registers through the
    // K loop except 1 / rho per row, which the epilogue multiplies by.  Every 32-row block lies in one sample (rows per
    // sample a multiple of 32).  The lower half-wave adds the first half of a row's slots in index order, the upper one
    // the rest, then the two sums are added - a fixed order.
    constexpr int kHalfSlots = 8;                          // up to 16 slots: rows of up to 2048 values
    [[maybe_unused]] float2 ln_p[kLnEpi ? TM : 1][kHalfSlots];
    [[maybe_unused]] float ln_c1[kLnEpi ? TM : 1][TN], ln_c0[kLnEpi ? TM : 1][TN];
    [[maybe_unused]] int ln_kn = 0;
    if constexpr (kLnEpi) {
        const int rps = ln.rows_per_sample;
        const int half = (ln.slots + 1) / 2;
        const int k0 = lhi ? half : 0;
        ln_kn = lhi ? ln.slots - half : half;              // this half-wave's slots
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int gm_blk = m0 + wm * TM * 32 + i * 32;
            const int gm = gm_blk + l32;
            // (rows past M and slots past the end re-read a valid entry with weight zero: no branches)
            const float2* st = reinterpret_cast<const float2*>(ln.stats) + static_cast<int64_t>(gm < M ? gm : M - 1) * ln.slots;
#pragma unroll
            for (int k = 0; k < kHalfSlots; ++k) ln_p[i][k] = st[k0 + (k < ln_kn ? k : 0)];
            // c1 / c0 of this block's sample: loaded again only where the sample changes (wave-uniform)
            const int smp = (gm_blk < M ? gm_blk : M - 1) / rps;
            const int smp_prev = i == 0 ? -1 : ((gm_blk - 32 < M ? gm_blk - 32 : M - 1) / rps);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (smp != smp_prev) {
                    const int n = n0 + wn * TN * 32 + j * 32 + l32;
                    const int64_t o = static_cast<int64_t>(smp) * ln.fold_stride + (n < N ? n : 0);
                    ln_c1[i][j] = ln.c1[o];
                    ln_c0[i][j] = ln.c0[o];
                } else {
                    ln_c1[i][j] = ln_c1[i > 0 ? i - 1 : 0][j];
                    ln_c0[i][j] = ln_c0[i > 0 ? i - 1 : 0][j];
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) dma(0, 0, i);
    if (nk > 1) {
#pragma unroll
        for (int i = 0; i < NL; ++i) dma(1, 1, i);
    }
    float ln_a[TM];                                        // folded LayerNorm: 1 / rho of this lane's rows
#pragma unroll
    for (int i = 0; i < TM; ++i) ln_a[i] = 1.0f;
    if constexpr (kLnEpi) {
        const auto split = [](float v, float* hi, float* lo) {
            *hi = __uint_as_float(pack2(v, 0.f) << 16);
            *lo = v - *hi;
        };
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int k = 0; k < kHalfSlots; ++k) {
                s1 += k < ln_kn ? ln_p[i][k].x : 0.f;
                s2 += k < ln_kn ? ln_p[i][k].y : 0.f;
            }
            const float o1 = __shfl_xor(s1, 32, 64), o2 = __shfl_xor(s2, 32, 64);
            s1 = lhi ? o1 + s1 : s1 + o1;                  // first half + second half in both lanes
            s2 = lhi ? o2 + s2 : s2 + o2;
            const float mean = s1 * ln.inv_width;
            const float var = fmaxf(s2 * ln.inv_width - mean * mean, 0.f);
            ln_a[i] = rsqrtf(var + kLnEps);
            float mh, ml, rh, rl;
            split(-mean, &mh, &ml);
            split(1.0f / ln_a[i], &rh, &rl);
            const u32x4_t xk = lhi ? u32x4_t{0, 0, 0, 0} : u32x4_t{pack2(mh, ml), pack2(mh, rh), pack2(rl, rh), 0};
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + wn * TN * 32 + j * 32 + l32;
                float c1h, c1l, c0h, c0l;
                split(n < N ? ln_c1[i][j] : 0.f, &c1h, &c1l);
                split(n < N ? ln_c0[i][j] : 0.f, &c0h, &c0l);
                const u32x4_t wk = lhi ? u32x4_t{0, 0, 0, 0} : u32x4_t{pack2(c1h, c1h), pack2(c1l, c0h), pack2(c0h, c0l), 0};
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wk),
                                                                    __builtin_bit_cast(bf16x8_t, xk), acc[i][j], 0, 0, 0);
            }
        }
    }
    if (nk > 1) wait_vm_barrier<NL>();
    else wait_vm_barrier<0>();

    // ---- K loop, one straight-line copy for wavefronts with and without products
    auto k_loop = [&](auto on) {
        if constexpr (decltype(on)::value) {
#pragma unroll
            for (int r = 0; r < FR; ++r) read(0, 0, r);
            __builtin_amdgcn_sched_barrier(0);
        }
        int kt = 0;
        for (; kt + 2 < nk; ++kt) {
            if constexpr (kSeg && decltype(on)::value) {
                if (kt == seg_end) {
                    add_part(false);
                    seg_end += seg;
                }
            }
            slice(kt, on, yes, yes);
        }
        if (kt + 1 < nk) {
            slice(kt, on, yes, no);
            ++kt;
        }
        slice(kt, on, no, no);
        if constexpr (decltype(on)::value) add_part(true);
    };
    if (n0 + wn * TN * 32 < N && m0 + wm * TM * 32 < M) k_loop(yes);
    else k_loop(no);

    // ---- epilogue: the stages are idle now, each wavefront transposes its output in a private piece of them
    __syncthreads();
    constexpr bool kResidEpi = EPI == FREE_EPI_GATE_RESID || kPrep || kSeg;
    constexpr int kWaveStage = kResidEpi ? 32 * (((TN % 2 == 0 ? 2 : 1) * 8 + 1) * 16)   // fp32 groups
                                         : 32 * (TN * 64 + 16);                          // bf16 rows
    constexpr int kSumBytes = kPrep ? BM * WGN * 2 * 4 : 0;
    static_assert(NW * kWaveStage + kSumBytes <= 2 * kStageBytes, "output staging must fit in the K-loop stages");
    float* row_sums = reinterpret_cast<float*>(lds + NW * kWaveStage);                   // kPrep: [BM][WGN][2]
    write_tile<bf16_t, TM, TN, (kSeg ? FREE_EPI_GATE_RESID : EPI), (NW == 8 ? 4 : 0)>(acc, m0 + wm * TM * 32 + l32, n0 + wn * TN * 32, lane, M, N, vec_ok, bias,
                                                       out, resid, gate, lds + wave * kWaveStage, ln, ln_a,
                                                       row_sums + (wm * TM * 32 * WGN + wn) * 2, WGN * 2);
    if constexpr (kPrep) {
        // the two 64-column halves of a slot, added in column order
        __syncthreads();
        constexpr int kSlots = WGN / 2;
        for (int e = tid; e < BM * kSlots * 2; e += NW * 64) {
            const int row = e / (kSlots * 2), slot = (e >> 1) % kSlots, k = e & 1;
            const int gm = m0 + row, gs = n0 / kLnSlotCols + slot;
            const float* h = row_sums + (row * WGN + 2 * slot) * 2 + k;
            if (gm < M && gs < ln.slots) ln.stats[(static_cast<int64_t>(gm) * ln.slots + gs) * 2 + k] = h[0] + h[2];
        }
    }
}

struct Args {
    const bf16_t *X, *W;
    const float* bias;
    int32_t M, N, K;
    bf16_t* out;
    float* resid;
    RowVec gate;
    hipStream_t s;
};

template <int BM, int BN, int WGM, int WGN, int EPI>
int32_t launch_one(const Args& a, const LnFold& ln) {
    const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    const size_t lds = 2 * static_cast<size_t>(BM + BN) * kRowBytes;
    auto kern = gemm_pipe_kernel<BM, BN, WGM, WGN, EPI>;
    static LdsLimit limit;
    if (!limit.allow(reinterpret_cast<const void*>(kern), lds)) return FREE_ERR_HIP;
    // the vector epilogue needs 16-byte aligned rows of out / resid / bias / gate
    auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    const bool vec = ((a.N & 7) == 0) && al16(a.bias) && al16(a.out) && al16(a.resid) && al16(a.gate.base) && ((a.gate.stride & 3) == 0);
    if (EPI >= FREE_EPI_LN_BIAS && EPI <= FREE_EPI_GATE_RESID_PREP && !vec) return FREE_ERR_SHAPE;     // the folded-LayerNorm epilogues have no element-wise form
    // Row tiles per group of the tile order.  Several rounds of workgroups: the 32 that run together on an XCD should cover
    // a x b tiles with a BM ~ b BN, the shape that needs the fewest distinct X and W panels (first-touch misses of that
    // XCD's L2).  A single round: every XCD holds total / 8 tiles for the whole kernel, and a group of exactly that many
    // tiles - whole tile rows - keeps each X panel in one L2.
    const int total = tiles_m * tiles_n;
    int group_m = BM > BN ? 4 : 8;
    if (total <= device_cus()) {
        const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
        group_m = std::max(1, (per_xcd + tiles_n / 2) / tiles_n);
    }
    hipLaunchKernelGGL(kern, dim3(total), dim3(WGM * WGN * 64), lds, a.s, a.X, a.W, a.bias, a.M, a.N, a.K, tiles_m, tiles_n,
                       group_m, vec ? 1 : 0, a.out, a.resid, a.gate, ln);
    return launch_ok() ? FREE_OK : FREE_ERR_HIP;
}

template <int BM, int BN, int WGM, int WGN>
int32_t launch_tile(const Args& a, int32_t epi, const LnFold& ln) {
    switch (epi) {
        case FREE_EPI_BIAS: return launch_one<BM, BN, WGM, WGN, FREE_EPI_BIAS>(a, ln);
        case FREE_EPI_BIAS_GELU: return launch_one<BM, BN, WGM, WGN, FREE_EPI_BIAS_GELU>(a, ln);
        case FREE_EPI_GATE_RESID: return launch_one<BM, BN, WGM, WGN, FREE_EPI_GATE_RESID>(a, ln);
        case FREE_EPI_LN_BIAS: return launch_one<BM, BN, WGM, WGN, FREE_EPI_LN_BIAS>(a, ln);
        case FREE_EPI_LN_BIAS_GELU: return launch_one<BM, BN, WGM, WGN, FREE_EPI_LN_BIAS_GELU>(a, ln);
        case FREE_EPI_GATE_RESID_PREP:
            if constexpr (BN == 256) return launch_one<BM, BN, WGM, WGN, FREE_EPI_GATE_RESID_PREP>(a, ln);
            return FREE_ERR_RANGE;
        case FREE_EPI_GATE_RESID_SEG:
            if constexpr (BM * BN <= kSegTileArea) return launch_one<BM, BN, WGM, WGN, FREE_EPI_GATE_RESID_SEG>(a, ln);
            return FREE_ERR_RANGE;
        default: return FREE_ERR_RANGE;
    }
}

}  // namespace

int32_t launch_linear_pipe(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                           bf16_t* out, float* resid, RowVec gate, hipStream_t s, PipeTile tile, const LnFold* ln) {
    const Args a{X, W, bias, M, N, K, out, resid, gate, s};
    const LnFold f = ln ? *ln : LnFold{};
    switch (tile) {
        case PIPE_256x256: return launch_tile<256, 256, 2, 4>(a, epi, f);
        case PIPE_384x192: return launch_tile<384, 192, 4, 2>(a, epi, f);
        case PIPE_256x192: return launch_tile<256, 192, 4, 2>(a, epi, f);
        case PIPE_192x256: return launch_tile<192, 256, 2, 4>(a, epi, f);
        case PIPE_192x128: return launch_tile<192, 128, 2, 4>(a, epi, f);
        case PIPE_160x128: return launch_tile<160, 128, 1, 4>(a, epi, f);
        case PIPE_128x128: return launch_tile<128, 128, 2, 4>(a, epi, f);
    }
    return FREE_ERR_RANGE;
}

}  // namespace freemi
