// GEMM of the dense projections for problems of few token rows (single guided steps, the drafter, short packs):
//   C[M,N] = X[M,K] . W[N,K]^T  (+bias, fused epilogue), bf16 or fp32 operands, fp32 accumulation, K a whole number of slices.
// (fp32: free_op_linear; the linear layers of fp32 models run on gemm_f32.hip.)
// Operand layout, accumulation order, LDS swizzle and results are those of gemm_mfma.hip bit for bit; this kernel is
// organised for latency.
//
// With few rows there are fewer large tiles than CUs, and a CU is limited by what it can load: about 32 KB are in flight
// whatever is asked for, i.e. 120 KB/us from its L2, 85 from the Infinity Cache, 46 from HBM (weights are used once per
// forward).  A 64 x 64 tile of MLP-2 (K = 4608) moves 1.2 MB, so its 72 slices of 64 take 21 us from HBM; what the kernel can
// do is use as many CUs as there are tiles and keep those 32 KB in flight from the first instruction to the last:
//  * small tiles: 64 x 64 (four wavefronts of 32 x 32), 128 x 64, and 128 x 128 on eight wavefronts;
//  * a ring of S stages in LDS filled by global-to-LDS loads, S slices ahead, one or two blocks of 1 KB behind every
//    group of products; one barrier per slice;
//  * fragments of slice t + 1 are read under the products of slice t (a whole slice in registers: the tiles are small);
//  * what the epilogue needs from memory (bias; gate and residual of the smallest tile) is requested before the first slice.
// K in parts (kSplitParts; narrow outputs of long K, where even small tiles leave CUs idle): one workgroup per tile and part with the
// fp32 sums to memory (FREE_EPI_PARTIAL), or one per tile that adds the same parts in the same order (FREE_EPI_GATE_RESID_SEG).
// Rows are walked fastest within an XCD, so every weight panel is fetched by one XCD only.
// Measured back to back, weights from HBM, against the 96 x 128 / 160 x 128 register-staged tiles (us; QKV, out-projection,
// MLP-1, MLP-2):   256 rows 13.3, 15.8, 14.5, 43.8 -> 8.2, 8.7, 11.2, 23.2
//                  512 rows 14.3, 16.0, 16.1, 44.3 -> 10.5, 8.8, 15.0, 23.3
//                 1024 rows 16.6, 16.4, 20.0, 44.7 -> 14.1, 11.2, 20.0, 31.7
// fp32 is bound by the matrix cores (0.43 us for the 16 products of a wavefront's slice; measured 0.57 with its waits), and
// what the small tiles buy is wavefronts: 512 rows 61, 59, 64, 217 -> 44, 26, 64, 89 (MLP-1 keeps its 96 x 128).
#include <algorithm>

#include "free_internal.h"
#include "gemm_dma.h"

namespace freemi {

namespace {

template <typename T, int BM, int BN, int WGM, int WGN, int S, int EPI>
__global__ __launch_bounds__(WGM * WGN * 64) void gemm_rows_kernel(
    const T* __restrict__ X, const T* __restrict__ W, const float* __restrict__ bias, int32_t M, int32_t N, int32_t K,
    int32_t tiles_m, int32_t tiles_n, T* __restrict__ out, float* __restrict__ resid, RowVec gate, int32_t from_zero) {
    constexpr bool kF32 = std::is_same<T, float>::value;
    constexpr bool kSeg = EPI == FREE_EPI_GATE_RESID_SEG, kResid = EPI == FREE_EPI_GATE_RESID || kSeg;
    constexpr bool kGelu = EPI == FREE_EPI_BIAS_GELU, kPart = EPI == FREE_EPI_PARTIAL;
    constexpr int kParts = kPart ? kSplitParts : 1;
    constexpr int ES = static_cast<int>(sizeof(T)), NW = WGM * WGN;
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
    constexpr int LA = BM / 8 / NW, NL = (BM + BN) / 8 / NW;            // 1 KB blocks per wavefront and slice: of X, of both
    constexpr int kStageBytes = (BM + BN) * kRowBytes;
    static_assert((BM / 8) % NW == 0 && (BN / 8) % NW == 0 && NW % 2 == 0, "whole blocks per wavefront, of one parity");
    static_assert(S >= 2 && S <= 6 && NL * (S - 1) < 64, "tail waits are written out; loads in flight can be counted");
    extern __shared__ __attribute__((aligned(16))) char lds[];

    // An XCD takes consecutive tiles, rows fastest, then columns, then parts of K: it keeps its rows of W (what was read ahead for it)
    // and, of X, mostly one part.  With the parts of a column next to each other every XCD read all of X, 9.4 MB through 4 MB of L2 at
    // 1024 rows of 4608: round of 4 x 256 states 2510 -> 2420 us, forward of 2 x 256 1853 -> 1830; 256 rows the same.
    const int tile = xcd_tile(blockIdx.x, tiles_m * tiles_n * kParts), column = tile / tiles_m;
    const int tile_m = tile - column * tiles_m, part = kParts > 1 ? column / tiles_n : 0, tile_n = column - part * tiles_n;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int nk = K / (kRowBytes / ES) / kParts;

    // ---- what the epilogue needs: register e of acc[i][j] is row gm_lane + 32 i, column gn_lane + 32 j + 8 (e / 4) + e % 4
    const int gm_lane = m0 + wm * TM * 32 + l32, gn_lane = n0 + wn * TN * 32 + 4 * lhi;
    f32x4_t pre_b[TN][4];
    [[maybe_unused]] f32x4_t pre_r[kResid ? TM : 1][TN][4], pre_g[kResid ? TM : 1][TN][4];
    constexpr bool kPreResid = kResid && TM * TN == 1;                   // (larger tiles have no registers for it)
    const f32x4_t zero4 = {0.f, 0.f, 0.f, 0.f};
    auto load_resid = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int gm = gm_lane + i * 32, gn = gn_lane + j * 32 + 8 * q;
                    const bool ok = gm < M && gn < N;
                    pre_r[i][j][q] = ok && !from_zero ? *reinterpret_cast<const f32x4_t*>(resid + static_cast<int64_t>(gm) * N + gn) : zero4;
                    pre_g[i][j][q] = ok ? *reinterpret_cast<const f32x4_t*>(gate.base + static_cast<int64_t>(gm / gate.rows_per_sample) * gate.stride + gn) : zero4;
                }
    };
    auto load_bias = [&]() {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int gn = gn_lane + j * 32 + 8 * q;                 // N % 8 == 0: four columns are all in or all out
                pre_b[j][q] = gn < N ? *reinterpret_cast<const f32x4_t*>(bias + gn) : zero4;
            }
    };
    constexpr bool kPreBias = !kPart && !(kSeg && !kPreResid);           // (nor for the bias beside two sets of accumulators)
    if constexpr (kPreBias) load_bias();
    if constexpr (kPreResid) load_resid();

    // ---- loads: block u holds tile rows 8 u .. 8 u + 7; lane -> row 8 u + lane / 8, LDS chunk lane % 8, which receives the
    // global 16-byte chunk (lane % 8) ^ ((row / 2) % 8); a wavefront's blocks w, w + NW, ... have the parity of w
    const int64_t k0 = static_cast<int64_t>(part) * nk * (kRowBytes / ES);
    const u32x4_t xsrd = make_rsrc(X + static_cast<int64_t>(m0) * K + k0, (static_cast<int64_t>(M - m0) * K - k0) * ES);
    const u32x4_t wsrd = make_rsrc(W + static_cast<int64_t>(n0) * K + k0, (static_cast<int64_t>(N - n0) * K - k0) * ES);
    const int voff = (lane >> 3) * K * ES + (((lane & 7) ^ (((wave & 1) << 2) | (lane >> 4))) << 4);
    const uint32_t lds_base = lds_address(lds);
    auto issue = [&](int kt, int stage, int lo, int hi) {               // blocks [lo, hi) of this wavefront's share
        const uint32_t dst = lds_base + stage * kStageBytes + wave * 1024;
        const int soff = wave * 8 * K * ES + kt * kRowBytes;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (i < lo || i >= hi) continue;
            if (i < LA) dma_1k(dst + i * NW * 1024, voff, xsrd, soff + i * NW * 8 * K * ES);
            else dma_1k(dst + BM * kRowBytes + (i - LA) * NW * 1024, voff, wsrd, soff + (i - LA) * NW * 8 * K * ES);
        }
    };

    const int sw = (l32 >> 1) & 7;
    const int x_row0 = (wm * TM * 32 + l32) * kRowBytes, w_row0 = (BM + wn * TN * 32 + l32) * kRowBytes;
    u32x4_t fx[2][4][TM], fw[2][4][TN];                                 // two slices of fragments
    f32x16_t acc[TM][TN];
    [[maybe_unused]] f32x16_t sum[kSeg ? TM : 1][TN];                   // kSeg: the finished parts of K
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[i][j][e] = 0.f;
                if constexpr (kSeg) sum[i][j][e] = 0.f;
            }
    auto load_frags = [&](int stage, int buf, int ks) {
        const char* base = lds + stage * kStageBytes;
        const int choff = (((ks << 1) | lhi) ^ sw) << 4;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fx[buf][ks][i] = *reinterpret_cast<const u32x4_t*>(base + x_row0 + i * 32 * kRowBytes + choff);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fw[buf][ks][j] = *reinterpret_cast<const u32x4_t*>(base + w_row0 + j * 32 * kRowBytes + choff);
    };
    auto mma = [&](int buf, int ks) {
        if constexpr (kF32) {
            // element e of the chunk: the lanes of group 0 / 1 hold the two k of one 32x32x2 product
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        // (copied out first: a bit cast applied directly to a vector element read element 0)
                        const uint32_t wbits = fw[buf][ks][j][e], xbits = fx[buf][ks][i][e];
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, wbits),
                                                                        __builtin_bit_cast(float, xbits), acc[i][j], 0, 0, 0);
                    }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fw[buf][ks][j]),
                                                                        __builtin_bit_cast(bf16x8_t, fx[buf][ks][i]),
                                                                        acc[i][j], 0, 0, 0);
        }
    };
    // the slice with r younger ones in flight has arrived, for the whole workgroup (r < S)
    auto arrive = [&](int r) {
        if (r == 0) wait_vm_barrier<0>();
        else if (r == 1) wait_vm_barrier<NL>();
        else if (r == 2) wait_vm_barrier<(S > 2 ? 2 : 0) * NL>();
        else if (r == 3) wait_vm_barrier<(S > 3 ? 3 : 0) * NL>();
        else if (r == 4) wait_vm_barrier<(S > 4 ? 4 : 0) * NL>();
        else wait_vm_barrier<(S > 5 ? 5 : 0) * NL>();
    };

#pragma unroll
    for (int p = 0; p < S; ++p)
        if (p < nk) issue(p, p, 0, NL);
    arrive(std::min(nk - 1, S - 1));
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) load_frags(0, 0, ks);
    __builtin_amdgcn_sched_barrier(0);
    int st_cur = 0, st_next = 1;
    // Slice kt is in fragment buffer `buf` (read from stage st_cur before this slice's barrier); slice kt + 1 is read from
    // stage st_next into the other buffer, slice kt + S replaces slice kt in LDS.
    auto step = [&](int kt, auto buf_c, auto steady) {
        constexpr int buf = decltype(buf_c)::value;
        if constexpr (decltype(steady)::value) {
            wait_vm_barrier<NL*(S - 2)>();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                issue(kt + S, st_cur, NL * q / 4, NL * (q + 1) / 4);
                load_frags(st_next, buf ^ 1, q);
                mma(buf, q);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            if (kt + 1 < nk) {
                arrive(std::min(nk - kt - 2, S - 2));
#pragma unroll
                for (int q = 0; q < 4; ++q) load_frags(st_next, buf ^ 1, q);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) mma(buf, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        st_cur = st_next;
        st_next = st_next + 1 == S ? 0 : st_next + 1;
    };
    const std::integral_constant<int, 0> b0{};
    const std::integral_constant<int, 1> b1{};
    const std::true_type yes{};
    const std::false_type no{};
    int kt = 0;
    const int n_steady = nk > S ? nk - S : 0;                           // slices whose stage is refilled
    if constexpr (kSeg) {
        // the parts before the last one: an even number of slices each, at least S (linear_split_covers)
        const int seg = nk / kSplitParts;
        for (int end = seg; end < nk; end += seg) {
            for (; kt < end; kt += 2) {
                step(kt, b0, yes);
                step(kt + 1, b1, yes);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        sum[i][j][e] += acc[i][j][e];
                        acc[i][j][e] = 0.f;
                    }
        }
    }
    for (; kt + 1 < n_steady; kt += 2) {
        step(kt, b0, yes);
        step(kt + 1, b1, yes);
    }
    if (kt < n_steady) {
        step(kt, b0, yes);
        ++kt;
        for (; kt < nk; kt += 2) {
            step(kt, b1, no);
            if (kt + 1 < nk) step(kt + 1, b0, no);
        }
    } else {
        for (; kt < nk; kt += 2) {
            step(kt, b0, no);
            if (kt + 1 < nk) step(kt + 1, b1, no);
        }
    }

    // ---- epilogue
    if constexpr (!kPart && !kPreBias) load_bias();
    if constexpr (kResid && !kPreResid) load_resid();
    if constexpr (kPart) {
        // 32-row blocks of the fp32 sums transposed through the idle stages: 128 TN bytes of a row per store, not 32
        __syncthreads();
        constexpr int CH = TN * 8, kStageRow = (CH + 1) * 16;
        static_assert(NW * 32 * kStageRow <= S * kStageBytes && (32 * CH) % 64 == 0, "output staging must fit in the stages");
        char* wave_lds = lds + wave * 32 * kStageRow;
        float* dst = resid + static_cast<int64_t>(part) * M * N;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4_t*>(wave_lds + l32 * kStageRow + ((8 * j + 2 * q + lhi) << 4)) =
                        f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
#pragma unroll
            for (int q = 0; q < 32 * CH / 64; ++q) {
                const int f = q * 64 + lane, row = f / CH, ch = f % CH;
                const f32x4_t o = *reinterpret_cast<const f32x4_t*>(wave_lds + row * kStageRow + (ch << 4));
                const int gm = m0 + wm * TM * 32 + i * 32 + row, gn = n0 + wn * TN * 32 + ch * 4;
                if (gm < M && gn < N) *reinterpret_cast<f32x4_t*>(dst + static_cast<int64_t>(gm) * N + gn) = o;
            }
        }
    } else if constexpr (kResid || kF32) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int gm = gm_lane + i * 32, gn = gn_lane + j * 32 + 8 * q;
                    if (gm >= M || gn >= N) continue;
                    f32x4_t o;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float a = acc[i][j][4 * q + c];
                        if constexpr (kSeg) a = sum[i][j][4 * q + c] + a;
                        const float v = a + pre_b[j][q][c];
                        if constexpr (kResid) o[c] = fmaf(pre_g[i][j][q][c], v, pre_r[i][j][q][c]);
                        else o[c] = kGelu ? gelu_fast(v) : v;
                    }
                    float* dst = kResid ? resid : reinterpret_cast<float*>(out);
                    *reinterpret_cast<f32x4_t*>(dst + static_cast<int64_t>(gm) * N + gn) = o;
                }
    } else {
        // bf16: 32-row blocks transposed through a wave-private piece of the idle stages, whole rows stored (write_tile)
        __syncthreads();
        constexpr int CH = TN * 4, kStageRow = (CH + 1) * 16;
        static_assert(NW * 32 * kStageRow <= S * kStageBytes && (32 * CH) % 64 == 0, "output staging must fit in the stages");
        char* wave_lds = lds + wave * 32 * kStageRow;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float v[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        v[c] = acc[i][j][8 * h + c] + pre_b[j][2 * h + (c >> 2)][c & 3];
                        if (kGelu) v[c] = gelu_fast(v[c]);
                    }
                    // runs of four columns of the two half-waves -> eight consecutive columns per lane
                    const u32x2_t s0 = __builtin_amdgcn_permlane32_swap(pack2(v[0], v[1]), pack2(v[4], v[5]), false, false);
                    const u32x2_t s1 = __builtin_amdgcn_permlane32_swap(pack2(v[2], v[3]), pack2(v[6], v[7]), false, false);
                    *reinterpret_cast<u32x4_t*>(wave_lds + l32 * kStageRow + ((4 * j + 2 * h + lhi) << 4)) = u32x4_t{s0[0], s1[0], s0[1], s1[1]};
                }
#pragma unroll
            for (int q = 0; q < 32 * CH / 64; ++q) {
                const int f = q * 64 + lane, row = f / CH, ch = f % CH;
                const u32x4_t o = *reinterpret_cast<const u32x4_t*>(wave_lds + row * kStageRow + (ch << 4));
                const int gm = m0 + wm * TM * 32 + i * 32 + row, gn = n0 + wn * TN * 32 + ch * 8;
                if (gm < M && gn < N) *reinterpret_cast<u32x4_t*>(reinterpret_cast<bf16_t*>(out) + static_cast<int64_t>(gm) * N + gn) = o;
            }
        }
    }
}

template <typename T>
struct Args {
    const T *X, *W;
    const float* bias;
    int32_t M, N, K;
    T* out;
    float* resid;
    RowVec gate;
    hipStream_t s;
    bool from_zero;                        // the residual stream counts as zero and is not read
};

template <typename T, int BM, int BN, int WGM, int WGN, int S, int EPI>
int32_t launch_one(const Args<T>& a) {
    const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    const size_t lds = S * static_cast<size_t>(BM + BN) * kRowBytes;
    auto kern = gemm_rows_kernel<T, BM, BN, WGM, WGN, S, EPI>;
    static LdsLimit limit;
    if (!limit.allow(reinterpret_cast<const void*>(kern), lds)) return FREE_ERR_HIP;
    constexpr int kParts = EPI == FREE_EPI_PARTIAL ? kSplitParts : 1;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * kParts), dim3(WGM * WGN * 64), lds, a.s, a.X, a.W, a.bias, a.M, a.N, a.K, tiles_m,
                       tiles_n, a.out, a.resid, a.gate, a.from_zero ? 1 : 0);
    return launch_ok() ? FREE_OK : FREE_ERR_HIP;
}

template <typename T, int BM, int BN, int WGM, int WGN, int S>
int32_t launch_tile(const Args<T>& a, int32_t epi) {
    switch (epi) {
        case FREE_EPI_BIAS: return launch_one<T, BM, BN, WGM, WGN, S, FREE_EPI_BIAS>(a);
        case FREE_EPI_BIAS_GELU: return launch_one<T, BM, BN, WGM, WGN, S, FREE_EPI_BIAS_GELU>(a);
        case FREE_EPI_GATE_RESID: return launch_one<T, BM, BN, WGM, WGN, S, FREE_EPI_GATE_RESID>(a);
        case FREE_EPI_PARTIAL:
            if constexpr (!std::is_same<T, float>::value) return launch_one<T, BM, BN, WGM, WGN, S, FREE_EPI_PARTIAL>(a);
            return FREE_ERR_RANGE;
        case FREE_EPI_GATE_RESID_SEG:
            if constexpr (!std::is_same<T, float>::value) return launch_one<T, BM, BN, WGM, WGN, S, FREE_EPI_GATE_RESID_SEG>(a);
            return FREE_ERR_RANGE;
        default: return FREE_ERR_RANGE;
    }
}

}  // namespace

bool linear_rows_covers(int32_t N, int32_t K, int32_t elem_bytes, const float* bias, const void* out, const float* resid,
                        const RowVec& gate) {
    auto aligned = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    return K % (kRowBytes / elem_bytes) == 0 && N % 8 == 0 && aligned(bias) && aligned(out) && aligned(resid) &&
           aligned(gate.base) && gate.stride % 4 == 0;
}

template <typename T>
static int32_t launch_rows(const Args<T>& a, int32_t epi, RowsTile tile) {
    if (!linear_rows_covers(a.N, a.K, sizeof(T), a.bias, a.out, a.resid, a.gate)) return FREE_ERR_SHAPE;
    if (tile == ROWS_64x64) return launch_tile<T, 64, 64, 2, 2, 4>(a, epi);
    if (tile == ROWS_128x64) return launch_tile<T, 128, 64, 2, 2, 3>(a, epi);
    // (fp32: as fast as the 128 x 128 tile of gemm_mfma.hip where either is the best one, so there is only that)
    if constexpr (!std::is_same<T, float>::value) {
        if (tile == ROWS_128x128) return launch_tile<T, 128, 128, 2, 4, 4>(a, epi);
    }
    return FREE_ERR_RANGE;
}

int32_t launch_linear_rows(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                           bf16_t* out, float* resid, RowVec gate, hipStream_t s, RowsTile tile, bool from_zero) {
    return launch_rows(Args<bf16_t>{X, W, bias, M, N, K, out, resid, gate, s, from_zero}, epi, tile);
}

int32_t launch_linear_rows(const float* X, const float* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                           float* out, float* resid, RowVec gate, hipStream_t s, RowsTile tile) {
    return launch_rows(Args<float>{X, W, bias, M, N, K, out, resid, gate, s, false}, epi, tile);
}

}  // namespace freemi
