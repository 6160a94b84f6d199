// fp32 GEMM of the dense projections (FREE_FP32): C[M,N] = X[M,K] . W[N,K]^T  (+bias, fused epilogue), K a multiple of 32.
//
// The fp32 matrix instructions run at 157 TFLOP/s, the bf16 ones at 2.5 PFLOP/s.  An fp32 value is the exact sum of three bf16
// values (its 24 significant bits cut in three eights, v = h + m + l, each part the leading bits of what is left; the technique is that of
// Henry, Tang and Heinecke, Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations, 2019), so that
//     x w = xh wh + (xh wm + xm wh + xm wm + xh wl + xl wh + xm wl + xl wm) + xl wl
// and the last product, below 2^-30 of the whole, is the only one left out: eight bf16 products, 256 cycles per 32 x 32 x 16 against
// 512.  (Without xm wl and xl wm, up to 2^-21 of a product, sums of few terms were further off than those of the fp32 instructions:
// one term 5.5e-8 against 2.5e-8; what the two cost: width 1152, MLP-2, 512 rows 58.5 -> 64.6 us, 12288 rows 689 -> 850.)  The leading
// products have an accumulator of their own, which is rounded once per 32 k and not at every second one, and the seven small ones
// another, whose rounding is 2^-7 of that.  2-norm error against 64 bits, fp32 instructions -> here: normal X and W, K = 32 1.0e-7 ->
// 4.2e-8, K = 96 1.8e-7 -> 5.2e-8, K = 1152 6.1e-7 -> 1.4e-7, K = 4608 1.2e-6 -> 2.9e-7; one non-zero per row 2.5e-8, both, and no element
// further off than one rounding; 5 % non-zeros over half a row, K = 32 2.9e-8 -> 2.5e-8, K = 96 3.7e-8 -> 3.3e-8.
// Values that are not finite have no such parts (inf - inf): they give a NaN.  And what is below the smallest bf16 (2^-133) has no
// part: values below 2^-110 lose bits, K values at most K 2^-132 max(|x|, |w|) of a sum, which counts in small sums only.  A wavefront
// that finds a sum that is not finite or below 2^-64 computes its tile again with fp32 products and takes those sums from there.  What is
// left: a value below 2^-110 in a sum of 2^-64 and more, which needs values of some 2^42 / K beside it to be seen in 24 bits; and values
// below 2^-133 where all of a sum consists of them, which are zero.
//
// A slice is 32 k.  Its fp32 values go through registers, two to four slices ahead, are cut there and stored to LDS as three planes
// of 64-byte rows (16-byte chunks swizzled by (row / 4) % 4: neither the stores nor the fragment reads of 16 lanes share a bank; the
// conflict counter reads zero); two stages, one barrier per slice.  Every value is cut once per workgroup, eleven instructions per
// pair.  Eight wavefronts: 2 x 2 parts of the tile, and of every slice one wavefront of a SIMD takes k-step 0, the other k-step 1 -
// with four wavefronts, one per SIMD, the cutting and the products of a wavefront hardly overlap (512 x 1152 x 4608 on 64 x 64 tiles
// six products: 76 us with four, 58 with eight; fp32 instructions 86).
// What bounds it now: the matrix pipe, 0.77 busy on 128 x 128 tiles at 12288 rows (vector pipe 0.37, LDS 0.29); on 64 x 64 tiles at 512
// rows matrix pipe 0.49, vector pipe 0.41, LDS 0.37, which overlap only in part.
#include <algorithm>
#include <cmath>
#include <utility>

#include "free_internal.h"
#include "gemm_dma.h"

namespace freemi {

namespace {

constexpr int kSlice = 32;                   // fp32 values per row and slice (kRowBytes of them)
constexpr int kPlaneRow = kSlice * 2;        // bytes of a row of one plane
constexpr float kSmall = 0x1p-64f;
constexpr int kProducts = 8;                 // of the nine products of two times three parts
constexpr int kWaves = 8;                    // 2 x 2 parts of the tile, each by two wavefronts: k-steps 0 and 1 of every slice

// two fp32 values -> their leading, middle and last eight bits as pairs of bf16
__device__ __forceinline__ void cut2(float v0, float v1, uint32_t (&out)[3]) {
    uint32_t r0 = __float_as_uint(v0), r1 = __float_as_uint(v1);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        out[p] = __builtin_amdgcn_perm(r1, r0, 0x07060302u);                    // the upper halves of r1, r0
        if (p == 2) break;
        r0 = __float_as_uint(__uint_as_float(r0) - __uint_as_float(r0 & 0xffff0000u));
        r1 = __float_as_uint(__uint_as_float(r1) - __uint_as_float(r1 & 0xffff0000u));
    }
}

template <typename F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

template <int BM, int BN, int SETS, int EPI>
__global__ __launch_bounds__(kWaves * 64) void gemm_f32_kernel(
    const float* __restrict__ X, const float* __restrict__ W, const float* __restrict__ bias, int32_t M, int32_t N, int32_t K,
    int32_t tiles_m, int32_t tiles_n, int32_t group_m, int32_t vec_ok, float* __restrict__ out, float* __restrict__ resid,
    RowVec gate) {
    constexpr int NW = kWaves, NT = NW * 64;
    constexpr int TM = BM / 64, TN = BN / 64;                           // 32 x 32 blocks of a wavefront
    constexpr int kRows = BM + BN, kPlane = kRows * kPlaneRow, kStage = 3 * kPlane;
    constexpr int UX = BM * 8 / NT, UP = kRows * 8 / NT;                // groups of four values per thread and slice: of X, of both
    static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0 && NW % 2 == 0, "whole passes: no branch in the K loop");
    extern __shared__ __attribute__((aligned(16))) char lds[];

    int tile_m, tile_n;
    tile_coords(group_m, blockIdx.x, tiles_m, tiles_n, &tile_m, &tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int nk = K / kSlice;

    // ---- loads: group i of this thread is row 8 (i NW + wave) + lane / 8 of the tile (X rows, then W rows), values
    // 4 (lane % 8) .. + 3 of the slice: the lanes walk whole lines.  Rows past the end of a matrix read as zero; a slice past the end
    // of a row reads the row behind (or zero) and is never multiplied.
    const int64_t x_left = static_cast<int64_t>(M - m0) * K * 4, w_left = static_cast<int64_t>(N - n0) * K * 4;
    const __amdgpu_buffer_rsrc_t xsrd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(X + static_cast<int64_t>(m0) * K), 0, static_cast<int>(std::min<int64_t>(x_left, 0x7fffffff)), 0x00020000);
    const __amdgpu_buffer_rsrc_t wsrd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(W + static_cast<int64_t>(n0) * K), 0, static_cast<int>(std::min<int64_t>(w_left, 0x7fffffff)), 0x00020000);
    const int voff = (lane >> 3) * K * 4 + (lane & 7) * 16;
    f32x4_t reg[SETS][UP];                                              // slice k goes through set k % SETS
    auto fetch = [&](int kt, auto set_c, int i) {
        constexpr int set = decltype(set_c)::value;
        const int soff = 8 * ((i < UX ? i : i - UX) * NW + wave) * K * 4 + kt * kRowBytes;
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(i < UX ? xsrd : wsrd, voff, soff, 0);
        reg[set][i] = __builtin_bit_cast(f32x4_t, v);
    };
    // (row / 4) % 4 of this lane's rows is 2 (wave % 2) + lane / 32
    const int st_off = (8 * wave + (lane >> 3)) * kPlaneRow + ((((lane >> 1) & 3) ^ (((wave & 1) << 1) | (lane >> 5))) << 4) + ((lane & 1) << 3);
    u32x2_t part[3];
    // half c of the cutting of group i; the second one stores it to its stage and requests the group of slice kt + SETS
    auto stash = [&](int kt, auto set_c, int i, int c) {
        constexpr int set = decltype(set_c)::value;
        uint32_t two[3];
        cut2(reg[set][i][2 * c], reg[set][i][2 * c + 1], two);
#pragma unroll
        for (int p = 0; p < 3; ++p) part[p][c] = two[p];
        if (c == 0) return;
        char* dst = lds + (kt & 1) * kStage + 8 * i * NW * kPlaneRow + st_off;
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2_t*>(dst + p * kPlane) = part[p];
        fetch(kt + SETS, set_c, i);
    };

    const int choff = (((ks << 1) | lhi) ^ ((l32 >> 2) & 3)) << 4;
    const int x_row = (wm * TM * 32 + l32) * kPlaneRow + choff, w_row = (BM + wn * TN * 32 + l32) * kPlaneRow + choff;
    // Fragments of two slices; the 64 x 64 blocks, short of registers, have two buffers for the leading plane only.
    constexpr bool kTwo = TM * TN < 4;
    u32x4_t fx[2][3][TM], fw[2][3][TN];
    f32x16_t hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                hi[i][j][e] = 0.f;
                lo[i][j][e] = 0.f;
            }
    constexpr int MF = kProducts * TM * TN, NR = 3 * (TM + TN);
    auto buffer = [](int buf, int p) { return p == 0 || kTwo ? buf : 0; };
    auto load_frag = [&](int stage, int buf, int r) {                   // fragment r of a slice: leading, last, middle plane
        const char* base = lds + stage * kStage;
        const int p = (3 - r / (TM + TN)) % 3, f = r % (TM + TN), at = buffer(buf, p);
        if (f < TM) fx[at][p][f] = *reinterpret_cast<const u32x4_t*>(base + p * kPlane + x_row + f * 32 * kPlaneRow);
        else fw[at][p][f - TM] = *reinterpret_cast<const u32x4_t*>(base + p * kPlane + w_row + (f - TM) * 32 * kPlaneRow);
    };
    // the reads of the next slice's fragments behind product t: evenly, or as the planes are used up (last 4, middle 7, of the eight)
    auto reads_until = [](int t) {
        if (kTwo) return t * NR / MF;
        constexpr int u = MF / kProducts, f = TM + TN;
        return t <= 4 * u ? t * f / (4 * u) : t <= 7 * u ? f + (t - 4 * u) * f / (3 * u) : 2 * f + (t - 7 * u) * f / u;
    };
    auto mma = [&](int buf, int t) {
        constexpr int pw[kProducts] = {2, 1, 0, 2, 1, 0, 1, 0}, px[kProducts] = {1, 2, 2, 0, 1, 1, 0, 0};
        const int p = t / (TM * TN), i = t / TN % TM, j = t % TN;
        f32x16_t& acc = p == kProducts - 1 ? hi[i][j] : lo[i][j];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fw[buffer(buf, pw[p])][pw[p]][j]),
                                                      __builtin_bit_cast(bf16x8_t, fx[buffer(buf, px[p])][px[p]][i]), acc, 0, 0, 0);
    };
    // Slice kt, its fragments in buffer `buf`.  Behind the barrier slice kt + 1 is complete in the other stage and every wavefront has
    // read slice kt: the fragments of slice kt + 1 are read, and slice kt + 2 is cut and stored in the place of slice kt, a share of
    // both behind every product (left to itself the compiler does all of the cutting between two products).
    using std::integral_constant;
    auto slice = [&](int kt, auto buf_c, auto set_c) {                  // register set of slice kt + 2
        constexpr int buf = decltype(buf_c)::value;
        wait_lds_barrier();
        // (a loop over t has too much in it for `#pragma unroll`)
        auto share = [&](auto t_c) {
            constexpr int t = decltype(t_c)::value;
            mma(buf, t);
#pragma unroll
            for (int r = reads_until(t); r < reads_until(t + 1); ++r) load_frag((kt + 1) & 1, buf ^ 1, r);
#pragma unroll
            for (int q = t * 2 * UP / MF; q < (t + 1) * 2 * UP / MF; ++q) stash(kt + 2, set_c, q / 2, q % 2);
            __builtin_amdgcn_sched_barrier(0);
        };
        unrolled(share, std::make_integer_sequence<int, MF>{});
    };
    const integral_constant<int, 0> c0{};
    const integral_constant<int, 1> c1{};
    const integral_constant<int, SETS == 4 ? 2 : 0> c2{};
    const integral_constant<int, SETS == 4 ? 3 : 1> c3{};
    auto fetch_all = [&](int kt, auto set_c) {
#pragma unroll
        for (int i = 0; i < UP; ++i) fetch(kt, set_c, i);
    };
    auto stash_all = [&](int kt, auto set_c) {
#pragma unroll
        for (int q = 0; q < 2 * UP; ++q) stash(kt, set_c, q / 2, q % 2);
    };
    fetch_all(0, c0);
    fetch_all(1, c1);
    if constexpr (SETS == 4) {
        fetch_all(2, c2);
        fetch_all(3, c3);
    }
    stash_all(0, c0);
    stash_all(1, c1);
    wait_lds_barrier();
#pragma unroll
    for (int r = 0; r < NR; ++r) load_frag(0, 0, r);
    __builtin_amdgcn_sched_barrier(0);
    int kt = 0;
    for (; kt + 3 < nk; kt += 4) {
        slice(kt, c0, c2);
        slice(kt + 1, c1, c3);
        slice(kt + 2, c0, c0);
        slice(kt + 3, c1, c1);
    }
    if (kt < nk) slice(kt, c0, c2);
    if (kt + 1 < nk) slice(kt + 1, c1, c3);
    if (kt + 2 < nk) slice(kt + 2, c0, c0);

    // ---- the two halves of K: the second wavefronts hand their sums to the first ones through the idle stages
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int e = 0; e < 16; ++e) hi[i][j][e] += lo[i][j][e];
            if (ks == 1) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4_t*>(lds + ((((wave & 3) * TM + i) * TN + j) * 4 + q) * 1024 + lane * 16) =
                        f32x4_t{hi[i][j][4 * q], hi[i][j][4 * q + 1], hi[i][j][4 * q + 2], hi[i][j][4 * q + 3]};
            }
        }
    static_assert(4 * TM * TN * 4096 <= 2 * kStage, "the sums of the second wavefronts must fit in the stages");
    __syncthreads();
    if (ks == 1) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(lds + (((wave * TM + i) * TN + j) * 4 + q) * 1024 + lane * 16);
#pragma unroll
                for (int c = 0; c < 4; ++c) hi[i][j][4 * q + c] += v[c];
            }

    // ---- epilogue
    // Sums that need fp32 products: not finite, or so small that bits below the parts (2^-133 of a value) may count.  Each on its own:
    // what a row is packed with has no part in it.
    auto needs = [](float v) { return !(fabsf(v) >= kSmall && fabsf(v) < INFINITY) && v != 0.f; };
    bool any = false;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) any |= needs(hi[i][j][e]);
    if (__builtin_expect(__any(any), 0)) {
        // (lane group 0 / 1 holds the two k of a product.)  Rows past the end repeat the last one: they are not stored, and a product has
        // its own row and column only.
#pragma unroll 1
        for (int i = 0; i < TM; ++i)
#pragma unroll 1
            for (int j = 0; j < TN; ++j) {
                const int gm = std::min(m0 + (wm * TM + i) * 32 + l32, M - 1), gn = std::min(n0 + (wn * TN + j) * 32 + l32, N - 1);
                const float* xr = X + static_cast<int64_t>(gm) * K + 4 * lhi;
                const float* wr = W + static_cast<int64_t>(gn) * K + 4 * lhi;
                f32x16_t acc;
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 0.f;
                for (int k = 0; k < K; k += 8) {
                    const f32x4_t xv = *reinterpret_cast<const f32x4_t*>(xr + k), wv = *reinterpret_cast<const f32x4_t*>(wr + k);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[e], xv[e], acc, 0, 0, 0);
                }
                // (indexes as constants: an accumulator indexed by a variable would live in scratch memory)
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b)
                        if (a == i && b == j)
#pragma unroll
                            for (int e = 0; e < 16; ++e) hi[a][b][e] = needs(hi[a][b][e]) ? acc[e] : hi[a][b][e];
            }
    }
    float ln_scale[TM];                                                 // (used by the folded-LayerNorm epilogues only)
#pragma unroll
    for (int i = 0; i < TM; ++i) ln_scale[i] = 1.0f;
    write_tile<float, TM, TN, EPI, 0>(hi, m0 + wm * TM * 32 + l32, n0 + wn * TN * 32, lane, M, N, vec_ok, bias, out, resid, gate, nullptr,
                                      LnFold{}, ln_scale);
}

struct Args {
    const float *X, *W, *bias;
    int32_t M, N, K;
    float *out, *resid;
    RowVec gate;
    hipStream_t s;
};

template <int BM, int BN, int SETS, int EPI>
int32_t launch_one(const Args& a) {
    const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN, total = tiles_m * tiles_n;
    const size_t lds = 2 * static_cast<size_t>(BM + BN) * 3 * kPlaneRow;
    auto kern = gemm_f32_kernel<BM, BN, SETS, EPI>;
    static LdsLimit limit;
    if (!limit.allow(reinterpret_cast<const void*>(kern), lds)) return FREE_ERR_HIP;
    // the vector epilogue needs 16-byte aligned rows of out / resid / bias / gate
    auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    const bool vec = ((a.N & 7) == 0) && al16(a.bias) && al16(a.out) && al16(a.resid) && al16(a.gate.base) && ((a.gate.stride & 3) == 0);
    // tile order as in gemm_pipe.hip; with few rows all row tiles of a column, so that a weight panel is fetched by one XCD
    int group_m = total <= 2 * device_cus() ? tiles_m : BM > BN ? 4 : 8;
    hipLaunchKernelGGL(kern, dim3(total), dim3(kWaves * 64), lds, a.s, a.X, a.W, a.bias, a.M, a.N, a.K, tiles_m, tiles_n, group_m,
                       vec ? 1 : 0, a.out, a.resid, a.gate);
    return launch_ok() ? FREE_OK : FREE_ERR_HIP;
}

template <int BM, int BN, int SETS>
int32_t launch_tile(const Args& a, int32_t epi) {
    switch (epi) {
        case FREE_EPI_BIAS: return launch_one<BM, BN, SETS, FREE_EPI_BIAS>(a);
        case FREE_EPI_BIAS_GELU: return launch_one<BM, BN, SETS, FREE_EPI_BIAS_GELU>(a);
        case FREE_EPI_GATE_RESID: return launch_one<BM, BN, SETS, FREE_EPI_GATE_RESID>(a);
        default: return FREE_ERR_RANGE;
    }
}

}  // namespace

bool linear_f32_covers(const float* X, const float* W, int32_t M, int32_t N, int32_t K) {
    // whole slices of 16-byte aligned rows; 32-bit byte offsets inside a tile and three slices past the end of its rows
    return M >= 1 && N >= 1 && K >= kSlice && K % kSlice == 0 && static_cast<int64_t>(K) * 4 * 130 < (1ll << 31) &&
           ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(W)) & 15u) == 0;
}

// Which tile: 128 x 128 takes half as many bytes from LDS per product, 64 x 64 gives few rows to more CUs (two or three share a
// CU).  Constants from both tiles, launches back to back, at 17 values of M from 64 to 12288 and the four layers at widths 384, 768 and
// 1152: the faster tile is chosen within 0.4 % everywhere (those fitted to six products at width 1152 alone chose tiles up to 26 %
// slower, 0.6 % on average: 4096 x 1152 x 1152 114 us for 90).  us at width 1152 (QKV, out-projection, MLP-1, MLP-2), 64 x 64 /
// 128 x 128; the fp32 instructions at the first:   256 rows 22 20 34 63 / 49 49 51 166 (25 24 42 83)
//      512 rows 36 22 53 65 / 52 49 55 167 (45 24 62 86)     2048 rows 125 53 164 190 / 117 55 176 174 (146 60 190 215)
//      12288 rows 717 250 953 931 / 650 245 850 841 (805 290 922 1045)
// Both add in the same order: the result does not depend on the choice.
int32_t launch_linear_f32(const float* X, const float* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                          float* out, float* resid, RowVec gate, hipStream_t s, int cu_share) {
    if (!linear_f32_covers(X, W, M, N, K)) return FREE_ERR_SHAPE;
    const Args a{X, W, bias, M, N, K, out, resid, gate, s};
    const double cus = std::max(1, device_cus() / std::max(1, cu_share)), nk = K / kSlice;
    const auto rounds = [&](int b) { return std::ceil(static_cast<double>((M + b - 1) / b) * ((N + b - 1) / b) / cus); };
    const double n64 = rounds(64), t64 = 4.4 + nk * (n64 <= 1.0 ? 0.526 : 0.499 * n64), t128 = rounds(128) * (7.5 + 1.455 * nk);
    return t64 <= t128 ? launch_tile<64, 64, 4>(a, epi) : launch_tile<128, 128, 2>(a, epi);
}

}  // namespace freemi
