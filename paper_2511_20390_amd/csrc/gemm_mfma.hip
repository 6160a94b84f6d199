// bf16 MFMA GEMM for the dense projections of the DiT blocks (QKV, attention
// out-projection, MLP FC1/FC2 of the packed target forward, Alg. 1):
//   C[M,N] = X[M,K] . W[N,K]^T  (+bias, fused epilogue), fp32 accumulation.
// Both operands are K-contiguous, which is exactly the per-lane operand layout of
// v_mfma_f32_32x32x16_bf16 (lane l: row/col l%32, 8 consecutive k at 8*(l/32)).
//
// Design for gfx950 (64-wide wavefronts, 160 KB LDS per CU, 512 registers per lane):
//  * used for fp32 operands (of models where K is no multiple of 32, else gemm_f32.hip; of free_op_linear always) and for bf16 with
//    K no multiple of the slice; bf16 problems of whole slices are chosen between
//    the tiles of gemm_pipe.hip and gemm_rows.hip at the end of this file.  Rates quoted below for bf16 were measured when
//    this kernel took those as well.
//  * workgroup = 4 or 8 wavefronts in a WGM x WGN grid, macro tile BM x BN (256x256 and
//    384x192 with 8 wavefronts - two per SIMD, so one wavefront's memory instructions issue
//    under the other's MFMAs - 256x128 / 128x128 / 96x128 / 160x128 with 4 for small problems), K slices of
//    64; each wavefront owns (BM/WGM) x (BN/WGN) as TM x TN MFMA tiles of 32x32 and keeps
//    the accumulators in registers for the whole K loop.
//  * the MFMA takes the WEIGHT rows as its A operand and the activation rows as its
//    B operand, i.e. it accumulates C^T tiles: a lane then owns one output ROW m
//    (lane % 32) and runs of 4 consecutive output columns n per register group.  Each
//    32-row block of output is transposed through a wave-private piece of the (by then idle)
//    LDS tiles so that global accesses cover whole rows of the wave's tile with consecutive
//    lanes - a row otherwise lives in two lanes, 32 bytes per row and instruction, and such
//    partial-line writes cost up to 1.8x the algorithmic write traffic at the memory
//    controller.  For bf16 output one v_permlane32_swap first pairs the two half-waves' runs
//    into 8 consecutive bf16; the fp32 residual update is a float4 read-modify-write on the
//    transposed block with all loads of a group issued before its first store.
//  * LDS: two stages of [BM + BN rows][64 bf16]; the 16-byte chunk index of a row is
//    XOR-swizzled with (row / 2) % 8: a ds_read_b128 is served 16 lanes at a time over 64
//    banks (256 bytes), and with this pattern the 16 rows of a pass hit 16 distinct 16-byte
//    bank groups (the conflict counter reads zero; swizzling with row % 8 leaves rows r and
//    r + 8 on the same banks, a 2-way conflict on every fragment read).  Global loads stay
//    128-byte coalesced.
//  * global loads are buffer loads (descriptor + one per-lane offset + scalar offsets):
//    no address registers, and rows past the end of a ragged edge tile read as zero.
//  * software pipeline: global loads run two slices ahead (slice kt+2 is in flight in
//    registers while slice kt+1 is written to the other LDS stage and slice kt is
//    multiplied); the LDS writes and the refills are spread over three of the four
//    k-steps; MFMA operand fragments are double-buffered in registers so every LDS read
//    is issued one k-step before its use; issue order is pinned with
//    sched_group_barrier.  One barrier per slice, placed before the last k-step so the
//    first fragments of the next slice are read under that step's MFMAs.
//  * workgroup ids are remapped so that each of the 8 XCDs (round-robin dispatch)
//    works on a compact, L2-friendly group of tiles.
//  * the tile configuration is chosen per problem from a measured time model (whole
//    rounds of workgroups x (K slices x time per slice + per-tile fixed cost)).
//  * FREE_FP32 mode runs the same kernel on fp32 operands: a K slice is still 128 bytes per row
//    (32 values), a fragment still one 16-byte chunk per lane, and each chunk pair feeds four
//    v_mfma_f32_32x32x2_f32 (one per element of the chunk: lane group 0 supplies k = 4 c + e,
//    group 1 supplies k = 4 (c + 1) + e, the same pairing for both operands); full fp32
//    products and accumulation, fp32 output through the LDS-staged row-major stores.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "free_internal.h"
#include "gemm_tile.h"

namespace freemi {

int device_cus() {
    static int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        return n;
    }();
    return cus;
}

namespace {

// T: bf16_t or float (operands and the output of the bias / GELU epilogues).  EVEN_K: K a multiple of the
// slice (64 bf16 or 32 fp32: no predicates in the K loop).  Rows past the end of a ragged M / N tile read
// as zero (extra rows are computed, never stored).
template <typename T, int BM, int BN, int WGM, int WGN, int EPI, bool EVEN_K>
__global__ __launch_bounds__(WGM * WGN * 64) void gemm_bf16_kernel(
    const T* __restrict__ X, const T* __restrict__ W, const float* __restrict__ bias, int32_t M,
    int32_t N, int32_t K, int32_t tiles_m, int32_t tiles_n, int32_t group_m, int32_t vec_ok,
    T* __restrict__ out, float* __restrict__ resid, RowVec gate) {
    static_assert(WGM * WGN == 4 || WGM * WGN == 8, "four or eight wavefronts per workgroup");
    constexpr bool kF32 = std::is_same<T, float>::value;
    constexpr int ES = static_cast<int>(sizeof(T));    // bytes per element
    constexpr int BKE = kRowBytes / ES;                // elements per K slice
    constexpr int CE = 16 / ES;                        // elements per 16-byte chunk
    constexpr int NT = WGM * WGN * 64;                 // threads per workgroup
    constexpr int RP = NT / 8;                         // tile rows covered by one pass of 16-byte loads
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
    constexpr int LA = BM / RP, LB = BN / RP;          // 16-byte loads per thread per slice
    constexpr int kStageBytes = (BM + BN) * kRowBytes;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    int tile_m, tile_n;
    tile_coords(group_m, blockIdx.x, tiles_m, tiles_n, &tile_m, &tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    // (the wavefront index as a scalar: the position of the wavefront's part of the tile, the test for an all-padding
    // wavefront and the LDS offsets that follow from it stay in scalar registers)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    // ---- global -> register staging: chunk idx = i*NT + tid, row = idx/8, chunk = idx%8
    const int ld_chunk = tid & 7;
    const int ld_row = tid >> 3;
    // Buffer descriptors over the rows of this tile: a load past the end of the matrix (rows
    // of a ragged edge tile) returns zeros, so no row clamping and no address registers -
    // one per-lane byte offset plus wave-uniform (scalar) offsets per load and per slice.
    const int64_t x_left = static_cast<int64_t>(M - m0) * K * ES, w_left = static_cast<int64_t>(N - n0) * K * ES;
    const __amdgpu_buffer_rsrc_t xsrd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(X + static_cast<int64_t>(m0) * K), 0,
        static_cast<int>(x_left < 0x7fffffff ? x_left : 0x7fffffff), 0x00020000);
    const __amdgpu_buffer_rsrc_t wsrd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(W + static_cast<int64_t>(n0) * K), 0,
        static_cast<int>(w_left < 0x7fffffff ? w_left : 0x7fffffff), 0x00020000);
    const int ld_voff = ld_row * K * ES + ld_chunk * 16;      // per-lane byte offset inside the tile
    const int pass_bytes = RP * K * ES;                       // RP rows further down per load index
    const int st_off = ld_row * kRowBytes + ((ld_chunk ^ ((ld_row >> 1) & 7)) << 4);   // + i*RP rows per load
    u32x4_t sreg[LA + LB];                              // staging registers: one K slice in flight
    const int nk = (K + BKE - 1) / BKE;

    // staging register idx in [0, LA + LB): the first LA hold X rows, the rest W rows
    constexpr int NS = LA + LB;
    auto fetch_range = [&](int kt, int lo, int hi) {
        const int kbyte = kt * kRowBytes;
        const bool in_k = EVEN_K || (kt * BKE + ld_chunk * CE) < K;   // K a multiple of the chunk: all in or all out
#pragma unroll
        for (int idx = 0; idx < NS; ++idx) {
            if (idx < lo || idx >= hi) continue;
            const u32x4_t v = (idx < LA)
                                  ? __builtin_amdgcn_raw_buffer_load_b128(xsrd, ld_voff, idx * pass_bytes + kbyte, 0)
                                  : __builtin_amdgcn_raw_buffer_load_b128(wsrd, ld_voff, (idx - LA) * pass_bytes + kbyte, 0);
            sreg[idx] = in_k ? v : u32x4_t{0, 0, 0, 0};
        }
    };
    auto stash_range = [&](int stage, int lo, int hi) {
        char* base = lds + stage * kStageBytes + st_off;
#pragma unroll
        for (int idx = 0; idx < NS; ++idx) {
            if (idx < lo || idx >= hi) continue;
            const int row = (idx < LA) ? idx * RP : BM + (idx - LA) * RP;
            *reinterpret_cast<u32x4_t*>(base + row * kRowBytes) = sreg[idx];
        }
    };

    // ---- MFMA operand fragments: row fixed per lane, chunk varies with the k step
    const int l32 = lane & 31, lhi = lane >> 5;
    const int sw = (l32 >> 1) & 7;                         // (row / 2) % 8 (tile row offsets are multiples of 32)
    const int x_row0 = (wm * TM * 32 + l32) * kRowBytes;           // + i*32 rows
    const int w_row0 = (BM + wn * TN * 32 + l32) * kRowBytes;      // + j*32 rows
    u32x4_t fx[2][TM], fw[2][TN];                      // one 16-byte chunk each: 8 bf16 or 4 fp32
    // A wavefront whose part of the tile lies wholly past N or M (N = 1152 is 4.5 tiles of 256 columns: the right
    // half of every fifth tile) takes part in the staging and the barriers only: its products would be thrown
    // away, and on a chip that runs at its power limit they are not free for the others.
    // (bf16 only: in the fp32 instantiation, whose K loop is matrix-bound, the branch costs 4 % on every launch)
    // How the test enters the K loop depends on the wavefronts a SIMD holds.  Eight-wavefront workgroups (two per
    // SIMD) keep it inside the loop: it splits the body into basic blocks, each k-step becomes "LDS traffic, wait
    // for all of it, eight products", and the two wavefronts of a SIMD alternate - measured faster than the
    // interleaved form.  Four-wavefront workgroups (one per SIMD: the tiles of problems with few rows) have nobody
    // to alternate with: there the wait for the NEXT step's fragments in front of every burst is pure latency
    // (measured 0.66 us per slice for 0.22 us of products), so they take one of two straight-line copies of the
    // loop (with / without products, chosen once), in which the compiler counts the LDS reads in flight and the
    // products of a step overlap the reads of the next.
    const bool wave_on = kF32 || ((n0 + wn * TN * 32 < N) && (m0 + wm * TM * 32 < M));
    constexpr bool kStraight = !kF32 && WGM * WGN <= 4;
    struct InLoop {};                                  // tag: test the flag inside the loop
    auto is_on = [&](auto tag) {
        if constexpr (std::is_same<decltype(tag), InLoop>::value) return wave_on;
        else return decltype(tag)::value;
    };
    auto load_frags = [&](const char* base, int ks, int buf, auto tag) {
        if (!is_on(tag)) return;
        const int choff = (((ks << 1) | lhi) ^ sw) << 4;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fx[buf][i] = *reinterpret_cast<const u32x4_t*>(base + x_row0 + i * 32 * kRowBytes + choff);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fw[buf][j] = *reinterpret_cast<const u32x4_t*>(base + w_row0 + j * 32 * kRowBytes + choff);
    };

    f32x16_t acc[TM][TN];                                  // acc[i][j]: rows n (tile j), columns m (tile i)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    auto mma = [&](int buf, auto tag) {
        if (!is_on(tag)) return;
        if constexpr (kF32) {
            // element e of the chunk: the lanes of group 0 / 1 hold the two k of one 32x32x2 product
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        // (copied out first: a bit cast applied directly to a vector element read element 0)
                        const uint32_t wbits = fw[buf][j][e], xbits = fx[buf][i][e];
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, wbits),
                                                                        __builtin_bit_cast(float, xbits),
                                                                        acc[i][j], 0, 0, 0);
                    }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fw[buf][j]),
                                                                        __builtin_bit_cast(bf16x8_t, fx[buf][i]),
                                                                        acc[i][j], 0, 0, 0);
        }
    };
    // One K slice.  Precondition: fragments of k-step 0 are in buffer 0.  The staging
    // registers hold slice kt+1; they are written to the other LDS stage in three
    // portions (k-steps 0..2), and each freed portion is immediately refilled with the
    // global loads of slice kt+2.  Spreading the LDS writes matters: the LDS write path
    // is much narrower than the read path, a burst of 16 writes per lane stalls issue.
    //   k-step 0..2: multiply | read fragments of the next step | write + refill a third
    //   barrier: the other stage is complete, this stage will not be read again
    //   k-step 3: multiply | read fragments of step 0 of slice kt+1 from the other stage
    constexpr int MF = TM * TN * (kF32 ? 4 : 1), NR = TM + TN;
    constexpr int C1 = (NS + 2) / 3, C2 = (2 * NS + 2) / 3;      // portion boundaries
    auto slice = [&](int kt, auto stash_next, auto fetch_ahead, auto tag) {
        constexpr bool kStash = decltype(stash_next)::value, kFetch = decltype(fetch_ahead)::value;
        const char* base = lds + (kt & 1) * kStageBytes;
        const int nst = (kt + 1) & 1;
        load_frags(base, 1, 1, tag);
        if (kStash) stash_range(nst, 0, C1);
        if (kFetch) fetch_range(kt + 2, 0, C1);
        mma(0, tag);
        sched_hints<0, MF, NR, kStash ? C1 : 0, kFetch ? C1 : 0>();
        load_frags(base, 2, 0, tag);
        if (kStash) stash_range(nst, C1, C2);
        if (kFetch) fetch_range(kt + 2, C1, C2);
        mma(1, tag);
        sched_hints<0, MF, NR, kStash ? C2 - C1 : 0, kFetch ? C2 - C1 : 0>();
        load_frags(base, 3, 1, tag);
        if (kStash) stash_range(nst, C2, NS);
        if (kFetch) fetch_range(kt + 2, C2, NS);
        mma(0, tag);
        sched_hints<0, MF, NR, kStash ? NS - C2 : 0, kFetch ? NS - C2 : 0>();
        __syncthreads();
        if (kStash) load_frags(lds + nst * kStageBytes, 0, 0, tag);
        mma(1, tag);
        sched_hints<0, MF, kStash ? NR : 0, 0, 0>();
    };
    const std::true_type yes{};
    const std::false_type no{};

    // ---- prologue: slice 0 through the registers into LDS stage 0, slice 1 into the registers
    fetch_range(0, 0, NS);
    stash_range(0, 0, NS);
    if (nk > 1) fetch_range(1, 0, NS);
    __syncthreads();
    // ---- steady state: slice kt multiplies while slice kt+1 moves registers -> LDS and
    //      slice kt+2 is requested from global memory
    auto k_loop = [&](auto tag) {
        load_frags(lds, 0, 0, tag);
        int kt = 0;
        for (; kt + 2 < nk; ++kt) slice(kt, yes, yes, tag);
        if (kt + 1 < nk) {
            slice(kt, yes, no, tag);
            ++kt;
        }
        slice(kt, no, no, tag);
    };
    if constexpr (kF32) {
        k_loop(yes);
    } else if constexpr (kStraight) {
        if (wave_on) k_loop(yes);
        else k_loop(no);
    } else {
        k_loop(InLoop{});
    }

    // ---- epilogue
    // after the barrier of the last slice no wavefront reads the LDS tiles any more: each wavefront
    // may use a private region of them to transpose its output
    constexpr bool kResidEpi = EPI == FREE_EPI_GATE_RESID;
    constexpr int kWaveStage = (kResidEpi || kF32) ? 32 * (((TN % 2 == 0 ? 2 : 1) * 8 + 1) * 16)   // fp32 groups
                                                   : 32 * (TN * 64 + 16);                            // bf16 rows
    static_assert(WGM * WGN * kWaveStage <= 2 * kStageBytes, "output staging must fit in the K-loop tiles");
    constexpr int kResidBatch = (WGM * WGN == 8) ? 4 : 0;
    float ln_scale[TM];                                    // (used by the folded-LayerNorm epilogues only)
#pragma unroll
    for (int i = 0; i < TM; ++i) ln_scale[i] = 1.0f;
    write_tile<T, TM, TN, EPI, kResidBatch>(acc, m0 + wm * TM * 32 + l32, n0 + wn * TN * 32, lane, M, N, vec_ok, bias, out, resid, gate,
                            lds + wave * kWaveStage, LnFold{}, ln_scale);
}

template <typename T, int BM, int BN, int WGM, int WGN, int EPI, bool EVEN_K>
int32_t launch_one(const T* X, const T* W, const float* bias, int32_t M, int32_t N, int32_t K, T* out,
                   float* resid, RowVec gate, hipStream_t s) {
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const size_t lds = 2 * static_cast<size_t>(BM + BN) * kRowBytes;
    auto kern = gemm_bf16_kernel<T, BM, BN, WGM, WGN, EPI, EVEN_K>;
    static LdsLimit limit;
    if (!limit.allow(reinterpret_cast<const void*>(kern), lds)) return FREE_ERR_HIP;
    // the vector epilogue needs 16-byte aligned rows of out / resid / bias / gate
    auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    const bool vec = ((N & 7) == 0) && al16(bias) && al16(out) && al16(resid) && al16(gate.base) &&
                     ((gate.stride & 3) == 0);
    const int32_t vec_ok = vec ? 1 : 0;
    // Row tiles per group of the tile order.  Several rounds of workgroups: the 32 that run together on an
    // XCD should cover a x b tiles with a BM ~ b BN, the shape that needs the fewest distinct X and W panels
    // (first-touch misses of that XCD's L2).  A single round: every XCD holds total / 8 tiles for the whole
    // kernel, and a group of exactly that many tiles - whole tile rows - keeps each X panel in one L2
    // (FC2 at 12288 rows: 361 MB fetched with groups of 8 row tiles, X read by two or three XCDs each).
    // This is about traffic, not time: the Infinity Cache served the repeats at no measurable cost.
    const int total = tiles_m * tiles_n;
    int group_m = BM > BN ? 4 : 8;
    if (total <= device_cus()) {
        const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
        group_m = std::max(1, (per_xcd + tiles_n / 2) / tiles_n);
    }
    hipLaunchKernelGGL(kern, dim3(total), dim3(WGM * WGN * 64), lds, s, X, W, bias, M, N, K, tiles_m, tiles_n, group_m,
                       vec_ok, out, resid, gate);
    return launch_ok() ? FREE_OK : FREE_ERR_HIP;
}

template <typename T, int BM, int BN, int WGM, int WGN>
int32_t launch_cfg(const T* X, const T* W, const float* bias, int32_t M, int32_t N, int32_t K,
                   int32_t epi, T* out, float* resid, RowVec gate, hipStream_t s) {
    // (bf16 problems of whole slices go to gemm_pipe.hip and gemm_rows.hip)
    constexpr bool kRaggedOnly = std::is_same<T, bf16_t>::value;
    const bool even = !kRaggedOnly && (K % (kRowBytes / static_cast<int>(sizeof(T)))) == 0;
#define FREE_GEMM_CASE(E)                                                                                              \
    case E:                                                                                                            \
        return even ? launch_one<T, BM, BN, WGM, WGN, E, !kRaggedOnly>(X, W, bias, M, N, K, out, resid, gate, s)       \
                    : launch_one<T, BM, BN, WGM, WGN, E, false>(X, W, bias, M, N, K, out, resid, gate, s)
    switch (epi) {
        FREE_GEMM_CASE(FREE_EPI_BIAS);
        FREE_GEMM_CASE(FREE_EPI_BIAS_GELU);
        FREE_GEMM_CASE(FREE_EPI_GATE_RESID);
        default: return FREE_ERR_RANGE;
    }
#undef FREE_GEMM_CASE
}

// Estimated time (us) of a tile configuration on `cus` compute units: workgroup rounds times
// (K slices x measured time per slice + per-tile prologue/epilogue), measured on MI355X in bf16 (one machine's
// microseconds: machines of the type differ by a few per cent, and half-share launches reuse them).  nk: 128-byte
// K slices; slice_scale: time of a slice relative to bf16 (fp32: 4.4 - four 16-pass MFMAs per chunk pair instead of
// one 8-pass MFMA, at the slightly higher clock the fp32 products leave).
double cfg_time(int M, int N, int nk, int bm, int bn, double us_per_slice, double us_fixed, int cus) {
    const double tiles = static_cast<double>((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    const double rounds = std::ceil(tiles / cus);
    return rounds * (nk * us_per_slice + us_fixed);
}

// The 128x128 configuration is small enough for two workgroups per CU: measured 0.6 us per slice for a
// workgroup that has its CU to itself and 1.05 us each for two that share one.  Used for problems of
// few rows, where it decides between half-empty rounds of large tiles and fuller rounds of small ones.
double small_tile_time(int M, int N, int nk, double sc, int cus) {
    const double tiles = static_cast<double>((M + 127) / 128) * ((N + 127) / 128);
    const double shared = nk * 1.05 * sc + 4.0, alone = nk * 0.6 * sc + 4.0;
    const double full = std::floor(tiles / (2.0 * cus));
    const double rest = tiles - full * 2.0 * cus;
    return full * shared + (rest == 0.0 ? 0.0 : (rest <= cus ? alone : shared));
}

enum StagedTile { STAGED_96x128, STAGED_128x128, STAGED_160x128, STAGED_256x128, STAGED_256x256, STAGED_384x192 };

// cus: compute units this launch can count on.  Tiles change how the output is cut, never the order in which a dot product is
// summed, so the result does not depend on the choice.
StagedTile choose_staged(int32_t M, int32_t N, int nk, double sc, int cus) {
    const double t256 = cfg_time(M, N, nk, 256, 256, 1.83 * sc, 9.0, cus);
    const double t384 = cfg_time(M, N, nk, 384, 192, 2.06 * sc, 10.0, cus);
    const double t2x1 = cfg_time(M, N, nk, 256, 128, 1.31 * sc, 6.0, cus);
    const double t128 = M <= 4096 ? small_tile_time(M, N, nk, sc, cus) : cfg_time(M, N, nk, 128, 128, 0.80 * sc, 4.0, cus);
    // 96 x 128 (one row of four wavefronts, each 96 x 32): for problems of few rows and few columns, where
    // 128 x 128 tiles leave compute units empty (2048 x 1152: 144 tiles on 256 CUs; 198 of three quarters the work)
    double t96 = 1e30;
    {
        const double tiles = static_cast<double>((M + 95) / 96) * ((N + 127) / 128);
        if (tiles <= cus && M <= 4096) t96 = nk * 0.47 * sc + 4.0;      // measured 0.47 us per slice
    }
    // 160 x 128 (same shape of workgroup, 160 x 32 per wavefront): for few rows and many columns, where 128 x 128
    // tiles spill into a second round (2048 x 4608: 576 tiles on 512 slots; 468 of 160 x 128).  Measured about
    // 1.25 x the slice time of 128 x 128, alone and shared.
    double t160 = 1e30;
    if (M <= 4096) {
        const double tiles = static_cast<double>((M + 159) / 160) * ((N + 127) / 128);
        if (tiles <= cus) t160 = nk * 0.80 * sc + 4.0;
        else if (tiles <= 2.0 * cus) t160 = nk * 1.40 * sc + 4.0;
    }
    const double best = std::fmin(std::fmin(std::fmin(t256, t384), std::fmin(t2x1, t128)), std::fmin(t96, t160));
    if (best == t160) return STAGED_160x128;
    if (best == t96) return STAGED_96x128;
    if (best == t384) return STAGED_384x192;
    if (best == t256) return STAGED_256x256;
    if (best == t2x1) return STAGED_256x128;
    return STAGED_128x128;
}

template <typename T>
int32_t launch_staged(StagedTile tile, const T* X, const T* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                      T* out, float* resid, RowVec gate, hipStream_t s) {
    switch (tile) {
        case STAGED_96x128: return launch_cfg<T, 96, 128, 1, 4>(X, W, bias, M, N, K, epi, out, resid, gate, s);
        case STAGED_128x128: return launch_cfg<T, 128, 128, 2, 2>(X, W, bias, M, N, K, epi, out, resid, gate, s);
        case STAGED_160x128: return launch_cfg<T, 160, 128, 1, 4>(X, W, bias, M, N, K, epi, out, resid, gate, s);
        case STAGED_256x128: return launch_cfg<T, 256, 128, 2, 2>(X, W, bias, M, N, K, epi, out, resid, gate, s);
        case STAGED_256x256: return launch_cfg<T, 256, 256, 4, 2>(X, W, bias, M, N, K, epi, out, resid, gate, s);
        case STAGED_384x192: return launch_cfg<T, 384, 192, 4, 2>(X, W, bias, M, N, K, epi, out, resid, gate, s);
    }
    return FREE_ERR_RANGE;
}

// A tile of one of the three kernels and the constants of its time.
enum TileFamily { TILE_STAGED, TILE_ROWS, TILE_PIPE };     // this file, gemm_rows.hip, gemm_pipe.hip
struct TileTime {
    TileFamily family;
    int tile, bm, bn;
    bool paired, paired_resid;    // two workgroups fit a CU (80 KB of LDS and the registers): bias epilogues, residual update
    double f;                     // per launch
    double e_bias, e_gelu, e_resid;    // per round of workgroups, by epilogue
    double a, b, d;               // per slice alone; per slice and per round for each of two that share a CU
};

// Tile choice for bf16 problems of whole slices.  Time of a launch: `f` + per round of workgroups (nk slices + `e`), with
// `a` us per slice for a workgroup that has its CU to itself, and `b` per slice and `d` more per round for each of two that
// share one.  Constants fitted to the times of every tile at 50 values of M from 64 to 12288 and the layer shapes at widths 384,
// 768 and 1152, weights from HBM and from the caches in equal parts, so that the tile chosen is close to the best one (a tile
// within some 3 % of the best counts in part: no choice hangs on the last digit); the times themselves are met to 14 % rms.
// The tile chosen is 0.2 % behind the best one on average, 15 % at worst (4095 x 384 x 768: 11.6 us for 10.1).  One `e` for all
// epilogues and both kinds of round, as the table had before, was 1.0 % behind on average and a third at worst (4000 x 768 x
// 768 with the residual update 15.2 us, now 11.3; 2048 x 4608 x 1152 with GELU 28.5 us, now 26.2): the epilogue of a
// residual update moves eight bytes per element where the others move two.
// Tiles change how the output is cut, never the order in which a dot product is summed, so the result does not depend on the
// choice.
constexpr TileTime kTiles[] = {
    {TILE_ROWS, ROWS_64x64, 64, 64, true, true, 1.1, 1.2, 1.6, 1.7, 0.215, 0.449, 0.0},
    {TILE_ROWS, ROWS_128x64, 128, 64, true, true, 0.9, 2.0, 2.4, 3.6, 0.256, 0.717, 0.7},
    {TILE_ROWS, ROWS_128x128, 128, 128, false, false, 0.1, 5.1, 5.8, 11.3, 0.318, 0.0, 0.0},
    {TILE_PIPE, PIPE_128x128, 128, 128, true, true, 0.0, 3.0, 3.7, 2.8, 0.567, 0.811, 1.1},
    {TILE_PIPE, PIPE_160x128, 160, 128, true, false, 1.0, 4.3, 6.0, 10.2, 0.475, 0.829, 1.8},
    {TILE_PIPE, PIPE_192x128, 192, 128, true, true, 0.0, 3.9, 4.6, 4.4, 0.627, 0.981, 3.8},
    {TILE_PIPE, PIPE_256x192, 256, 192, false, false, 1.7, 1.6, 4.7, 4.2, 1.188, 0.0, 0.0},
    {TILE_PIPE, PIPE_192x256, 192, 256, false, false, 0.0, 7.6, 10.7, 9.6, 0.958, 0.0, 0.0},
    {TILE_PIPE, PIPE_256x256, 256, 256, false, false, 1.4, 5.7, 8.5, 12.4, 1.135, 0.0, 0.0},
    {TILE_PIPE, PIPE_384x192, 384, 192, false, false, 1.8, 6.9, 9.9, 12.6, 1.300, 0.0, 0.0},
};

// The same for fp32 (slices of 32, whole ones).  A slice of a 32 x 32 block is 16 products of 64 cycles, so the matrix cores
// decide as soon as every SIMD has a wavefront, and below that the number of tiles does: 512 x 1152 x 4608 is 54 tiles of
// 96 x 128 (217 us) or 144 of 64 x 64 (89 us).  Fitted to every tile at 18 values of M from 64 to 4096 and the four layer
// shapes at widths 384, 768 and 1152 (rms error 2-5 %); the chosen tile is within 1 % of the best one on average, 5 % at
// worst, up to kFewRowsF32 rows.  Above that the rule of choose_staged is as good.  us, old rule -> this one, at width
// 1152 (QKV, out-projection, MLP-1, MLP-2):  64 rows 57 56 56 208 -> 24 24 23 82;  512 rows 61 59 64 217 -> 44 26 64 89;
// 1024 rows 77 60 96 218 -> 75 44 96 153;  2048 rows 142 63 179 229 -> 141 63 179 229.
constexpr int kFewRowsF32 = 2048;
constexpr TileTime kTilesF32[] = {
    {TILE_ROWS, ROWS_64x64, 64, 64, true, true, 2.0, 2.3, 2.3, 2.3, 0.572, 1.082, 0.0},
    {TILE_ROWS, ROWS_128x64, 128, 64, true, true, 3.9, 1.7, 1.7, 1.7, 1.038, 2.043, 0.0},
    {TILE_STAGED, STAGED_96x128, 96, 128, true, true, 3.5, 2.8, 2.8, 2.8, 1.455, 2.872, 0.0},
    {TILE_STAGED, STAGED_128x128, 128, 128, true, true, 8.0, 0.0, 0.0, 0.0, 1.881, 3.739, 0.0},
    {TILE_STAGED, STAGED_160x128, 160, 128, true, true, 0.0, 8.6, 8.6, 8.6, 2.329, 4.623, 0.0},
    {TILE_STAGED, STAGED_256x256, 256, 256, false, false, 0.6, 9.9, 9.9, 9.9, 7.039, 0.0, 0.0},
};

// Time of a launch of `u` workgroups per CU.  last_alone: up to this many workgroups per CU left over after the full pairs
// run as if they had a CU each.
double launch_time(const TileTime& t, int32_t epi, double u, int nk, double last_alone) {
    const bool resid = epi == FREE_EPI_GATE_RESID || epi == FREE_EPI_GATE_RESID_PREP || epi == FREE_EPI_PARTIAL ||
                       epi == FREE_EPI_GATE_RESID_SEG;       // (fp32 sums out: as many bytes per element as a residual update's)
    const bool gelu = epi == FREE_EPI_BIAS_GELU || epi == FREE_EPI_LN_BIAS_GELU;
    const double e = resid ? t.e_resid : gelu ? t.e_gelu : t.e_bias;
    const double alone = nk * t.a + e, shared = nk * t.b + e + t.d;
    if (!(resid ? t.paired_resid : t.paired)) return t.f + std::ceil(u) * alone;
    const double full = std::floor(u / 2.0), rest = u - 2.0 * full;
    return t.f + full * shared + (rest <= 0.0 ? 0.0 : rest <= (full > 0.0 ? last_alone : 1.0) ? alone : shared);
}

// What a problem is launched on.  rows_ok: linear_rows_covers holds.  cu_share: how many launches of this size are expected to
// run side by side (the parts of a packed batch on several streams); the tile is chosen for that share of the compute units.
struct Choice {
    TileFamily family;
    int tile, bm, bn;
};
Choice choose(int32_t M, int32_t N, int32_t K, int elem_bytes, int32_t epi, bool rows_ok, int cu_share, double* time = nullptr) {
    const int cus = std::max(1, device_cus() / std::max(1, cu_share));
    const int slice = kRowBytes / elem_bytes, nk = (K + slice - 1) / slice;
    const bool f32 = elem_bytes == 4;
    if (K % slice != 0 || (f32 && M > kFewRowsF32)) {
        static constexpr int dims[][2] = {{96, 128}, {128, 128}, {160, 128}, {256, 128}, {256, 256}, {384, 192}};
        const StagedTile t = choose_staged(M, N, nk, f32 ? 4.4 : 1.0, cus);
        return {TILE_STAGED, t, dims[t][0], dims[t][1]};
    }
    const TileTime* best = nullptr;
    double t_best = 0.0;
    auto consider = [&](const TileTime& t, double last_alone) {
        if (t.family == TILE_ROWS && (!rows_ok || (epi > FREE_EPI_GATE_RESID && epi != FREE_EPI_GATE_RESID_SEG))) return;
        if (epi == FREE_EPI_GATE_RESID_SEG && t.bm * t.bn > kSegTileArea) return;
        if (epi == FREE_EPI_GATE_RESID_PREP && t.bn != 256) return;          // whole 128-column slots of row sums
        const double u = static_cast<double>((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) / cus;
        const double t_launch = launch_time(t, epi, u, nk, last_alone);
        if (best == nullptr || t_launch < t_best) {
            best = &t;
            t_best = t_launch;
        }
    };
    if (f32)
        for (const TileTime& t : kTilesF32) consider(t, 0.75);
    else
        for (const TileTime& t : kTiles) consider(t, 1.0);
    if (time) *time = t_best;
    return {best->family, best->tile, best->bm, best->bn};
}

}  // namespace

bool mfma_linear_supported(int32_t M, int32_t N, int32_t K) {
    // 32-bit byte offsets inside a tile: up to 384 rows of K bf16
    return M >= 1 && N >= 1 && K >= 8 && (K % 8) == 0 && static_cast<int64_t>(K) * 2 * 384 < (1ll << 31);
}

bool mfma_linear_f32_supported(int32_t M, int32_t N, int32_t K) {
    // whole 16-byte chunks of fp32; 32-bit byte offsets inside a tile: up to 384 rows of K fp32
    return M >= 1 && N >= 1 && K >= 4 && (K % 4) == 0 && static_cast<int64_t>(K) * 4 * 384 < (1ll << 31);
}

int32_t launch_linear_mfma(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K,
                           int32_t epi, bf16_t* out, float* resid, RowVec gate, hipStream_t s, int cu_share,
                           const LnFold* ln) {
    if (!mfma_linear_supported(M, N, K)) return FREE_ERR_SHAPE;
    if (ln != nullptr) {
        // producer: the rows being normalised are this GEMM's output rows (width N); consumer: its input rows (width K)
        const int32_t width = epi == FREE_EPI_GATE_RESID_PREP ? N : K;
        const auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
        if (width % kLnSlotCols != 0 || ln->slots != width / kLnSlotCols || ln->stats == nullptr ||
            (reinterpret_cast<uintptr_t>(ln->stats) & 7u))
            return FREE_ERR_SHAPE;
        if (epi == FREE_EPI_GATE_RESID_PREP) {
            if (ln->z == nullptr || ln->scale_next == nullptr || !al16(ln->z) || !al16(ln->scale_next)) return FREE_ERR_SHAPE;
        } else {
            if (ln->c1 == nullptr || ln->c0 == nullptr || !al16(ln->c1) || !al16(ln->c0) || (ln->fold_stride & 3) ||
                ln->rows_per_sample < 32 || ln->rows_per_sample % 32 != 0)
                return FREE_ERR_SHAPE;
        }
    }
    if ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(W)) & 15u) return FREE_ERR_SHAPE;
    if (ln != nullptr ? K % BK != 0 || epi > FREE_EPI_GATE_RESID_PREP : epi > FREE_EPI_GATE_RESID) return FREE_ERR_SHAPE;
    const Choice c = choose(M, N, K, 2, epi, linear_rows_covers(N, K, 2, bias, out, resid, gate), cu_share);
    switch (c.family) {
        case TILE_ROWS: return launch_linear_rows(X, W, bias, M, N, K, epi, out, resid, gate, s, static_cast<RowsTile>(c.tile));
        case TILE_PIPE: return launch_linear_pipe(X, W, bias, M, N, K, epi, out, resid, gate, s, static_cast<PipeTile>(c.tile), ln);
        default: return launch_staged(static_cast<StagedTile>(c.tile), X, W, bias, M, N, K, epi, out, resid, gate, s);
    }
}

// A part has at least twelve slices: below that a workgroup is all prologue and epilogue, and with one part less to wait for there
// is little to gain (K = 1536 to 384 columns 8.6 -> 7.6 us at 2250 rows, which the LayerNorm behind gives back).  And an even number:
// gemm_rows_kernel takes two per pass.  So K is a multiple of 384 from 2304 on: the second layer of four-fold MLPs at widths that are
// multiples of 96 from 576 on; at width 1024 (64 slices) K stays in one.
bool linear_split_covers(int32_t N, int32_t K) {
    return N % 8 == 0 && N <= 2048 && K % (kSplitParts * 2 * BK) == 0 && K >= kSplitParts * 12 * BK;
}

namespace {

const TileTime* best_split_tile(int32_t M, int32_t N, int32_t K, double* t_best) {
    const TileTime* best = nullptr;
    for (const TileTime& t : kTiles) {
        if (t.family != TILE_ROWS) continue;
        const double u = static_cast<double>((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * kSplitParts / device_cus();
        const double time = launch_time(t, FREE_EPI_PARTIAL, u, K / BK / kSplitParts, 1.0);
        if (best == nullptr || time < *t_best) {
            best = &t;
            *t_best = time;
        }
    }
    return best;
}

}  // namespace

// The next kernel reads the parts and updates the residual stream, out of the caches at 8.5 TB/s, and takes a microsecond longer; a
// launch of its own takes three more.  Second layer of the MLP at width 1152, one launch -> parts, and the LayerNorm behind it (us):
// 256 rows 17 -> 8.4, 4.2 -> 6.2; 512 rows 16.6 -> 11.8, 6.0 -> 8.2; 2048 rows 36 -> 36, 5.6 -> 10.8 (not taken).
// Where it does not pay one workgroup adds the same parts for the sake of equal bits alone, with a second set of accumulators.  Forward
// of a target, K in one -> in parts, us: width 1152 1536 rows 3015 -> 3018, 2048 3591 -> 3622, 3072 4459 -> 4431, 3840 5063 -> 5070;
// width 768 1536 905 -> 916, 2048 1007 -> 1018, 3072 1227 -> 1229 (256 rows 590 -> 536, 512 645 -> 621, 1024 729 -> 716).
bool linear_split_pays(int32_t M, int32_t N, int32_t K, bool own_launch) {
    if (M > kMaxPartRows) return false;
    double t_split = 0.0, t_one = 0.0;
    best_split_tile(M, N, K, &t_split);
    choose(M, N, K, 2, FREE_EPI_GATE_RESID_SEG, true, 1, &t_one);
    const double t_join = (own_launch ? 4.0 : 1.0) + 16.0 * M * N / 8.5e6;
    return t_split + t_join < t_one;
}

bool linear_split_from_zero(int32_t M, int32_t N, int32_t K, bool own_launch) {
    return linear_split_pays(M, N, K, own_launch) || choose(M, N, K, 2, FREE_EPI_GATE_RESID_SEG, true, 1).family == TILE_ROWS;
}

int32_t launch_linear_split(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K, float* resid,
                            RowVec gate, float* part, bool own_launch, ResidJoin* join, hipStream_t s, bool from_zero) {
    if (!mfma_linear_supported(M, N, K) || !linear_split_covers(N, K) || !linear_rows_covers(N, K, 2, bias, part, resid, gate))
        return FREE_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(W)) & 15u) return FREE_ERR_SHAPE;
    if (linear_split_pays(M, N, K, own_launch)) {
        double t;
        const TileTime* tile = best_split_tile(M, N, K, &t);
        *join = ResidJoin{part, bias, gate, from_zero};
        return launch_linear_rows(X, W, nullptr, M, N, K, FREE_EPI_PARTIAL, nullptr, part, RowVec{nullptr, 0, 1}, s,
                                  static_cast<RowsTile>(tile->tile));
    }
    const Choice c = choose(M, N, K, 2, FREE_EPI_GATE_RESID_SEG, true, 1);
    if (c.family == TILE_ROWS)
        return launch_linear_rows(X, W, bias, M, N, K, FREE_EPI_GATE_RESID_SEG, nullptr, resid, gate, s, static_cast<RowsTile>(c.tile),
                                  from_zero);
    if (from_zero) return FREE_ERR_SHAPE;
    return launch_linear_pipe(X, W, bias, M, N, K, FREE_EPI_GATE_RESID_SEG, nullptr, resid, gate, s, static_cast<PipeTile>(c.tile),
                              nullptr);
}

bool mfma_ln_fold_supported(int32_t M, int32_t D, int32_t rows_per_sample) {
    // (a 32-row block of a tile then lies in one sample; up to 16 slots of partial sums per row)
    return M >= 1 && D % kLnSlotCols == 0 && D <= 16 * kLnSlotCols && rows_per_sample >= 32 && rows_per_sample % 32 == 0;
}

int32_t launch_linear_mfma_f32(const float* X, const float* W, const float* bias, int32_t M, int32_t N, int32_t K,
                               int32_t epi, float* out, float* resid, RowVec gate, hipStream_t s, int cu_share) {
    if (!mfma_linear_f32_supported(M, N, K)) return FREE_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(W)) & 15u) return FREE_ERR_SHAPE;
    if (epi > FREE_EPI_GATE_RESID) return FREE_ERR_RANGE;
    const Choice c = choose(M, N, K, 4, epi, linear_rows_covers(N, K, 4, bias, out, resid, gate), cu_share);
    if (c.family == TILE_ROWS)
        return launch_linear_rows(X, W, bias, M, N, K, epi, out, resid, gate, s, static_cast<RowsTile>(c.tile));
    return launch_staged(static_cast<StagedTile>(c.tile), X, W, bias, M, N, K, epi, out, resid, gate, s);
}

int32_t mfma_linear_tile(int32_t M, int32_t N, int32_t K, int32_t dtype, int32_t epi) {
    const int es = dtype == FREE_BF16 ? 2 : 4;
    if (!(es == 2 ? mfma_linear_supported(M, N, K) : mfma_linear_f32_supported(M, N, K))) return FREE_ERR_SHAPE;
    if (epi > FREE_EPI_GATE_RESID && (es == 4 || K % BK != 0 || epi > FREE_EPI_GATE_RESID_PREP)) return FREE_ERR_SHAPE;
    const Choice c = choose(M, N, K, es, epi, linear_rows_covers(N, K, es, nullptr, nullptr, nullptr, RowVec{nullptr, 0, 1}), 1);
    return c.family * 1000000 + c.bm * 1000 + c.bn;
}

}  // namespace freemi
