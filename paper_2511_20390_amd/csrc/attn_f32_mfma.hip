// Flash-style softmax attention in full fp32 on the matrix cores, for the FREE_FP32 mode of the
// packed target forward (Alg. 1): per (sample, head), out = softmax(q k^T / sqrt(dh)) v,
// non-causal, fp32 operands, products and online softmax (v_mfma_f32_32x32x2_f32).
//
// Same formulation as the bf16 kernel of attn_mfma.hip: the score tile is computed TRANSPOSED,
// S^T = K Q^T (rows = keys, columns = queries), so that in the accumulator layout a lane owns one
// query column (lane % 32) and half of the key rows: the softmax statistics are lane-local (one
// exchange with lane ^ 32), and the probabilities are already the B operand of the second
// product O^T = V^T P^T - register e of the score tile holds key 8 (e / 4) + 4 (lane / 32) + e % 4,
// and one 32x32x2 product contracts over exactly the two keys that the two half-waves hold in
// register e.  The matching A operand is one float per lane, V[key][d = lane % 32 (+ 32 per row
// tile of O^T)], read from a row-major V tile in LDS (32 consecutive floats per half-wave).
// The contraction over the head dim uses 16-byte fragments like the fp32 GEMM: lane group g reads
// chunk 2 j + g of its K row (and holds the same chunks of its Q row in registers); element e of
// the chunk pair (2 j, 2 j + 1) is one 32x32x2 product.
// One workgroup = 32 queries of one head; its four wavefronts take the key tiles (32 keys) t = wave, wave + 4, ... with an LDS tile
// and an online softmax of their own - no barrier in the loop - and their maxima, sums and O^T are put together at the end in
// wavefront order, whatever the batch.  (Head dim 128 has no LDS for that with two workgroups per CU: four query blocks that share the
// tiles.)  What bounds it: a key tile is 36 + 32 products of 64 cycles at head dim 72, so that a wavefront with all 256 keys of a state
// is a chain of 15 us, and such a state has 8 x heads query blocks, on 1024 SIMDs; with many samples the matrix pipe, which wants three
// wavefronts per SIMD: the queries are in LDS, which the four wavefronts share, K and V take turns in one LDS tile (a wavefront's own, so
// that no barrier is needed), and no register is spilled.  us per launch, all keys in each wavefront, the third 32-row tile of O^T at head
// dim 72 in products too / keys over four wavefronts with two of them per SIMD / here:
//   16 heads of 72   2 x 256 tokens 30.5 / 11.4 / 11.5   16 x 256 61 / 62 / 58   64 x 256 211 / 229 / 200   2 x 450 54 / 29 / 29   12 x 1024 580 / 524 / 495
//   12 heads of 64   2 x 256 23.5 / 8.8 / 8.6   16 x 256 44 / 41 / 38   32 x 256 65 / 75 / 69   64 x 256 114 / 139 / 124   12 x 1024 350 / 326 / 309
//   16 heads of 64   8 x 256 30 / 32 / 33.5 (1024 workgroups on 256, 512, 768 places)
//   8 heads of 128 (two per SIMD, tiles shared)   2 x 256 41.5 / 39.7 / 39.6   64 x 256 178 / 144 / 144
//   16 heads of 72, one to 16 tokens of one to nine samples 6.0 / 6.4 / 6.7: the last barriers of a workgroup
// A wavefront has two of the eight tiles at 256 tokens, and what it does once - queries, first tile, the sums of the four put together - is then
// 4 to 8 % more than all keys in one, at 32 samples of head dim 64 and more, 12 % there; by the batch the choice cannot go, or a state would
// have other bits in a pack.  2-norm error against 64 bits 4.1e-7 -> 3.4e-7 (256 tokens), 6.6e-7 -> 4.2e-7 (1024).
#include <algorithm>
#include <cmath>

#include "free_internal.h"
#include "lanes.h"

namespace freemi {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kWaves = 4, kThreads = kWaves * 64;
constexpr int BQ = 32;                    // queries per workgroup
constexpr int BKV = 32;                   // keys per tile

// KS: wavefronts that share the keys of a query block, 4 (an LDS tile each) or 1 (four query blocks, one tile and a barrier).
template <int DH, int KS>
struct Tile {
    static constexpr int NC = DH / 4;            // 16-byte chunks per row
    static constexpr int NP = DH / 8;            // chunk pairs: groups of four 32x32x2 products
    static constexpr int kRest = DH > 32 && DH % 32 <= 8 ? DH % 32 : 0;   // last columns of O, on the vector ALU
    static constexpr int DT = (DH - kRest + 31) / 32;         // 32-row tiles of O^T
    static constexpr int KP = DH + 4;            // K row pitch in floats: an odd number of chunks (conflict-free b128 reads)
    static constexpr int VP = (DH % 16 == 8) ? DH : DH + 8;   // V row pitch = 8 mod 16: rows 4 apart land on the other 32 banks
    // floats per wavefront: K and V take turns in one tile with KS > 1; the pad rows of O^T read past a row's end
    static constexpr int kV = KS > 1 ? 0 : BKV * KP, kKeys = KS > 1 ? std::max(BKV * KP, BKV * VP + 32 * DT) : BKV * (KP + VP) + 32 * DT;
    static constexpr int kSums = KS > 1 ? 32 * DH : 0;        // floats of O^T
    static constexpr int kWaveFloats = kKeys > kSums ? kKeys : kSums;
    static constexpr int kQ = KS * (kWaveFloats + (KS > 1 ? 2 * BQ : 0));       // where Q is, with KS > 1
    static constexpr size_t kLds = sizeof(float) * (kQ + (KS > 1 ? BQ * KP : 0));
};

template <int DH, int KS>
__global__ __launch_bounds__(kThreads, KS > 1 ? 3 : 2) void attn_f32_mfma_kernel(const float* __restrict__ qkv, int32_t N,
                                                                 int32_t heads, float scale_log2,
                                                                 float* __restrict__ out) {
    static_assert(DH % 8 == 0 && DH <= 128, "whole chunk pairs");
    static_assert(KS == 1 || KS == kWaves, "whole workgroups");
    using L = Tile<DH, KS>;
    constexpr int NC = L::NC, NP = L::NP, DT = L::DT, KP = L::KP, VP = L::VP, kRest = L::kRest;
    constexpr int kGroup = kThreads / KS;            // threads that fill a tile
    constexpr int NLD = BKV * NC / kGroup;           // chunks per thread of a K (and a V) tile
    constexpr int kPieces = NC / 8, kRows = kGroup / 8, kWhole = BKV / kRows * kPieces;    // 128-byte pieces of a row; passes of them
    constexpr bool kEarlyK = KS == 1 || DH <= 64;    // (with head dim 72 three wavefronts per SIMD have no registers for K and V)
    constexpr int kTail = NC % 8 ? NC % 8 : 8;       // chunks behind the last piece
    static_assert(BKV * NC % kGroup == 0 && kGroup % kTail == 0 && kRest % 4 == 0, "whole passes");
    extern __shared__ __attribute__((aligned(16))) float lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    constexpr int kQueries = BQ * kWaves / KS;
    const int nq = (N + kQueries - 1) / kQueries, group = KS > 1 ? wave : 0, in_group = KS > 1 ? lane : tid;
    // all query tiles of one (sample, head) on one XCD, back to back (attn_mfma.hip)
    const int id = blockIdx.x;
    const bool by_xcd = gridDim.x / nq % 8 == 0;
    const int pair_idx = by_xcd ? (id & 7) + 8 * (id / (8 * nq)) : id / nq, q_tile = by_xcd ? (id >> 3) % nq : id % nq;
    const int h = pair_idx % heads, b = pair_idx / heads;
    const int D = heads * DH;
    const int64_t row0 = static_cast<int64_t>(b) * N;
    const int64_t row_stride = static_cast<int64_t>(3) * D;       // floats
    const int q_base = q_tile * kQueries + (KS > 1 ? 0 : wave * BQ);
    float* const sK = lds + group * L::kWaveFloats;
    float* const sV = sK + L::kV;

    // staging of a K or V tile: whole 128-byte pieces of kRows rows per pass, then what is left of the rows.  Rows past N read as zero, also
    // in a pass that has no other (a load whose scalar offset alone is past the descriptor's end returns zero on gfx950, measured): their
    // scores are masked, and their probabilities are zero
    const int row_bytes = 12 * D;
    const int piece = (in_group >> 3) * row_bytes + (in_group & 7) * 16, tail = (in_group / kTail) * row_bytes + (kPieces * 8 + in_group % kTail) * 16;
    auto fetch = [&](f32x4_t (&reg)[NLD], int t, int which) {         // 1: K, 2: V
        const int left = N - t * BKV;
        const float* base = qkv + (row0 + t * BKV) * row_stride + which * D + h * DH;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0,
            (std::min(left, BKV) - 1) * row_bytes + DH * 4, 0x00020000);
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const bool whole = i < kWhole;
            const int soff = whole ? i / std::max(kPieces, 1) * kRows * row_bytes + i % std::max(kPieces, 1) * 128 : (i - kWhole) * (kGroup / kTail) * row_bytes;
            reg[i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, whole ? piece : tail, soff, 0));
        }
    };
    // K of the wavefront's first tile and the queries: lane holds query column l32, chunks 2 j + g, with one query block (KS > 1) in LDS for
    // all four wavefronts
    const int ntiles = (N + BKV - 1) / BKV;
    f32x4_t kreg[NLD], vreg[NLD], qf[KS > 1 ? 1 : NP];
    const float* const qrow = lds + L::kQ + l32 * KP + 4 * g;
    if constexpr (KS > 1) {
        constexpr int kChunks = BQ * NC, kLoads = (kChunks + kThreads - 1) / kThreads;
        f32x4_t own[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int idx = std::min(tid + i * kThreads, kChunks - 1), r = idx / NC;
            own[i] = *reinterpret_cast<const f32x4_t*>(qkv + (row0 + std::min(q_base + r, N - 1)) * row_stride + h * DH + 4 * (idx - r * NC));
        }
        if (group < ntiles) fetch(kreg, group, 1);
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int idx = tid + i * kThreads, r = idx / NC;
            if (idx < kChunks) *reinterpret_cast<f32x4_t*>(lds + L::kQ + r * KP + 4 * (idx - r * NC)) = own[i];
        }
        __syncthreads();
    } else {
        fetch(kreg, group, 1);
        const float* src = qkv + (row0 + std::min(q_base + l32, N - 1)) * row_stride + h * DH;
#pragma unroll
        for (int j = 0; j < NP; ++j) qf[j] = *reinterpret_cast<const f32x4_t*>(src + 4 * (2 * j + g));
    }

    // With KS > 1 a wavefront's LDS operations keep their order, and the fences keep the compiler's.  With KS == 1 the barrier behind
    // the K tile says that every wavefront is done with the V tile before, the one behind the V tile the same of the K tile.
    auto stash = [&](const f32x4_t (&reg)[NLD], float* dst, int pitch) {
        if constexpr (KS > 1) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            float* at = i < kWhole ? dst + ((in_group >> 3) + i / std::max(kPieces, 1) * kRows) * pitch + (in_group & 7) * 4 + i % std::max(kPieces, 1) * 32
                                   : dst + (in_group / kTail + (i - kWhole) * (kGroup / kTail)) * pitch + (kPieces * 8 + in_group % kTail) * 4;
            *reinterpret_cast<f32x4_t*>(at) = reg[i];
        }
        if constexpr (KS > 1) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        else __syncthreads();
    };

    f32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    // columns DH - kRest .. DH - 1 of this lane's query over its keys (g): a third product of 32 rows per key pair, of which head dim
    // 72 uses 8, would be a fifth of the matrix pipe's time; the vector ALU does them beside it
    [[maybe_unused]] float rest[kRest > 0 ? kRest : 1] = {};
    float m_run = -INFINITY, l_run = 0.f;

    // K of a tile is on its way while the tile before is multiplied with V, V while the scores are computed
    for (int t = group; t < ntiles; t += KS) {
        fetch(vreg, t, 2);
        stash(kreg, sK, KP);

        // ---- S^T = K Q^T for the 32 keys of the tile
        f32x16_t st;
#pragma unroll
        for (int e = 0; e < 16; ++e) st[e] = 0.f;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const f32x4_t kf = *reinterpret_cast<const f32x4_t*>(sK + l32 * KP + 4 * (2 * j + g));
            const f32x4_t qv4 = KS > 1 ? *reinterpret_cast<const f32x4_t*>(qrow + 8 * j) : qf[KS > 1 ? 0 : j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float kv = kf[e], qv = qv4[e];
                st = __builtin_amdgcn_mfma_f32_32x32x2f32(kv, qv, st, 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (kEarlyK && t + KS < ntiles) fetch(kreg, t + KS, 1);
        if ((t + 1) * BKV > N) {              // ragged last tile: keys past N
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (t * BKV + 8 * (e >> 2) + 4 * g + (e & 3) >= N) st[e] = -INFINITY;
        }

        // ---- online softmax of the query column
        float mx = st[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, st[e]);
        mx = max_lane_xor32(mx);
        const float m_new = fmaxf(m_run, mx);
        // (scores of -inf only, so far: they weigh nothing, and the keys of the other wavefronts may be finite)
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_ref) * scale_log2);
        const float mb = m_ref * scale_log2;
        float p[16], sum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            p[e] = __builtin_amdgcn_exp2f(fmaf(st[e], scale_log2, -mb));
            sum += p[e];
        }
        l_run = fmaf(l_run, alpha, sum);
        m_run = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
        if constexpr (kRest > 0)
#pragma unroll
            for (int d = 0; d < kRest; ++d) rest[d] *= alpha;

        __builtin_amdgcn_sched_barrier(0);
        stash(vreg, sV, VP);
        if (!kEarlyK && t + KS < ntiles) fetch(kreg, t + KS, 1);
        // ---- O^T += V^T P^T: register e pairs the keys 8 (e / 4) + e % 4 (+ 4 for the upper half-wave)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float* vrow = sV + (8 * (e >> 2) + 4 * g + (e & 3)) * VP;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const float vv = vrow[l32 + 32 * dt];
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv, p[e], o[dt], 0, 0, 0);
            }
            if constexpr (kRest > 0)
#pragma unroll
                for (int c = 0; c < kRest / 4; ++c) {
                    const f32x4_t vv = *reinterpret_cast<const f32x4_t*>(vrow + 32 * DT + 4 * c);
#pragma unroll
                    for (int i = 0; i < 4; ++i) rest[4 * c + i] = fmaf(vv[i], p[e], rest[4 * c + i]);
                }
        }
    }

    l_run = add_lane_xor<32>(l_run);
    if constexpr (kRest > 0)
#pragma unroll
        for (int d = 0; d < kRest; ++d) rest[d] = add_lane_xor<32>(rest[d]);
    // ---- register e of O^T tile dt is row d = 32 dt + 8 (e / 4) + 4 g + e % 4, column l32: groups of eight columns of a query, four in
    // either half-wave
    auto columns = [&](int c) -> f32x4_t {
        const int dt = c >> 2, e4 = c & 3;
        if constexpr (kRest > 0) {
            if (c * 8 >= 32 * DT)
                return g == 0 ? f32x4_t{rest[0], rest[1], rest[2], rest[3]} : f32x4_t{rest[4 % kRest], rest[5 % kRest], rest[6 % kRest], rest[7 % kRest]};
        }
        return f32x4_t{o[dt][4 * e4], o[dt][4 * e4 + 1], o[dt][4 * e4 + 2], o[dt][4 * e4 + 3]};
    };
    const int q = q_base + l32;
    float* dst = out + (row0 + q) * D + h * DH + 4 * g;
    if constexpr (KS == 1) {
        if (q >= N) return;
        const float inv = 1.0f / l_run;
#pragma unroll
        for (int c = 0; c < DH / 8; ++c) *reinterpret_cast<f32x4_t*>(dst + 8 * c) = columns(c) * inv;
        return;
    }
    // ---- the four parts: every wavefront scales its sums to the common maximum (one without keys has weight zero) and leaves them
    // in its LDS tile
    float* const maxima = lds + KS * L::kWaveFloats;
    float* const sums = maxima + KS * BQ;
    if (g == 0) {
        maxima[wave * BQ + l32] = m_run;
        sums[wave * BQ + l32] = l_run;
    }
    __syncthreads();
    float m_all = maxima[l32];
#pragma unroll
    for (int w = 1; w < KS; ++w) m_all = fmaxf(m_all, maxima[w * BQ + l32]);
    auto weight = [&](float m) { return __builtin_amdgcn_exp2f((m - m_all) * scale_log2); };
    const float own = weight(m_run);
#pragma unroll
    for (int c = 0; c < DH / 8; ++c) *reinterpret_cast<f32x4_t*>(sK + c * 256 + lane * 4) = columns(c) * own;
    float l_tot = 0.f;
#pragma unroll
    for (int w = 0; w < KS; ++w) l_tot = fmaf(sums[w * BQ + l32], weight(maxima[w * BQ + l32]), l_tot);
    __syncthreads();
    if (q >= N) return;
    const float inv = 1.0f / l_tot;
    for (int c = wave; c < DH / 8; c += KS) {
        f32x4_t v = *reinterpret_cast<const f32x4_t*>(lds + c * 256 + lane * 4);
#pragma unroll
        for (int w = 1; w < KS; ++w) v += *reinterpret_cast<const f32x4_t*>(lds + w * L::kWaveFloats + c * 256 + lane * 4);
        *reinterpret_cast<f32x4_t*>(dst + 8 * c) = v * inv;
    }
}

template <int DH, int KS>
int32_t launch_dh(const float* qkv, int32_t B, int32_t N, int32_t heads, float* out, hipStream_t s) {
    constexpr int kQueries = BQ * kWaves / KS;
    const float scale_log2 = 1.4426950408889634f / std::sqrt(static_cast<float>(DH));
    const int64_t total = static_cast<int64_t>((N + kQueries - 1) / kQueries) * heads * B;
    if (total > 0x7fffffff) return FREE_ERR_SHAPE;
    auto kern = attn_f32_mfma_kernel<DH, KS>;
    static LdsLimit limit;
    if (!limit.allow(reinterpret_cast<const void*>(kern), Tile<DH, KS>::kLds)) return FREE_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(total)), dim3(kThreads), (Tile<DH, KS>::kLds), s, qkv, N, heads, scale_log2, out);
    return launch_ok() ? FREE_OK : FREE_ERR_HIP;
}

}  // namespace

bool mfma_attention_f32_supported(int32_t N, int32_t dh) {
    return N >= 1 && (dh == 16 || dh == 64 || dh == 72 || dh == 128);
}

int32_t launch_attention_mfma_f32(const float* qkv, int32_t B, int32_t N, int32_t heads, int32_t dh, float* out,
                                  hipStream_t s) {
    if ((reinterpret_cast<uintptr_t>(qkv) | reinterpret_cast<uintptr_t>(out)) & 15u) return FREE_ERR_SHAPE;
    switch (dh) {
        case 16: return launch_dh<16, 4>(qkv, B, N, heads, out, s);
        case 64: return launch_dh<64, 4>(qkv, B, N, heads, out, s);
        case 72: return launch_dh<72, 4>(qkv, B, N, heads, out, s);
        case 128: return launch_dh<128, 1>(qkv, B, N, heads, out, s);
        default: return FREE_ERR_SHAPE;
    }
}

}  // namespace freemi
