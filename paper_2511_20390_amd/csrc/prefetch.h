// Device side of Prefetch: what the extra workgroups of a launch do.
#pragma once

#include "free_internal.h"

namespace freemi {

// Workgroups first .. gridDim.x - 1 of a launch (first and their number multiples of 8) read one word of every
// 128-byte line of the matrices.  Workgroup ids are dealt round-robin to the 8 XCDs, and the few-row GEMMs give each XCD a
// contiguous eighth of the weight rows (where K is summed in parts: of the rows of part 0, then of part 1, ...), so XCD x reads eighth x.
// What it buys: a CU takes in 46 KB/us from HBM, 85 from the Infinity Cache, 120 from its L2, and the few-row GEMMs are bound
// by that.  The LayerNorm in front of QKV (latency-bound, 5 us) loads the QKV and out-projection weights of its block, the
// attention kernel (idle CUs at few rows) those of the MLP.  512 rows at width 1152, us per launch without -> with: QKV 10.7
// -> 8.5, out-projection 8.9 -> 7.0, MLP-1 15.0 -> 11.6, MLP-2 23.5 -> 17.0 against LayerNorm 5.1 -> 6.0 and attention
// 8.9 -> 11.6; forward 2.30 -> 1.99 ms.  1024 rows: round 2.99 -> 2.69 ms.
// From some 1500 rows on QKV and MLP-1 run on tiles whose order gives every XCD all of the weights: what the read-ahead brings
// then is in the Infinity Cache rather than in the right L2, and buys 6 to 9 % of the forward instead of 11 to 14 (2560 to 3840
// against 256 to 1024 rows).  LayerNorm and attention each contribute: 4 and 8 % of those 11 to 14.
// A thread has two lines over both matrices (Prefetch::blocks), at most two of one and mostly no second round; its loads are in
// flight together, and the share of a workgroup takes a 32-bit division per matrix (a wait behind every load and four 64-bit
// divisions before: at 512 rows LayerNorm 6.15 -> 6.03, attention 12.0 -> 11.9 us).  Where a matrix is taken in parts of K, each of its
// lines takes two more, in front of its load.
__device__ inline void prefetch_lines(const Prefetch& pf, int first) {
    const uint32_t xcd = blockIdx.x & 7, rank = (blockIdx.x - first) >> 3, n = (gridDim.x - first) >> 3;
    const char* base[2];
    uint32_t at[2], end[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const uint32_t eighth = static_cast<uint32_t>((pf.bytes[m] >> 7) + 7) >> 3, per = (eighth + n - 1) / n;
        const uint32_t lo = rank * per < eighth ? rank * per : eighth, hi = lo + per < eighth ? lo + per : eighth;
        const uint32_t lines = static_cast<uint32_t>(pf.bytes[m] >> 7);
        base[m] = static_cast<const char*>(pf.p[m]);
        at[m] = xcd * eighth + lo + threadIdx.x;
        end[m] = xcd * eighth + hi < lines ? xcd * eighth + hi : lines;
    }
    // line i of a matrix; where its GEMM takes it in parts of K: the lines of part 0 of all rows, then those of part 1, ...
    auto where = [&](int m, uint32_t i) -> int64_t {
        if (m == 0 || pf.part_lines == 0) return static_cast<int64_t>(i) << 7;
        const uint32_t per = pf.part_lines, lines = static_cast<uint32_t>(pf.bytes[1] >> 7) / kSplitParts;
        const uint32_t part = i / lines, in_part = i - part * lines, row = in_part / per;
        return static_cast<int64_t>((row * kSplitParts + part) * per + (in_part - row * per)) << 7;
    };
    uint32_t acc = 0;
    while (at[0] < end[0] || at[1] < end[1]) {
        uint32_t v[2][2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int k = 0; k < 2; ++k, at[m] += blockDim.x)
                v[m][k] = at[m] < end[m] ? *reinterpret_cast<const uint32_t*>(base[m] + where(m, at[m])) : 0u;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int k = 0; k < 2; ++k) acc ^= v[m][k];
    }
    asm volatile("" ::"v"(acc));                             // the loads are for the caches: keep them, drop the value
}

}  // namespace freemi
