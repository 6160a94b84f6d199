// Internal declarations shared by the translation units of libfree_mi355x.
// Host-side launch wrappers only; every kernel lives in exactly one .hip file.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "../../include/free_mi355x.h"

namespace freemi {

// ---- bf16 storage type: raw bits, round-to-nearest-even conversion ----------
struct bf16_t {
    uint16_t v;
};

__host__ __device__ inline float bf16_to_float(bf16_t h) {
    union { uint32_t u; float f; } c;
    c.u = static_cast<uint32_t>(h.v) << 16;
    return c.f;
}

__host__ __device__ inline bf16_t float_to_bf16(float f) {
    union { uint32_t u; float f; } c;
    c.f = f;
    uint32_t u = c.u;
    bf16_t r;
    if ((u & 0x7fffffffu) > 0x7f800000u) {          // NaN stays NaN
        r.v = static_cast<uint16_t>((u >> 16) | 0x40u);
        return r;
    }
    u += 0x7fffu + ((u >> 16) & 1u);
    r.v = static_cast<uint16_t>(u >> 16);
    return r;
}

#if defined(__HIPCC__)
// two floats -> packed bf16 pair (low half = first), hardware round-to-nearest-even
__device__ inline uint32_t pack_bf16_pair(float lo, float hi) {
    typedef float f2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    const f2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t));
}
#endif

__device__ inline float load_f(const float* p) { return *p; }
__device__ inline float load_f(const bf16_t* p) { return bf16_to_float(*p); }
__device__ inline void store_f(float* p, float v) { *p = v; }
__device__ inline void store_f(bf16_t* p, float v) { *p = float_to_bf16(v); }

__host__ __device__ inline float gelu_tanh_f(float v) {
    const float k = 0.7978845608028654f;            // sqrt(2/pi)
    float inner = k * (v + 0.044715f * v * v * v);
    return 0.5f * v * (1.0f + tanhf(inner));
}

__host__ __device__ inline float silu_f(float v) { return v / (1.0f + expf(-v)); }

constexpr float kLnEps = 1e-6f;

// Per-sample modulation / gate vector of an epilogue or a LayerNorm:
// value for (row m, column n) = base[(m / rows_per_sample) * stride + n].
struct RowVec {
    const float* base;
    int32_t stride;
    int32_t rows_per_sample;
};

// LayerNorm + modulate folded into the GEMMs on both sides of it (bf16 matrix-core path only).
// With z = x (1 + scale) rounded to bf16, row mean mu and r = 1 / sqrt(var + eps):
//   (LN(x) (1 + scale) + shift) W^T + b = r (z W^T) - r mu c1 + c0,
//   c1[n] = sum_k (1 + scale[k]) W[n, k],  c0[n] = sum_k shift[k] W[n, k] + b[n]   (per sample).
// The GEMM that updates the residual stream (producer, FREE_EPI_GATE_RESID_PREP) also writes z for the
// next LayerNorm and, per row and per 128-column slot, the sums of x and x^2; the GEMM that consumes the
// normalised rows (FREE_EPI_LN_BIAS / FREE_EPI_LN_BIAS_GELU) multiplies z and applies r, mu, c1, c0 in
// its epilogue.  No separate pass over the residual stream, no atomics: every partial sum has one writer
// and the consumer adds the slots of a row in a fixed order.
constexpr int FREE_EPI_LN_BIAS = 3, FREE_EPI_LN_BIAS_GELU = 4, FREE_EPI_GATE_RESID_PREP = 5;
// sums over one part of K, no bias, fp32 to resid[part][M][N] (gemm_rows.hip); see ResidJoin
constexpr int FREE_EPI_PARTIAL = 6;
// the residual update of FREE_EPI_GATE_RESID with the sums over those parts of K added in the same order in one workgroup; tiles
// of up to kSegTileArea elements (a second set of accumulators)
constexpr int FREE_EPI_GATE_RESID_SEG = 7;
constexpr int kSegTileArea = 192 * 128;
constexpr int kLnSlotCols = 128;           // columns of the residual stream per partial-sum slot
struct LnFold {
    // producer: scale vector of the NEXT LayerNorm (indexed like the gate: same stride and rows per sample),
    // z [M, N] bf16 and stats [M, slots, 2] fp32 are outputs.  consumer: stats is an input.
    const float* scale_next = nullptr;
    void* z = nullptr;
    float* stats = nullptr;
    int32_t slots = 0;                     // width of the normalised rows / kLnSlotCols
    // consumer: c1 / c0 of sample s start at c1[s * fold_stride] (N entries each, 16-byte aligned)
    const float* c1 = nullptr;
    const float* c0 = nullptr;
    int64_t fold_stride = 0;
    int32_t rows_per_sample = 1;
    float inv_width = 0.f;                 // 1 / width of the normalised rows
};

// Few rows, bf16: a linear layer of long K and few columns sums K in kSplitParts parts, always in this order, so that it can be
// one workgroup per tile (FREE_EPI_GATE_RESID_SEG) or one per tile and part (FREE_EPI_PARTIAL).  In the second case the residual
// update is left to the next kernel:
//   x = gate (((part 0 + part 1) + part 2) + bias) + x        (x taken as zero with from_zero).
constexpr int kSplitParts = 3;
constexpr int32_t kMaxPartRows = 4095;     // rows of a layer whose parts may be left to the next kernel: what workspaces have room for
struct ResidJoin {
    const float* part = nullptr;           // [kSplitParts, M, D]; nullptr: nothing to add
    const float* bias = nullptr;
    RowVec gate{nullptr, 0, 1};
    int32_t from_zero = 0;
};

// Weight matrices that the launches after the next one read: the launch of a short kernel carries extra workgroups that
// load them, so that the GEMMs find them in the L2 of their XCD or in the Infinity Cache (prefetch.h).
struct Prefetch {
    const void* p[2] = {nullptr, nullptr};
    int64_t bytes[2] = {0, 0};
    int32_t part_lines = 0;                                  // p[1] is used in kSplitParts parts of its rows: 128-byte lines of each; 0: whole
    int blocks(int threads = 256) const {                    // workgroups of that many threads, a multiple of 8
        const int64_t per_block = static_cast<int64_t>(threads) << 8;
        return static_cast<int>(((bytes[0] + bytes[1] + per_block - 1) / per_block + 7) / 8 * 8);
    }
};

// Thread-local HIP error memo (free_last_hip_error).
void note_hip_error(hipError_t e);
inline bool hip_ok(hipError_t e) {
    if (e != hipSuccess) { note_hip_error(e); return false; }
    return true;
}
inline bool launch_ok() { return hip_ok(hipGetLastError()); }

// More than 64 KB of dynamic LDS has to be allowed per kernel and device.  One object per kernel, asked in front of every launch, from
// any thread.
class LdsLimit {
public:
    bool allow(const void* kernel, size_t bytes) {
        int dev = 0;
        if (!hip_ok(hipGetDevice(&dev))) return false;
        const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;
        if (allowed.load(std::memory_order_relaxed) & bit) return true;
        if (!hip_ok(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)))) return false;
        allowed.fetch_or(bit, std::memory_order_relaxed);
        return true;
    }

private:
    std::atomic<uint64_t> allowed{0};
};

// ---- optional per-kernel timing (free_profile_begin / free_profile_end) --------
// A Profiler belongs to a model handle.  While it is on, a ProfScope records a HIP event on the
// launch stream before and after the launches it brackets; with a null or idle profiler it does nothing.
enum ProfCat {
    PROF_COND = 0, PROF_ADALN, PROF_PATCH, PROF_LN_MOD, PROF_GEMM_QKV, PROF_ATTN, PROF_GEMM_PROJ,
    PROF_GEMM_FC1, PROF_GEMM_FC2, PROF_FINAL, PROF_EPS2MEAN, PROF_VERIFY,
    PROF_NCAT
};
static_assert(PROF_NCAT == FREE_PROF_NCAT, "category count is part of the ABI");
struct Profiler;
struct ProfScope {
    ProfScope(Profiler* p, int cat, hipStream_t s);
    ~ProfScope();
    Profiler* prof;
    int slot;
    hipStream_t stream;
};

// ---- verification (verify.hip) -------------------------------------------------
struct VerifyArgs {
    const float* m_target;   // [n_traj, K, d]
    const float* m_draft;    // [n_traj, K, d]
    const float* x_draft;    // [n_traj, K, d]; or, when x_last != nullptr, the K packed
                             // states of ONE trajectory: draft k is x_draft + (k+1) d
    const float* x_last;     // nullptr, or the K-th draft of the single trajectory
    const float* sigma; const float* u; const float* lambda;   // sigma [n_traj, K]; nullptr with sigma_elem
    int32_t n_traj, K; int64_t d;
    float* log_ratio; uint8_t* accept; int32_t* n_accept; float* x_out;
    Profiler* prof;          // nullptr, or the profiler of the handle the call belongs to
    const float* sigma_elem = nullptr;   // nullptr, or one standard deviation per element [n_traj, K, d]
};
size_t verify_workspace_bytes(int32_t n_traj, int32_t K, int64_t d);
// device address, on the current device, of the library's static scratch array (FREE_STATIC_SCRATCH_BYTES);
// looked up once per device with hipGetSymbolAddress, no allocation
int32_t static_verify_scratch(void** ptr);
// ev4 (nullable): four events, attached as start / stop to the dispatches of the two launches (benchmark timing)
int32_t launch_verify(const VerifyArgs& a, void* ws, size_t ws_bytes, hipStream_t s, hipEvent_t* ev4 = nullptr);

// ---- simple DiT kernels, both dtypes (dit_kernels.hip) ---------------------------
// Timestep and label of every sample of a batch: t[b] and y[b], or, with steps > 0, those of a guided pack [conditional x steps | null
// x steps]: t[b % steps], and label or null_label.
struct CondIn {
    const int32_t *t, *y;
    int32_t steps = 0, label = 0, null_label = 0;
    __host__ __device__ int32_t timestep(int b) const { return t[steps > 0 ? b % steps : b]; }
    __host__ __device__ int32_t label_of(int b) const { return steps == 0 ? y[b] : b < steps ? label : null_label; }
};
int32_t launch_conditioning(const CondIn& in, int32_t B, int32_t D, int32_t tfreq,
                            const float* w1, const float* b1, const float* w2, const float* b2,
                            const float* ytab, float* h1, float* sc, hipStream_t s);
// mod[b, r] = sum_i sc[b, i] W_r[i] + bias_r; rows r come from n_mats matrices of
// rows_per_mat rows each (device pointer tables), plus they are laid out back to
// back in mod with the given offsets.
int32_t launch_adaln(const float* sc, int32_t B, int32_t D, const void* const* w_tab,
                     const float* const* b_tab, const int32_t* row_start, int32_t n_mats,
                     int32_t total_rows, int32_t dtype, float* mod, hipStream_t s);
int32_t launch_patch_embed(const float* x, int32_t x_mod, int32_t B, int32_t C, int32_t H, int32_t W,
                           int32_t p, int32_t D, const float* pw, const float* pb, const float* pos,
                           float* out, hipStream_t s);
int32_t launch_ln_modulate(const float* x, RowVec shift, RowVec scale, int32_t M, int32_t D,
                           int32_t dtype, void* out, hipStream_t s, const Prefetch& pf = Prefetch{});
// the same in bf16 on the residual stream after `join`, which it writes back to x; and the join alone.  D % 4 == 0, D <= 2048,
// 16-byte aligned rows
int32_t launch_ln_modulate_join(float* x, const ResidJoin& join, RowVec shift, RowVec scale, int32_t M, int32_t D, bf16_t* out,
                                hipStream_t s, const Prefetch& pf);
int32_t launch_resid_join(float* x, const ResidJoin& join, int32_t M, int32_t D, hipStream_t s);
int32_t launch_linear_simple(const void* A, const void* W, const float* bias, int32_t M, int32_t N,
                             int32_t K, int32_t dtype, int32_t epi, void* out, float* resid,
                             RowVec gate, hipStream_t s);
int32_t launch_attention_simple(const void* qkv, int32_t B, int32_t N, int32_t heads, int32_t dh,
                                int32_t dtype, void* out, hipStream_t s);
// What follows the output layer in a drafting step, on the one latent x [C, H, W]: the guided noise estimate (dup = 2: conditional and
// null state, cfg_scale), m = coef_x x + coef_eps eps and x_next = m + sigma xi.  x_copy: nullptr, or where x goes too.
struct FinalMean {
    const float* x;
    const float *coef_x, *coef_eps, *sigma;
    float cfg_scale;
    int32_t dup, C;
    const float* xi;
    float *m, *x_next, *x_copy;
};
// mean: nullptr (the noise estimates go to out), or the step's mean and next draft, out being room for the estimates of dup states
int32_t launch_final_layer(const float* x, RowVec shift, RowVec scale, int32_t B, int32_t gh, int32_t gw,
                           int32_t p, int32_t c_out, int32_t D, const void* w, const float* bias,
                           int32_t dtype, float* out, hipStream_t s, const FinalMean* mean = nullptr);
int32_t launch_eps_to_mean(const float* eps_out, const float* x_states, const float* coef_x,
                           const float* coef_eps, float cfg_scale, int32_t K, int32_t C, int32_t c_out,
                           int64_t hw, float* m_out, hipStream_t s, float* eps_guided = nullptr,
                           const float* sigma_step = nullptr, const float* xi = nullptr, float* x_next = nullptr);

// drafter: fin = [emb | feat] in the compute type with emb the patch embedding, zero_out (nullable, may be feat) cleared.  One
// launch where the patch embedding has its 16-byte form, else emb goes through `emb_buf`.
int32_t launch_draft_embed(const float* x, int32_t x_mod, int32_t B, int32_t C, int32_t H, int32_t W, int32_t p, int32_t D,
                           const float* pw, const float* pb, const float* pos, const float* feat, int32_t dtype, void* fin,
                           float* zero_out, float* emb_buf, hipStream_t s);
// fin = [emb | feat], zero_out (nullable) cleared
int32_t launch_fuse_pack(const float* emb, const float* feat, int64_t M, int32_t D, int32_t dtype, void* fin,
                         float* zero_out, hipStream_t s);
// blocking range check of device-resident inputs (any pointer may be null); bit mask of violations
int32_t run_validate(const int32_t* t, int64_t n_t, int32_t T, const float* sigma, const float* u,
                     const float* lambda, int64_t n, uint32_t* violations, hipStream_t s);
// calib.hip: register-only MFMA loop on every CU; sustained TFLOP/s and shader clock (MHz) while it runs
int32_t run_mfma_ceiling(int32_t iters, double* tflops, double* mhz, hipStream_t s);

// frozen-target drafting of K steps from one noise estimate e [d]; out[k] = ||a_k - b_k||^2 (fp64)
int32_t launch_frozen_draft(const float* x_a, const float* e, const float* coef_x, const float* coef_eps,
                            const float* sigma, const float* xi, int32_t K, int64_t d, float* x_states, float* x_last,
                            float* m_draft, hipStream_t s);
int32_t launch_sqdist(const float* a, const float* b, int32_t K, int64_t d, double* out, hipStream_t s);

// ---- MFMA adaLN modulation GEMV, bf16 or fp32 weights as `mode` says (adaln_mfma.hip)
bool adaln_mfma_supported(int32_t D, int32_t total_rows);
// final_mfma.hip: final layer on the matrix cores (weights of type `dtype`, DiT-S/B/L/XL widths)
bool final_mfma_supported(int32_t D, int32_t P);
int32_t launch_final_layer_mfma(const float* x, RowVec shift, RowVec scale, int32_t M, int32_t gh, int32_t gw,
                                int32_t p, int32_t c_out, int32_t D, const void* w, int32_t dtype, const float* bias,
                                float* out, hipStream_t s, const FinalMean* mean);
int32_t launch_adaln_mfma(const float* sc, int32_t B, int32_t D, const void* const* w_tab,
                          const float* const* b_tab, const int32_t* row_start, int32_t n_mats,
                          int32_t total_rows, int32_t mode, float* mod, hipStream_t s);

// ---- MFMA kernels, bf16 only (gemm_mfma.hip, attn_mfma.hip) ------------------------
// compute units of the device (256 where there is none): asked once
int device_cus();
bool mfma_linear_supported(int32_t M, int32_t N, int32_t K);
int32_t launch_linear_mfma(const bf16_t* A, const bf16_t* W, const float* bias, int32_t M, int32_t N,
                           int32_t K, int32_t epi, bf16_t* out, float* resid, RowVec gate, hipStream_t s, int cu_share = 1,
                           const LnFold* ln = nullptr);
// the same product, K a whole number of slices, by two kernels that launch_linear_mfma chooses between:
// gemm_pipe.hip (many rows; bf16, all epilogues) ...
enum PipeTile { PIPE_256x256, PIPE_384x192, PIPE_256x192, PIPE_192x256, PIPE_192x128, PIPE_160x128, PIPE_128x128 };
int32_t launch_linear_pipe(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                           bf16_t* out, float* resid, RowVec gate, hipStream_t s, PipeTile tile, const LnFold* ln);
// ... and gemm_rows.hip (few rows; N % 8 == 0 and 16-byte aligned operands, checked by linear_rows_covers)
enum RowsTile { ROWS_64x64, ROWS_128x64, ROWS_128x128 };
int32_t launch_linear_rows(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                           bf16_t* out, float* resid, RowVec gate, hipStream_t s, RowsTile tile, bool from_zero = false);
int32_t launch_linear_rows(const float* X, const float* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                           float* out, float* resid, RowVec gate, hipStream_t s, RowsTile tile);
bool linear_rows_covers(int32_t N, int32_t K, int32_t elem_bytes, const float* bias, const void* out, const float* resid,
                        const RowVec& gate);
// resid = gate (X W^T + bias) + resid with K summed in kSplitParts parts (shapes: linear_split_covers, whatever M is).  Either at
// once, or, where that is faster (linear_split_pays), the parts go to part[kSplitParts][M][N] and *join is set for the next kernel.
// own_launch: the join has a launch of its own.
bool linear_split_covers(int32_t N, int32_t K);
bool linear_split_pays(int32_t M, int32_t N, int32_t K, bool own_launch);
int32_t launch_linear_split(const bf16_t* X, const bf16_t* W, const float* bias, int32_t M, int32_t N, int32_t K, float* resid,
                            RowVec gate, float* part, bool own_launch, ResidJoin* join, hipStream_t s, bool from_zero = false);
// whether it can take resid as zero instead of reading it (from_zero; where the parts are left, the next kernel can)
bool linear_split_from_zero(int32_t M, int32_t N, int32_t K, bool own_launch);
// fp32 operands and results, K a multiple of 32, products on the bf16 matrix instructions (gemm_f32.hip)
bool linear_f32_covers(const float* X, const float* W, int32_t M, int32_t N, int32_t K);
int32_t launch_linear_f32(const float* X, const float* W, const float* bias, int32_t M, int32_t N, int32_t K, int32_t epi,
                          float* out, float* resid, RowVec gate, hipStream_t s, int cu_share = 1);
// shapes the folded-LayerNorm epilogues cover: M rows of width D normalised, rows_per_sample tokens per sample
bool mfma_ln_fold_supported(int32_t M, int32_t D, int32_t rows_per_sample);
// the same kernel on fp32 operands (v_mfma_f32_32x32x2_f32), fp32 output
bool mfma_linear_f32_supported(int32_t M, int32_t N, int32_t K);
int32_t launch_linear_mfma_f32(const float* A, const float* W, const float* bias, int32_t M, int32_t N,
                               int32_t K, int32_t epi, float* out, float* resid, RowVec gate, hipStream_t s,
                               int cu_share = 1);
// the kernel and tile the two launches above pick for a problem with aligned operands that has the device to itself, encoded
// as free_linear_tile returns it; negative: not theirs
int32_t mfma_linear_tile(int32_t M, int32_t N, int32_t K, int32_t dtype, int32_t epi);
// fold vectors of all blocks in one launch (lnfold_mfma.hip); see LnFold
bool ln_fold_supported(int32_t D, int32_t rows_qkv, int32_t rows_fc1);
int32_t launch_ln_fold(const float* mod, int32_t B, int32_t D, int32_t mod_stride, int32_t depth, int32_t rows_qkv,
                       int32_t rows_fc1, const void* const* w_tab, const float* const* b_tab, float* fold,
                       int64_t fold_stride, hipStream_t s);
bool mfma_attention_supported(int32_t N, int32_t dh);
int32_t launch_attention_mfma(const bf16_t* qkv, int32_t B, int32_t N, int32_t heads, int32_t dh,
                              bf16_t* out, hipStream_t s, const Prefetch& pf = Prefetch{}, bool split_keys = false);
// fp32 operands and softmax on the matrix cores (attn_f32_mfma.hip); qkv and out 16-byte aligned
bool mfma_attention_f32_supported(int32_t N, int32_t dh);
int32_t launch_attention_mfma_f32(const float* qkv, int32_t B, int32_t N, int32_t heads, int32_t dh,
                                  float* out, hipStream_t s);

}  // namespace freemi
