// Internal helpers of the HIP library (gfx950 only).  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "moe.h"

namespace moe {

// Element storage types: bf16 is kept as its 16-bit pattern.
typedef uint16_t bf16_t;

// MFMA operand / accumulator vector types.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_to_f32(bf16_t h) {
    return __uint_as_float(((uint32_t)h) << 16);
}

// fp32 -> bf16, round to nearest, ties to even (v_cvt_pk_bf16_f32); NaN stays a
// quiet NaN.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)pack_bf16x2(f, f); }

// SiLU(a) = a / (1 + exp(-a)), the quotient correctly rounded: by the division, or for
// |a| < SILU_NEAR by the hardware reciprocal and one residual step, which for every one of
// the 2^31 floats in that range gives the division's bits (-0 gives +0) at under half its
// instructions (DeepSeek-V2-Lite prefill, 8192 tokens: divisions 548 us a step, this 537.5,
// the reciprocal alone, an ulp off for 4.6 % of the floats, 534.5).  Past the range the
// reciprocal goes subnormal, which the hardware gives as zero, from a = -87.3 down, and an
// infinity has no residual.
constexpr float SILU_NEAR = 87.0f;

__device__ __forceinline__ float silu_near(float a) {
    const float d = 1.0f + __expf(-a), r = __builtin_amdgcn_rcpf(d), q = a * r;
    return fmaf(fmaf(-d, q, a), r, q);
}

__device__ __forceinline__ float silu_div(float a) { return a / (1.0f + __expf(-a)); }

template <int N>
__device__ __forceinline__ void silu(float (&a)[N]) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) m = fmaxf(m, fabsf(a[i]));
    if (m < SILU_NEAR) {
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = silu_near(a[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = silu_div(a[i]);
    }
}

// Inclusive prefix sum across the 64 lanes of a wave (every lane active), by DPP
// moves: within rows of 16 lanes (row_shr 1, 2, 4, 8), then each row's last lane added
// to the row after it (row_bcast 15) and lane 31 to the upper half (row_bcast 31).  A
// shuffle per step goes through LDS, six dependent round trips.
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Largest s in [0, n) with a[s] <= v, for non-decreasing a with a[0] <= v.
__device__ __forceinline__ int last_le(const int* a, int n, int v) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__host__ __device__ constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Launch-error check shared by the host wrappers.  Reading the error clears it, so a
// status that a caller drops is lost: it and the launchers below are [[nodiscard]].
[[nodiscard]] inline int launch_status() {
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? MOE_OK : MOE_ERR_DEVICE;
}

// Raise a kernel's dynamic-LDS limit to `bytes` on the current device.  The
// setting persists, so each device is configured once per size increase and
// later launches skip the runtime call.  The check, the runtime call and the
// record of the granted size happen under one lock per kernel, so concurrent
// callers never leave a smaller limit set than the one recorded.
struct LdsGrant {
    static constexpr int kMaxDevices = 64;
    std::mutex lock;
    int granted[kMaxDevices] = {};
};

[[nodiscard]] inline int allow_dynamic_lds(const void* kernel, size_t bytes, LdsGrant& g) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= LdsGrant::kMaxDevices)
        return MOE_ERR_DEVICE;
    std::lock_guard<std::mutex> guard(g.lock);
    if (g.granted[dev] >= (int)bytes) return MOE_OK;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) !=
        hipSuccess)
        return MOE_ERR_DEVICE;
    g.granted[dev] = (int)bytes;
    return MOE_OK;
}

template <auto F>
[[nodiscard]] inline int allow_dynamic_lds(size_t bytes) {
    static LdsGrant grant;
    return allow_dynamic_lds((const void*)F, bytes, grant);
}

// ---------------------------------------------------------------------------
// Internal launchers (one translation unit each); arguments already validated.
// ---------------------------------------------------------------------------
[[nodiscard]]
int launch_route_topk(const void* x, int dtype, const void* w, const float* bias, int64_t T, int d,
                      int E, int k, int flags, float* logits, int32_t* idx, float* gate, void* ws,
                      hipStream_t s);
// bf16 scores of a short batch (route.hip): whether a batch takes them, in how many K
// chunks, and the launch (one chunk: scores + bias to out[T][E]; more: the chunks' sums to
// out[chunk][T][E], bias left to the top-k)
bool route_short(int64_t T, int d, int E);
int route_chunks(int64_t T, int d, int E);
[[nodiscard]]
int launch_scores_short(const void* x, const void* w, const float* bias, int64_t T, int d, int E,
                        float* out, hipStream_t s);
size_t route_ws_bytes(int dtype, int64_t T, int d, int E, int flags);

[[nodiscard]]
int launch_quantize_e4m3(const void* x, int dtype, int64_t rows, int cols, uint8_t* q, float* scales,
                         hipStream_t s);
[[nodiscard]]
int launch_route_topk_e4m3(const uint8_t* xq, const float* sx, const uint8_t* wq, const float* sw,
                           const float* bias, int64_t T, int d, int E, int k, int flags,
                           float* logits, int32_t* idx, float* gate, hipStream_t s);

// Tiled score kernel (score.hip): whether a batch takes it, and the launch over more than
// SCORE_TOPK_MAX_E experts (scores + bias to out[T][E]).
bool score_tiled(int64_t T, int rowbytes, int E);
[[nodiscard]]
int launch_score_tiles(bool fp8, const void* x, const void* w, const float* sx, const float* sw,
                       const float* bias, int64_t T, int rowbytes, int E, float* out,
                       hipStream_t s);
// The tiled score kernel over 33 .. SCORE_TOPK_MAX_E experts
// (MOE_ERR_SHAPE otherwise), finishing with the top-k and gates of its tokens
// (logits nullable: scores + bias stored there when given).
// Wider batches keep the top-k launch of their own (its lanes per token double and the
// workgroup's passes over its tokens cost more than the launch).  Fused at 65-128
// experts: 16384 x 128 routing 25.3 -> 23.0 us, E4M3 20.6 -> 18.3; 8192 x 128 even.
constexpr int SCORE_TOPK_MAX_E = 128;
[[nodiscard]]
int launch_score_tiles_topk(bool fp8, const void* x, const void* w, const float* sx,
                            const float* sw, const float* bias, int64_t T, int rowbytes, int E,
                            int k, int renorm, float* logits, int32_t* idx, float* gate,
                            hipStream_t s);
// Top-k and gates of given scores (route.hip): scores[T][E] read in place.
[[nodiscard]]
int launch_topk_given(const float* scores, int64_t T, int E, int k, int flags, int32_t* idx,
                      float* gate, hipStream_t s);

[[nodiscard]]
int launch_histogram(const int32_t* idx, int64_t T, int k, int E, int32_t* counts, int32_t* coact,
                     hipStream_t s);
// co-activation counts added to coact (already cleared)
[[nodiscard]]
int launch_coact(const int32_t* idx, int64_t T, int k, int E, int32_t* coact, hipStream_t s);

struct PermuteTables {
    uint64_t hosts[MOE_MAX_E];          // bit j set iff GPU j hosts expert e
    int16_t slot_of[MOE_MAX_E];         // local slot of expert e, or -1
    int16_t expert_of_slot[MOE_MAX_GROUPS];
};

[[nodiscard]]
int launch_permute(const void* x, int dtype, const int32_t* idx, const float* gate,
                   const int32_t* counts, int64_t T, int d, int k, int E, const PermuteTables& tab,
                   int n_local, int G, int dev, void* x_perm, int64_t cap_rows,
                   int32_t* group_offsets, int32_t* row_token, float* row_gate, int32_t* token_row,
                   int32_t* send_counts, void* ws, hipStream_t s);
size_t permute_ws_bytes(int64_t T, int k, int E);
// route_topk, histogram and permute in one call (x_perm null: no row copy)
[[nodiscard]]
int launch_route_package(const void* x, int dtype, const void* w, const float* bias, int64_t T,
                         int d, int E, int k, int flags, float* logits, int32_t* idx, float* gate,
                         void* ws_route, int32_t* counts, int32_t* coact, const PermuteTables& tab,
                         int n_local, int G, int dev, void* x_perm, int64_t cap_rows,
                         int32_t* group_offsets, int32_t* row_token, float* row_gate,
                         int32_t* token_row, int32_t* send_counts, void* ws_perm, hipStream_t s);
// Device address of the library's own permute scratch on the current device
// (MOE_PERMUTE_NOALLOC_MAX_WS bytes, 256-byte aligned).
[[nodiscard]]
int permute_scratch(void** ptr);

// a_rows (nullable): row p of the first product's input is row a_rows[p] of
// x_perm, which then holds a_total rows (the token rows; no packaged copy).
// lead > 0: the first `lead` of the n_groups groups hold lead_rows rows each,
// and offsets (n_groups - lead + 1 entries) counts the others' rows from row
// lead * lead_rows.
[[nodiscard]]
int launch_grouped_ffn(const void* x_perm, int dtype, const int32_t* offsets, int n_groups,
                       const void* const* w13, const void* const* w2, int d, int f,
                       int64_t cap_rows, void* y_perm, void* ws, hipStream_t s,
                       const int32_t* a_rows = nullptr, int64_t a_total = 0,
                       int products = MOE_FFN_GATE_UP | MOE_FFN_DOWN,
                       const void* combine = nullptr, int lead = 0, int lead_rows = 0);
// moe_grouped_ffn with every group streamed and the down product's chunk sum
// writing the gate-weighted combine (bf16)
[[nodiscard]]
int launch_grouped_ffn_combine(const void* x_perm, const int32_t* offsets, int n_groups,
                               const void* const* w13, const void* const* w2, int d, int f,
                               int64_t cap_rows, const int32_t* token_row, const float* gate,
                               const void* y_shared, int64_t T, int k, void* y, void* ws,
                               hipStream_t s);
// the fp32 products (ffn_f32.hip); h: [cap_rows][f] scratch
[[nodiscard]]
int launch_ffn_f32(const float* x, const int32_t* offsets, int n_groups, const void* const* w13,
                   const void* const* w2, int d, int f, int64_t cap_rows, float* y, float* h,
                   const int32_t* a_rows, int products, int lead, int lead_rows, int cus,
                   hipStream_t s);
size_t grouped_ffn_ws_bytes(int dtype, int64_t cap_rows, int d, int f, int n_groups);

// y_shared: n_shared slices of [T][d] (nullable: none)
[[nodiscard]]
int launch_combine(const void* y_perm, int dtype, const int32_t* token_row, const float* gate,
                   const void* y_shared, int n_shared, int64_t T, int d, int k, void* y,
                   hipStream_t s);

}  // namespace moe
