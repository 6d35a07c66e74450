// Gate scores of long batches over many experts (Sec. II-A: the gating network
// scores every expert for every token), as a tiled GEMM:
//
//   bf16:  S[t][e] = sum_i x[t][i] w[e][i]
//   E4M3:  S[t][e] = s_x[t] s_w[e] sum_i q_x[t][i] q_w[e][i]    (the quantized
//          predictor's gate, Sec. V-A)
//
// plus bias.  The kernel streams the hidden states once: a workgroup
// owns 64 tokens x all experts (2 token halves x 2 or 4 groups of expert columns), so
// each router row is read once per 64 tokens instead of once per 32 or 16, and
// both operands go straight from HBM/L2 into a ring of R LDS stages (128 bytes of
// K per row per stage, `buffer_load ... lds`), which keeps enough bytes moving per CU:
// a stage's fragments are read while the stage before it multiplies, and its slot is
// refilled at once.  Rows past the
// batch or past E fall outside the buffer descriptors and read as zero.  The
// LDS rows are XOR-swizzled in 16-byte chunks (the loading lane fetches the
// chunk that belongs in its slot), so fragment reads are free of bank
// conflicts without padding.  Bound by the launch, the first loads and the epilogue
// (about 8 us at any d), then by the latency of a stage; with a ring that truly stays
// in flight a 64-token block of 128 experts takes 0.27 us per 128 bytes of K in E4M3
// (0.85 before), 0.27 in bf16 (0.39).  Routing calls, top-k included: 8192 x 64, d = 2048
// bf16 17.5 -> 13.9 us, E4M3 17.2 -> 11.8; 16384 x 128 27.7 -> 23.0 and 25.3 -> 18.3.
//
// The workgroup stores its scores (bias added), and up to 128 experts finishes with the
// top-k of its own 64 tokens (KM > 0): the scores go through LDS to the same
// top-k as for given scores, so no second launch reads them back.
#include "common.h"
#include "topk.h"

namespace moe {
namespace {

typedef __attribute__((address_space(3))) void lds_void;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int SC_BKB = 128;        // bytes of K per row per stage
constexpr uint32_t SC_RSRC_WORD3 = 0x00020000;
constexpr int SC_OOB = 0x7fffff00;  // an offset past every descriptor's range: the store is dropped

// chunk position of 16-byte chunk c of LDS row r: c ^ sc_swz(r)
__device__ __forceinline__ int sc_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// wait until at most N of this wave's vector-memory loads are outstanding
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// KM > 0: top-k (k <= KM, top-k class C) of the workgroup's tokens
// into idx / gate after the scores; out (the scores) may then be null.
template <bool FP8, int WM, int WN, int NTW, int R, int KM = 0, int C = 0>
__global__ __launch_bounds__(64 * WM * WN) void score_tiles_kernel(
    const uint8_t* __restrict__ x, const uint8_t* __restrict__ w, const float* __restrict__ sx,
    const float* __restrict__ sw, const float* __restrict__ bias, int64_t T, int rowbytes, int E,
    float* __restrict__ out, int k = 0, int renorm = 0, int32_t* __restrict__ idx = nullptr,
    float* __restrict__ gate = nullptr) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    constexpr int NW = WM * WN, BM = 32 * WM;         // waves, tokens
    static_assert(NW % 2 == 0, "sc_swz of a load's rows");
    constexpr int A_BYTES = BM * SC_BKB;
    constexpr int NB = 32 * WN * NTW;                 // router rows per tile
    constexpr int B_BYTES = NB * SC_BKB;
    constexpr int STAGE = A_BYTES + B_BYTES;
    constexpr int A_LOADS = A_BYTES / 1024 / NW;      // 1 KB direct loads per wave per stage
    constexpr int B_LOADS = B_BYTES / 1024 / NW;
    constexpr int P = A_LOADS + B_LOADS;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int64_t t0 = (int64_t)blockIdx.x * BM;
    const int nt = (int)((T - t0) < BM ? (T - t0) : BM);
    const int nst = rowbytes / SC_BKB;

    const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(x + t0 * rowbytes), (short)0, nt * rowbytes, SC_RSRC_WORD3);
    const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)w, (short)0, E * rowbytes, SC_RSRC_WORD3);
    const __amdgpu_buffer_rsrc_t none =
        __builtin_amdgcn_make_buffer_rsrc((void*)x, (short)0, 0, SC_RSRC_WORD3);
    // stage s into slot s % R; past the last stage from an empty range, loads without
    // traffic, so that the counts the waits rely on stay the same
    // load i of a wave fills LDS rows 8 (NW i + wave) + (lane / 8), chunk slot lane % 8,
    // from the operand row of the same index (row offsets in the per-lane offset, so
    // the descriptor's range check sees them), chunk (lane % 8) ^ sc_swz(row)
    const int drow = lane >> 3;
    const int voff0 = (8 * wave + drow) * rowbytes + (((lane & 7) ^ (drow ^ (wave & 1))) * 16);
    const int vstep = 8 * NW * rowbytes;
    auto dma = [&](int s) {
        char* base = lds + (s % R) * STAGE;
        const int so = s * SC_BKB;
        const bool in = s < nst;
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                in ? arsrc : none, (lds_void*)(base + (NW * i + wave) * 1024), 16, voff0 + i * vstep, so, 0, 0);
#pragma unroll
        for (int i = 0; i < B_LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                in ? brsrc : none, (lds_void*)(base + A_BYTES + (NW * i + wave) * 1024), 16, voff0 + i * vstep,
                so, 0, 0);
    };

    // fragments: lane row r = lane % 32 of its 32-row tile, half h = lane / 32.
    // bf16 (32x32x16): sub-step q reads chunk 4h + q (elements 32h + 8q ..);
    // E4M3 (32x32x64): sub-step q reads chunks 4h + 2q, 4h + 2q + 1.  The same
    // K order for both operands, so the products sum over all of K.
    const int fr = lane & 31, h = lane >> 5;
    const int swz = sc_swz(fr);
    const int a_row = (wm * 32 + fr) * SC_BKB;
    const int b_row = A_BYTES + (wn * 32 * NTW + fr) * SC_BKB;
    int coff[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) coff[c] = ((4 * h + c) ^ swz) * 16;

    f32x16 acc[NTW];
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

    // the lane's column terms (bias; the FP8 router-row scales), loaded before the
    // K loop: a load still pending at the stores made the compiler wait for every
    // earlier store before each one, serialising the epilogue
    float b_c[NTW], s_c[NTW];
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        const int col = wn * 32 * NTW + j * 32 + fr;
        const int cc = col < E ? col : E - 1;
        b_c[j] = bias ? bias[cc] : 0.0f;
        s_c[j] = FP8 ? sw[cc] : 1.0f;
    }

    // fragments of a stage: 16-byte chunks, of the tokens and of each router tile
    struct Frags {
        u32x4 a[4], b[NTW][4];
    };
    auto read = [&](int s, Frags& f) {
        const char* st = lds + (s % R) * STAGE;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f.a[c] = *(const u32x4*)(st + a_row + coff[c]);
#pragma unroll
            for (int j = 0; j < NTW; ++j)
                f.b[j][c] = *(const u32x4*)(st + b_row + j * 32 * SC_BKB + coff[c]);
        }
    };
    auto mma = [&](const Frags& f) {
        if constexpr (FP8) {
            auto pair = [](const u32x4& u, const u32x4& v) {
                return i32x8{(int)u.x, (int)u.y, (int)u.z, (int)u.w,
                             (int)v.x, (int)v.y, (int)v.z, (int)v.w};
            };
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < NTW; ++j)
                    acc[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        pair(f.a[2 * q], f.a[2 * q + 1]), pair(f.b[j][2 * q], f.b[j][2 * q + 1]),
                        acc[j], 0, 0, 0, 127, 0, 127);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < NTW; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8, f.a[q]), __builtin_bit_cast(bf16x8, f.b[j][q]),
                        acc[j], 0, 0, 0);
        }
    };
    // stage t + 1 has landed (the R - 2 after it may still fly) and every wave holds its
    // fragments of stage t, so that stage's slot takes stage t + R: the next fragments
    // come from LDS and the ring refills while stage t multiplies.  A bare barrier: the
    // fence of __syncthreads would wait for all the stages in flight.  The compiler
    // waits for every load in flight before an LDS read it cannot tell apart from the
    // loads' writes: with the reads after the loads, or through HIP's struct uint4, it
    // drained the ring in every stage.
    auto step = [&](int t, const Frags& f, Frags& next) {
        wait_vm<(R - 2) * P>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        read(t + 1, next);
        dma(t + R);
        mma(f);
    };

    Frags f0, f1;
#pragma unroll
    for (int s = 0; s < R; ++s) dma(s);
    wait_vm<(R - 1) * P>();
    asm volatile("s_barrier" ::: "memory");
    read(0, f0);
    int t = 0;
    for (; t + 1 < nst; t += 2) {
        step(t, f0, f1);
        step(t + 1, f1, f0);
    }
    if (t < nst) step(t, f0, f1);
    wait_vm<0>();                          // no load outlives the ring

    // accumulator element r of a 32x32 tile: row 8 (r / 4) + 4 h + r % 4, column fr;
    // out[t][e] = score + bias[e].
    // Branch-free stores through a descriptor over the block's rows: an element past
    // the batch or past E gets an offset outside it and is dropped.
    float* o = out ? out + t0 * E : nullptr;
    const __amdgpu_buffer_rsrc_t orsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)o, (short)0, o ? nt * E * 4 : 0, SC_RSRC_WORD3);
    // fused top-k: the scores also go to an LDS tile [64][E_pad + 1] over the
    // ring, which every wave has finished reading and loading once past this barrier
    const int ldS = ((E + 15) & ~15) + 1;
    float* const sc = (float*)lds;
    if constexpr (KM > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    float sx_r[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = wm * 32 + (r >> 2) * 8 + 4 * h + (r & 3);
        sx_r[r] = FP8 ? sx[t0 + (row < nt ? row : nt - 1)] : 1.0f;
    }
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        const int col = wn * 32 * NTW + j * 32 + fr;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = wm * 32 + (r >> 2) * 8 + 4 * h + (r & 3);
            float v = acc[j][r];
            if (FP8) v = v * sx_r[r] * s_c[j];
            if (bias) v += b_c[j];
            const int off = (row < nt && col < E) ? (row * E + col) * 4 : SC_OOB;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), orsrc, off, 0, 0);
            if constexpr (KM > 0)
                if (row < nt && col < E) sc[row * ldS + col] = v;
        }
    }
    if constexpr (KM > 0) {
        __syncthreads();
        topk_tokens<KM, C>(sc, ldS, nt, t0, E, k, renorm, idx, gate);
    }
}

template <bool FP8, int WM, int WN, int NTW, int R, int KM, int C>
int launch_tiles_topk(const uint8_t* x, const uint8_t* w, const float* sx, const float* sw,
                      const float* bias, int64_t T, int rowbytes, int E, int k, int renorm,
                      float* logits, int32_t* idx, float* gate, hipStream_t s) {
    constexpr size_t ring = (size_t)R * 32 * (WM + WN * NTW) * SC_BKB;
    constexpr size_t tile = (size_t)32 * WM * (32 * WN * NTW + 1) * sizeof(float);
    constexpr size_t lds = ring > tile ? ring : tile;
    static_assert(lds <= 160 * 1024, "ring fits the LDS of a CU");
    if (lds > 65536 &&
        allow_dynamic_lds<score_tiles_kernel<FP8, WM, WN, NTW, R, KM, C>>(lds) != MOE_OK)
        return MOE_ERR_DEVICE;
    hipLaunchKernelGGL((score_tiles_kernel<FP8, WM, WN, NTW, R, KM, C>),
                       dim3((unsigned)ceil_div(T, 32 * WM)), dim3(64 * WM * WN), lds, s, x, w, sx, sw,
                       bias, T, rowbytes, E, logits, k, renorm, idx, gate);
    return launch_status();
}

template <bool FP8, int KM>
int launch_topk_by_width(const uint8_t* x, const uint8_t* w, const float* sx, const float* sw,
                         const float* bias, int64_t T, int rowbytes, int E, int k, int renorm,
                         float* logits, int32_t* idx, float* gate, hipStream_t s) {
    if (E <= 64)
        return launch_tiles_topk<FP8, 2, 2, 1, 4, KM, 2>(x, w, sx, sw, bias, T, rowbytes, E, k,
                                                         renorm, logits, idx, gate, s);
    return launch_tiles_topk<FP8, 2, 4, 1, 6, KM, 3>(x, w, sx, sw, bias, T, rowbytes, E, k, renorm,
                                                     logits, idx, gate, s);
}

}  // namespace

// Whether a batch takes the tiled score kernel:
// E > 32 (smaller E is cheap for the K-split kernel), whole 128-byte stages,
// and at least 128 token tiles (half a tile per CU or more; the DeepSeek-V2-Lite
// prefill batch of 8192 tokens: 22.1 -> 20.2 us against the block kernel).  One
// K chunk: summing K-chunk partials in a second pass cost more than the
// parallelism it bought (that batch split in two: 27.1 us), and with fewer tiles
// the K-split kernel, which spreads a batch over more workgroups, measured faster
// (Qwen1.5-shaped batches).
bool score_tiled(int64_t T, int rowbytes, int E) {
    if (E <= 32 || E > MOE_MAX_E || rowbytes % SC_BKB != 0 || T <= 0) return false;
    if ((int64_t)MOE_MAX_E * rowbytes >= ((int64_t)1 << 31)) return false;   // 32-bit buffer offsets
    return ceil_div(T, 64) >= 128;
}

// Waves and ring by tile width.  Up to 64 experts: 4 waves, 4 stages, two workgroups a
// CU (8 stages, one a CU: 13.8 against 15.5 us at 8192 x 64, d = 2048); up to 128: 8
// waves (4: 22.4 against 22.7 us at 12000 x 100, even at 16384 x 128), 6 stages, both with
// the top-k (launch_score_tiles_topk); wider: as many stages as the LDS holds.
template <bool FP8>
static int launch_wide(const void* x, const void* w, const float* sx, const float* sw,
                       const float* bias, int64_t T, int rowbytes, int E, float* out, hipStream_t s) {
    constexpr int WM = 2, WN = 2, NTW = 4, R = 3;
    constexpr size_t lds = (size_t)R * 32 * (WM + WN * NTW) * SC_BKB;
    static_assert(lds <= 160 * 1024, "ring fits the LDS of a CU");
    if (allow_dynamic_lds<score_tiles_kernel<FP8, WM, WN, NTW, R>>(lds) != MOE_OK)
        return MOE_ERR_DEVICE;
    hipLaunchKernelGGL((score_tiles_kernel<FP8, WM, WN, NTW, R>),
                       dim3((unsigned)ceil_div(T, 32 * WM)), dim3(64 * WM * WN), lds, s,
                       (const uint8_t*)x, (const uint8_t*)w, sx, sw, bias, T, rowbytes, E, out);
    return launch_status();
}

int launch_score_tiles(bool fp8, const void* x, const void* w, const float* sx, const float* sw,
                       const float* bias, int64_t T, int rowbytes, int E, float* out,
                       hipStream_t s) {
    if (E <= SCORE_TOPK_MAX_E) return MOE_ERR_SHAPE;
    return fp8 ? launch_wide<true>(x, w, sx, sw, bias, T, rowbytes, E, out, s)
               : launch_wide<false>(x, w, sx, sw, bias, T, rowbytes, E, out, s);
}

int launch_score_tiles_topk(bool fp8, const void* x, const void* w, const float* sx,
                            const float* sw, const float* bias, int64_t T, int rowbytes, int E,
                            int k, int renorm, float* logits, int32_t* idx, float* gate,
                            hipStream_t s) {
    if (E <= 32 || E > SCORE_TOPK_MAX_E) return MOE_ERR_SHAPE;
    const uint8_t* xb = (const uint8_t*)x;
    const uint8_t* wb = (const uint8_t*)w;
#define MOE_ST(KM)                                                                               \
    (fp8 ? launch_topk_by_width<true, KM>(xb, wb, sx, sw, bias, T, rowbytes, E, k, renorm, logits, \
                                          idx, gate, s)                                          \
         : launch_topk_by_width<false, KM>(xb, wb, sx, sw, bias, T, rowbytes, E, k, renorm,      \
                                           logits, idx, gate, s))
    if (k <= 2) return MOE_ST(2);
    if (k <= 4) return MOE_ST(4);
    if (k <= 8) return MOE_ST(8);
    return MOE_ST(MOE_MAX_K);
#undef MOE_ST
}

}  // namespace moe
