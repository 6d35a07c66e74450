// Gate scores and top-k routing (Sec. II-A of the Director paper: the gating
// network scores each expert for every token and the token is sent to the k
// best; the gate is replicated on every GPU, Sec. II-B).
//
// Each workgroup owns a block of tokens:
//   phase 1  scores for its tokens x all E experts into LDS
//            bf16: MFMA 16x16x32, K split over 16 waves, fixed-order reduction
//            (long batches over more than 32 experts use the tiled kernel of
//            score.hip instead; short batches score_small_kernel and a top-k
//            launch);
//            f32:  MFMA 16x16x4 (fp32 operands and sums), K split over waves;
//            logits-in: read in place from global memory
//   phase 2  bias added, scores written back coalesced (if requested)
//   phase 3  a group of lanes per token: k rounds of a group-wide maximum, gates.
#include "common.h"
#include "topk.h"

namespace moe {
namespace {

constexpr int ROUTE_THREADS = TOPK_THREADS;

// bf16 gate scores on MFMA 16x16x32.  A workgroup of 16 waves owns 16*RT
// tokens; wave w takes the K steps w, w+16, w+32, ... (32 elements each) for
// all RT token tiles and up to NTM expert tiles, with operand fragments loaded
// straight from global memory (the router matrix stays L2-resident), two K
// steps of loads in flight per wave.  Partial scores are reduced in LDS in a fixed order
// (four slices, each summed over its four waves in turn, then the slices in
// turn), so the scores are deterministic.
constexpr int RB_WAVES = 16;
constexpr int RB_THREADS = RB_WAVES * 64;
constexpr uint32_t RB_RSRC_WORD3 = 0x00020000;     // raw buffer, 32-bit data format
constexpr int RB_OOB = 0x7ffffff0;                 // an offset past every descriptor's range

__device__ __forceinline__ uint4 rb_load16(__amdgpu_buffer_rsrc_t r, int voff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
}

template <int RT, int NTM, int KM, int C>
__global__ __launch_bounds__(RB_THREADS) void route_bf16_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, const float* __restrict__ bias,
    int64_t T, int d, int E, int k, int renorm, float* __restrict__ logits,
    int32_t* __restrict__ idx, float* __restrict__ gate) {
    extern __shared__ __attribute__((aligned(16))) float smem[];
    constexpr int ROWS = 16 * RT;
    const int E_pad = (E + 15) & ~15;
    const int ldS = E_pad + 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * ROWS;
    const int nt = (int)((T - t0) < ROWS ? (T - t0) : ROWS);
    const int NT = E_pad / 16;
    const int row = lane & 15, kq = (lane >> 4) * 8;

    // operands through buffer descriptors: rows past the block's tokens or past E
    // fall outside them and read as zero, and a masked lane (K past d, a tile past
    // the experts) gets an offset outside them too, so every load is issued
    // unconditionally and the compiler can keep several in flight
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(X + t0 * d), (short)0, nt * d * 2, RB_RSRC_WORD3);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)W, (short)0, E * d * 2, RB_RSRC_WORD3);
    int xoff[RT], woff[NTM];
#pragma unroll
    for (int i = 0; i < RT; ++i) xoff[i] = ((i * 16 + row) * d + kq) * 2;
#pragma unroll
    for (int j = 0; j < NTM; ++j) woff[j] = ((j * 16 + row) * d + kq) * 2;   // j >= NT: rows >= E
    f32x4 acc[RT][NTM];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NTM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nsteps = (d + 31) / 32;                  // 32 elements each
    if (NTM <= 4) {
        // all tiles' fragments of one K step fit in registers: keep two steps of
        // loads in flight (ring of two register sets, alternating by step parity).
        // Loads past this wave's last step get out-of-range offsets (zeros, no
        // memory traffic), so the loop has no branches and the waits are exact.
        uint4 av[2][RT], bv[2][NTM];
        const int n_mine = wave < nsteps ? (nsteps - wave + RB_WAVES - 1) / RB_WAVES : 0;
        const int s0 = wave;
        auto load = [&](int i, uint4* a_, uint4* b_) {
            const int k0 = (s0 + i * RB_WAVES) * 32;
            const bool kin = i < n_mine && k0 + kq < d;
#pragma unroll
            for (int r = 0; r < RT; ++r) a_[r] = rb_load16(xrsrc, kin ? xoff[r] + k0 * 2 : RB_OOB);
#pragma unroll
            for (int j = 0; j < NTM; ++j) b_[j] = rb_load16(wrsrc, kin ? woff[j] + k0 * 2 : RB_OOB);
        };
        // every tile, also those past the experts (their operands read as zero):
        // a branch here would make the compiler wait for every load in flight
        auto mma = [&](const uint4* a_, const uint4* b_) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < NTM; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, a_[i]), __builtin_bit_cast(bf16x8, b_[j]),
                        acc[i][j], 0, 0, 0);
        };
        load(0, av[0], bv[0]);
        load(1, av[1], bv[1]);
        for (int i = 0; i < n_mine; i += 2) {
            mma(av[0], bv[0]);
            load(i + 2, av[0], bv[0]);
            mma(av[1], bv[1]);                    // zeros when i + 1 == n_mine
            load(i + 3, av[1], bv[1]);
        }
    } else {
        for (int step = wave; step < nsteps; step += RB_WAVES) {
            const int k0 = step * 32;
            const bool kin = k0 + kq < d;
            bf16x8 a[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i)
                a[i] = __builtin_bit_cast(bf16x8, rb_load16(xrsrc, kin ? xoff[i] + k0 * 2 : RB_OOB));
#pragma unroll
            for (int jc = 0; jc < NTM; jc += 4) {
                if (jc >= NT) break;
                bf16x8 b[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    b[jj] = __builtin_bit_cast(bf16x8,
                                               rb_load16(wrsrc, kin ? woff[jc + jj] + k0 * 2 : RB_OOB));
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
                        if (jc + jj < NT)
                            acc[i][jc + jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                a[i], b[jj], acc[i][jc + jj], 0, 0, 0);
            }
        }
    }

    // fixed-order reduction in the MFMA output layout (one 16-byte LDS access per
    // tile and lane): slice g = wave & 3 receives waves g, g+4, g+8, g+12 in turn,
    // the four slices are added in order into slice 0, and the sums are laid out
    // row-major (over slices 1..3) for the epilogue.
    const int g = wave & 3, q = wave >> 2;
    const int nslice = ROWS * E_pad;                  // floats per slice
    f32x4* Sg = (f32x4*)smem + g * (nslice / 4);
    for (int pass = 0; pass < 4; ++pass) {
        if (q == pass) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < NTM; ++j) {
                    if (j >= NT) continue;
                    f32x4* p = Sg + (i * NT + j) * 64 + lane;
                    *p = pass == 0 ? acc[i][j] : *p + acc[i][j];
                }
        }
        __syncthreads();
    }
    {
        f32x4* s4 = (f32x4*)smem;
        const int n4 = nslice / 4;
        for (int c = tid; c < n4; c += RB_THREADS)
            s4[c] = ((s4[c] + s4[n4 + c]) + s4[2 * n4 + c]) + s4[3 * n4 + c];
    }
    __syncthreads();
    float* Sm = smem + nslice;
    for (int c = tid; c < ROWS * E_pad; c += RB_THREADS) {
        const int r = c / E_pad, e = c % E_pad;
        const int rr = r & 15;
        const int o = (((r >> 4) * NT + (e >> 4)) * 64 + (rr >> 2) * 16 + (e & 15)) * 4 + (rr & 3);
        Sm[r * ldS + e] = smem[o];
    }
    __syncthreads();
    // 1024 threads hold at least one lane group per token: one token per group
    finish_tokens<KM, C, 1>(Sm, ldS, nt, t0, E, k, renorm, bias, logits, idx, gate);
}

// bf16 gate scores of short batches (few token blocks, e.g. decode): one 8-wave
// workgroup per (16 tokens, 16 experts, K chunk) on MFMA 16x16x32, the waves splitting
// the chunk, every operand load of a wave's slice issued before its first product (up to 8
// K steps at a time), the 8 partial tiles summed in wave order through LDS.  Rows
// past the batch or past E, and K past d, read as zero through the buffer
// descriptors.  Bound by load latency, and past 2048 K elements by what one CU can
// load.  With one chunk the scores leave finished, bias added; with more the chunks'
// sums go to out[chunk][T][E] for the top-k to add (route_chunks).
constexpr int SS_WAVES = 8;
constexpr int SS_STEPS = 8;            // 32-wide K steps of loads issued at once

__global__ __launch_bounds__(SS_WAVES * 64) void score_small_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, const float* __restrict__ bias,
    int64_t T, int d, int E, int chunks, float* __restrict__ out) {
    __shared__ f32x4 part[SS_WAVES][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int e0 = blockIdx.x * 16;
    const int64_t t0 = (int64_t)blockIdx.y * 16;
    const int nt = (int)((T - t0) < 16 ? (T - t0) : 16);
    const int ne = E - e0 < 16 ? E - e0 : 16;
    const int row = lane & 15, kq = (lane >> 4) * 8;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(X + t0 * d), (short)0, nt * d * 2, RB_RSRC_WORD3);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(W + (int64_t)e0 * d), (short)0, ne * d * 2, RB_RSRC_WORD3);
    // the thread that finishes (token r, expert e): its bias, loaded beside the operands
    const int r = (tid >> 4) & 15, e = tid & 15;
    const float b = chunks == 1 && bias && e < ne ? bias[e0 + e] : 0.f;
    const int nall = (d + 31) / 32, chunk = blockIdx.z;       // chunk * nall < 2^31
    const int cbeg = chunks == 1 ? 0 : chunk * nall / chunks;
    const int nsteps = chunks == 1 ? nall : (chunk + 1) * nall / chunks - cbeg;
    const int sbeg = cbeg + wave * nsteps / SS_WAVES, send = cbeg + (wave + 1) * nsteps / SS_WAVES;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = sbeg; s0 < send; s0 += SS_STEPS) {
        uint4 a[SS_STEPS], w[SS_STEPS];
#pragma unroll
        for (int i = 0; i < SS_STEPS; ++i) {
            const int k = (s0 + i) * 32 + kq;
            const int off = (s0 + i < send && k < d) ? (row * d + k) * 2 : RB_OOB;
            a[i] = rb_load16(xr, off);
            w[i] = rb_load16(wr, off);
        }
#pragma unroll
        for (int i = 0; i < SS_STEPS; ++i)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]),
                                                          __builtin_bit_cast(bf16x8, w[i]), acc,
                                                          0, 0, 0);
    }
    part[wave][lane] = acc;
    __syncthreads();
    // accumulator element i of lane L: token 4 (L / 16) + i, expert L % 16
    if (tid < 256 && r < nt && e < ne) {
        const float* p = (const float*)&part[0][(r >> 2) * 16 + e] + (r & 3);
        float sum = p[0];
#pragma unroll
        for (int v = 1; v < SS_WAVES; ++v) sum += p[v * 256];
        out[(chunk * T + t0 + r) * E + e0 + e] = chunks == 1 ? sum + b : sum;
    }
}

// fp32 gate scores on v_mfma_f32_16x16x4_f32 (fp32 operands, fp32 sums) and their
// top-k: 16 tokens per workgroup of 16 waves; the waves are dealt over the
// experts' 16-column tiles (P = their number rounded up to a power of two) and
// 16 / P K slices, so a small layer's short dot products still run on every wave.
// In a 16-wide K block a lane loads 4 consecutive K elements of its row (16 bytes
// when rows allow it) and the j-th MFMA sums element j of the four lane groups,
// A and B in the same K order; loads past the slice or past d read zero.  The
// slices' sums are added in slice order.  Bound by load latency: four blocks of
// loads are issued together.  A thread per score walking its dot product took
// 11 us at 64 tokens x 8 experts, d = 128, and 23 us at 1000 x 8, d = 256; this
// kernel 5.7 and 6.8 us.
constexpr int RF_WAVES = 16;
constexpr int RF_TOKENS = 16;
constexpr int RF_U = 4;                // K blocks of loads issued together

template <bool VEC>
__device__ __forceinline__ f32x4 route_f32_slice(const float* __restrict__ xr,
                                                 const float* __restrict__ wr, int d, int b0,
                                                 int b1, int kq) {
    auto load = [&](const float* __restrict__ p, int k) {
        f32x4 v;
        if (VEC) {
            const bool ok = k < d;
            v = *(const f32x4*)(p + (ok ? k : 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = ok ? v[j] : 0.f;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = k + j < d;
                const float e = p[ok ? k + j : 0];
                v[j] = ok ? e : 0.f;
            }
        }
        return v;
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int b = b0; b < b1; b += RF_U) {
        f32x4 xa[RF_U], wb[RF_U];
#pragma unroll
        for (int u = 0; u < RF_U; ++u) {
            const int k = b + u < b1 ? (b + u) * 16 + kq : d;
            xa[u] = load(xr, k);
            wb[u] = load(wr, k);
        }
#pragma unroll
        for (int u = 0; u < RF_U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[u][j], wb[u][j], acc, 0, 0, 0);
    }
    return acc;
}

template <int KM, int C>
__global__ __launch_bounds__(RF_WAVES * 64) void route_f32_kernel(
    const float* __restrict__ X, const float* __restrict__ W, const float* __restrict__ bias,
    int64_t T, int d, int E, int k, int renorm, int vec, float* __restrict__ logits,
    int32_t* __restrict__ idx, float* __restrict__ gate) {
    constexpr int P = 1 << C;                            // E <= 16 P
    constexpr int KS = RF_WAVES / P;                     // K slices
    constexpr int ldS = 16 * P + 1;
    __shared__ f32x4 part[RF_WAVES * 64];
    __shared__ float Sm[RF_TOKENS * ldS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * RF_TOKENS;
    const int nt = (int)((T - t0) < RF_TOKENS ? (T - t0) : RF_TOKENS);
    const int ct = wave % P, ks = wave / P;
    const int nblk = (d - 1) / 16 + 1;
    const int b0 = (int)((int64_t)ks * nblk / KS), b1 = (int)((int64_t)(ks + 1) * nblk / KS);
    if (ct * 16 < E) {
        // rows past the batch and experts past E re-read the last one (not used)
        const int r = min(lane & 15, nt - 1), e = min(ct * 16 + (lane & 15), E - 1);
        const float* xr = X + (t0 + r) * d;
        const float* wr = W + (int64_t)e * d;
        const int kq = (lane >> 4) * 4;
        part[wave * 64 + lane] = vec ? route_f32_slice<true>(xr, wr, d, b0, b1, kq)
                                     : route_f32_slice<false>(xr, wr, d, b0, b1, kq);
    }
    __syncthreads();
    // accumulator element i of lane l: token 4 (l / 16) + i, expert l % 16
    for (int c = tid; c < RF_TOKENS * E; c += RF_WAVES * 64) {
        const int r = c / E, e = c - r * E;
        const float* p = (const float*)&part[(e >> 4) * 64 + (r >> 2) * 16 + (e & 15)] + (r & 3);
        float sum = p[0];
#pragma unroll
        for (int s = 1; s < KS; ++s) sum += p[s * P * 64 * 4];
        Sm[r * ldS + e] = sum;
    }
    __syncthreads();
    finish_tokens<KM, C, 1>(Sm, ldS, nt, t0, E, k, renorm, bias, logits, idx, gate);
}

// Top-k of given scores: `tpb` tokens per workgroup of 256 threads, straight from
// global memory.
template <int KM, int C>
__global__ __launch_bounds__(ROUTE_THREADS) void topk_given_kernel(
    const float* __restrict__ scores, int64_t T, int E, int k, int renorm,
    int32_t* __restrict__ idx, float* __restrict__ gate, int tpb) {
    const int64_t t0 = (int64_t)blockIdx.x * tpb;
    const int nt = (int)((T - t0) < tpb ? (T - t0) : tpb);
    topk_tokens<KM, C>(scores + t0 * E, E, nt, t0, E, k, renorm, idx, gate);
}

// Top-k of scores in K chunks (part[chunk][T][E]): a token's chunks summed in chunk
// order, then as for scores of its own (finish_tokens).
template <int KM, int C>
__global__ __launch_bounds__(ROUTE_THREADS) void topk_chunks_kernel(
    const float* __restrict__ part, int chunks, const float* __restrict__ bias, int64_t T, int E,
    int k, int renorm, float* __restrict__ logits, int32_t* __restrict__ idx,
    float* __restrict__ gate, int tpb) {
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int ldS = ((E + 15) & ~15) + 1;
    const int64_t t0 = (int64_t)blockIdx.x * tpb;
    const int nt = (int)((T - t0) < tpb ? (T - t0) : tpb);
    for (int c = threadIdx.x; c < nt * E; c += ROUTE_THREADS) {
        const int r = c / E, e = c - r * E;
        smem[r * ldS + e] = sum_chunks(part + t0 * E + c, T * E, chunks);
    }
    __syncthreads();
    finish_tokens<KM, C>(smem, ldS, nt, t0, E, k, renorm, bias, logits, idx, gate);
}

// Token rows per workgroup of the bf16 score kernel, by expert count.
int route_rows(int E) {
    const int E_pad = (E + 15) & ~15;
    // E <= 16: 16 tokens per workgroup (the router rows are a few KB, so small
    // token blocks cost little re-reading, and a long batch then fills the chip
    // without splitting K and a second launch)
    return 16 * (E_pad <= 16 ? 1 : (E_pad <= 128 ? 2 : 1));
}

// Tokens per workgroup of topk_given_kernel: at most one pass of the top-k
// lane groups, and few enough that a short batch still spreads over >= 128
// workgroups (the top-k is latency-bound per workgroup).
int simple_tokens_per_block(int64_t T, int E) {
    const int cap = topk_tokens_per_block(E);
    const int64_t want = ceil_div(T, 128);
    return want >= cap ? cap : (want < 1 ? 1 : (int)want);
}

template <int KM, int C>
int launch_kmv(const void* x, int dtype, const void* w, const float* bias, int64_t T, int d,
              int E, int k, int flags, float* logits, int32_t* idx, float* gate, void* ws,
              hipStream_t s) {
    const int renorm = (flags & MOE_RENORM) ? 1 : 0;
    const int E_pad = (E + 15) & ~15;
    const float* given = logits;
    if (!(flags & MOE_LOGITS_IN) && dtype == MOE_F32) {
        const int vec = d % 4 == 0 && (((uintptr_t)x | (uintptr_t)w) & 15u) == 0;
        hipLaunchKernelGGL((route_f32_kernel<KM, C>), dim3((unsigned)ceil_div(T, RF_TOKENS)),
                           dim3(RF_WAVES * 64), 0, s, (const float*)x, (const float*)w, bias, T, d, E,
                           k, renorm, vec, logits, idx, gate);
        return launch_status();
    }
    if (!(flags & MOE_LOGITS_IN)) {
        const bool tiled = score_tiled(T, 2 * d, E);
        if (tiled && E <= SCORE_TOPK_MAX_E)
            return launch_score_tiles_topk(false, x, w, nullptr, nullptr, bias, T, 2 * d, E, k,
                                           renorm, logits, idx, gate, s);
        const int chunks = route_short(T, d, E) ? route_chunks(T, d, E) : 1;
        if (chunks > 1) {
            const int st = launch_scores_short(x, w, nullptr, T, d, E, (float*)ws, s);
            if (st != MOE_OK) return st;
            const int tpb = simple_tokens_per_block(T, E);
            hipLaunchKernelGGL((topk_chunks_kernel<KM, C>), dim3((unsigned)ceil_div(T, tpb)),
                               dim3(ROUTE_THREADS), (size_t)tpb * (E_pad + 1) * sizeof(float), s,
                               (const float*)ws, chunks, bias, T, E, k, renorm, logits, idx, gate, tpb);
            return launch_status();
        }
        float* out = logits ? logits : (float*)ws;
        given = out;
        if (tiled) {
            const int st = launch_score_tiles(false, x, w, nullptr, nullptr, bias, T, 2 * d, E, out, s);
            if (st != MOE_OK) return st;
        } else if (route_short(T, d, E)) {
            const int st = launch_scores_short(x, w, bias, T, d, E, out, s);
            if (st != MOE_OK) return st;
        } else {
            const int rows = route_rows(E);
            const size_t lds = (size_t)4 * rows * (E_pad + 1) * sizeof(float);
#define MOE_RB_LAUNCH(RT, NTM)                                                                  \
    do {                                                                                        \
        if (lds > 65536 && allow_dynamic_lds<route_bf16_kernel<RT, NTM, KM, C>>(lds) != MOE_OK)  \
            return MOE_ERR_DEVICE;                                                              \
        hipLaunchKernelGGL((route_bf16_kernel<RT, NTM, KM, C>),                                 \
                           dim3((unsigned)ceil_div(T, rows)), dim3(RB_THREADS), lds, s,         \
                           (const bf16_t*)x, (const bf16_t*)w, bias, T, d, E, k, renorm, logits, \
                           idx, gate);                                                          \
    } while (0)
            if constexpr (C == 0) MOE_RB_LAUNCH(1, 1);          // E <= 16
            else if constexpr (C <= 2) MOE_RB_LAUNCH(2, 4);     // E <= 64
            else if constexpr (C == 3) MOE_RB_LAUNCH(2, 8);     // E <= 128
            else MOE_RB_LAUNCH(1, 16);
#undef MOE_RB_LAUNCH
            return launch_status();
        }
    }
    const int tpb = simple_tokens_per_block(T, E);
    hipLaunchKernelGGL((topk_given_kernel<KM, C>), dim3((unsigned)ceil_div(T, tpb)),
                       dim3(ROUTE_THREADS), 0, s, given, T, E, k, renorm, idx, gate, tpb);
    return launch_status();
}

}  // namespace

// Short batches: too few token blocks for the one-launch kernel (fewer than 128), K
// long enough to be worth splitting over 8 waves, and no more rounds of 16 x 16
// workgroups over the CUs than half the expert tiles: a round takes about 7.6 us at d =
// 4096, the one-launch kernel, which reads the tokens once for all experts, 30, 41 and 46 us
// in its single round at 64, 100 and 128 experts (d = 4096, 128 experts: 2000 tokens 38.5
// against 46.4, 2500 46.3 against 46.6, 4000 66.5 against 47.2; 64 experts: 2000 23.3
// against 29.8, 3500 37.9 against 30.2).  Their scores come from score_small_kernel, the
// top-k from a launch of its own (or from the packaging launch).
bool route_short(int64_t T, int d, int E) {
    const int64_t et = ceil_div(E, 16), tiles = ceil_div(T, 16) * et;
    return T > 0 && ceil_div(T, route_rows(E)) < 128 && (d + 31) / 32 >= (E <= 16 ? 8 : 4) &&
           ceil_div(tiles, 256) <= (et + (et <= 8)) / 2 && !score_tiled(T, 2 * d, E);
}

// K chunks of a short batch's scores: past 2048 elements one per 1024 of them, as long as
// they make no more than a workgroup a CU (beyond that every CU is loading already, and the
// chunks' way through memory costs more: 300 tokens, d = 4096, 128 experts 14.8 us in one
// chunk, 16.5 in two).  moe_route_topk of 64 tokens in one chunk, chunks of 2048 and of 1024:
// d = 4096, 8 experts 10.4, 8.7 and 7.8 us; d = 14336 24.6, 9.0 and 8.9; d = 4096, 16
// experts 9.3 and 8.0 (the K chunks of one wave each that this kernel replaced: 7.9, 8.7
// and 8.0); chunks of 512 are even with 1024.
int route_chunks(int64_t T, int d, int E) {
    const int64_t tiles = ceil_div(T, 16) * ceil_div(E, 16);
    int64_t chunks = d <= 2048 ? 1 : ceil_div(d, 1024);
    if (chunks > 256 / tiles) chunks = 256 / tiles;
    if (chunks > 16) chunks = 16;
    return chunks < 1 ? 1 : (int)chunks;
}

int launch_scores_short(const void* x, const void* w, const float* bias, int64_t T, int d, int E,
                        float* out, hipStream_t s) {
    const int chunks = route_chunks(T, d, E);
    hipLaunchKernelGGL(score_small_kernel,
                       dim3((unsigned)ceil_div(E, 16), (unsigned)ceil_div(T, 16), (unsigned)chunks),
                       dim3(SS_WAVES * 64), 0, s, (const bf16_t*)x, (const bf16_t*)w, bias, T, d, E,
                       chunks, out);
    return launch_status();
}

// Scores kept for the top-k: a short batch's K chunks, or its scores and those of a tiled
// batch when the caller wants none stored.
size_t route_ws_bytes(int dtype, int64_t T, int d, int E, int flags) {
    if ((flags & MOE_LOGITS_IN) || dtype != MOE_BF16 || T <= 0) return 0;
    const size_t scores = (size_t)T * (size_t)E * sizeof(float);
    if (route_short(T, d, E)) return route_chunks(T, d, E) * scores;
    return score_tiled(T, 2 * d, E) ? scores : 0;
}

int launch_topk_given(const float* scores, int64_t T, int E, int k, int flags, int32_t* idx,
                      float* gate, hipStream_t s) {
    return launch_route_topk(nullptr, MOE_F32, nullptr, nullptr, T, 0, E, k,
                             (flags & MOE_RENORM) | MOE_LOGITS_IN, (float*)scores, idx, gate,
                             nullptr, s);
}

int launch_route_topk(const void* x, int dtype, const void* w, const float* bias, int64_t T, int d,
                      int E, int k, int flags, float* logits, int32_t* idx, float* gate, void* ws,
                      hipStream_t s) {
    if (T == 0) return MOE_OK;
#define MOE_KC(KM, C) launch_kmv<KM, C>(x, dtype, w, bias, T, d, E, k, flags, logits, idx, gate, ws, s)
#define MOE_KMV(KM)                                                                              \
    switch (topk_class(E)) {                                                                     \
        case 0: return MOE_KC(KM, 0);                                                            \
        case 1: return MOE_KC(KM, 1);                                                            \
        case 2: return MOE_KC(KM, 2);                                                            \
        case 3: return MOE_KC(KM, 3);                                                            \
        default: return MOE_KC(KM, 4);                                                           \
    }
    if (k <= 2) MOE_KMV(2);
    if (k <= 4) MOE_KMV(4);
    if (k <= 8) MOE_KMV(8);
    MOE_KMV(16);
#undef MOE_KMV
#undef MOE_KC
}

}  // namespace moe
