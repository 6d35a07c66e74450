// fp32 grouped SwiGLU FFN over ragged groups of rows (the fp32 path of
// moe_grouped_ffn), on v_mfma_f32_16x16x4_f32: fp32 operands, fp32
// accumulation.
//
// What bounds it: the layers run in fp32 are small, so first the latency of the
// operand loads, then the L2 reads.  Every wave therefore multiplies a 32-row
// tile straight from global memory, with no LDS staging and no barrier in the
// loop: in a block of 16 consecutive K a lane loads 4 consecutive K elements of
// its row (lane q = l / 16 those from 4 q, one 16-byte load), and the j-th MFMA
// of the block takes element j of every lane, i.e. sums K = 16 b + 4 q + j over
// q.  A and B use the same order, so each product sums over the same K.  The
// loads of the next two blocks are in flight while two blocks multiply.  The
// four waves of a workgroup split K of one tile (short K chains, four times the
// waves; partial sums added in wave order through LDS) unless there are enough
// tiles, when they take a 2 x 2 arrangement of tiles and share operands in L1, each
// adding the same four partial sums in the same order: an output's bits depend on
// neither the arrangement, nor the call's capacity, nor the operands' alignment.
// It replaced 16 x 16 output tiles staged through LDS and multiplied on the
// vector unit: 1000 tokens, d = 256, f = 512, 8 experts, top-2: gate/up 74 -> 30
// us, down 73 -> 19 us; 64 tokens, d = 128, f = 256: 12.7 -> 7.3 and 20.7 -> 5.9 us.
#include <type_traits>

#include "common.h"

namespace moe {
namespace {

constexpr int F_THREADS = 256;
constexpr int F_MT = 2;                  // 16-row tiles per wave
constexpr int F_U = 2;                   // 16-wide K blocks per load batch

struct F32Args {
    const float* w[MOE_MAX_GROUPS];      // per group: [2N][K] (gate rows, up rows) or [N][K]
    const float* x;                      // [rows][K], or the token rows of a_rows
    const int32_t* a_rows;               // row p of the input is x[a_rows[p]]; nullptr: x[p]
    const int32_t* offsets;              // row offsets of the groups after the first `lead`
    float* out;                          // [rows][N]
    int K, N;
    int n_groups, lead, lead_rows;
};

// Four floats at any float's address: one 16-byte load (global loads need no more than
// the element's alignment).  Rows off a 16-byte boundary and odd widths took an element a
// load before, behind the vector kernel these products replaced (1500 rows of 5 groups, d
// = 73, f = 41: that 14.6 us, so 22.2, now 9.7; 4500 rows, d = 1023, f = 513: 972, 532, 234).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// 4 consecutive K elements from k of a row, as they come and before zero_past.  The
// address is moved down so that all four lie in the row; with K < 4 (TINY), where that
// is not possible, every element has an address of its own.
template <bool TINY>
__device__ __forceinline__ f32x4 load_k4(const float* __restrict__ row, unsigned k, unsigned K) {
    f32x4 v;
    if (TINY) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = row[k + j < K ? k + j : 0];
    } else {
        v = *(const f32x4_any*)(row + min(k, K - 4));
    }
    return v;
}

// Element j of load_k4 is K element k + j, or zero from K on.
template <bool TINY>
__device__ __forceinline__ void zero_past(f32x4& v, unsigned k, unsigned K) {
    if (TINY) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = k + j < K ? v[j] : 0.f;
    } else {
        const unsigned s = k - min(k, K - 4);                // by how many the address was moved
        v[0] = s == 0 ? v[0] : s == 1 ? v[1] : s == 2 ? v[2] : s == 3 ? v[3] : 0.f;
        v[1] = s == 0 ? v[1] : s == 1 ? v[2] : s == 2 ? v[3] : 0.f;
        v[2] = s == 0 ? v[2] : s == 1 ? v[3] : 0.f;
        v[3] = s == 0 ? v[3] : 0.f;
    }
}

// NT: 16-column tiles per wave (SWIGLU: of gate and of up each).  KS: waves that
// split K of one tile (4), or 1: the waves take 2 x 2 tiles.
template <bool SWIGLU, bool TINY, int NT, int KS>
__global__ __launch_bounds__(F_THREADS, KS == 4 ? 3 : 2) void ffn_f32_kernel(F32Args args) {
    static_assert(KS == 1 || KS == 4, "wave arrangement");
    constexpr int WM = KS == 1 ? 2 : 1, WN = KS == 1 ? 2 : 1;
    constexpr int TM = 16 * F_MT * WM, TN = 16 * NT * WN;
    constexpr int NP = SWIGLU ? 2 : 1;                   // products: gate, up
    __shared__ int s_off[MOE_MAX_GROUPS + 1], s_tstart[MOE_MAX_GROUPS + 1];
    __shared__ f32x4 red[KS == 4 ? 4 * F_MT * NT * NP * 64 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_groups = args.n_groups;
    const int N = args.N;
    const unsigned K = (unsigned)args.K;
    for (int s = tid; s <= n_groups; s += F_THREADS)
        s_off[s] = s < args.lead ? s * args.lead_rows
                                 : args.lead * args.lead_rows + args.offsets[s - args.lead];
    __syncthreads();
    const int ncol = (N + TN - 1) / TN;
    if (wave == 0) {
        int carry = 0;
        for (int g0 = 0; g0 < n_groups; g0 += 64) {
            const int g = g0 + lane;
            const int rows = g < n_groups ? s_off[g + 1] - s_off[g] : 0;
            const int incl = wave_incl_scan((rows + TM - 1) / TM * ncol);
            if (g < n_groups) s_tstart[g + 1] = carry + incl;
            carry += __shfl(incl, 63, 64);
        }
        if (lane == 0) s_tstart[0] = 0;
    }
    __syncthreads();
    const int nblk = (int)((K + 15) / 16);               // K < 2^31
    auto quarter = [&](int i) { return (int)((int64_t)i * nblk / 4); };   // of K, in blocks
    const int b0 = KS == 4 ? quarter(wave) : 0, b1 = KS == 4 ? quarter(wave + 1) : nblk;
    const int wm = KS == 1 ? wave & 1 : 0, wn = KS == 1 ? wave >> 1 : 0;
    const int fr = lane & 15, kq = (lane >> 4) * 4;

    for (int tile = blockIdx.x; tile < s_tstart[n_groups]; tile += gridDim.x) {
        const int g = last_le(s_tstart, n_groups, tile);
        const int rows = s_off[g + 1] - s_off[g];
        const int mt = (rows + TM - 1) / TM;
        const int local = tile - s_tstart[g];
        const int m0 = (local % mt) * TM + wm * 16 * F_MT;   // this wave's first row and column
        const int n0 = (local / mt) * TN + wn * 16 * NT;
        // rows past the group and columns past N re-read its last one; their sums are
        // not stored
        const float* ap[F_MT];
        const float* bp[NP][NT];
#pragma unroll
        for (int i = 0; i < F_MT; ++i) {
            const int p = s_off[g] + min(m0 + i * 16 + fr, rows - 1);
            ap[i] = args.x + (int64_t)(args.a_rows ? args.a_rows[p] : p) * args.K;
        }
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                bp[q][j] = args.w[g] + ((int64_t)q * N + min(n0 + j * 16 + fr, N - 1)) * args.K;

        f32x4 acc[NP][F_MT][NT], sum[NP][F_MT][NT];      // sum: KS == 1
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int i = 0; i < F_MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[q][i][j] = sum[q][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 a[2][F_U][F_MT], b[2][F_U][NP][NT];
        unsigned kb[2][F_U];                             // a slot's blocks: their first K element
        // blocks at or past b1 count as past K: zeros, so the products need no branch
        auto load = [&](int slot, int blk) {
#pragma unroll
            for (int u = 0; u < F_U; ++u) {
                kb[slot][u] = blk + u < b1 ? (unsigned)(blk + u) * 16 : K;
                const unsigned k = kb[slot][u] + kq;
#pragma unroll
                for (int i = 0; i < F_MT; ++i) a[slot][u][i] = load_k4<TINY>(ap[i], k, K);
#pragma unroll
                for (int q = 0; q < NP; ++q)
#pragma unroll
                    for (int j = 0; j < NT; ++j) b[slot][u][q][j] = load_k4<TINY>(bp[q][j], k, K);
            }
        };
        // f(q, i, j) for every accumulator
        auto each = [&](auto f) {
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int i = 0; i < F_MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) f(q, i, j);
        };
        auto mma = [&](auto whole, int slot, int blk) {
#pragma unroll
            for (int u = 0; u < F_U; ++u) {
                if constexpr (!decltype(whole)::value) {
                    const unsigned k = kb[slot][u] + kq;
#pragma unroll
                    for (int i = 0; i < F_MT; ++i) zero_past<TINY>(a[slot][u][i], k, K);
#pragma unroll
                    for (int q = 0; q < NP; ++q)
#pragma unroll
                        for (int j = 0; j < NT; ++j) zero_past<TINY>(b[slot][u][q][j], k, K);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    each([&](int q, int i, int j) {
                        acc[q][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            a[slot][u][i][e], b[slot][u][q][j][e], acc[q][i][j], 0, 0, 0);
                    });
                // whole K in one wave: the sums of the quarters that four waves would take,
                // added in the same order, so the sums are the same bits either way
                if constexpr (KS == 1) {
                    const int done = blk + u + 1;
                    if (done == quarter(1) || done == quarter(2) || done == quarter(3))
                        each([&](int q, int i, int j) {
                            sum[q][i][j] += acc[q][i][j];
                            acc[q][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                        });
                }
            }
        };
        // turns of blocks that all lie in the rows, then the last ones a batch at a time, so
        // that a short K loads and multiplies no batch for its zeros (12000 rows, d = 128, f
        // = 256: 81 -> 57 us)
        const int full = min(b1, (int)(K / 16));
        int blk = b0;
        load(0, b0);
        if constexpr (!TINY)
            for (; blk + 2 * F_U <= full; blk += 2 * F_U) {
                load(1, blk + F_U);
                mma(std::true_type{}, 0, blk);
                load(0, blk + 2 * F_U);
                mma(std::true_type{}, 1, blk + F_U);
            }
        for (; blk < b1; blk += F_U) {
            mma(std::false_type{}, 0, blk);
            if (blk + F_U < b1) load(0, blk + F_U);
        }
        if constexpr (KS == 1)
            each([&](int q, int i, int j) { acc[q][i][j] = sum[q][i][j] + acc[q][i][j]; });

        // accumulator element r of lane l: row 4 (l / 16) + r, column l % 16
        auto store = [&](int i, int j, const f32x4& x, const f32x4& y) {
            const int col = n0 + j * 16 + fr;
            if (col >= N) return;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + i * 16 + (lane >> 4) * 4 + r;
                const float v = SWIGLU ? x[r] / (1.0f + expf(-x[r])) * y[r] : x[r];
                if (row < rows) args.out[(int64_t)(s_off[g] + row) * N + col] = v;
            }
        };
        if constexpr (KS == 4) {
            constexpr int TILES = F_MT * NT;
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int i = 0; i < F_MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        red[((wave * NP + q) * TILES + i * NT + j) * 64 + lane] = acc[q][i][j];
            __syncthreads();
            if (wave < TILES) {
                f32x4 s[NP];
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    s[q] = red[(q * TILES + wave) * 64 + lane];
#pragma unroll
                    for (int w = 1; w < 4; ++w) s[q] += red[((w * NP + q) * TILES + wave) * 64 + lane];
                }
                store(wave / NT, wave % NT, s[0], s[NP - 1]);
            }
            __syncthreads();                             // red is reused by the next tile
        } else {
#pragma unroll
            for (int i = 0; i < F_MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) store(i, j, acc[0][i][j], acc[NP - 1][i][j]);
        }
    }
}

template <bool SWIGLU>
int launch_product(const F32Args& a, int64_t cap_rows, int cus, hipStream_t s) {
    // tiles of a TM-row, TN-column split: at most cap_rows / TM + n_groups row tiles
    auto tiles = [&](int TM, int TN) {
        return (cap_rows / TM + a.n_groups) * ceil_div(a.N, TN);
    };
    auto grid = [&](int64_t n) { return dim3((unsigned)(n < 16 * cus ? n : 16 * cus)); };
    // 64 x 64 tiles of whole-K waves when there are at least four of them per CU;
    // below that K is split over the waves, and with fewer than two 32 x 32 tiles
    // per CU the tile is 16 columns wide (twice the workgroups)
    const int64_t t64 = tiles(64, 64), t32 = tiles(32, 32);
    if (a.K < 4)
        hipLaunchKernelGGL((ffn_f32_kernel<SWIGLU, true, 2, 4>), grid(t32), dim3(F_THREADS), 0, s, a);
    else if (t64 >= 4 * cus)
        hipLaunchKernelGGL((ffn_f32_kernel<SWIGLU, false, 2, 1>), grid(t64), dim3(F_THREADS), 0, s, a);
    else if (t32 >= 2 * cus)
        hipLaunchKernelGGL((ffn_f32_kernel<SWIGLU, false, 2, 4>), grid(t32), dim3(F_THREADS), 0, s, a);
    else
        hipLaunchKernelGGL((ffn_f32_kernel<SWIGLU, false, 1, 4>), grid(tiles(32, 16)), dim3(F_THREADS),
                           0, s, a);
    return launch_status();
}

}  // namespace

// h = SiLU(x W1^T) * (x W3^T) into ws ([cap_rows][f]), then y = h W2^T.
int launch_ffn_f32(const float* x, const int32_t* offsets, int n_groups, const void* const* w13,
                   const void* const* w2, int d, int f, int64_t cap_rows, float* y, float* h,
                   const int32_t* a_rows, int products, int lead, int lead_rows, int cus,
                   hipStream_t s) {
    F32Args a;
    a.offsets = offsets;
    a.n_groups = n_groups;
    a.lead = lead;
    a.lead_rows = lead_rows;
    if (products & MOE_FFN_GATE_UP) {
        for (int i = 0; i < MOE_MAX_GROUPS; ++i)
            a.w[i] = i < n_groups ? (const float*)w13[i] : nullptr;
        a.x = x;
        a.a_rows = a_rows;
        a.out = h;
        a.K = d;
        a.N = f;
        const int st = launch_product<true>(a, cap_rows, cus, s);
        if (st != MOE_OK) return st;
    }
    if (products & MOE_FFN_DOWN) {
        for (int i = 0; i < MOE_MAX_GROUPS; ++i)
            a.w[i] = i < n_groups ? (const float*)w2[i] : nullptr;
        a.x = h;
        a.a_rows = nullptr;
        a.out = y;
        a.K = f;
        a.N = d;
        const int st = launch_product<false>(a, cap_rows, cus, s);
        if (st != MOE_OK) return st;
    }
    return MOE_OK;
}

}  // namespace moe
