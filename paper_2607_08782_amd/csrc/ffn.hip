// Grouped SwiGLU expert FFN over ragged groups of rows (Sec. II-A of the
// Director paper: each expert is an FFN sub-network; Eq. 2 prices this step
// as the per-GPU compute latency f_comp of the rows a GPU receives).
//
// bf16 path, two products, each "NT": every operand row is contiguous along K, so
// global loads and MFMA fragment reads are all 16-byte vectors.
//   1. H = SiLU(X W1^T) * (X W3^T)   gate and up rows side by side in one weight
//                                     tile, fused epilogue
//   2. Y = H W2^T
// Groups of many rows run as 256 x 256 tiles of a persistent grid
// (grouped_gemm_kernel: bound by the matrix rate under the board's power limit).
// A short call's groups of up to 256 rows stream their weights instead (bound by
// latency and the weight reads): as strips that walk all of K (strip_gemm_kernel),
// or, where K is long, split over workgroups (stream_gemm_kernel) and summed in
// chunk order (split_reduce_kernel, which also sums the tiled kernel's split
// tiles).  Which groups stream is decided on the device from the group sizes
// (small_limits), which form streams on the host (strip_product).  All use
// v_mfma_f32_16x16x32_bf16 but the split kernel (32x32x16): under sustained load
// the part runs at its board power limit, so the clock follows the energy per
// flop, and 16x16x32 moves half the accumulator bytes per flop.  Work is cut into
// eight contiguous chunks, one per XCD (workgroups are dispatched round-robin
// over the XCDs), so the workgroups sharing an L2 also share weights.  Group
// sizes are read on the device; empty groups produce no tiles, so their weights
// are never read.
#include <type_traits>

#include "common.h"

namespace moe {
namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = 256;          // rows per tile
constexpr int BNW = 256;         // weight rows per tile
constexpr int BK = 64;           // K granularity of a tile's range
constexpr int LDK = BK + 8;      // streaming kernel: LDS row stride in elements (144 B)
constexpr int WAVES_M = 2, WAVES_N = 2;
constexpr int GEMM_THREADS = WAVES_M * WAVES_N * 64;
constexpr int MS = BM / WAVES_M / 16;              // 16-row accumulator tiles per wave
constexpr int NS = BNW / WAVES_N / 16;             // 16-column accumulator tiles per wave
// ring of K stages in LDS, filled by direct loads
constexpr int SK = 32;                             // K per stage: 64-byte LDS rows
constexpr int ROWB = SK * 2;
constexpr int RING = 4;
constexpr int A_BYTES = BM * ROWB, STAGE_BYTES = (BM + BNW) * ROWB;
constexpr int RING_BYTES = RING * STAGE_BYTES;     // 128 KB
constexpr int A_LOADS = A_BYTES / 1024 / 4;        // 1 KB direct loads per wave per stage
constexpr int B_LOADS = BNW * ROWB / 1024 / 4;
constexpr int LOADS = A_LOADS + B_LOADS;
constexpr int TILE_LIST = 256;                     // tiles of a workgroup listed at a time
constexpr int NUM_XCD = 8;
constexpr uint32_t RSRC_WORD3 = 0x00020000;        // raw buffer: 32-bit data format
constexpr int A_OOB = 0x7fffff00;                  // offset past any descriptor: reads zero

typedef __attribute__((address_space(3))) void lds_void;

// wait until at most N of this wave's vector-memory operations are outstanding
// (they complete in issue order); no memory access moves across it
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// First row of group g.  The first `lead` groups hold lead_rows rows each (the
// shared experts' groups of moe_grouped_ffn_rows_shared, every token once); the
// offsets array gives the row ranges of the groups after them, counted from
// row lead * lead_rows, as moe_permute writes them.
__device__ __forceinline__ int group_start(const int32_t* offsets, int lead, int lead_rows, int g) {
    return g < lead ? g * lead_rows : lead * lead_rows + offsets[g - lead];
}

struct GemmArgs {
    const bf16_t* w[MOE_MAX_GROUPS];   // per-group weight matrix, rows contiguous along K
    const int32_t* offsets;            // [n_groups - lead + 1] row offsets (device), see group_start
    const bf16_t* a;                   // [rows][K]
    bf16_t* out;                       // [rows][ldo]
    int n_groups;                      // lead groups included
    int lead, lead_rows;               // leading groups of lead_rows rows each (group_start)
    int K;                             // contraction length
    int N;                             // output columns per group (f for SWIGLU, d for PLAIN)
    int ldo;
    int up_row;                        // SWIGLU: first row of W3 inside w[s] (= f)
    int n_tiles;                       // output-column tiles per group
    int* limits;                       // [2] row limits of the streamed groups of the gate/up and
                                       // the down product (small_limits): the gate/up launch
                                       // writes both, later launches read theirs; nullptr: the
                                       // limit is lim0
    int product;                       // 0 gate/up, 1 down
    int lim0;                          // row limit of streamed groups when limits is nullptr
    int down_tiles;                    // gate/up launch: the down product's column tiles
    float* part;                       // fp32 partial tiles for split K (nullptr: never split)
    int* split_info;                   // the kernel records its split factor here for the reduce
    int split_units;                   // workgroups split K aims to occupy (<= TILE_SPLIT_UNITS)
    const int32_t* a_rows;             // gather: row p of A is a[a_rows[p]] (a holds a_total rows)
    int a_total;
};

// With fewer tiles than half the workgroups (mid-sized groups: a few 256-row
// tiles, long K), each tile's K range may be cut into S chunks of at least
// TILE_SPLIT_MIN_STEPS stages; every (tile, chunk) unit writes an fp32 partial
// tile and split_reduce_kernel sums the chunks in order and applies the epilogue.
// S minimises (rounds of units) x (K stages per unit) plus the partial-tile
// round trip, about 1/20 of a stage per unit (256 KB written and read back).
constexpr int TILE_SPLIT_UNITS = 256;
constexpr int TILE_SPLIT_MIN_STEPS = 8;

// A short call none of whose groups holds more than SMALL_ROWS_MAX rows streams every
// group (see small_limits, which decides for each product); any other call tiles every
// group, but for some with a long K, which stream those of up to SMALL_ROWS_MAX rows.
// Without the row limits in the workspace (a call of at most SMALL_ROWS rows in all)
// every group is streamed.
constexpr int SMALL_ROWS = 64;
constexpr int SMALL_ROWS_MAX = 256;

__host__ __device__ __forceinline__ int tile_split(int total, int KT, int split_units) {
    if (total <= 0 || 2 * total > split_units) return 1;
    const int smax = min(split_units / total, KT / TILE_SPLIT_MIN_STEPS);
    int best = 1;
    int64_t best_cost = 20 * (int64_t)KT;
    for (int S = 2; S <= smax; ++S) {
        const int64_t rounds = ((int64_t)total * S + split_units - 1) / split_units;
        const int64_t cost = 20 * rounds * ((KT + S - 1) / S) + (int64_t)S * total;
        if (cost < best_cost) { best_cost = cost; best = S; }
    }
    return best;
}

// Which tiles split: with few tiles all of them; otherwise only the tiles of a
// last round that would fill at most half the workgroups (the round every
// other workgroup waits for).  Tiles [0, head) run whole; tiles
// [head, head + tail) run as S chunks each.
struct SplitPlan {
    int head, tail, S;
};

__host__ __device__ __forceinline__ SplitPlan split_plan(int total, int KT, int split_units) {
    SplitPlan p = {total, 0, 1};
    if (total <= 0) return p;
    const int rounds = total / split_units;
    const int rest = total - rounds * split_units;
    const int S = tile_split(rest, KT, split_units);
    if (S > 1) {
        p.head = total - rest;
        p.tail = rest;
        p.S = S;
    }
    return p;
}

__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// s_tstart[g] = tiles of the groups before g, for g = 0..n_groups (a group of
// more than small_rows rows has ceil(rows / BM) * n_tiles tiles, others none);
// run by one whole wave.
__device__ __forceinline__ void tile_starts(const int* s_off, int n_groups, int small_rows,
                                            int n_tiles, int* s_tstart, int lane) {
    int carry = 0;
    for (int g0 = 0; g0 < n_groups; g0 += 64) {
        const int g = g0 + lane;
        const int rows = g < n_groups ? s_off[g + 1] - s_off[g] : 0;
        const int v = rows > small_rows ? (int)ceil_div(rows, BM) * n_tiles : 0;
        const int incl = wave_incl_scan(v);
        if (g < n_groups) s_tstart[g + 1] = carry + incl;
        carry += __shfl(incl, 63, 64);
    }
    if (lane == 0) s_tstart[0] = 0;
}

// Tile `local` of a group of mt x n_tiles tiles: the row tiles in blocks of at most
// 8 (of equal size, give or take one), each block running through all column tiles,
// rows first.  The 32 tiles an XCD works on at once then span about 8 row and 4
// column slabs of operands, whatever the group's height (rows first over a whole
// group of 32 row tiles, they span 32 + 1: an 8192-row expert's gate/up product at
// d = f = 2048 x 2816 fetched twice the bytes).
struct TilePos {
    int m, n;
};

__device__ __forceinline__ TilePos tile_pos(int local, int mt, int n_tiles) {
    const int nb = (mt + 7) >> 3;
    const int base = mt / nb, extra = mt - base * nb;      // the first `extra` blocks have one more
    const int big = extra * (base + 1) * n_tiles;
    TilePos p;
    if (local < big) {
        const int b = local / ((base + 1) * n_tiles), l = local - b * (base + 1) * n_tiles;
        p.n = l / (base + 1);
        p.m = b * (base + 1) + l - p.n * (base + 1);
    } else {
        const int l0 = local - big, b = l0 / (base * n_tiles), l = l0 - b * base * n_tiles;
        p.n = l / base;
        p.m = extra * (base + 1) + b * base + l - p.n * base;
    }
    return p;
}

// Row limits of the streamed groups of the two products, run by one whole wave.
// When the groups above SMALL_ROWS rows make so few tiles (a quarter of the
// split units or fewer) that the tiled kernel would split K over them, its
// launch is short and latency-bound: every workgroup still runs several K
// stages of a 256 x 256 tile, on a fraction of the CUs.  Streaming every group
// of up to SMALL_ROWS_MAX rows instead spreads the weight reads over all CUs
// (a DeepSeek-V2-Lite-shaped decode step: 219 -> 188 us).  As a rule only when no
// group is larger still: a call that tiles one group anyway tiles them all, in one
// launch's rounds instead of two launches (777 tokens of the Mixtral shape, groups
// of about 500 and 120 rows: step 344 -> 325 us).  Not where all of the groups
// make too many tiles to split K over (more than half the units) and K is past
// MIXED_MIN_K: whole tiles then walk all of a long K in a round or two, and the
// streamed groups beside split tiles of the large ones are ahead (FFN, one group of
// 500 rows and small ones, all tiled against both: 8 groups at d = 4096, f = 14336 805
// and 700 us, 16 at d = 12288, f = 1024 446 and 361, 32 at d = 1024, f = 10240 583 and
// 510), by less the shorter K is (the second launch and its chunk sum cost about 20 us
// at any K): 8 groups at d = 5120, f = 8256 616 and 603, and 514 and 524 with 300 rows;
// 16 at d = 5120, f = 1536 250 and 255, and 215 and 226.  Otherwise the small
// groups join the tiled launch, whose rounds leave CUs free for their tiles,
// rather than stream in a launch of their own after it (the two run one after
// the other): DeepSeek-V2-Lite prefill FFN 364 -> 332 us, Qwen1.5 batch 137 ->
// 129 us, Qwen3 prefill 466 -> 459 us.
constexpr int MIXED_MIN_K = 8192;

__device__ __forceinline__ void small_limits(const int* s_off, int n_groups, int tiles_up,
                                             int tiles_down, int k_up, int k_down,
                                             int split_units, int lane, int& lim_up,
                                             int& lim_down) {
    int mt = 0;                                      // 256-row tiles of the groups > SMALL_ROWS
    int all = 0;                                     // of every group
    int most = 0;
    for (int g0 = 0; g0 < n_groups; g0 += 64) {
        const int g = g0 + lane;
        const int rows = g < n_groups ? s_off[g + 1] - s_off[g] : 0;
        mt += rows > SMALL_ROWS ? (int)ceil_div(rows, BM) : 0;
        all += (int)ceil_div(rows, BM);
        most = max(most, rows);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mt += __shfl_xor(mt, o, 64);
        all += __shfl_xor(all, o, 64);
        most = max(most, __shfl_xor(most, o, 64));
    }
    auto limit = [&](int tiles, int k) {
        const bool mixed = k > MIXED_MIN_K && 2 * all * tiles > split_units;
        return (most <= SMALL_ROWS_MAX || mixed) && 4 * mt * tiles <= split_units ? SMALL_ROWS_MAX : 0;
    };
    lim_up = limit(tiles_up, k_up);
    lim_down = limit(tiles_down, k_down);
}

// Persistent grouped NT GEMM: 4 waves (2 x 2), one per SIMD, each a 128 x 128
// tile of the 256 x 256 macro tile (the fewest LDS bytes per flop that the
// accumulators allow: 128 KB of fragment reads per 64 K against 192 KB for eight
// 64 x 128 wave tiles).  Both operands go straight from global memory into a ring
// of four 32-wide K stages (no staging registers, no LDS store instructions),
// three stages in flight: a stage's loads have three stages of MFMAs to arrive.
// One barrier per stage: at the barrier of stage t every wave holds its fragments
// of stage t in registers, so stage t's buffer is free for stage t + 4, and stage
// t + 1 has landed, so its fragments are read during stage t's MFMAs.  The stages
// of a workgroup's tiles form one stream: a tile's last four stages load the next
// tile's first four, and its first fragments are in registers before the epilogue.
// LDS rows are 64 bytes; 16-byte chunk c of row r sits at c ^ ((r >> 1) & 3)
// (conflict-free for the 16-row fragment reads).
// The weights are the MFMA's A operand, the token rows its B operand, so a lane
// holds 4 consecutive output columns of one row per accumulator tile; the weight
// rows of a 32-row block are laid out in LDS in the order that makes two tiles'
// columns 8 consecutive ones (w_order), stored as one 16-byte vector.
// GATHER: row p of A is row a_rows[p] of args.a (the token rows themselves, so
// the packaged copy of them is never materialised).
struct TileRec {
    int g, row0, rows_valid, n0, kt0, nsteps, u, split;   // kt0, nsteps in stages
};

// weight row, within its 32-row block, of LDS row r: MFMA tile (r >> 4) & 1, row
// i = r & 15 holds output column 8 (i >> 2) + 4 tile + (i & 3)
__device__ __forceinline__ int w_order(int r) {
    return (r & ~31) + 8 * ((r >> 2) & 3) + 4 * ((r >> 4) & 1) + (r & 3);
}

// d += w x^T on v_mfma_f32_16x16x32_bf16 with d in AGPRs or in VGPRs, and the same
// placement for a value between MFMAs (the register constraints exist in the device
// pass only, so these and the kernel's body are compiled there alone)
#ifdef __HIP_DEVICE_COMPILE__
__device__ __forceinline__ void mfma_agpr(f32x4& d, const bf16x8& w, const bf16x8& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(w), "v"(x));
}
__device__ __forceinline__ void mfma_vgpr(f32x4& d, const bf16x8& w, const bf16x8& x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(w), "v"(x));
}
__device__ __forceinline__ void pin_agpr(f32x4& d) { asm volatile("" : "+a"(d)); }
__device__ __forceinline__ void pin_vgpr(f32x4& d) { asm volatile("" : "+v"(d)); }
__device__ __forceinline__ void opaque(int& x) { asm volatile("" : "+v"(x)); }
#endif

template <bool SWIGLU, bool GATHER = false>
__global__ __launch_bounds__(GEMM_THREADS, 1) void grouped_gemm_kernel(GemmArgs args) {
#ifdef __HIP_DEVICE_COMPILE__
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    __shared__ int s_off[MOE_MAX_GROUPS + 1];
    __shared__ int s_tstart[MOE_MAX_GROUPS + 1];
    __shared__ TileRec s_tile[TILE_LIST];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int n_groups = args.n_groups;
    constexpr int BN_OUT = SWIGLU ? BNW / 2 : BNW;      // output columns per tile

    // the down launch reads its row limit from the gate/up launch (no group can
    // exceed SMALL_ROWS when there is nowhere to keep it)
    int lim = args.limits != nullptr && args.product == 1 ? args.limits[1] : args.lim0;
    for (int s = tid; s <= n_groups; s += GEMM_THREADS)
        s_off[s] = group_start(args.offsets, args.lead, args.lead_rows, s);
    __syncthreads();
    if (wave == 0) {
        if (args.limits != nullptr && args.product == 0) {
            int lim_down;
            // the gate/up product's N is the down product's K
            small_limits(s_off, n_groups, args.n_tiles, args.down_tiles, args.K, args.N,
                         args.split_units, lane, lim, lim_down);
            if (blockIdx.x == 0 && lane == 0) {
                args.limits[0] = lim;
                args.limits[1] = lim_down;
            }
        }
        tile_starts(s_off, n_groups, lim, args.n_tiles, s_tstart, lane);
    }
    __syncthreads();
    const int KT = args.K / BK;
    const int K = args.K;
    const int total_tiles = s_tstart[n_groups];
    SplitPlan plan = {total_tiles, 0, 1};
    if (args.part != nullptr) plan = split_plan(total_tiles, KT, args.split_units);
    if (args.part != nullptr && blockIdx.x == 0 && tid == 0) *args.split_info = plan.S;
    // each XCD takes a contiguous chunk of the whole tiles and a contiguous
    // chunk of the split units, so every XCD carries the same share of both
    const int nper = gridDim.x / NUM_XCD;
    const int xcd = blockIdx.x % NUM_XCD;
    const int widx = blockIdx.x / NUM_XCD;
    const int hchunk = (plan.head + NUM_XCD - 1) / NUM_XCD;
    const int h_begin = min(xcd * hchunk, plan.head), h_end = min(h_begin + hchunk, plan.head);
    const int n_units = plan.tail * plan.S;
    const int uchunk = (n_units + NUM_XCD - 1) / NUM_XCD;
    const int s_begin = min(xcd * uchunk, n_units), s_end = min(s_begin + uchunk, n_units);
    const int n_head = h_end - h_begin, n_mine = n_head + (s_end - s_begin);
    if (widx >= n_mine) return;
    const int n_list = (n_mine - widx + nper - 1) / nper;   // this workgroup's tiles

    // Tile q of this workgroup: a whole tile, or unit u = (split tile, K chunk).
    // Each thread works out one of the next TILE_LIST, so a tile's start costs one
    // LDS read instead of a search over the groups.
    auto list_tiles = [&](int q0) {
        const int q = q0 + tid;
        if (tid < TILE_LIST && q < n_list) {
            const int i = widx + q * nper;
            TileRec c;
            const bool split = i >= n_head;
            const int u = split ? s_begin + (i - n_head) : 0;
            const int L = split ? plan.head + u / plan.S : h_begin + i;
            const int S = split ? plan.S : 1;
            const int kchunk = split ? u - (u / plan.S) * plan.S : 0;
            const int kt0 = (int)((int64_t)kchunk * KT / S);
            const int s = last_le(s_tstart, n_groups, L);
            const int mt = (int)ceil_div(s_off[s + 1] - s_off[s], BM);
            const TilePos pos = tile_pos(L - s_tstart[s], mt, args.n_tiles);
            const int nt = pos.n;
            c.g = s;
            c.row0 = s_off[s] + pos.m * BM;
            c.rows_valid = min(BM, s_off[s + 1] - c.row0);
            c.n0 = nt * BN_OUT;
            c.kt0 = kt0 * (BK / SK);
            c.nsteps = ((int)((int64_t)(kchunk + 1) * KT / S) - kt0) * (BK / SK);
            c.u = u;
            c.split = split ? 1 : 0;
            s_tile[tid] = c;
        }
    };
    auto tile_at = [&](int q) {
        TileRec c = s_tile[q % TILE_LIST];
        c.g = __builtin_amdgcn_readfirstlane(c.g);
        c.row0 = __builtin_amdgcn_readfirstlane(c.row0);
        c.rows_valid = __builtin_amdgcn_readfirstlane(c.rows_valid);
        c.n0 = __builtin_amdgcn_readfirstlane(c.n0);
        c.kt0 = __builtin_amdgcn_readfirstlane(c.kt0);
        c.nsteps = __builtin_amdgcn_readfirstlane(c.nsteps);
        c.u = __builtin_amdgcn_readfirstlane(c.u);
        c.split = __builtin_amdgcn_readfirstlane(c.split);
        return c;
    };
    // operand descriptors of a tile: rows past the group's end or past the output
    // columns fall outside them (their products are not stored); gate and up halves
    // of a SwiGLU weight tile.  live = false: empty ranges, loads without traffic
    struct Rsrc {
        __amdgpu_buffer_rsrc_t a, lo, hi;
    };
    auto rsrc_of = [&](const TileRec& c, bool live) {
        Rsrc r;
        r.a = GATHER ? __builtin_amdgcn_make_buffer_rsrc((void*)args.a, (short)0,
                                                         live ? args.a_total * K * 2 : 0, RSRC_WORD3)
                     : __builtin_amdgcn_make_buffer_rsrc((void*)(args.a + (int64_t)c.row0 * K),
                                                         (short)0, live ? c.rows_valid * K * 2 : 0,
                                                         RSRC_WORD3);
        const bf16_t* __restrict__ W = args.w[c.g];
        const int bvalid = live ? min(BN_OUT, args.N - c.n0) : 0;
        const int bup = SWIGLU ? args.up_row + c.n0 : c.n0;
        r.lo = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (int64_t)c.n0 * K), (short)0,
                                                 bvalid * K * 2, RSRC_WORD3);
        r.hi = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (int64_t)bup * K), (short)0,
                                                 bvalid * K * 2, RSRC_WORD3);
        return r;
    };
    // load i of a wave fills LDS rows 64 i + 16 wave + (lane / 4) of A or B, chunk
    // slot lane % 4
    const int lrow = 16 * wave + (lane >> 2);
    const int kc = (((lane & 3) ^ ((lane >> 3) & 3)) * 8);
    const int avoff = (lrow * K + kc) * 2;
    const int bvoff = (w_order(lrow) * K + kc) * 2;
    const int vstep = 64 * K * 2;
    // GATHER: the token rows of a tile's loads (-1: past the group), and their offsets
    auto a_tokens = [&](const TileRec& c, int* tok) {
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i) {
            const int rin = lrow + 64 * i;
            tok[i] = GATHER && rin < c.rows_valid ? args.a_rows[c.row0 + rin] : -1;
        }
    };
    auto a_offsets = [&](const int* tok, int* av) {
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i)
            av[i] = !GATHER ? avoff + i * vstep : tok[i] >= 0 ? (tok[i] * K + kc) * 2 : A_OOB;
    };
    // direct load i of a wave's share of stage kt (A's loads, then B's)
    auto load1 = [&](const Rsrc& r, const int* av, int kt, int slot, int i) {
        char* base = ring + slot * STAGE_BYTES + wave * 1024 + i * 4096;
        if (i < A_LOADS) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r.a, (lds_void*)base, 16, av[i], kt * ROWB, 0, 0);
        } else {
            const int b = i - A_LOADS;
            const bool up = SWIGLU && b >= B_LOADS / 2;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(up ? r.hi : r.lo, (lds_void*)base, 16,
                                                     bvoff + (up ? b - B_LOADS / 2 : b) * vstep,
                                                     kt * ROWB, 0, 0);
        }
    };

    f32x4 acc[MS][NS];
    // v_mfma_f32_16x16x32_bf16 fragments: lane l holds row l % 16 of a 16-row block
    // and the 8 K elements 8 (l / 16) .. of the stage, for both operands alike
    const int frow = lane & 15;
    const int fchunk = ((lane >> 4) ^ ((frow >> 1) & 3)) * 16;
    const int a_frag = (wm * (BM / WAVES_M) + frow) * ROWB + fchunk;
    // SwiGLU tiles hold 128 gate rows then the matching 128 up rows; a wave takes the
    // same columns from both halves, so gate and up meet in its registers
    const int b_frag = A_BYTES + (wn * (SWIGLU ? BNW / 2 / WAVES_N : BNW / WAVES_N) + frow) * ROWB +
                       fchunk;
    auto b_tile = [](int j) { return SWIGLU && j >= NS / 2 ? BNW / 2 + (j - NS / 2) * 16 : j * 16; };
    // MFMA u of a stage.  The accumulators of row blocks 0..6 are pinned to 224 AGPRs,
    // those of the last block to VGPRs (filling all 256 AGPRs left the register
    // allocator moving some in and out of VGPRs in every stage, and so did the
    // compiler's own choice)
    auto mfma = [&](int u, const bf16x8* fa, const bf16x8* fb) {
        const int m = u / NS, j = u % NS;
        if (m < MS - 1) mfma_agpr(acc[m][j], fb[j], fa[m]);
        else mfma_vgpr(acc[m][j], fb[j], fa[m]);
    };
    // accumulators cross between MFMAs and other instructions only behind enough idle
    // cycles (the compiler does not see the MFMAs inside the assembly): settle() before
    // or after all MFMAs, then use(m) where row block m is first set or read (it also
    // keeps the compiler from copying all accumulators out at once)
    auto settle = []() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); };
    auto use = [&](int m) {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            if (m < MS - 1) pin_agpr(acc[m][j]);
            else pin_vgpr(acc[m][j]);
        }
    };
    constexpr int STORES = SWIGLU ? MS * NS / 4 : MS * NS / 2;   // 16-byte stores of an epilogue
    unsigned c = 0;                              // stages run so far: stage slot c % RING
    struct Source {                              // what the stages of a tile load
        Rsrc own, next;
        int av[A_LOADS], an[A_LOADS];
        int kt_own, kt_next, own_end;            // stage t loads own K stage kt_own + t below
    };                                           // own_end, then next's kt_next + t
    // one stage: multiply the fragments fa, fb (stage t), read those of stage t + 1
    // into na, nb, load stage t + 4 (past the tile's end: of the next tile).  WAIT:
    // what may be outstanding once stage t + 1 has landed: the loads of the two stages
    // after it, and in the first three stages of a tile the last epilogue's stores
    auto stage = [&](auto wait, int t, const bf16x8* fa, const bf16x8* fb, bf16x8* na, bf16x8* nb,
                     const Source& src) {
        wait_vm<decltype(wait)::value>();
        // this wave's fragment reads of stage t are done
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const unsigned slot = c % RING;
        ++c;
        const char* st = ring + (c % RING) * STAGE_BYTES;
        // issue order, fixed: one fragment read of the next stage before every three
        // MFMAs (the reads are back well before the next barrier waits for them), a
        // load before every six, each with the selection of its descriptor
        const bool own = t < src.own_end;
        const int kt = t + (own ? src.kt_own : src.kt_next);
        Rsrc r;
#pragma unroll
        for (int i = 0; i < MS + NS; ++i) {
            if (i < NS) nb[i] = *(const bf16x8*)(st + b_frag + b_tile(i) * ROWB);
            else na[i - NS] = *(const bf16x8*)(st + a_frag + (i - NS) * 16 * ROWB);
            if (i == 1) r.a = own ? src.own.a : src.next.a;
            if (i == 2 * A_LOADS + 1) r.lo = own ? src.own.lo : src.next.lo;
            if (i == 2 * A_LOADS + B_LOADS + 1) r.hi = own ? src.own.hi : src.next.hi;
            if (i & 1) {
                const int q = i >> 1;
                int av[A_LOADS];
                if (q < A_LOADS) av[q] = !GATHER || own ? src.av[q] : src.an[q];
                load1(r, av, kt, slot, q);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 3 * i; u < 3 * i + 3; ++u) mfma(u, fa, fb);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 3 * (MS + NS); u < MS * NS; ++u) mfma(u, fa, fb);
    };

    list_tiles(0);
    __syncthreads();
    // with fewer than four stages a tile (K = 64) cannot hold the next tile's loads:
    // every tile then starts its own ring
    const bool chain = KT * (BK / SK) >= RING;
    bf16x8 fa0[MS], fa1[MS], fb0[NS], fb1[NS];
    int q = 0;
    TileRec cur = tile_at(0);
    Rsrc rc = rsrc_of(cur, true);
    int avc[A_LOADS], tok[A_LOADS];
    a_tokens(cur, tok);
    a_offsets(tok, avc);
    bool start = true;
    for (;;) {
        if (start) {
#pragma unroll
            for (int s = 0; s < RING; ++s)
#pragma unroll
                for (int i = 0; i < LOADS; ++i)
                    load1(rc, avc, cur.kt0 + min(s, cur.nsteps - 1), (c + s) % RING, i);
            // all four have landed: the first stages' waits allow for more
            wait_vm<0>();
            asm volatile("s_barrier" ::: "memory");
            const char* st = ring + (c % RING) * STAGE_BYTES;
#pragma unroll
            for (int j = 0; j < NS; ++j) fb0[j] = *(const bf16x8*)(st + b_frag + b_tile(j) * ROWB);
#pragma unroll
            for (int m = 0; m < MS; ++m) fa0[m] = *(const bf16x8*)(st + a_frag + m * 16 * ROWB);
        }
        const int qn = q + 1;
        const bool has_next = qn < n_list;
        if (has_next && qn % TILE_LIST == 0) {
            __syncthreads();
            list_tiles(qn);
            __syncthreads();
        }
        const TileRec nxt = has_next ? tile_at(qn) : cur;
        a_tokens(nxt, tok);                      // used by the last stages' loads
        const int nsteps = cur.nsteps;
#pragma unroll
        for (int m = 0; m < MS; ++m)
#pragma unroll
            for (int j = 0; j < NS; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < MS; ++m) use(m);
        settle();

        Source src;
        src.own = rc;
        src.next = rsrc_of(nxt, has_next && chain);
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i) src.av[i] = avc[i];
        a_offsets(tok, src.an);
        src.own_end = nsteps - RING;
        src.kt_own = cur.kt0 + RING;
        src.kt_next = nxt.kt0 - src.own_end;
        constexpr std::integral_constant<int, 2 * LOADS> loads{};
        constexpr std::integral_constant<int, 2 * LOADS + STORES> loads_stores{};
        stage(loads_stores, 0, fa0, fb0, fa1, fb1, src);
        stage(loads_stores, 1, fa1, fb1, fa0, fb0, src);
        if (nsteps > 2) {
            stage(loads_stores, 2, fa0, fb0, fa1, fb1, src);
            stage(loads, 3, fa1, fb1, fa0, fb0, src);
        }
        for (int t = 4; t < nsteps; t += 2) {
            stage(loads, t, fa0, fb0, fa1, fb1, src);
            stage(loads, t + 1, fa1, fb1, fa0, fb0, src);
        }
        settle();
        rc = src.next;
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i) avc[i] = src.an[i];

        // accumulator element r of tile (m, j) sits at output row m * 16 + lane % 16 of
        // the wave's rows; elements 0..3 of tiles 2 p and 2 p + 1 are columns 32 p + 8
        // (lane / 16) + 0..3 and + 4..7.  The lane's offset is made opaque per tile: the
        // compiler otherwise keeps every store's offset live across the K loop, in scratch
        int lrow_out = wm * (BM / WAVES_M) + frow, colq = (lane >> 4) * 8;
        opaque(lrow_out);
        opaque(colq);
        if (cur.split) {
            // fp32 partial tile of this K chunk, laid out [row][weight row of the tile]
            // (rows past the group inside the last 16-row block hold unused sums)
            const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(args.part + (int64_t)cur.u * BM * BNW), (short)0, BM * BNW * 4, RSRC_WORD3);
            const int wcol = wn * (SWIGLU ? BNW / 2 / WAVES_N : BNW / WAVES_N);
            const int vo = (lrow_out * BNW + wcol + colq) * 4;
#pragma unroll
            for (int m = 0; m < MS; ++m) {
                if (wm * (BM / WAVES_M) + m * 16 >= cur.rows_valid) break;
                use(m);
#pragma unroll
                for (int j = 0; j < NS; ++j)
                    __builtin_amdgcn_raw_buffer_store_b128(
                        __builtin_bit_cast(u32x4, acc[m][j]), prsrc,
                        vo + (b_tile(j & ~1) + (j & 1) * 4) * 4, m * 16 * BNW * 4, 0);
            }
            wait_vm<0>();                        // more stores than the stage waits allow for
        } else {
            // rows past the group are dropped by the descriptor, and so are 32-column
            // blocks past the output (N is a multiple of 64), by an empty one
            const int wcol = cur.n0 + wn * (BN_OUT / WAVES_N);
            auto orsrc = [&](int p) {
                return __builtin_amdgcn_make_buffer_rsrc(
                    (void*)(args.out + (int64_t)cur.row0 * args.ldo), (short)0,
                    wcol + 32 * p < args.N ? cur.rows_valid * args.ldo * 2 : 0, RSRC_WORD3);
            };
            // NEAR: SiLU by the short form, the largest gate value to `most`
            float most = 0.f;
            auto store_tile = [&](auto near) {
                constexpr bool NEAR = decltype(near)::value;
                constexpr int NP = SWIGLU ? NS / 4 : NS / 2;
                int vo = (lrow_out * args.ldo + wcol + colq) * 2;
#pragma unroll
                for (int m = 0; m < MS; ++m) {
                    use(m);
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        float v[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int j = 2 * p + (e >> 2);
                            v[e] = acc[m][j][e & 3];
                            if constexpr (SWIGLU) {
                                if (NEAR) most = fmaxf(most, fabsf(v[e]));
                                v[e] = (NEAR ? silu_near(v[e]) : silu_div(v[e])) *
                                       acc[m][NS / 2 + j][e & 3];
                            }
                        }
                        const u32x4 w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                         pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
                        __builtin_amdgcn_raw_buffer_store_b128(w, orsrc(p), vo + 64 * p, 0, 0);
                    }
                    vo += 32 * args.ldo;
                }
            };
            store_tile(std::true_type{});
            // some gate value out of the short form's range: the tile again (the stores are
            // then more than the stage waits allow for, which only makes them wait longer).
            // One test a tile: a branch per eight values cost as much as the divisions
            if constexpr (SWIGLU)
                if (__any(!(most < SILU_NEAR))) store_tile(std::false_type{});
        }
        if (!has_next) break;
        q = qn;
        cur = nxt;
        start = !chain;
        if (start) {
            // the ring is idle before it is refilled
            wait_vm<0>();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            rc = rsrc_of(cur, true);
        }
    }
    wait_vm<0>();                                // no direct load outlives the workgroup's LDS
#endif
}

// ---------------------------------------------------------------------------
// Small groups (those of a short call up to SMALL_ROWS_MAX rows, see
// small_limits; every group of a call with the MOE_FFN_SMALL_GROUPS statement or
// of at most SMALL_ROWS rows in all): weight streaming with split-K.  Here the
// weights dominate the traffic (each weight byte is used by a handful of rows), so
// the aim is to read every weight byte once, from all CUs at once.  This kernel runs
// the products that strip_product leaves it (the long K).  Work item = (group, 128
// weight rows, K chunk, 64 rows); one workgroup per item, three per CU with three K
// steps of loads in flight each (four per CU cannot hold that ring without
// spilling), fp32 partial sums per K chunk.  HBM reads reach their rate only with
// many independent streams in flight (a read-only probe over 448 MiB: 4.3-5.1 TB/s
// with 224-448 workgroups, 5.4-5.7 TB/s with 896 or more), so the item is narrow in
// weight rows and covers a whole decode-sized group (a group of up to 64 rows reads
// its weights once).  A second kernel adds the chunks in a fixed order (so results
// are deterministic) and, for the gate/up product, applies SiLU(a) * b.
// The split factor S is derived on the device from the group sizes; both
// kernels derive the same plan from the same inputs.
// ---------------------------------------------------------------------------
constexpr int ST_M = 64;                 // rows per item (two 32-row MFMA tiles per wave)
constexpr int ST_N = 128;                // weight rows per item (32 per wave)
constexpr int ST_THREADS = 256;
constexpr int ST_WG_PER_CU = 3;
constexpr int ST_RING = 2;               // K steps of loads in flight beyond the one in LDS
constexpr int ST_A_PER = ST_M * 64 / 8 / ST_THREADS;   // 16-byte loads per thread per K step
constexpr int ST_B_PER = ST_N * 64 / 8 / ST_THREADS;
constexpr int SPLIT_MAX = 32;
constexpr int PART_FACTOR = 8;           // partial capacity = PART_FACTOR x bound on small rows
static_assert(ST_A_PER == 2 && ST_B_PER == 4, "streaming tile");

struct StreamArgs {
    const bf16_t* w[MOE_MAX_GROUPS];     // per group [N][K]
    const int32_t* offsets;              // as GemmArgs::offsets
    const bf16_t* a;                     // [rows][K]
    float* part;                         // [S][n_small][N]
    bf16_t* out;                         // reduce output [rows][ldo]
    int n_groups;                        // lead groups included
    int lead, lead_rows;                 // as in GemmArgs
    int K;
    int N;                               // weight rows (2f for gate/up, d for down)
    int ldo;
    int part_rows;                       // capacity of `part` in rows (S * n_small <= part_rows)
    int grid;                            // workgroups of the streaming launch
    const int32_t* a_rows;               // gather: row p of A is a[a_rows[p]] (a holds a_total rows)
    int a_total;
    const int* limits;                   // row limits written by the gate/up tiled launch (nullptr:
    int product;                         // lim0); this product's index, 0 gate/up, 1 down
    int lim0;                            // row limit of streamed groups when limits is nullptr
    int zero_big;                        // strips: rows of groups above the limit get zeros
};

struct StreamPlan {
    int off[MOE_MAX_GROUPS + 1];
    int qbase[MOE_MAX_GROUPS + 1];       // compact row base of each small group
    int istart[MOE_MAX_GROUPS + 1];      // first work item of each group
    int n_small, S, total, n_tiles;
};

// Row limit of the streamed groups.  Most calls of a few hundred rows a group stream
// none (limit 0): the streaming launches and the chunk sums look at it first and leave
// out their plans.
__device__ __forceinline__ int stream_limit(const StreamArgs& a) {
    return a.limits != nullptr ? a.limits[a.product] : a.lim0;
}

__device__ void make_stream_plan(const StreamArgs& a, StreamPlan& P, int nthreads) {
    const int lim = stream_limit(a);
    for (int g = threadIdx.x; g <= a.n_groups; g += nthreads)
        P.off[g] = group_start(a.offsets, a.lead, a.lead_rows, g);
    __syncthreads();
    if (threadIdx.x < 64) {                          // one wave: prefix sums over the groups
        const int lane = threadIdx.x;
        const int nt = (int)ceil_div(a.N, ST_N);
        const int KT = a.K / 64;
        int rows_small = 0, base = 0;
        for (int g0 = 0; g0 < a.n_groups; g0 += 64) {
            const int g = g0 + lane;
            const int rows = g < a.n_groups ? P.off[g + 1] - P.off[g] : 0;
            const bool small = rows > 0 && rows <= lim;
            const int rs = small ? rows : 0;
            const int items = small ? (int)ceil_div(rows, ST_M) * nt : 0;
            const int irs = wave_incl_scan(rs), iit = wave_incl_scan(items);
            if (g < a.n_groups) {
                P.qbase[g] = rows_small + irs - rs;
                P.istart[g] = base + iit - items;    // scaled by S below
            }
            rows_small += __shfl(irs, 63, 64);
            base += __shfl(iit, 63, 64);
        }
        // split factor: as many K chunks as fit the grid in one round (every
        // workgroup streams one item; a partly filled extra round would leave
        // most of HBM idle)
        int S = base > 0 ? a.grid / base : 1;
        S = min(S, SPLIT_MAX);
        S = min(S, KT);
        if (rows_small > 0) S = min(S, a.part_rows / rows_small);
        S = max(S, 1);
        for (int g = lane; g < a.n_groups; g += 64) P.istart[g] *= S;
        if (lane == 0) {
            P.qbase[a.n_groups] = rows_small;
            P.istart[a.n_groups] = base * S;
            P.n_small = rows_small;
            P.S = S;
            P.total = base * S;
            P.n_tiles = nt;
        }
    }
    __syncthreads();
}

// One workgroup per item (64 rows x 128 weight rows x one K chunk); each wave
// takes 32 of the weight rows against both 32-row halves of the rows.  Loads
// are coalesced (8 lanes read one 128-byte row segment) and run ST_RING K
// steps ahead in registers; one LDS stage holds the step being multiplied.
// The partial-sum epilogue adds a uniform row offset per accumulator element to
// one per-lane pointer: with a 64-bit row offset per element and lane, the
// compiler kept all of them live across the item loop and spilled them to
// scratch (decode steps 5 % slower).
template <bool GATHER = false>
__global__ __launch_bounds__(ST_THREADS, ST_WG_PER_CU) void stream_gemm_kernel(StreamArgs args) {
    __shared__ __attribute__((aligned(16))) bf16_t As[ST_M * LDK];
    __shared__ __attribute__((aligned(16))) bf16_t Bs[ST_N * LDK];
    __shared__ StreamPlan P;
    __shared__ int s_item[4];
    if (stream_limit(args) <= 0) return;
    make_stream_plan(args, P, ST_THREADS);
    if (P.total == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wg_per_xcd = gridDim.x / NUM_XCD;
    const int xcd = blockIdx.x % NUM_XCD;
    const int widx = blockIdx.x / NUM_XCD;
    const int chunk = (P.total + NUM_XCD - 1) / NUM_XCD;
    const int i_begin = xcd * chunk, i_end = min(i_begin + chunk, P.total);
    const int K = args.K, KT = K / 64, S = P.S;
    const int kc = (tid & 7) * 8;
    const int lrow = tid >> 3;                          // 0..31: row of this thread's loads
    const int voff = (lrow * K + kc) * 2;
    const int vstep = 32 * K * 2;
    const int frag_col = (lane >> 5) * 32, frag_row = lane & 31;

    for (int it = i_begin + widx; it < i_end; it += wg_per_xcd) {
        if (tid == 0) {
            const int lo = last_le(P.istart, args.n_groups, it);   // the item's group
            s_item[0] = lo;
            s_item[1] = it - P.istart[lo];
        }
        __syncthreads();
        const int g = __builtin_amdgcn_readfirstlane(s_item[0]);
        int local = __builtin_amdgcn_readfirstlane(s_item[1]);
        const int rows = __builtin_amdgcn_readfirstlane(P.off[g + 1] - P.off[g]);
        const int mt = (int)ceil_div(rows, ST_M);
        const int m = local % mt;
        local /= mt;
        const int c = local % S;
        const int n0 = (local / S) * ST_N;
        const int row0 = __builtin_amdgcn_readfirstlane(P.off[g]) + m * ST_M;
        const int rows_valid = min(ST_M, rows - m * ST_M);
        const int bvalid = min(ST_N, args.N - n0);
        const int kt0 = (int)((int64_t)c * KT / S), kt1 = (int)((int64_t)(c + 1) * KT / S);

        const __amdgpu_buffer_rsrc_t ar =
            GATHER ? __builtin_amdgcn_make_buffer_rsrc((void*)args.a, (short)0, args.a_total * K * 2,
                                                      RSRC_WORD3)
                   : __builtin_amdgcn_make_buffer_rsrc((void*)(args.a + (int64_t)row0 * K), (short)0,
                                                      rows_valid * K * 2, RSRC_WORD3);
        int avoff[ST_A_PER];
#pragma unroll
        for (int q = 0; q < ST_A_PER; ++q) {
            const int rin = lrow + 32 * q;
            avoff[q] = !GATHER ? voff + q * vstep
                       : rin < rows_valid ? (args.a_rows[row0 + rin] * K + kc) * 2 : A_OOB;
        }
        const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(args.w[g] + (int64_t)n0 * K), (short)0, bvalid * K * 2, RSRC_WORD3);

        uint4 ring_a[ST_RING + 1][ST_A_PER], ring_b[ST_RING + 1][ST_B_PER];
        auto load = [&](int kt, uint4* ra, uint4* rb) {
            const int so = kt * 128;
#pragma unroll
            for (int q = 0; q < ST_A_PER; ++q) ra[q] = buffer_load16(ar, avoff[q], so);
#pragma unroll
            for (int i = 0; i < ST_B_PER; ++i) rb[i] = buffer_load16(br, voff + i * vstep, so);
        };
        f32x16 acc0, acc1;
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc0[r] = 0.f; acc1[r] = 0.f; }
        const int nsteps = kt1 - kt0;
#pragma unroll
        for (int u = 0; u <= ST_RING; ++u)
            if (u < nsteps) load(kt0 + u, ring_a[u], ring_b[u]);
        for (int t0 = 0; t0 < nsteps; t0 += ST_RING + 1) {
#pragma unroll
            for (int u = 0; u <= ST_RING; ++u) {
                const int t = t0 + u;
                if (t < nsteps) {
                    __syncthreads();                 // previous step's fragment reads are done
#pragma unroll
                    for (int q = 0; q < ST_A_PER; ++q)
                        *(uint4*)&As[(lrow + 32 * q) * LDK + kc] = ring_a[u][q];
#pragma unroll
                    for (int i = 0; i < ST_B_PER; ++i)
                        *(uint4*)&Bs[(lrow + 32 * i) * LDK + kc] = ring_b[u][i];
                    __syncthreads();
                    if (t + ST_RING + 1 < nsteps) load(kt0 + t + ST_RING + 1, ring_a[u], ring_b[u]);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        const bf16x8 a0 = *(const bf16x8*)&As[frag_row * LDK + frag_col + kk * 8];
                        const bf16x8 a1 = *(const bf16x8*)&As[(32 + frag_row) * LDK + frag_col + kk * 8];
                        const bf16x8 bw = *(const bf16x8*)&Bs[(wave * 32 + frag_row) * LDK + frag_col + kk * 8];
                        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, bw, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, bw, acc1, 0, 0, 0);
                    }
                }
            }
        }

        // partial store: element r of a 32x32 tile is row 8*(r/4) + 4*(lane/32) + r%4, col lane%32
        float* prow = args.part + ((int64_t)c * P.n_small + P.qbase[g] + m * ST_M) * args.N + n0 +
                      wave * 32;
        const int cw = bvalid - wave * 32;           // valid columns of this wave
        if (frag_row < cw) {
            // one per-lane base pointer; the row offset of each r is uniform
            const int lr = (lane >> 5) * 4;
            float* pl = prow + (int64_t)lr * args.N + frag_row;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rc = (r >> 2) * 8 + (r & 3);
                const int64_t o = (int64_t)__builtin_amdgcn_readfirstlane(rc * args.N);
                const int64_t o32 = (int64_t)__builtin_amdgcn_readfirstlane((rc + 32) * args.N);
                if (rc + lr < rows_valid) pl[o] = acc0[r];
                if (rc + 32 + lr < rows_valid) pl[o32] = acc1[r];
            }
        }
        __syncthreads();                             // s_item and LDS reuse by the next item
    }
}

// ---------------------------------------------------------------------------
// Strips: the streamed groups' products where K is short (strip_product): one
// launch, no split of K over workgroups, no partial sums and no launch to add
// them.  A workgroup takes up to 64 rows of a group x 64 weight rows (SwiGLU: 32 gate
// and the matching 32 up rows) over the whole of K; both operands go straight into an
// LDS ring of R 64-wide K stages.  What bounds it: at decode the latency of the launch
// and of the first loads, then the weight stream; an item of the split kernel reads a
// few K steps only and pays for the partial sums' round trip and the second launch.
// At the barrier of stage t the fragments of stage t are in registers and stage t + 1
// has landed: its fragments come from LDS and stage t + R into the ring while stage t
// multiplies.  The tile is as high as its rows need (32 or 64: fewer LDS bytes per
// stage and more stages in the same LDS; one token, DeepSeek-V2-Lite: 40.3 -> 34.4 us
// a step; a third height of 16 gained nothing); three workgroups fit a CU.  128-byte LDS
// rows, 16-byte chunk c of row r at c ^ (r & 7) (conflict-free for the fragment
// reads); weights as the MFMA's A operand, so a lane holds 4 consecutive output
// columns of one row.  Every sum runs over K in ascending stages, whatever the height.
// ---------------------------------------------------------------------------
constexpr int SP_M = 64;                 // rows per tile, at most
constexpr int SP_N = 64;                 // weight rows per tile
constexpr int SP_THREADS = 256;
constexpr int SP_ROWB = 128;             // LDS row bytes: 64 K
constexpr int SP_WG_PER_CU = 3;
constexpr int strip_lds(int M, int R) { return R * (M + SP_N) * SP_ROWB; }
constexpr int SP_R32 = 4, SP_R64 = 3;    // ring stages by tile height
constexpr int SP_LDS = strip_lds(64, SP_R64);
static_assert(strip_lds(32, SP_R32) <= SP_LDS, "ring size");
constexpr int STRIP_ANY_K = 2048, STRIP_MAX_K = 4096;   // see strip_product

template <bool SWIGLU, bool GATHER>
__global__ __launch_bounds__(SP_THREADS, SP_WG_PER_CU) void strip_gemm_kernel(StreamArgs args) {
#ifdef __HIP_DEVICE_COMPILE__
    extern __shared__ __attribute__((aligned(1024))) char strip_ring[];
    __shared__ int s_off[MOE_MAX_GROUPS + 1], s_tstart[MOE_MAX_GROUPS + 1];
    constexpr int OUT = SWIGLU ? SP_N / 2 : SP_N;              // output columns per tile
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_groups = args.n_groups, K = args.K;
    const int n_out = SWIGLU ? args.N / 2 : args.N;
    const int nt = n_out / OUT;
    const int lim = stream_limit(args);
    if (lim <= 0 && !args.zero_big) return;                    // nothing streamed
    for (int g = tid; g <= n_groups; g += SP_THREADS)
        s_off[g] = group_start(args.offsets, args.lead, args.lead_rows, g);
    __syncthreads();
    if (wave == 0) {
        int carry = 0;
        for (int g0 = 0; g0 < n_groups; g0 += 64) {
            const int g = g0 + lane;
            const int rows = g < n_groups ? s_off[g + 1] - s_off[g] : 0;
            const int v = rows <= lim || args.zero_big ? (int)ceil_div(rows, SP_M) * nt : 0;
            const int incl = wave_incl_scan(v);
            if (g < n_groups) s_tstart[g + 1] = carry + incl;
            carry += __shfl(incl, 63, 64);
        }
        if (lane == 0) s_tstart[0] = 0;
    }
    __syncthreads();
    // contiguous tiles per XCD: the row tiles of a weight strip share its L2
    const int total = s_tstart[n_groups];
    const int per = (total + NUM_XCD - 1) / NUM_XCD;
    const int t_begin = (blockIdx.x % NUM_XCD) * per, t_end = min(t_begin + per, total);
    // load i of a wave fills LDS rows 32 i + 8 wave + lane / 8, chunk slot lane % 8
    const int lrow = 8 * wave + (lane >> 3);
    const int kc = ((lane & 7) ^ ((lane >> 3) & 7)) * 8;
    const int frow = lane & 15;
    const int c0 = ((lane >> 4) ^ (frow & 7)) * 16;

    for (int tile = t_begin + blockIdx.x / NUM_XCD; tile < t_end; tile += gridDim.x / NUM_XCD) {
        const int g = __builtin_amdgcn_readfirstlane(last_le(s_tstart, n_groups, tile));
        const int start = __builtin_amdgcn_readfirstlane(s_off[g]);
        const int rows = __builtin_amdgcn_readfirstlane(s_off[g + 1]) - start;
        const int mt = (rows + SP_M - 1) / SP_M;
        const int local = tile - __builtin_amdgcn_readfirstlane(s_tstart[g]);
        // the row tiles of a strip in another order from turn to turn: a workgroup's turns
        // are gridDim.x / NUM_XCD tiles apart, a multiple of mt for most mt, and a group's
        // last row tile is the short one, so in a fixed order some workgroups would take
        // short tiles only and others none (8 groups of 65 rows, d = 4096, f = 14336: FFN
        // 924 us, in turn 684)
        const int strip = local / mt;
        const int m = (local + strip * mt / (int)(gridDim.x / NUM_XCD)) % mt, n0 = strip * OUT;
        const int row0 = start + m * SP_M, rows_valid = min(SP_M, rows - m * SP_M);
        // uniform (the compiler loops over the lanes' values for a descriptor it cannot
        // prove to be)
        const int nst = __builtin_amdgcn_readfirstlane(rows <= lim ? K / 64 : 0);
        // rows past the group read as zero or leave LDS as it is: not stored either way
        const __amdgpu_buffer_rsrc_t ar =
            GATHER ? __builtin_amdgcn_make_buffer_rsrc((void*)args.a, (short)0, args.a_total * K * 2,
                                                      RSRC_WORD3)
                   : __builtin_amdgcn_make_buffer_rsrc((void*)(args.a + (int64_t)row0 * K), (short)0,
                                                      rows_valid * K * 2, RSRC_WORD3);
        const bf16_t* W = args.w[g] + (int64_t)n0 * K;
        const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc(
            (void*)W, (short)0, (SWIGLU ? 32 : SP_N) * K * 2, RSRC_WORD3);
        const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(W + (int64_t)(SWIGLU ? n_out : 0) * K), (short)0, (SWIGLU ? 32 : SP_N) * K * 2,
            RSRC_WORD3);
        const __amdgpu_buffer_rsrc_t none =
            __builtin_amdgcn_make_buffer_rsrc((void*)args.a, (short)0, 0, RSRC_WORD3);
        const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(args.out + (int64_t)row0 * args.ldo), (short)0, rows_valid * args.ldo * 2,
            RSRC_WORD3);

        // the tile at a height of M rows: waves 2 x 2, each M / 2 rows x 32 weight rows
        // (SwiGLU: 16 gate, 16 up)
        auto run = [&](auto height, auto ring) {
            constexpr int M = decltype(height)::value, R = decltype(ring)::value;
            constexpr int SA = M * SP_ROWB, STAGE = SA + SP_N * SP_ROWB;
            constexpr int NA = M / 32, NB = SP_N / 32, P = NA + NB;   // 1 KB loads a wave a stage
            constexpr int MT = M / 32;                             // 16-row tiles per wave
            const int wm = wave & 1, wn = wave >> 1;
            const int a_frag = (wm * (M / 2) + frow) * SP_ROWB;
            const int b_frag = SA + (wn * (SWIGLU ? 16 : 32) + frow) * SP_ROWB;
            constexpr int B_STEP = (SWIGLU ? 32 : 16) * SP_ROWB;   // second column tile
            const int wvoff = ((SWIGLU ? lrow : w_order(lrow)) * K + kc) * 2;
            int av[NA];
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int rin = lrow + 32 * i;
                av[i] = !GATHER ? (rin * K + kc) * 2
                        : rin < rows_valid ? (args.a_rows[row0 + rin] * K + kc) * 2 : A_OOB;
            }
            // stage s into slot s % R; past the tile's K: empty ranges, loads without
            // traffic, so that the counts the waits rely on stay the same
            auto dma = [&](int s) {
                char* base = strip_ring + (s % R) * STAGE + wave * 1024;
                const int so = s * SP_ROWB;
                const bool in = s < nst;
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(
                        in ? (SWIGLU && i ? ur : br) : none, (lds_void*)(base + SA + i * 4096), 16,
                        wvoff + (SWIGLU ? 0 : i * 64 * K), so, 0, 0);
#pragma unroll
                for (int i = 0; i < NA; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(in ? ar : none,
                                                             (lds_void*)(base + i * 4096), 16, av[i],
                                                             so, 0, 0);
            };
            f32x4 acc[MT][2];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            struct Frags {
                bf16x8 a[2][MT], b[2][2];                   // two 32-wide K steps
            };
            auto read = [&](int s, Frags& f) {
                const char* st = strip_ring + (s % R) * STAGE;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int cq = c0 ^ (q * 64);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        f.b[q][j] = *(const bf16x8*)(st + b_frag + j * B_STEP + cq);
#pragma unroll
                    for (int i = 0; i < MT; ++i)
                        f.a[q][i] = *(const bf16x8*)(st + a_frag + i * 16 * SP_ROWB + cq);
                }
            };
            auto step = [&](int t, const Frags& f, Frags& next) {
                // stage t + 1 has landed (the R - 2 after it may still fly), and every
                // wave holds its fragments of stage t
                wait_vm<(R - 2) * P>();
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                read(t + 1, next);
                dma(t + R);
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                f.b[q][j], f.a[q][i], acc[i][j], 0, 0, 0);
            };
            if (nst > 0) {
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
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int row_in = wm * (M / 2) + i * 16 + frow;
                const int quad = lane >> 4;
                if constexpr (SWIGLU) {
                    float v[4] = {acc[i][0][0], acc[i][0][1], acc[i][0][2], acc[i][0][3]};
                    silu(v);
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] *= acc[i][1][r];
                    const u32x2 w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                    __builtin_amdgcn_raw_buffer_store_b64(
                        w, orsrc, (row_in * args.ldo + n0 + wn * 16 + quad * 4) * 2, 0, 0);
                } else {
                    const u32x4 w = {pack_bf16x2(acc[i][0][0], acc[i][0][1]),
                                     pack_bf16x2(acc[i][0][2], acc[i][0][3]),
                                     pack_bf16x2(acc[i][1][0], acc[i][1][1]),
                                     pack_bf16x2(acc[i][1][2], acc[i][1][3])};
                    __builtin_amdgcn_raw_buffer_store_b128(
                        w, orsrc, (row_in * args.ldo + n0 + wn * 32 + quad * 8) * 2, 0, 0);
                }
            }
        };
        if (rows_valid <= 32)
            run(std::integral_constant<int, 32>{}, std::integral_constant<int, SP_R32>{});
        else
            run(std::integral_constant<int, 64>{}, std::integral_constant<int, SP_R64>{});
        // every wave is done with the ring, and no load for it is on its way, before the
        // next tile (of another height, perhaps) refills it or the workgroup ends
        wait_vm<0>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
#endif
}

// Adds chunks [c, c + RU) of a partial sum to x (SWIGLU: the up half, `up`
// floats further on, to y), in chunk order.  All RU loads are issued before the
// first add: a chunk at or past S reads chunk S - 1 and its add is skipped, so
// a short split costs one load round trip instead of one per chunk.
template <bool SWIGLU, int RU>
__device__ __forceinline__ void add_chunk_batch(const float* pr, int64_t cstride, int up, int c,
                                                int S, float4& x, float4& y) {
    float4 v[RU], u[RU];
#pragma unroll
    for (int j = 0; j < RU; ++j) {
        const int cc = c + j < S ? c + j : S - 1;
        v[j] = *(const float4*)(pr + cc * cstride);
        if (SWIGLU) u[j] = *(const float4*)(pr + cc * cstride + up);
    }
#pragma unroll
    for (int j = 0; j < RU; ++j)
        if (c + j < S) {
            x.x += v[j].x; x.y += v[j].y; x.z += v[j].z; x.w += v[j].w;
            if (SWIGLU) { y.x += u[j].x; y.y += u[j].y; y.z += u[j].z; y.w += u[j].w; }
        }
}

// x (and y) = the sum of chunks 0 .. S-1 (S >= 1) in chunk order: batches of 8
// loads, the rest as one batch of 4 or 8.
template <bool SWIGLU>
__device__ __forceinline__ void add_chunks(const float* pr, int64_t cstride, int up, int S,
                                           float4& x, float4& y) {
    x = make_float4(0.f, 0.f, 0.f, 0.f);
    y = x;
    int c = 0;
    for (; c + 8 <= S; c += 8) add_chunk_batch<SWIGLU, 8>(pr, cstride, up, c, S, x, y);
    if (S - c > 4) add_chunk_batch<SWIGLU, 8>(pr, cstride, up, c, S, x, y);
    else if (c < S) add_chunk_batch<SWIGLU, 4>(pr, cstride, up, c, S, x, y);
}

// Four summed columns in bf16 (SWIGLU: SiLU(x) * y).
template <bool SWIGLU>
__device__ __forceinline__ uint2 pack_sum(const float4& x, const float4& y) {
    float o[4] = {x.x, x.y, x.z, x.w};
    if constexpr (SWIGLU) {
        silu(o);
        o[0] *= y.x;
        o[1] *= y.y;
        o[2] *= y.z;
        o[3] *= y.w;
    }
    return make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
}

// Sums, in chunk order, the K chunks of the tiled kernel's split tiles (fp32
// partial tiles [row][weight row]; SWIGLU: gate in tile columns [0, 128), up
// in [128, 256)) and applies the epilogue: out = SiLU(gate) * up, or the sum.
template <bool SWIGLU>
__device__ void tile_split_reduce(const GemmArgs& t, int* s_off, int* s_tstart) {
    const int n_groups = t.n_groups;
    for (int g = threadIdx.x; g <= n_groups; g += ST_THREADS)
        s_off[g] = group_start(t.offsets, t.lead, t.lead_rows, g);
    __syncthreads();
    const int lim = t.limits != nullptr ? t.limits[t.product] : t.lim0;
    if (threadIdx.x < 64) tile_starts(s_off, n_groups, lim, t.n_tiles, s_tstart, threadIdx.x);
    __syncthreads();
    const SplitPlan plan = split_plan(s_tstart[n_groups], t.K / BK, t.split_units);
    const int S = plan.S;
    if (S == 1) return;
    constexpr int BN_OUT = SWIGLU ? BNW / 2 : BNW;
    constexpr int C4 = BN_OUT / 4;
    const int64_t items = (int64_t)plan.tail * BM * C4;
    for (int64_t i = (int64_t)blockIdx.x * ST_THREADS + threadIdx.x; i < items;
         i += (int64_t)gridDim.x * ST_THREADS) {
        const int q = (int)(i / (BM * C4));          // split tile, counted from plan.head
        const int L = plan.head + q;
        const int rem = (int)(i - (int64_t)q * BM * C4);
        const int row = rem / C4, j = (rem - row * C4) * 4;
        const int g = last_le(s_tstart, n_groups, L);
        const int rows = s_off[g + 1] - s_off[g];
        const TilePos pos = tile_pos(L - s_tstart[g], (int)ceil_div(rows, BM), t.n_tiles);
        const int nt = pos.n;
        const int m0 = pos.m * BM;
        if (m0 + row >= rows) continue;
        const int n0 = nt * BN_OUT;
        if (n0 + j >= t.N) continue;
        float4 x, y;
        add_chunks<SWIGLU>(t.part + ((int64_t)q * S * BM + row) * BNW + j, (int64_t)BM * BNW,
                           BNW / 2, S, x, y);
        const uint2 pk = pack_sum<SWIGLU>(x, y);
        *(uint2*)(t.out + (int64_t)(s_off[g] + m0 + row) * t.ldo + n0 + j) = pk;
    }
}

template <bool SWIGLU>
__device__ __forceinline__ void stream_reduce(const StreamArgs& args, const StreamPlan& P);

// Fixed-order sum of the K chunks; SWIGLU: out[p][j] = SiLU(sum gate_j) * sum up_j
// with gate in partial columns [0, N/2) and up in [N/2, N).  The same launch
// finishes the tiled kernel's split tiles (tile_split_reduce).
template <bool SWIGLU>
__global__ __launch_bounds__(ST_THREADS) void split_reduce_kernel(StreamArgs args, GemmArgs targs) {
    __shared__ StreamPlan P;
    __shared__ int t_off[MOE_MAX_GROUPS + 1], t_tstart[MOE_MAX_GROUPS + 1];
    const int tsplit = targs.part != nullptr ? *targs.split_info : 1;   // used at the end
    if (stream_limit(args) > 0) {
        make_stream_plan(args, P, ST_THREADS);
        stream_reduce<SWIGLU>(args, P);
    }
    if (tsplit > 1) tile_split_reduce<SWIGLU>(targs, t_off, t_tstart);
}

template <bool SWIGLU>
__device__ __forceinline__ void stream_reduce(const StreamArgs& args, const StreamPlan& P) {
    const int n_small = P.n_small;
    if (n_small == 0) return;
    const int S = P.S;
    const int cols = SWIGLU ? args.N / 2 : args.N;
    const int chunks = cols / 4;                     // 4 output columns per item
    const int64_t total = (int64_t)n_small * chunks;
    const int64_t cstride = (int64_t)n_small * args.N;
    for (int64_t i = (int64_t)blockIdx.x * ST_THREADS + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * ST_THREADS) {
        const int q = (int)(i / chunks);
        const int c4 = (int)(i - (int64_t)q * chunks) * 4;
        // the row's group: groups without small rows share qbase with the next one
        const int g = last_le(P.qbase, args.n_groups, q);
        const int p = P.off[g] + (q - P.qbase[g]);
        float4 x, y;
        add_chunks<SWIGLU>(args.part + (int64_t)q * args.N + c4, cstride, cols, S, x, y);
        const uint2 pk = pack_sum<SWIGLU>(x, y);
        *(uint2*)(args.out + (int64_t)p * args.ldo + c4) = pk;
    }
}

// The down product's chunk sum fused with the gate-weighted combine, for calls
// in which every group is streamed (no group above SMALL_ROWS_MAX rows): one
// thread per token and 4 output columns.  For each assignment r of token t, in
// ascending r, the row's output is summed over the K chunks in chunk order and
// rounded to bf16 (the value the chunk sum would store in y_perm), then added
// with its gate by fmaf; the shared experts' output is added last and the sum
// stored in bf16 -- the arithmetic of split_reduce_kernel followed by the
// combine, so the outputs are the same bits, without y_perm being written and
// read back or the combine's launch.
struct CombineArgs {
    const int32_t* token_row;            // [T][k]
    const float* gate;                   // [T][k]
    const bf16_t* y_shared;              // [T][d], nullable
    bf16_t* y;                           // [T][d]
    int64_t T;
    int k;
};

template <int KM>
__global__ __launch_bounds__(ST_THREADS) void stream_reduce_combine_kernel(StreamArgs args,
                                                                           CombineArgs cb) {
    __shared__ StreamPlan P;
    make_stream_plan(args, P, ST_THREADS);
    const int lim = stream_limit(args);
    const int S = P.S;
    const int d = args.N;
    const int chunks = d / 4;
    const int64_t cstride = (int64_t)P.n_small * d;
    const int64_t total = cb.T * chunks;
    // CB chunks of every assignment are loaded together, KM * CB loads in flight
    constexpr int CB = 32 / KM > 0 ? 32 / KM : 1;
    for (int64_t i = (int64_t)blockIdx.x * ST_THREADS + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * ST_THREADS) {
        const int64_t t = i / chunks;
        const int c4 = (int)(i - t * chunks) * 4;
        // the partial row of each assignment here, or none
        int64_t off[KM];
        float g[KM];
        bool ok[KM];
        int64_t first = -1;
#pragma unroll
        for (int r = 0; r < KM; ++r) {
            const int rr = r < cb.k ? r : cb.k - 1;
            const int32_t p = r < cb.k ? cb.token_row[t * cb.k + rr] : -1;
            g[r] = cb.gate[t * cb.k + rr];
            ok[r] = false;
            off[r] = 0;
            if (p >= 0) {
                const int grp = last_le(P.off, args.n_groups, p);
                // a group above the streaming limit has no partial rows (outside the contract)
                ok[r] = P.off[grp + 1] - P.off[grp] <= lim;
                off[r] = (int64_t)(P.qbase[grp] + p - P.off[grp]) * d + c4;
            }
            if (ok[r] && first < 0) first = off[r];
        }
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        if (first >= 0) {
            float4 x[KM];
#pragma unroll
            for (int r = 0; r < KM; ++r) x[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int c = 0; c < S; c += CB) {
                float4 v[KM][CB];
                // every load issued before the first add: an assignment not here
                // reads the first one's row and a chunk past S the last chunk,
                // both dropped below
#pragma unroll
                for (int r = 0; r < KM; ++r)
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        const int cc = c + j < S ? c + j : S - 1;
                        v[r][j] = *(const float4*)(args.part + (ok[r] ? off[r] : first) + cc * cstride);
                    }
#pragma unroll
                for (int r = 0; r < KM; ++r)
#pragma unroll
                    for (int j = 0; j < CB; ++j)
                        if (c + j < S) {
                            x[r].x += v[r][j].x; x[r].y += v[r][j].y;
                            x[r].z += v[r][j].z; x[r].w += v[r][j].w;
                        }
            }
            // each row's bf16 value, as y_perm would hold it, added with its gate in
            // ascending r
#pragma unroll
            for (int r = 0; r < KM; ++r) {
                if (!ok[r]) continue;
                acc[0] = fmaf(g[r], bf16_to_f32(f32_to_bf16(x[r].x)), acc[0]);
                acc[1] = fmaf(g[r], bf16_to_f32(f32_to_bf16(x[r].y)), acc[1]);
                acc[2] = fmaf(g[r], bf16_to_f32(f32_to_bf16(x[r].z)), acc[2]);
                acc[3] = fmaf(g[r], bf16_to_f32(f32_to_bf16(x[r].w)), acc[3]);
            }
        }
        if (cb.y_shared) {
            const uint2 w = *(const uint2*)(cb.y_shared + t * d + c4);
            acc[0] += __uint_as_float(w.x << 16);
            acc[1] += __uint_as_float(w.x & 0xffff0000u);
            acc[2] += __uint_as_float(w.y << 16);
            acc[3] += __uint_as_float(w.y & 0xffff0000u);
        }
        uint2 pk;
        pk.x = pack_bf16x2(acc[0], acc[1]);
        pk.y = pack_bf16x2(acc[2], acc[3]);
        *(uint2*)(cb.y + t * d + c4) = pk;
    }
}

int num_cus() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cached[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

}  // namespace

static int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

static int64_t small_rows_bound(int64_t cap_rows, int n_groups) {
    const int64_t b = (int64_t)n_groups * SMALL_ROWS;
    return cap_rows < b ? cap_rows : b;
}

// fp32 partial tiles of the tiled kernel's split K (none when no group can be
// big enough for the tiled kernel)
static int64_t tile_part_bytes(int64_t cap_rows) {
    return cap_rows > SMALL_ROWS ? 256 + (int64_t)TILE_SPLIT_UNITS * BM * BNW * 4 : 0;
}

// workspace: [H: cap_rows x f bf16][streaming partials][tiled partial tiles]
size_t grouped_ffn_ws_bytes(int dtype, int64_t cap_rows, int d, int f, int n_groups) {
    if (dtype != MOE_BF16) return (size_t)cap_rows * (size_t)f * 4 + 256;
    const int64_t h = align256(cap_rows * (int64_t)f * 2);
    const int64_t ncols = 2 * (int64_t)f > d ? 2 * (int64_t)f : d;
    const int64_t part = align256((int64_t)PART_FACTOR * small_rows_bound(cap_rows, n_groups) * ncols * 4);
    return (size_t)(h + part + tile_part_bytes(cap_rows) + 256);
}

// Whether the streamed groups of a product run as strips (n_out output columns in
// strips of `out`).  Only in a call whose rows may all lie in streamed groups, which also
// bounds the rows the fused combine keeps in the workspace.  Up to K = 2048 strips are
// ahead at every group size.  Past it a strip is a long chain, and a group above 64 rows
// reads its weight strip once per 64 rows through LDS where the split kernel's items are
// twice as wide: ahead while groups hold up to 64 rows (K = 4096, f = 14336, FFN of 2 and
// 4 groups of 64 rows: split 169 and 310 us, strips 158 and 291) in up to 9 rounds of
// workgroups (8 groups: 585 against 607), behind above (4 groups of 128 and 256 rows: 404
// and 641 against 410 and 693; 16 groups of 128 at f = 4096: 458 against 492), and so
// taken by the rows a group may hold on average.
// With one or two groups that bound says little (a batch's capacity is then its tokens
// in every group): there also above, if the strips make more than two rounds of
// workgroups (Mixtral-shaped step, 2 of 8 experts here, 256 tokens: split 246 us, strips
// 233; at two rounds or less f = 8192, 2 groups of 128 rows: 134 against 159).  Past
// K = 4096 the chain is too long (Mixtral-shaped down product, K = 14336: step 176 us
// split, 216 as strips).
static bool strip_product(int K, int n_out, int out, int64_t cap_rows, int n_groups, int cus) {
    if (K > STRIP_MAX_K || cap_rows > (int64_t)SMALL_ROWS_MAX * n_groups) return false;
    if (K <= STRIP_ANY_K) return true;
    const int64_t tiles = (cap_rows / SP_M + n_groups) * (n_out / out);
    const int64_t round = (int64_t)SP_WG_PER_CU * cus;
    if (cap_rows <= (int64_t)SP_M * n_groups && tiles <= 9 * round) return true;
    return n_groups <= 2 && tiles > 2 * round;
}

template <bool SWIGLU, bool GATHER>
static int launch_strips(const StreamArgs& a, int cus, hipStream_t s) {
    hipLaunchKernelGGL((strip_gemm_kernel<SWIGLU, GATHER>),
                       dim3((unsigned)(SP_WG_PER_CU * cus / NUM_XCD * NUM_XCD)), dim3(SP_THREADS),
                       SP_LDS, s, a);
    return launch_status();
}

int launch_grouped_ffn(const void* x_perm, int dtype, const int32_t* offsets, int n_groups,
                       const void* const* w13, const void* const* w2, int d, int f,
                       int64_t cap_rows, void* y_perm, void* ws, hipStream_t s,
                       const int32_t* a_rows, int64_t a_total, int products,
                       const void* combine, int lead, int lead_rows) {
    if (cap_rows == 0) return MOE_OK;
    const bool up = (products & MOE_FFN_GATE_UP) != 0, down = (products & MOE_FFN_DOWN) != 0;
    // every group within SMALL_ROWS_MAX rows (the caller's statement): all of them are
    // streamed, so no tile, no split tile and no row limit to pass on, and the tiled
    // launches are left out
    const bool small = (products & MOE_FFN_SMALL_GROUPS) != 0;
    // every non-empty group above SMALL_ROWS_MAX rows (the caller's statement): none is
    // streamed, every group is tiled (row limit 0) and the streaming launches are left out
    const bool large = (products & MOE_FFN_LARGE_GROUPS) != 0;
    const int cus = num_cus();
    if (dtype == MOE_F32)
        return launch_ffn_f32((const float*)x_perm, offsets, n_groups, w13, w2, d, f, cap_rows,
                              (float*)y_perm, (float*)ws, a_rows, products, lead, lead_rows, cus, s);
    const int grid = (cus / NUM_XCD) * NUM_XCD;
    bf16_t* h = (bf16_t*)ws;
    float* part = (float*)((char*)ws + align256(cap_rows * (int64_t)f * 2));
    const int64_t rmax = small_rows_bound(cap_rows, n_groups);
    const int64_t ncols = 2 * (int64_t)f > d ? 2 * (int64_t)f : d;
    // tiled split K: two split factors (one per product) and the two products'
    // streamed-group row limits in a 256-byte header, then the partial tiles
    char* tbase = tile_part_bytes(cap_rows) > 0
                      ? (char*)part + align256((int64_t)PART_FACTOR * rmax * ncols * 4)
                      : nullptr;
    float* tpart = tbase && !small ? (float*)(tbase + 256) : nullptr;
    int* tinfo = tbase && !small ? (int*)tbase : nullptr;
    const int sgrid = ((cus * ST_WG_PER_CU) / NUM_XCD) * NUM_XCD;
    const int64_t red_items = rmax * ((f > d ? f : d) / 4);
    int rgrid = (int)ceil_div(red_items, ST_THREADS);
    if (tpart != nullptr && rgrid < 2 * cus) rgrid = 2 * cus;   // room for split tiles
    if (rgrid > 4096) rgrid = 4096;
    // only split tiles to sum: four workgroups per CU, each thread a few items
    // (the idle workgroups of a larger grid cost more than the loop; gate/up
    // products 1-2 % faster at the Mixtral and Qwen3 prefill shapes)
    if (large) rgrid = 4 * cus;
    if (rgrid < 1) rgrid = 1;

    // gate/up product: tiled launch, then the streaming launch (the small groups of a
    // short call), then the chunk sums
    GemmArgs a1;
    for (int i = 0; i < MOE_MAX_GROUPS; ++i)
        a1.w[i] = up && i < n_groups ? (const bf16_t*)w13[i] : nullptr;
    a1.offsets = offsets;
    a1.lead = lead;
    a1.lead_rows = lead_rows;
    a1.a = (const bf16_t*)x_perm;
    a1.out = h;
    a1.n_groups = n_groups;
    a1.K = d;
    a1.N = f;
    a1.ldo = f;
    a1.up_row = f;
    a1.n_tiles = (int)ceil_div(f, BNW / 2);
    a1.limits = tinfo && !large ? tinfo + 2 : nullptr;
    a1.product = 0;
    a1.lim0 = small ? SMALL_ROWS_MAX : large ? 0 : SMALL_ROWS;
    a1.down_tiles = (int)ceil_div(d, BNW);
    a1.part = tpart;
    a1.split_info = tinfo;
    a1.split_units = grid < TILE_SPLIT_UNITS ? grid : TILE_SPLIT_UNITS;
    a1.a_rows = a_rows;
    a1.a_total = (int)a_total;
    // the ring is dynamic LDS above the default limit
#define MOE_TILED(SWIGLU, GATHER, args)                                                          \
    do {                                                                                         \
        static LdsGrant grant;                                                                   \
        if (allow_dynamic_lds((const void*)grouped_gemm_kernel<SWIGLU, GATHER>, RING_BYTES,      \
                              grant) != MOE_OK)                                                  \
            return MOE_ERR_DEVICE;                                                               \
        hipLaunchKernelGGL((grouped_gemm_kernel<SWIGLU, GATHER>), dim3(grid),                    \
                           dim3(GEMM_THREADS), RING_BYTES, s, args);                             \
    } while (0)
    if (up && !small && a_rows) MOE_TILED(true, true, a1);
    else if (up && !small) MOE_TILED(true, false, a1);
    StreamArgs s1;
    for (int i = 0; i < MOE_MAX_GROUPS; ++i) s1.w[i] = a1.w[i];
    s1.offsets = offsets;
    s1.lead = lead;
    s1.lead_rows = lead_rows;
    s1.a = (const bf16_t*)x_perm;
    s1.part = part;
    s1.out = h;
    s1.n_groups = n_groups;
    s1.K = d;
    s1.N = 2 * f;
    s1.ldo = f;
    s1.part_rows = (int)(PART_FACTOR * rmax);
    s1.grid = sgrid;
    s1.a_rows = a_rows;
    s1.a_total = (int)a_total;
    s1.limits = a1.limits;
    s1.product = 0;
    s1.lim0 = a1.lim0;
    s1.zero_big = 0;
    // the chunk sums' launch: nothing streamed to add up when the strips did it
    auto reduce_args = [](StreamArgs r, bool strips) {
        if (strips) {
            r.limits = nullptr;
            r.lim0 = 0;
        }
        return r;
    };
    const bool strips1 = strip_product(d, f, SP_N / 2, cap_rows, n_groups, cus);
    if (up) {
        if (!large && strips1) {
            const int st = a_rows ? launch_strips<true, true>(s1, cus, s)
                                  : launch_strips<true, false>(s1, cus, s);
            if (st != MOE_OK) return st;
        } else if (!large && a_rows)
            hipLaunchKernelGGL(stream_gemm_kernel<true>, dim3(sgrid), dim3(ST_THREADS), 0, s, s1);
        else if (!large)
            hipLaunchKernelGGL(stream_gemm_kernel<false>, dim3(sgrid), dim3(ST_THREADS), 0, s, s1);
        if (!strips1 || tpart != nullptr)
            hipLaunchKernelGGL(split_reduce_kernel<true>, dim3(rgrid), dim3(ST_THREADS), 0, s,
                               reduce_args(s1, strips1), a1);
    }
    if (!down) return launch_status();

    // down product
    GemmArgs a2 = a1;
    for (int i = 0; i < MOE_MAX_GROUPS; ++i) a2.w[i] = i < n_groups ? (const bf16_t*)w2[i] : nullptr;
    a2.a = h;
    a2.out = (bf16_t*)y_perm;
    a2.K = f;
    a2.N = d;
    a2.ldo = d;
    a2.up_row = 0;
    a2.n_tiles = (int)ceil_div(d, BNW);
    a2.split_info = tinfo ? tinfo + 1 : nullptr;
    a2.product = 1;
    a2.a_rows = nullptr;
    if (!small) MOE_TILED(false, false, a2);
#undef MOE_TILED
    StreamArgs s2 = s1;
    for (int i = 0; i < MOE_MAX_GROUPS; ++i) s2.w[i] = a2.w[i];
    s2.a = h;
    s2.out = (bf16_t*)y_perm;
    s2.K = f;
    s2.N = d;
    s2.ldo = d;
    s2.a_rows = nullptr;
    s2.product = 1;
    const bool strips2 = strip_product(f, d, SP_N, cap_rows, n_groups, cus);
    if (strips2 && !large) {
        if (combine != nullptr) {
            // the fused combine's y_perm: the partial sums' place (at most 256 rows a
            // group: 512 n d bytes of at least 2048 n d, or 2 of 32 d bytes a row), rows
            // of groups above the limit zeroed, which leaves them out of the sum
            s2.out = (bf16_t*)part;
            s2.zero_big = 1;
        }
        const int st = launch_strips<false, false>(s2, cus, s);
        if (st != MOE_OK) return st;
        if (combine != nullptr) {
            const CombineArgs& cb = *(const CombineArgs*)combine;
            return launch_combine(part, MOE_BF16, cb.token_row, cb.gate, cb.y_shared, 1, cb.T, d,
                                  cb.k, cb.y, s);
        }
    } else if (!large)
        hipLaunchKernelGGL(stream_gemm_kernel<false>, dim3(sgrid), dim3(ST_THREADS), 0, s, s2);
    if (combine == nullptr) {
        if (!strips2 || tpart != nullptr)
            hipLaunchKernelGGL(split_reduce_kernel<false>, dim3(rgrid), dim3(ST_THREADS), 0, s,
                               reduce_args(s2, strips2), a2);
        return launch_status();
    }
    // the down product's chunk sum writes the combined output (every group streamed)
    const CombineArgs& cb = *(const CombineArgs*)combine;
    int64_t cgrid = ceil_div(cb.T * (d / 4), ST_THREADS);
    if (cgrid > 4096) cgrid = 4096;
    if (cgrid < 1) cgrid = 1;
#define MOE_RC(KM)                                                                               \
    hipLaunchKernelGGL(stream_reduce_combine_kernel<KM>, dim3((unsigned)cgrid), dim3(ST_THREADS), \
                       0, s, s2, cb)
    if (cb.k <= 2) MOE_RC(2);
    else if (cb.k <= 4) MOE_RC(4);
    else if (cb.k <= 8) MOE_RC(8);
    else MOE_RC(MOE_MAX_K);
#undef MOE_RC
    return launch_status();
}

int launch_grouped_ffn_combine(const void* x_perm, const int32_t* offsets, int n_groups,
                               const void* const* w13, const void* const* w2, int d, int f,
                               int64_t cap_rows, const int32_t* token_row, const float* gate,
                               const void* y_shared, int64_t T, int k, void* y, void* ws,
                               hipStream_t s) {
    if (T == 0) return MOE_OK;
    CombineArgs cb;
    cb.token_row = token_row;
    cb.gate = gate;
    cb.y_shared = (const bf16_t*)y_shared;
    cb.y = (bf16_t*)y;
    cb.T = T;
    cb.k = k;
    if (cap_rows == 0) {
        // no local row: y is the shared experts' output (or zero), as the combine gives
        return launch_combine(nullptr, MOE_BF16, token_row, gate, y_shared, 1, T, d, k, y, s);
    }
    return launch_grouped_ffn(x_perm, MOE_BF16, offsets, n_groups, w13, w2, d, f, cap_rows,
                              nullptr, ws, s, nullptr, 0,
                              MOE_FFN_GATE_UP | MOE_FFN_DOWN | MOE_FFN_SMALL_GROUPS, &cb);
}

}  // namespace moe
