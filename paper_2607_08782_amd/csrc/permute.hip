// Packaging of tokens for the experts placed on this GPU (Sec. II-B of the
// Director paper: tokens are packaged and sent to the GPUs that host their
// experts; Sec. VI-A: placement x[e][j], Eq. 1 load and Eq. 3 volume).
//
// A stable counting sort of the T*k assignments into local-expert groups,
// with no host round trip:
//   count    one wave per 64 tokens: per-slot membership bitmaps in LDS,
//            popcounts -> per-block counts (or, in moe_route_package, one
//            workgroup per 64 tokens: counts of every expert, a byte each)
//   scan     one workgroup: replica ranges [lo, hi) per slot from the global
//            counts, group offsets, per-slot exclusive scan over blocks,
//            send counts per GPU
//   scatter  one wave per 64 tokens: rank = block base + popcount of the
//            lower lanes' bits; kept ranks get a row
//   gather   x_perm[p] = x[row_token[p]], 16-byte vector copies
// Every step is integer arithmetic, so the result is exact and unique.
#include "common.h"
#include "topk.h"

namespace moe {
namespace {

constexpr int PERM_TOKENS = 64;          // one wave per block of 64 tokens

struct SlotTable {
    int16_t slot_of[MOE_MAX_E];
};

struct HostTable {
    uint64_t hosts[MOE_MAX_E];
    int16_t expert_of_slot[MOE_MAX_GROUPS];
};

// The k expert ids (and gates) of token t, every load issued before the first
// use: k ids behind one wait instead of k dependent round trips.  Lanes past
// k re-read id k-1 of the same row.
__device__ __forceinline__ void load_ids(const int32_t* __restrict__ idx, int64_t t, int k,
                                         int (&ev)[MOE_MAX_K]) {
#pragma unroll
    for (int r = 0; r < MOE_MAX_K; ++r) ev[r] = idx[t * k + (r < k ? r : k - 1)];
}

__device__ __forceinline__ void load_gates(const float* __restrict__ gate, int64_t t, int k,
                                           float (&gv)[MOE_MAX_K]) {
#pragma unroll
    for (int r = 0; r < MOE_MAX_K; ++r) gv[r] = gate[t * k + (r < k ? r : k - 1)];
}

// Bit `lane` of bits[s] set iff this lane's token has an assignment to local slot s.
__device__ __forceinline__ void set_bits(const int (&ev)[MOE_MAX_K], bool valid, int k, int E,
                                         const int16_t* slot_of, unsigned long long* bits,
                                         int lane) {
    if (!valid) return;
#pragma unroll
    for (int r = 0; r < MOE_MAX_K; ++r) {
        if (r >= k) break;
        const int e = ev[r];
        const int s = (unsigned)e < (unsigned)E ? (int)slot_of[e] : -1;
        if (s >= 0) atomicOr(&bits[s], 1ull << lane);
    }
}

// Rows of the replica range: of expert e's c assignments, the host of rank q
// among its n hosts takes [q c / n, (q+1) c / n).
__device__ __forceinline__ int64_t replica_lo(int q, int64_t c, int n) {
    return (int64_t)q * c / n;
}

// send_s[j] += rows GPU j receives from every expert it hosts; the counts of
// the E experts sit in cnt_s.  Integer adds, so the order does not matter.
__device__ __forceinline__ void add_send_counts(const int32_t* cnt_s, const uint64_t* hosts,
                                                int E, int tid, int nthr, int32_t* send_s) {
    for (int e = tid; e < E; e += nthr) {
        uint64_t h = hosts[e];
        const int64_t c = cnt_s[e];
        const int n = __popcll(h);
        for (int q = 0; h; ++q, h &= h - 1ull) {
            const int j = __builtin_ctzll(h);
            atomicAdd(&send_s[j], (int32_t)(replica_lo(q + 1, c, n) - replica_lo(q, c, n)));
        }
    }
}

// off[0] = 0, off[i + 1] = size[0] + ... + size[i] for i < n; one whole wave.
__device__ __forceinline__ void wave_offsets(const int32_t* size, int n, int32_t* off, int lane) {
    int32_t carry = 0;
    for (int c0 = 0; c0 < n; c0 += 64) {
        const int i = c0 + lane;
        const int32_t v = i < n ? size[i] : 0;
        int32_t incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (i < n) off[i + 1] = carry + incl;
        carry += __shfl(incl, 63, 64);
    }
    if (lane == 0) off[0] = 0;
}

__global__ __launch_bounds__(PERM_TOKENS) void perm_count_kernel(
    const int32_t* __restrict__ idx, int64_t T, int k, int E, SlotTable tab, int n_local,
    int32_t* __restrict__ blk_counts) {
    __shared__ unsigned long long bits[MOE_MAX_GROUPS];
    __shared__ int16_t slot_lds[MOE_MAX_E];
    const int lane = threadIdx.x;
    const int64_t blk = blockIdx.x;
    const int64_t t = blk * PERM_TOKENS + lane;
    int ev[MOE_MAX_K];
    if (t < T) load_ids(idx, t, k, ev);
    for (int e = lane; e < E; e += PERM_TOKENS) slot_lds[e] = tab.slot_of[e];
    for (int s = lane; s < n_local; s += PERM_TOKENS) bits[s] = 0ull;
    __syncthreads();
    set_bits(ev, t < T, k, E, slot_lds, bits, lane);
    __syncthreads();
    for (int s = lane; s < n_local; s += PERM_TOKENS)
        blk_counts[blk * n_local + s] = __popcll(bits[s]);
}

// Counts of all E experts per block of 64 tokens, a byte each (ids distinct within a
// token: at most 64), in rows of Es = E rounded up to 4; clears coact[0, ncoact).
constexpr int ALL_THREADS = 256;

__global__ __launch_bounds__(ALL_THREADS) void perm_count_all_kernel(
    const int32_t* __restrict__ idx, int64_t T, int k, int E, int Es, uint32_t* __restrict__ table,
    int32_t* __restrict__ coact, int ncoact) {
    __shared__ uint32_t cnt[MOE_MAX_E];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * PERM_TOKENS;
    const int n = (int)(T - t0 < PERM_TOKENS ? T - t0 : PERM_TOKENS) * k;
    const int32_t* ids = idx + t0 * k;
    int e[MOE_MAX_K * PERM_TOKENS / ALL_THREADS];
#pragma unroll
    for (int u = 0; u < MOE_MAX_K * PERM_TOKENS / ALL_THREADS; ++u) {
        const int i = u * ALL_THREADS + tid;
        e[u] = ids[i < n ? i : 0];
        if (i >= n) e[u] = -1;
    }
    for (int i = tid; i < MOE_MAX_E; i += ALL_THREADS) cnt[i] = 0;
    for (int i = (int)blockIdx.x * ALL_THREADS + tid; i < ncoact; i += (int)gridDim.x * ALL_THREADS)
        coact[i] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MOE_MAX_K * PERM_TOKENS / ALL_THREADS; ++u)
        if ((unsigned)e[u] < (unsigned)E) atomicAdd(&cnt[e[u]], 1u);
    __syncthreads();
    for (int w = tid; w < Es / 4; w += ALL_THREADS)
        table[(int64_t)blockIdx.x * (Es / 4) + w] =
            cnt[4 * w] | cnt[4 * w + 1] << 8 | cnt[4 * w + 2] << 16 | cnt[4 * w + 3] << 24;
}

constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_WAVES = SCAN_THREADS / 64;
constexpr int SCAN_TILE = 8192;          // block counts staged in LDS per pass

// ALL: the block counts come from perm_count_all_kernel's table, which also gives the
// expert counts, stored to counts_out (at most ALL_MAX_BLOCKS blocks).
constexpr int ALL_MAX_BLOCKS = 512;

template <bool ALL>
__global__ __launch_bounds__(SCAN_THREADS) void perm_scan_kernel(
    const int32_t* __restrict__ counts, HostTable tab, int E, int n_local, int G, int dev,
    int64_t nblk, int32_t* __restrict__ blk_counts, int32_t* __restrict__ group_offsets,
    int32_t* __restrict__ lo_out, int32_t* __restrict__ send_counts,
    const uint8_t* __restrict__ table, int Es, int32_t* __restrict__ counts_out) {
    __shared__ uint64_t hosts_s[MOE_MAX_E];
    __shared__ int32_t cnt_s[MOE_MAX_E];
    __shared__ int32_t size_s[MOE_MAX_GROUPS], carry_s[MOE_MAX_GROUPS];
    __shared__ int32_t send_s[MOE_MAX_G];
    __shared__ int32_t tile[SCAN_TILE];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    __shared__ int16_t expert_s[ALL ? MOE_MAX_GROUPS : 1];
    for (int e = tid; e < E; e += SCAN_THREADS) {
        cnt_s[e] = ALL ? 0 : counts[e];
        hosts_s[e] = tab.hosts[e];
    }
    if (tid < MOE_MAX_G) send_s[tid] = 0;
    if (tid < MOE_MAX_GROUPS) {
        carry_s[tid] = 0;
        if (ALL) expert_s[tid] = tab.expert_of_slot[tid];
    }
    __syncthreads();
    if constexpr (ALL) {
        // a thread sums one word (four experts) over every P-th block, in 16-bit halves
        // (at most 512 blocks of at most 64)
        const int nw = Es / 4, P = SCAN_THREADS / nw;
        const int w = tid % nw, part = tid / nw;
        const uint32_t* tw = (const uint32_t*)table;
        if (part < P) {
            uint32_t lo = 0, hi = 0;
#pragma unroll 8
            for (int b = part; b < (int)nblk; b += P) {
                const uint32_t v = tw[b * nw + w];
                lo += v & 0x00ff00ffu;
                hi += (v >> 8) & 0x00ff00ffu;
            }
            // padding words past E hold zeros
            const int32_t c[4] = {(int32_t)(lo & 0xffffu), (int32_t)(hi & 0xffffu),
                                  (int32_t)(lo >> 16), (int32_t)(hi >> 16)};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c[i]) atomicAdd(&cnt_s[4 * w + i], c[i]);
        }
        __syncthreads();
        for (int e = tid; e < E; e += SCAN_THREADS) counts_out[e] = cnt_s[e];
    }
    if (tid < n_local) {
        const int e = tab.expert_of_slot[tid];
        const uint64_t h = hosts_s[e];
        const int n = __popcll(h);
        const int q = dev == 0 ? 0 : __popcll(h & (~0ull >> (64 - dev)));
        const int64_t lo = replica_lo(q, cnt_s[e], n);
        size_s[tid] = (int32_t)(replica_lo(q + 1, cnt_s[e], n) - lo);
        lo_out[tid] = (int32_t)lo;
    }
    if (send_counts) add_send_counts(cnt_s, hosts_s, E, tid, SCAN_THREADS, send_s);
    __syncthreads();
    if (wave == 0) wave_offsets(size_s, n_local, group_offsets, lane);
    if (send_counts && tid < G) send_counts[tid] = send_s[tid];

    // Per-slot exclusive scan of the block counts [nblk][n_local], a tile of
    // whole block rows at a time: coalesced loads into LDS, one wave per slot
    // (each lane a run of rows), coalesced stores.
    if (n_local <= 0 || nblk <= 0) return;
    const int64_t rows_per = SCAN_TILE / n_local;
    for (int64_t r0 = 0; r0 < nblk; r0 += rows_per) {
        const int rows = (int)(nblk - r0 < rows_per ? nblk - r0 : rows_per);
        const int n = rows * n_local;
        int32_t* g = blk_counts + r0 * n_local;
        int32_t v[SCAN_TILE / SCAN_THREADS];
#pragma unroll
        for (int u = 0; u < SCAN_TILE / SCAN_THREADS; ++u) {
            const int i = u * SCAN_THREADS + tid;
            if constexpr (ALL) {
                const int ii = i < n ? i : 0, row = (int)((unsigned)ii / (unsigned)n_local);
                v[u] = table[(r0 + row) * Es + expert_s[ii - row * n_local]];
            } else {
                v[u] = g[i < n ? i : 0];
            }
        }
#pragma unroll
        for (int u = 0; u < SCAN_TILE / SCAN_THREADS; ++u) tile[u * SCAN_THREADS + tid] = v[u];
        __syncthreads();
        const int per = (rows + 63) / 64;
        for (int s = wave; s < n_local; s += SCAN_WAVES) {
            const int b0 = lane * per;
            int32_t sum = 0;
            for (int i = 0; i < per; ++i)
                if (b0 + i < rows) sum += tile[(b0 + i) * n_local + s];
            int32_t incl = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int32_t u = __shfl_up(incl, o, 64);
                if (lane >= o) incl += u;
            }
            int32_t run = carry_s[s] + incl - sum;
            for (int i = 0; i < per; ++i) {
                if (b0 + i < rows) {
                    int32_t* p = &tile[(b0 + i) * n_local + s];
                    const int32_t c = *p;
                    *p = run;
                    run += c;
                }
            }
            const int32_t total = __shfl(incl, 63, 64);
            if (lane == 0) carry_s[s] += total;
        }
        __syncthreads();
        for (int i = tid; i < n; i += SCAN_THREADS) g[i] = tile[i];
        __syncthreads();
    }
}

__global__ __launch_bounds__(PERM_TOKENS) void perm_scatter_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ gate, int64_t T, int k, int E,
    SlotTable tab, int n_local, const int32_t* __restrict__ blk_base,
    const int32_t* __restrict__ lo_in, const int32_t* __restrict__ group_offsets,
    int32_t* __restrict__ row_token, float* __restrict__ row_gate,
    int32_t* __restrict__ token_row) {
    __shared__ unsigned long long bits[MOE_MAX_GROUPS];
    __shared__ int16_t slot_lds[MOE_MAX_E];
    __shared__ int32_t base_s[MOE_MAX_GROUPS], lo_s[MOE_MAX_GROUPS], off_s[MOE_MAX_GROUPS + 1];
    const int lane = threadIdx.x;
    const int64_t blk = blockIdx.x;
    const int64_t t = blk * PERM_TOKENS + lane;
    int ev[MOE_MAX_K];
    float gv[MOE_MAX_K];
    if (t < T) {
        load_ids(idx, t, k, ev);
        load_gates(gate, t, k, gv);
    }
    for (int e = lane; e < E; e += PERM_TOKENS) slot_lds[e] = tab.slot_of[e];
    for (int s = lane; s < n_local; s += PERM_TOKENS) {
        bits[s] = 0ull;
        base_s[s] = blk_base[blk * n_local + s];
        lo_s[s] = lo_in[s];
    }
    for (int s = lane; s <= n_local; s += PERM_TOKENS) off_s[s] = group_offsets[s];
    __syncthreads();
    set_bits(ev, t < T, k, E, slot_lds, bits, lane);
    __syncthreads();
    if (t >= T) return;
    const unsigned long long lower = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < MOE_MAX_K; ++r) {
        if (r >= k) break;
        const int e = ev[r];
        int32_t p = -1;
        const int s = (unsigned)e < (unsigned)E ? (int)slot_lds[e] : -1;
        if (s >= 0) {
            const int32_t rank = base_s[s] + __popcll(bits[s] & lower);
            const int32_t lo = lo_s[s];
            if (rank >= lo && rank < lo + (off_s[s + 1] - off_s[s])) {
                p = off_s[s] + (rank - lo);
                row_token[p] = (int32_t)t;
                row_gate[p] = gv[r];
            }
        }
        token_row[t * k + r] = p;
    }
}

// Short batches (at most SMALL_T tokens): count, scan and scatter in one
// workgroup, one wave per 64-token block, the same arithmetic as the three
// kernels above (so the same unique result), one launch instead of three.
// COUNT: the expert counts (and, with coact, the co-activation counts, E * E bins in
// dynamic LDS) are taken here too instead of read from `counts`: one launch instead
// of the histogram's and this one.  KM > 0 (COUNT, at most PLAN_IDS assignments): the
// top-k (k <= KM, top-k class C) of `scores` as well, so a decode step's routing is
// this launch after the scores.  Bound by the latency of one workgroup's chain of
// loads and barriers; each launch saved is 4-8 us of a decode step.
constexpr int SMALL_T = 1024;
constexpr int SMALL_BLK = SMALL_T / PERM_TOKENS;
constexpr int PLAN_IDS = 4096;
constexpr int PLAN_U = 4;                // assignments a thread loads at a time

// replica_lo for a short batch's counts (q <= 64, c <= SMALL_T): 32-bit, and no
// division for an expert with one host
__device__ __forceinline__ uint32_t replica_lo_small(int q, uint32_t c, int n) {
    return n == 1 ? (q ? c : 0u) : (uint32_t)q * c / (uint32_t)n;
}

struct SmallArgs {
    const int32_t* idx;                  // [T][k] (KM == 0)
    const float* gate;
    const int32_t* counts_in;            // [E] (!COUNT)
    int32_t* counts;                     // [E] (COUNT)
    int32_t* coact;                      // [E][E], nullable (COUNT)
    const float* scores;                 // [T][E], bias added (KM > 0)
    int chunks;                          // > 1: scores come in K chunks [chunk][T][E], without
    const float* bias;                   // the bias; their sums + bias go to sums (which may be
    float* sums;                         // chunk 0 itself), read by the top-k
    int32_t* idx_out;                    // [T][k] (KM > 0)
    float* gate_out;
    int renorm;
    int T, k, E, n_local, G, dev;
    int32_t* group_offsets;
    int32_t* row_token;
    float* row_gate;
    int32_t* token_row;
    int32_t* send_counts;
};

template <bool COUNT, int KM = 0, int C = 0>
__global__ __launch_bounds__(SMALL_T) void perm_small_kernel(SmallArgs a, SlotTable st,
                                                             HostTable ht) {
    __shared__ unsigned long long bits[SMALL_BLK][MOE_MAX_GROUPS];
    __shared__ int32_t base[SMALL_BLK][MOE_MAX_GROUPS];
    __shared__ int16_t slot_lds[MOE_MAX_E];
    __shared__ uint64_t hosts_s[MOE_MAX_E];
    __shared__ int32_t cnt_s[MOE_MAX_E], send_s[MOE_MAX_G];
    __shared__ int32_t lo_s[MOE_MAX_GROUPS], size_s[MOE_MAX_GROUPS], off_s[MOE_MAX_GROUPS + 1];
    __shared__ int32_t ids_s[KM > 0 ? PLAN_IDS : 1];
    __shared__ float gates_s[KM > 0 ? PLAN_IDS : 1];
    extern __shared__ __attribute__((aligned(16))) int32_t co_s[];   // [E][E] with coact
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int T = a.T, k = a.k, E = a.E, n_local = a.n_local;
    const int nblk = (int)ceil_div(T, PERM_TOKENS);
    // slots of wave 0's lanes, read before the first wait
    int my_expert[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
        my_expert[c] = wave == 0 && lane + 64 * c < n_local ? ht.expert_of_slot[lane + 64 * c] : 0;
    for (int e = tid; e < E; e += SMALL_T) {
        slot_lds[e] = st.slot_of[e];
        cnt_s[e] = COUNT ? 0 : a.counts_in[e];
        hosts_s[e] = ht.hosts[e];
    }
    if (tid < MOE_MAX_G) send_s[tid] = 0;
    for (int i = tid; i < nblk * MOE_MAX_GROUPS; i += SMALL_T)
        bits[i / MOE_MAX_GROUPS][i % MOE_MAX_GROUPS] = 0ull;
    const bool coact = COUNT && a.coact != nullptr;
    if (coact)
        for (int i = tid; i < E * E; i += SMALL_T) co_s[i] = 0;
    if constexpr (KM > 0) {
        const float* scores = a.scores;
        if (a.chunks > 1) {
            for (int i = tid; i < T * E; i += SMALL_T) {
                const float v = sum_chunks(a.scores + i, (int64_t)T * E, a.chunks);
                a.sums[i] = a.bias ? v + a.bias[i % E] : v;
            }
            __syncthreads();
            scores = a.sums;
        }
        topk_tokens<KM, C, 1>(scores, E, T, 0, E, k, a.renorm, ids_s, gates_s);
    }
    __syncthreads();
    // The assignments i = t k + r, one per thread and PLAN_U per thread at a time: f(i,
    // token, expert).  A loop over a token's k assignments by one thread each waited
    // for k dependent LDS round trips.  (i + 0.5) / k truncates to the token exactly: n
    // is at most 2^14.
    const int n = T * k;
    const int32_t* ids = KM > 0 ? ids_s : a.idx;
    const float rk = 1.0f / (float)k;
    auto each = [&](auto f) {
        for (int i0 = tid; i0 < n; i0 += PLAN_U * SMALL_T) {
            int e[PLAN_U];
#pragma unroll
            for (int u = 0; u < PLAN_U; ++u) {
                const int i = i0 + u * SMALL_T;
                e[u] = ids[i < n ? i : i0];
            }
#pragma unroll
            for (int u = 0; u < PLAN_U; ++u) {
                const int i = i0 + u * SMALL_T;
                if (i < n) f(i, (int)(((float)i + 0.5f) * rk), e[u]);
            }
        }
    };
    each([&](int i, int t, int e) {
        // out-of-range expert ids are ignored rather than counted out of bounds
        if ((unsigned)e >= (unsigned)E) return;
        const int s = slot_lds[e];
        if (s >= 0) atomicOr(&bits[t / PERM_TOKENS][s], 1ull << (t % PERM_TOKENS));
        if (COUNT) atomicAdd(&cnt_s[e], 1);
        if (coact)
            for (int q = 0; q < k; ++q) {
                const int e2 = ids[t * k + q];
                if ((unsigned)e2 < (unsigned)E) atomicAdd(&co_s[e * E + e2], 1);
            }
    });
    __syncthreads();
    if (wave == 0) {
        // replica range, group size and offset of every slot (at most 128)
        int32_t carry = 0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int s = lane + 64 * c;
            int32_t size = 0;
            if (s < n_local) {
                const uint64_t h = hosts_s[my_expert[c]];
                const int hosts = __popcll(h);
                const int q = a.dev == 0 ? 0 : __popcll(h & (~0ull >> (64 - a.dev)));
                const uint32_t cnt = (uint32_t)cnt_s[my_expert[c]];
                const uint32_t lo = replica_lo_small(q, cnt, hosts);
                lo_s[s] = (int32_t)lo;
                size = (int32_t)(replica_lo_small(q + 1, cnt, hosts) - lo);
                size_s[s] = size;
            }
            const int32_t incl = wave_incl_scan(size);
            if (s < n_local) off_s[s + 1] = carry + incl;
            carry += __shfl(incl, 63, 64);
        }
        if (lane == 0) off_s[0] = 0;
    } else if (wave < 3) {
        for (int s = tid - 64; s < n_local; s += 128) {
            int32_t run = 0;
            for (int b = 0; b < nblk; ++b) {
                base[b][s] = run;
                run += __popcll(bits[b][s]);
            }
        }
    } else if (a.send_counts) {
        for (int e = tid - 192; e < E; e += SMALL_T - 192) {
            uint64_t h = hosts_s[e];
            const uint32_t c = (uint32_t)cnt_s[e];
            const int hosts = __popcll(h);
            for (int q = 0; h; ++q, h &= h - 1ull)
                atomicAdd(&send_s[__builtin_ctzll(h)],
                          (int32_t)(replica_lo_small(q + 1, c, hosts) - replica_lo_small(q, c, hosts)));
        }
    }
    __syncthreads();
    // the stores come after the last barrier: a barrier waits for those before it
    each([&](int i, int t, int e) {
        int32_t p = -1;
        const int s = (unsigned)e < (unsigned)E ? (int)slot_lds[e] : -1;
        if (s >= 0) {
            const int b = t / PERM_TOKENS;
            const int32_t rank =
                base[b][s] + __popcll(bits[b][s] & ((1ull << (t % PERM_TOKENS)) - 1ull));
            const int32_t lo = lo_s[s];
            if (rank >= lo && rank < lo + size_s[s]) {
                p = off_s[s] + (rank - lo);
                a.row_token[p] = t;
                a.row_gate[p] = KM > 0 ? gates_s[i] : a.gate[i];
            }
        }
        a.token_row[i] = p;
        if (KM > 0) {
            a.idx_out[i] = e;
            a.gate_out[i] = gates_s[i];
        }
    });
    for (int sl = tid; sl <= n_local; sl += SMALL_T) a.group_offsets[sl] = off_s[sl];
    if (a.send_counts && tid < a.G) a.send_counts[tid] = send_s[tid];
    if (COUNT)
        for (int e = tid; e < E; e += SMALL_T) a.counts[e] = cnt_s[e];
    if (coact)
        for (int i = tid; i < E * E; i += SMALL_T) a.coact[i] = co_s[i];
}

template <typename U>
__global__ __launch_bounds__(256) void gather_rows_kernel(
    const U* __restrict__ x, const int32_t* __restrict__ row_token,
    const int32_t* __restrict__ total, int units_per_row, U* __restrict__ x_perm) {
    const int32_t N = *total;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int64_t p = (int64_t)blockIdx.x * 4 + wave; p < N; p += (int64_t)gridDim.x * 4) {
        const int64_t t = row_token[p];
        const U* src = x + t * units_per_row;
        U* dst = x_perm + p * units_per_row;
        for (int u = lane; u < units_per_row; u += 64) dst[u] = src[u];
    }
}

// Scratch of moe_permute_noalloc: the per-block slot counts and replica
// offsets that moe_permute keeps in the caller's workspace, held instead in a
// device array of this library (one copy per GPU, kept until the process
// ends).  Every byte the kernels read is written earlier in the same call, so
// nothing needs clearing; calls that overlap on one GPU race on it.
static __device__ __align__(256) unsigned char scratch[MOE_PERMUTE_NOALLOC_MAX_WS];

}  // namespace

// Device address of `scratch` on the current device.  The array's name in host
// code is a host-side stand-in, not a device address, so the address is looked
// up once per device, with that device current, and kept.
int permute_scratch(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static void* addr[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_ERR_DEVICE;
    std::lock_guard<std::mutex> guard(lock);
    if (addr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr)
            return MOE_ERR_DEVICE;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return MOE_OK;
}

size_t permute_ws_bytes(int64_t T, int k, int E) {
    (void)k;
    const int64_t nblk = ceil_div(T, PERM_TOKENS);
    const int64_t slots = E < MOE_MAX_GROUPS ? E : MOE_MAX_GROUPS;
    return (size_t)(nblk * slots + MOE_MAX_GROUPS) * sizeof(int32_t) + 256;
}

static void fill_tables(const PermuteTables& tabs, SlotTable& st, HostTable& ht) {
    for (int e = 0; e < MOE_MAX_E; ++e) {
        st.slot_of[e] = tabs.slot_of[e];
        ht.hosts[e] = tabs.hosts[e];
    }
    for (int i = 0; i < MOE_MAX_GROUPS; ++i) ht.expert_of_slot[i] = tabs.expert_of_slot[i];
}

// x_perm[p] = x[row_token[p]] for the rows the maps hold (nothing when d = 0)
static void launch_gather_rows(const void* x, int dtype, int64_t T, int d, int k, int n_local,
                               void* x_perm, int64_t cap_rows, const int32_t* group_offsets,
                               const int32_t* row_token, hipStream_t s) {
    if (T <= 0 || n_local <= 0 || d <= 0) return;
    const size_t row_bytes = (size_t)d * (dtype == MOE_BF16 ? 2 : 4);
    int64_t max_rows = cap_rows;
    if (max_rows > T * (int64_t)k) max_rows = T * (int64_t)k;
    int64_t blocks = ceil_div(max_rows, 4);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    const int32_t* total = group_offsets + n_local;
    if (row_bytes % 16 == 0)
        hipLaunchKernelGGL(gather_rows_kernel<uint4>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const uint4*)x, row_token, total, (int)(row_bytes / 16),
                           (uint4*)x_perm);
    else if (row_bytes % 4 == 0)
        hipLaunchKernelGGL(gather_rows_kernel<uint32_t>, dim3((unsigned)blocks), dim3(256), 0,
                           s, (const uint32_t*)x, row_token, total, (int)(row_bytes / 4),
                           (uint32_t*)x_perm);
    else
        hipLaunchKernelGGL(gather_rows_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0,
                           s, (const uint16_t*)x, row_token, total, (int)(row_bytes / 2),
                           (uint16_t*)x_perm);
}

int launch_permute(const void* x, int dtype, const int32_t* idx, const float* gate,
                   const int32_t* counts, int64_t T, int d, int k, int E, const PermuteTables& tabs,
                   int n_local, int G, int dev, void* x_perm, int64_t cap_rows,
                   int32_t* group_offsets, int32_t* row_token, float* row_gate, int32_t* token_row,
                   int32_t* send_counts, void* ws, hipStream_t s) {
    const int64_t nblk = ceil_div(T, PERM_TOKENS);
    int32_t* lo_ws = (int32_t*)ws;
    int32_t* blk = lo_ws + MOE_MAX_GROUPS;
    SlotTable st;
    HostTable ht;
    fill_tables(tabs, st, ht);

    if (T <= SMALL_T) {
        SmallArgs a = {};
        a.idx = idx;
        a.gate = gate;
        a.counts_in = counts;
        a.T = (int)T, a.k = k, a.E = E, a.n_local = n_local, a.G = G, a.dev = dev;
        a.group_offsets = group_offsets;
        a.row_token = row_token;
        a.row_gate = row_gate;
        a.token_row = token_row;
        a.send_counts = send_counts;
        hipLaunchKernelGGL(perm_small_kernel<false>, dim3(1), dim3(SMALL_T), 0, s, a, st, ht);
    } else {
        if (n_local > 0)
            hipLaunchKernelGGL(perm_count_kernel, dim3((unsigned)nblk), dim3(PERM_TOKENS), 0, s,
                               idx, T, k, E, st, n_local, blk);
        hipLaunchKernelGGL(perm_scan_kernel<false>, dim3(1), dim3(SCAN_THREADS), 0, s, counts, ht, E,
                           n_local, G, dev, n_local > 0 ? nblk : (int64_t)0, blk, group_offsets,
                           lo_ws, send_counts, (const uint8_t*)nullptr, 0, (int32_t*)nullptr);
        hipLaunchKernelGGL(perm_scatter_kernel, dim3((unsigned)nblk), dim3(PERM_TOKENS), 0, s,
                           idx, gate, T, k, E, st, n_local, blk, lo_ws, group_offsets, row_token,
                           row_gate, token_row);
    }
    launch_gather_rows(x, dtype, T, d, k, n_local, x_perm, cap_rows, group_offsets, row_token, s);
    return launch_status();
}

namespace {

// The packaging launch with the counts, and with the top-k when scores are given;
// KM, C as topk_group.
template <int KM, int C>
int launch_small_plan(const SmallArgs& a, const SlotTable& st, const HostTable& ht, hipStream_t s) {
    const size_t lds = a.coact ? (size_t)a.E * a.E * sizeof(int32_t) : 0;
    if (lds > 0 && allow_dynamic_lds<perm_small_kernel<true, KM, C>>(lds) != MOE_OK)
        return MOE_ERR_DEVICE;
    hipLaunchKernelGGL((perm_small_kernel<true, KM, C>), dim3(1), dim3(SMALL_T), lds, s, a, st, ht);
    return launch_status();
}

template <int KM>
int launch_small_topk(const SmallArgs& a, const SlotTable& st, const HostTable& ht, hipStream_t s) {
    switch (topk_class(a.E)) {
        case 0: return launch_small_plan<KM, 0>(a, st, ht, s);
        case 1: return launch_small_plan<KM, 1>(a, st, ht, s);
        case 2: return launch_small_plan<KM, 2>(a, st, ht, s);
        case 3: return launch_small_plan<KM, 3>(a, st, ht, s);
        default: return launch_small_plan<KM, 4>(a, st, ht, s);
    }
}

// Whether the packaging launch also takes the top-k: at most one pass of its 1024
// threads (L lanes a token), and the ids within PLAN_IDS.  Measured per step against
// the top-k launch of its own, see launch_route_package.
bool plan_topk(int64_t T, int k, int E) {
    const int C = topk_class(E);
    const int L = C == 0 ? 4 : C <= 2 ? 8 : C == 3 ? 16 : 32;
    return T * L <= SMALL_T && T * k <= PLAN_IDS;
}

}  // namespace

// Routing, counts and packaging of one batch: moe_route_topk, moe_expert_histogram and
// moe_permute, in fewer launches where the batch is short (at most SMALL_T tokens;
// co-activation bins that fit LDS): the counts move into the packaging launch, and
// for decode-sized bf16 batches the top-k too.
int launch_route_package(const void* x, int dtype, const void* w, const float* bias, int64_t T,
                         int d, int E, int k, int flags, float* logits, int32_t* idx, float* gate,
                         void* ws_route, int32_t* counts, int32_t* coact, const PermuteTables& tabs,
                         int n_local, int G, int dev, void* x_perm, int64_t cap_rows,
                         int32_t* group_offsets, int32_t* row_token, float* row_gate,
                         int32_t* token_row, int32_t* send_counts, void* ws_perm, hipStream_t s) {
    const bool small = T > 0 && T <= SMALL_T && (!coact || E <= 128);
    const bool given = (flags & MOE_LOGITS_IN) != 0;
    const bool topk = small && plan_topk(T, k, E) &&
                      (given || (dtype == MOE_BF16 && route_short(T, d, E)));
    const int dcopy = x_perm ? d : 0;
    int st = MOE_OK, chunks = 1;
    const float* scores = logits;
    if (!topk) {
        st = launch_route_topk(x, dtype, w, bias, T, d, E, k, flags, logits, idx, gate, ws_route, s);
    } else if (!given) {
        chunks = route_chunks(T, d, E);
        float* out = chunks > 1 || !logits ? (float*)ws_route : logits;
        scores = out;
        st = launch_scores_short(x, w, bias, T, d, E, out, s);
    }
    if (st != MOE_OK) return st;
    // long batches of up to 512 blocks: one count of every expert per block serves the
    // expert counts and the slots' scan, and clears coact (the histogram's clearing and
    // counting launches left out: DeepSeek-V2-Lite prefill step 540 -> 534 us, 4096 tokens
    // of the Qwen1.5 shape 396 -> 392, 16384 of the Qwen3 shape, with coact, even); the
    // table lies behind the scan's block counts where the workspace has room for both.
    // Longer batches: the one workgroup of the scan would read the whole table
    const int64_t nblk = ceil_div(T, PERM_TOKENS);
    const int Es = (E + 3) & ~3, max_slots = E < MOE_MAX_GROUPS ? E : MOE_MAX_GROUPS;
    if (!small && T > 0 && nblk <= ALL_MAX_BLOCKS && n_local > 0 && Es + 4 * n_local <= 4 * max_slots) {
        int32_t* lo_ws = (int32_t*)ws_perm;
        int32_t* blk = lo_ws + MOE_MAX_GROUPS;
        uint32_t* table = (uint32_t*)(blk + nblk * n_local);
        SlotTable stab;
        HostTable htab;
        fill_tables(tabs, stab, htab);
        hipLaunchKernelGGL(perm_count_all_kernel, dim3((unsigned)nblk), dim3(ALL_THREADS), 0, s, idx,
                           T, k, E, Es, table, coact, coact ? E * E : 0);
        if (coact) {
            st = launch_coact(idx, T, k, E, coact, s);
            if (st != MOE_OK) return st;
        }
        hipLaunchKernelGGL(perm_scan_kernel<true>, dim3(1), dim3(SCAN_THREADS), 0, s,
                           (const int32_t*)nullptr, htab, E, n_local, G, dev, nblk, blk,
                           group_offsets, lo_ws, send_counts, (const uint8_t*)table, Es, counts);
        hipLaunchKernelGGL(perm_scatter_kernel, dim3((unsigned)nblk), dim3(PERM_TOKENS), 0, s, idx,
                           gate, T, k, E, stab, n_local, blk, lo_ws, group_offsets, row_token,
                           row_gate, token_row);
        launch_gather_rows(x, dtype, T, dcopy, k, n_local, x_perm, cap_rows, group_offsets,
                           row_token, s);
        return launch_status();
    }
    if (!small) {
        st = launch_histogram(idx, T, k, E, counts, coact, s);
        if (st != MOE_OK) return st;
        return launch_permute(x, dtype, idx, gate, counts, T, dcopy, k, E, tabs, n_local, G, dev,
                              x_perm, cap_rows, group_offsets, row_token, row_gate, token_row,
                              send_counts, ws_perm, s);
    }
    SlotTable slots;
    HostTable hosts;
    fill_tables(tabs, slots, hosts);
    SmallArgs a = {};
    a.idx = idx;
    a.gate = gate;
    a.counts = counts;
    a.coact = coact;
    a.scores = scores;
    a.chunks = chunks;
    a.bias = bias;
    a.sums = logits ? logits : (float*)ws_route;
    a.idx_out = idx;
    a.gate_out = gate;
    a.renorm = (flags & MOE_RENORM) ? 1 : 0;
    a.T = (int)T, a.k = k, a.E = E, a.n_local = n_local, a.G = G, a.dev = dev;
    a.group_offsets = group_offsets;
    a.row_token = row_token;
    a.row_gate = row_gate;
    a.token_row = token_row;
    a.send_counts = send_counts;
    if (!topk) st = launch_small_plan<0, 0>(a, slots, hosts, s);
    else if (k <= 2) st = launch_small_topk<2>(a, slots, hosts, s);
    else if (k <= 4) st = launch_small_topk<4>(a, slots, hosts, s);
    else if (k <= 8) st = launch_small_topk<8>(a, slots, hosts, s);
    else st = launch_small_topk<MOE_MAX_K>(a, slots, hosts, s);
    if (st != MOE_OK) return st;
    launch_gather_rows(x, dtype, T, dcopy, k, n_local, x_perm, cap_rows, group_offsets, row_token, s);
    return launch_status();
}

}  // namespace moe
