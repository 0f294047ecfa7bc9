// build.hip -- graph builder: raw edge list -> degree-ordered directed graph
// with co-located metadata, its in-edge index and the survey's tile plan.
//
// Phases (all device-resident after the upload):
//   0 canonicalise: (u,v,t) -> key (min<<b | max), self-loops to a sentinel
//   1 radix sort of (key, t)
//   2 dedup: one edge per pair with the minimum time (the chronologically
//     first copy, Datasets subsection)
//   3 degree d(v) of the simple graph, then the order <+ (Preliminaries):
//     sort of (d(v), hash(v)) gives every vertex its rank
//   4 orient each edge from the lower to the higher rank and sort by
//     (source rank, target rank): rows ascend in the order <+
//   5 CSR with the time of each edge and the label of its target stored
//     beside it (Adj+^m of the Graph Storage subsection)
//   6 in-edge index: for every target q the list of (p, slot of q in p's row)
//     whose remaining row is non-empty -- the work the survey streams
//   7 plan: split each target's list into tiles and class targets by d+(q)
#include <algorithm>
#include <memory>
#include <vector>

#include "graph.hpp"
#include "plan.hpp"

using namespace tp;

namespace {

constexpr int kB = 256;

__device__ __forceinline__ uint64_t pair_key(uint32_t lo, uint32_t hi, int nb)
{
    return ((uint64_t)lo << nb) | hi;
}

// ------------------------------------------------------------ phase 0

// Graphs of a batch: graph g owns edges [eoff[g], eoff[g+1]) with local
// vertex ids < vcnt[g], which map to global ids voff[g] + local.
struct BatchMap {
    uint32_t n_graphs;
    const uint64_t *eoff;  // [n_graphs + 1]
    const uint32_t *voff;  // [n_graphs + 1]
};

// Pair keys through the two pair sorts: (g << 2 lb) | (a << lb) | b for two
// ids (vertices, then ranks) a, b local to graph g.  A batch's ranks are
// graph-major like its ids (graph g holds ranks voff[g] .. voff[g+1] - 1),
// so local ids and local ranks share the layout.  With local ids a batch's
// keys take 2 lb + gb bits (lb: bits of the largest graph's ids, gb: bits of
// the graph index) instead of 2 nb (nb: bits of all ids together): 47
// against 56 bits for the 20,000-graph batch, one radix pass fewer in each
// sort.  voff null: global ids, g = 0, lb = nb (single graphs, and batches
// whose local layout would be longer).
struct PairCode {
    int lb;
    const uint32_t *voff;
    __device__ __forceinline__ uint64_t pack(uint32_t g, uint32_t a, uint32_t b) const
    {
        return ((uint64_t)g << (2 * lb)) | ((uint64_t)a << lb) | b;
    }
    // first global id (or rank) of the key's graph
    __device__ __forceinline__ uint32_t base(uint64_t k) const { return voff ? voff[k >> (2 * lb)] : 0u; }
    __device__ __forceinline__ uint32_t hi(uint64_t k) const { return base(k) + (uint32_t)((k >> lb) & ((1ull << lb) - 1)); }
    __device__ __forceinline__ uint32_t lo(uint64_t k) const { return base(k) + (uint32_t)(k & ((1ull << lb) - 1)); }
};

__device__ __forceinline__ uint32_t graph_of_edge(const BatchMap &bm, size_t i)
{
    uint32_t a = 0, b = bm.n_graphs;  // eoff[a] <= i < eoff[b]
    while (b - a > 1) {
        const uint32_t mid = (a + b) >> 1;
        if (bm.eoff[mid] <= i) a = mid;
        else b = mid;
    }
    return a;
}

// Each workgroup canonicalises one contiguous span of `per_block` raw edges,
// so in a batch a thread finds the graph of its first edge by binary search
// and then only steps forward through the edge offsets.
// dbit = 1 (directed inputs) appends the direction of the raw edge to its
// key: 0 for lower id -> higher id, 1 for the reverse.
__global__ __launch_bounds__(kB) void k_canon(const uint32_t *src, const uint32_t *dst, const uint32_t *ts, size_t M, uint32_t n,
                        PairCode pc, int dbit, uint64_t sentinel, uint64_t *keys, uint32_t *vals,
                        unsigned long long *bad, unsigned long long *loops, BatchMap bm, size_t per_block)
{
    __shared__ unsigned long long tmp[kB / kWave];
    unsigned long long nbad = 0, nloop = 0;
    const size_t begin = blockIdx.x * per_block;
    const size_t end = begin + per_block < M ? begin + per_block : M;
    size_t i = begin + threadIdx.x;
    uint32_t g = 0;
    if (bm.n_graphs && i < end) g = graph_of_edge(bm, i);
    for (; i < end; i += blockDim.x) {
        uint32_t a = src[i], b = dst[i];
        bool ok;
        uint32_t kg = 0;  // graph index of the key (local layout)
        if (bm.n_graphs) {
            // local ids of graph g: kept local with the graph in the key, or
            // made global
            while (bm.eoff[g + 1] <= i) ++g;
            const uint32_t base = bm.voff[g], cnt = bm.voff[g + 1] - base;
            ok = a < cnt && b < cnt;
            if (pc.voff) {
                kg = g;
            } else {
                a += base;
                b += base;
            }
        } else {
            ok = a < n && b < n;
        }
        nbad += ok ? 0 : 1;
        uint64_t k;
        if (!ok || a == b) {
            k = sentinel;
            nloop += (ok && a == b) ? 1 : 0;
        } else {
            k = a < b ? pc.pack(kg, a, b) : pc.pack(kg, b, a);
            k = (k << dbit) | (uint64_t)(dbit && a > b);
        }
        keys[i] = k;
        vals[i] = ts ? ts[i] : 0u;
    }
    block_add<kB>(nbad, tmp, bad);
    block_add<kB>(nloop, tmp, loops);
}

// ------------------------------------------------------------ phase 2

// A block takes a tile of kCompTile consecutive sorted pairs and wave w the
// tile's w-th part, 64 consecutive pairs at a time (lane l takes pair
// 64 j + l), so that every load is coalesced; the unique pairs leave in the
// same order.
constexpr int kCompItems = 16;
constexpr size_t kCompTile = (size_t)kB * kCompItems;
constexpr size_t kCompWave = (size_t)kWave * kCompItems;

// Is pair i the first of its run?  `k` is keys[i]; the previous key comes
// from the lane below, or from memory for lane 0.
// Keys carry dbit direction bits below the pair, which runs ignore.
__device__ __forceinline__ bool run_head(const uint64_t *keys, size_t i, size_t n, uint64_t k, int dbit)
{
    uint64_t prev = __shfl_up(k, 1, kWave);
    if (lane_id() == 0 && i < n) prev = i ? keys[i - 1] : ~k;
    return i < n && (prev >> dbit) != (k >> dbit);
}

// Unique pairs of this wave's part of the tile.
__device__ __forceinline__ uint64_t wave_heads(const uint64_t *keys, size_t n, size_t wbase, int dbit)
{
    uint64_t c = 0;
    for (int j = 0; j < kCompItems; ++j) {
        const size_t i = wbase + (size_t)j * kWave + lane_id();
        const uint64_t k = i < n ? keys[i] : 0ull;
        c += (uint64_t)__popcll(__ballot(run_head(keys, i, n, k, dbit)));
    }
    return c;
}

// (The self-loops, at the end of the M sorted keys, are counted on the device
// and left out.)
__global__ __launch_bounds__(kB) void k_dedup_count(const uint64_t *keys, const unsigned long long *loops, size_t M,
                                                    int dbit, uint64_t *tile_cnt)
{
    __shared__ uint64_t tmp[kB / kWave];
    const size_t n = M - (size_t)*loops;
    const int w = threadIdx.x / kWave;
    const uint64_t c = wave_heads(keys, n, blockIdx.x * kCompTile + (size_t)w * kCompWave, dbit);
    if (lane_id() == 0) tmp[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int x = 0; x < kB / kWave; ++x) t += tmp[x];
        tile_cnt[blockIdx.x] = t;
    }
}

// Lane l's 64-bit value, in a scalar register (the builtin returns a signed
// 32-bit int: each half is widened as unsigned).
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l)
{
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    return ((uint64_t)hi << 32) | lo;
}

// One pair per run with its earliest time; with direction bits (dbit = 1)
// also the directions of its copies (bit 0: lower -> higher id, bit 1: the
// reverse) into udir.  The wave keeps its 16 rounds of keys and times in
// registers and reduces the runs of a round by shuffles, as many steps as its
// longest run needs (few rounds of a large graph hold a run above 2); a run
// that goes on is carried from the round after it, and past the wave's part
// it is walked by the whole wave.  (Walked copy by copy by its head's lane, the
// 100 copies of a small graph's hub pair took 86 of its build's 1200 us, now
// 14.)
__global__ __launch_bounds__(kB) void k_dedup_write(const uint64_t *keys, const uint32_t *vals,
                                                    const unsigned long long *loops, size_t M, int dbit,
                                                    const uint64_t *tile_off, uint64_t *ukey, uint32_t *uts,
                                                    uint8_t *udir)
{
    __shared__ uint64_t tmp[kB / kWave];
    const size_t n = M - (size_t)*loops;
    const int w = threadIdx.x / kWave;
    const unsigned lane = lane_id();
    const size_t wbase = blockIdx.x * kCompTile + (size_t)w * kCompWave;
    uint64_t kk[kCompItems];
    uint64_t hm[kCompItems];  // each round's heads
    uint32_t tt[kCompItems];
    uint64_t c = 0;
#pragma unroll
    for (int j = 0; j < kCompItems; ++j) {
        const size_t i = wbase + (size_t)j * kWave + lane;
        kk[j] = i < n ? keys[i] : 0ull;
        tt[j] = i < n ? vals[i] : 0xffffffffu;
    }
#pragma unroll
    for (int j = 0; j < kCompItems; ++j) {
        const size_t i = wbase + (size_t)j * kWave + lane;
        uint64_t prev = __shfl_up(kk[j], 1, kWave);
        if (j > 0) {
            const uint64_t last = readlane64(kk[j - 1], kWave - 1);
            if (lane == 0) prev = last;
        } else if (lane == 0 && i < n) {
            prev = i ? keys[i - 1] : ~kk[j];
        }
        hm[j] = __ballot(i < n && (prev >> dbit) != (kk[j] >> dbit));
        c += (uint64_t)__popcll(hm[j]);
    }
    if (lane == 0) tmp[w] = c;
    __syncthreads();
    uint64_t pos = tile_off[blockIdx.x] + c;  // past this wave's heads
    for (int x = 0; x < w; ++x) pos += tmp[x];
    if (c == 0) return;
    // the part of the wave's last run past its part
    uint32_t carry_t = 0xffffffffu, carry_d = 0;
    const size_t wend = wbase + kCompWave;
    if (wend < n) {
        const uint64_t pk = readlane64(kk[kCompItems - 1], kWave - 1) >> dbit;
        for (size_t b = wend;; b += kWave) {
            const size_t x = b + lane;
            const uint64_t k = x < n ? keys[x] : 0ull;
            const bool same = x < n && (k >> dbit) == pk;
            if (same) {
                carry_t = min(carry_t, vals[x]);
                carry_d |= 1u << (k & (uint64_t)dbit);
            }
            if (__ballot(same) != ~0ull) break;
        }
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) {
            carry_t = min(carry_t, (uint32_t)__shfl_xor(carry_t, d, kWave));
            carry_d |= (uint32_t)__shfl_xor(carry_d, d, kWave);
        }
    }
    // rounds from the last to the first
#pragma unroll
    for (int j = kCompItems - 1; j >= 0; --j) {
        const size_t base = wbase + (size_t)j * kWave;
        if (base >= n) continue;
        const uint32_t valid = (uint32_t)min((size_t)kWave, n - base);
        const uint64_t k = kk[j], b = hm[j];
        uint32_t t = tt[j];
        uint32_t d = lane < valid ? 1u << (k & (uint64_t)dbit) : 0u;
        // lanes after this one in its run, in this round
        const uint64_t above = lane == kWave - 1 ? 0ull : (b & (~0ull << (lane + 1)));
        const uint32_t end = above ? (uint32_t)__ffsll((long long)above) - 1 : valid;
        const uint32_t rest = lane < valid ? end - lane - 1 : 0u;
        for (uint32_t step = 1; __ballot(rest >= step); step <<= 1) {
            const uint32_t ot = __shfl_down(t, step, kWave);
            if (rest >= step) t = min(t, ot);
            if (udir) {
                const uint32_t od = __shfl_down(d, step, kWave);
                if (rest >= step) d |= od;
            }
        }
        // the round's last run goes on after it
        if (end == valid) {
            t = min(t, carry_t);
            d |= carry_d;
        }
        pos -= (uint64_t)__popcll(b);
        if ((b >> lane) & 1ull) {
            const uint64_t at = pos + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
            ukey[at] = k >> dbit;
            uts[at] = t;
            if (udir) udir[at] = (uint8_t)d;
        }
        // carried into the round before: this round's first run, unless it
        // starts here
        const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)t, 0);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, 0);
        carry_t = (b & 1ull) ? 0xffffffffu : t0;
        carry_d = (b & 1ull) ? 0u : d0;
    }
}

// ------------------------------------------------------------ phase 3

// Add the lengths of the runs of equal values among a wave's 64 values
// (sorted; lanes with ok == false form a suffix) to cnt[value]: one atomic
// per run, to increasing addresses.
__device__ __forceinline__ void add_runs(uint64_t v, bool ok, uint32_t *cnt)
{
    const unsigned lane = lane_id();
    const uint64_t prev = __shfl_up(v, 1, kWave);
    const bool head = ok && (lane == 0 || prev != v);
    const uint64_t heads = __ballot(head);
    const uint32_t valid = (uint32_t)__popcll(__ballot(ok));
    if (head) {
        const uint64_t above = lane == 63 ? 0ull : (heads & (~0ull << (lane + 1)));
        const uint32_t next = above ? (uint32_t)__ffsll((long long)above) - 1 : valid;
        atomicAdd(&cnt[v], next - lane);
    }
}

// d(v) counts each unique pair at both ends.  The pairs are sorted by their
// lower end, so that half is counted by runs; the higher ends are written
// out here (one read of the pairs for both), sorted on their own (a 32-bit
// radix sort) and counted the same way by k_degree_runs, instead of one
// scattered atomic per pair.
__global__ void k_degree_low(const uint64_t *ukey, size_t m, PairCode pc, uint32_t *deg, uint32_t *hi)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t base = blockIdx.x * (size_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); base < m; base += stride) {
        const size_t i = base + lane_id();
        const bool ok = i < m;
        const uint64_t k = ok ? ukey[i] : 0ull;
        add_runs(ok ? pc.hi(k) : ~0ull, ok, deg);
        if (ok) hi[i] = pc.lo(k);
    }
}

__global__ void k_degree_runs(const uint32_t *v, size_t m, uint32_t *deg)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t base = blockIdx.x * (size_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); base < m; base += stride) {
        const size_t i = base + lane_id();
        const bool ok = i < m;
        add_runs(ok ? v[i] : ~0ull, ok, deg);
    }
}

// The largest degree and the largest label (vlab null: 0).
__global__ __launch_bounds__(kB) void k_vertex_max(const uint32_t *deg, const uint8_t *vlab, size_t n,
                                                   unsigned long long *dmax, unsigned long long *lmax)
{
    __shared__ unsigned long long tmp[kB / kWave];
    uint32_t d = 0, l = 0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        d = max(d, deg[i]);
        if (vlab) l = max(l, (uint32_t)vlab[i]);
    }
    block_max<kB>(d, tmp, dmax);
    block_max<kB>(l, tmp, lmax);
}

// The higher ends counted in LDS: they are first partitioned by their top bits
// (one radix pass, in place of the three or four of a sort), each part an id
// range of 2^log_range.  A workgroup takes `chunk` consecutive ends, and for
// every part among them counts the ends of 2^kCountLog ids at a time, then adds
// the counts to deg.  (1.05e9 ends: 11.2 ms with the partition, 17.9 with the
// sort; 231e6 ends of a 1200-graph batch 2.1 against 4.1 ms.)
constexpr int kCountBlock = 1024;
constexpr int kCountLog = 15;  // 32-bit counters, 128 KB of the compute unit's 160
__global__ __launch_bounds__(kCountBlock) void k_degree_count(const uint32_t *v, size_t m, const uint64_t *start,
                                                              uint32_t parts, int log_range, size_t chunk, uint32_t *deg)
{
    extern __shared__ uint32_t cnt[];
    const size_t lo = blockIdx.x * chunk, hi = lo + chunk < m ? lo + chunk : m;
    const int log_span = log_range < kCountLog ? log_range : kCountLog;
    const uint32_t span = 1u << log_span;
    // the part that holds `lo`: start[d] <= lo < start[d + 1]
    uint32_t d = 0;
    for (uint32_t e = parts; e - d > 1;) {
        const uint32_t mid = (d + e) >> 1;
        if (start[mid] <= lo) d = mid;
        else e = mid;
    }
    for (; d < parts && start[d] < hi; ++d) {
        const size_t a = start[d] > lo ? start[d] : lo, b = start[d + 1] < hi ? start[d + 1] : hi;
        if (a >= b) continue;
        const size_t first = (size_t)d << log_range;
        for (uint32_t part = 0; part < (1u << (log_range - log_span)); ++part) {
            for (uint32_t i = threadIdx.x; i < span; i += kCountBlock) cnt[i] = 0;
            __syncthreads();
            for (size_t i = a + threadIdx.x; i < b; i += kCountBlock) {
                const uint32_t x = v[i] & ((1u << log_range) - 1u);
                if ((x >> log_span) == part) atomicAdd(&cnt[x & (span - 1u)], 1u);
            }
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < span; i += kCountBlock)
                if (cnt[i]) atomicAdd(&deg[first + ((size_t)part << log_span) + i], cnt[i]);
            __syncthreads();
        }
    }
}

// Whether the ends are counted so: ids of 13 to 26 bits, whose parts are at
// most two LDS ranges (2^28 vertices with 4.2e9 ends have eight, each a reading
// of the part: the degree phase took 143 ms so, 119 with the sort; 2^27 with
// 1.07e9 ends have four: 28.5 so, 31.7 with the sort, and 13.2 against 13.3 with
// 1.3e8), and enough ends for each part's counters to be worth clearing and
// adding up.
bool degree_by_count(size_t m, uint32_t n, int nb) { return nb >= 13 && nb <= 26 && m >= (size_t)1 << 20 && m >= n; }

// A bijection of [0, 2^nb): xor-shifts and odd multiplications modulo 2^nb.
__device__ __forceinline__ uint32_t tie_mix(uint32_t x, int nb)
{
    const uint64_t mask = (nb >= 32) ? 0xffffffffull : ((1ull << nb) - 1);
    const int s = (nb + 1) / 2;
    uint64_t y = x;
    y ^= y >> s;
    y = (y * 0x9e3779b1ull) & mask;
    y ^= y >> s;
    y = (y * 0x85ebca6bull) & mask;
    y ^= y >> s;
    return (uint32_t)y;
}

// graph of vertex v in a batch: voff[g] <= v < voff[g + 1]
__device__ __forceinline__ uint32_t graph_of_vertex(const uint32_t *voff, uint32_t n_graphs, uint32_t v)
{
    uint32_t a = 0, b = n_graphs;
    while (b - a > 1) {
        const uint32_t mid = (a + b) >> 1;
        if (voff[mid] <= v) a = mid;
        else b = mid;
    }
    return a;
}

// Sort key of the degree order: (d(v), hash(v)).  In a batch the graph id
// sits above them, so that every graph owns a contiguous range of ranks (the
// graphs share no edge, so the order between graphs is free).
__global__ void k_rank_keys(const uint32_t *deg, uint32_t n, int nb, int gshift, const uint32_t *voff,
                            uint32_t n_graphs, uint32_t tie, uint64_t *rkey, uint32_t *rval)
{
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < n; v += (size_t)gridDim.x * blockDim.x) {
        const uint32_t h = tie == TP_TIE_ID ? (uint32_t)v : tie_mix((uint32_t)v, nb);
        uint64_t key = ((uint64_t)deg[v] << nb) | h;
        if (voff) key |= (uint64_t)graph_of_vertex(voff, n_graphs, (uint32_t)v) << gshift;
        rkey[v] = key;
        rval[v] = (uint32_t)v;
    }
}

__global__ void k_rank_scatter(const uint32_t *perm, uint32_t n, const uint8_t *vlab, uint32_t *rank, uint8_t *rlab)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const uint32_t v = perm[i];
        rank[v] = (uint32_t)i;
        rlab[i] = vlab ? vlab[v] : 0;
    }
}

// ceil(log2 d) for d >= 2 (the bit length of d - 1); 0 for d <= 1; cap 31
__device__ __forceinline__ uint32_t degree_bin(uint32_t d)
{
    if (d <= 1) return 0;
    const uint32_t b = 32u - (uint32_t)__clz(d - 1);
    return b > 31 ? 31 : b;
}

// Ranks are in degree order, so the degree bins are ranges of ranks:
// first[k] = the first rank whose bin is >= k (first[] is pre-filled with
// 2^32 - 1 for bins above the largest).  Rank i writes the bins it opens.
// In a batch each graph's ranks are a range of their own in degree order,
// so each graph g gets its own 32 bounds at first[32 g + k], and a graph's
// first rank opens every bin up to its own.  Rank i's degree (bits
// [nb, gshift)) and graph (bits from gshift) are read from its sorted order
// key, in rank order.
__global__ void k_dbin_rank(const uint64_t *skey, uint32_t n, int nb, int gshift, bool batch, uint32_t *first)
{
    const uint64_t dmask = (1ull << (gshift - nb)) - 1;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const uint64_t key = skey[i];
        const uint32_t b = degree_bin((uint32_t)((key >> nb) & dmask));
        const uint32_t g = batch ? (uint32_t)(key >> gshift) : 0u;
        uint64_t pkey = 0;
        if (i) pkey = skey[i - 1];
        const bool opens = i == 0 || (batch && (uint32_t)(pkey >> gshift) != g);
        const int prev = opens ? -1 : (int)degree_bin((uint32_t)((pkey >> nb) & dmask));
        for (int k = prev + 1; k <= (int)b; ++k) first[(size_t)g * 32 + k] = (uint32_t)i;
    }
}

// The same boundaries as CSR slots: rows are laid out by rank.
__global__ void k_dbin_slot(const uint32_t *first, const uint64_t *rowptr, size_t count, uint64_t *slot)
{
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < count; k += (size_t)gridDim.x * blockDim.x)
        slot[k] = first[k] == 0xffffffffu ? ~0ull : rowptr[first[k]];
}

__global__ void fill_u32(uint32_t *p, size_t n, uint32_t v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// graph id of every rank in a batch: the bits above gshift of its sorted
// order key
__global__ void k_rank_graph(const uint64_t *skey, uint32_t n, int gshift, uint32_t *rank_gid)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        rank_gid[i] = (uint32_t)(skey[i] >> gshift);
}

// ------------------------------------------------------------ phase 4

// With directions (udir set), the oriented key carries two bits below the
// pair: bit 0 for the arc source -> target of the oriented edge, bit 1 for
// the reverse.
// (The times stay where the dedup wrote them: the orientation sort takes
// them as its values in place, so that they are not copied here.)
__global__ void k_orient(const uint64_t *ukey, const uint8_t *udir, size_t m, PairCode pc, const uint32_t *rank,
                         uint64_t *okey)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < m; i += (size_t)gridDim.x * blockDim.x) {
        const uint64_t k = ukey[i];
        const uint32_t base = pc.base(k);
        const uint32_t a = rank[pc.hi(k)], b = rank[pc.lo(k)];
        const uint32_t s = min(a, b), t = max(a, b);
        // local ranks of the key's graph (its ranks start at its first id)
        uint64_t o = pc.pack((uint32_t)(pc.voff ? k >> (2 * pc.lb) : 0u), s - base, t - base);
        if (udir) {
            // udir is relative to lower id -> higher id; a is the lower id's rank
            const uint32_t d = udir[i];
            o = (o << 2) | (a < b ? d : (((d & 1u) << 1) | (d >> 1)));
        }
        okey[i] = o;
    }
}



// ------------------------------------------------------------ phase 5

// The oriented pairs sorted by source: position i is CSR slot i.  One read
// of them writes each slot's target, its label, its source and (directed
// builds) the two direction bits below the pair into edir, and counts d+(s):
// each wave adds one count per run of equal sources among its 64 pairs, to
// increasing addresses.  The first block clears the pads of col, ets and edir.
__global__ void k_csr(const uint64_t *okey, size_t m, PairCode pc, const uint8_t *rlab, uint32_t *col, uint32_t *ets,
                      uint8_t *tlab, uint32_t *srow, uint8_t *edir, uint32_t *dplus)
{
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < kRowPad; i += blockDim.x) {
            col[m + i] = 0;
            ets[m + i] = 0;
        }
        if (edir)
            for (uint32_t i = threadIdx.x; i < 4 * kRowPad; i += blockDim.x) edir[m + i] = 0;
    }
    const int dshift = edir ? 2 : 0;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t base = blockIdx.x * (size_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); base < m; base += stride) {
        const size_t i = base + lane_id();
        const bool ok = i < m;
        const uint64_t k = ok ? okey[i] : 0ull;
        const uint32_t src = pc.hi(k >> dshift);
        add_runs(ok ? (uint64_t)src : ~0ull, ok, dplus);
        if (ok) {
            const uint32_t t = pc.lo(k >> dshift);
            col[i] = t;
            tlab[i] = rlab[t];
            srow[i] = src;
            if (edir) edir[i] = (uint8_t)(k & 3u);
        }
    }
}

// (One atomic per block and value: with one per wave the scale-22 graph's
// pass took 780 us, nearly all of it the atomics.)
__global__ __launch_bounds__(kB) void k_row_stats(const uint64_t *rowptr, uint32_t n, unsigned long long *wedges,
                                                  unsigned long long *dplus_max)
{
    __shared__ unsigned long long tmp[kB / kWave];
    unsigned long long w = 0, mx = 0;
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < n; v += (size_t)gridDim.x * blockDim.x) {
        const uint64_t d = rowptr[v + 1] - rowptr[v];
        w += d ? d * (d - 1) / 2 : 0;
        mx = max(mx, (unsigned long long)d);
    }
    block_add<kB>(w, tmp, wedges);
    block_max<kB>(mx, tmp, dplus_max);
}

// ------------------------------------------------------------ phase 6

// The wedges (p, q, r) of the oriented edge p -> q at slot k are the slots
// after k in p's row; they can close only if q has out-neighbours.
__device__ __forceinline__ uint32_t rest_len(const uint64_t *rowptr, uint32_t s, size_t k)
{
    return (uint32_t)(rowptr[s + 1] - k - 1);
}

// One bit per vertex: whether its row is non-empty (bit v & 63 of word
// v >> 6).  At one bit per vertex the array stays in cache, where the row
// pointers of random targets would not.
__global__ void k_has_out(const uint64_t *rowptr, uint32_t n, uint64_t *bits)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t base = blockIdx.x * (size_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); base < n; base += stride) {
        const size_t v = base + lane_id();
        const bool b = v < n && rowptr[v + 1] > rowptr[v];
        const uint64_t word = __ballot(b);
        if (lane_id() == 0) bits[base >> 6] = word;
    }
}

// Key of each oriented edge for the in-edge sort: (q << kbits) | k, with q
// replaced by n (sorted past every target) when the edge has no wedge to
// check; and the record payload that travels with it through the sort: the
// length of the rest of p's row after slot k (< 2^22) | label(p) << 24.
// Counts the edges kept.  Slots are in row order, so every read here walks
// memory forwards, but for the bit of q.
// (The count leaves with one atomic per block, as in k_row_stats.)
__global__ __launch_bounds__(kB) void k_in_keys(const uint32_t *srow, const uint32_t *col, const uint64_t *rowptr, const uint64_t *has_out,
                          const uint8_t *rlab, size_t m, int kbits, uint32_t n, uint64_t *key, uint32_t *pay,
                          unsigned long long *kept)
{
    __shared__ unsigned long long tmp[kB / kWave];
    unsigned long long c = 0;
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < m; k += (size_t)gridDim.x * blockDim.x) {
        const uint32_t s = srow[k], t = col[k];
        const uint32_t rest = rest_len(rowptr, s, k);
        const bool ok = rest > 0 && ((has_out[t >> 6] >> (t & 63)) & 1ull);
        key[k] = ((uint64_t)(ok ? t : n) << kbits) | k;
        pay[k] = rest | ((uint32_t)rlab[s] << 24);
        c += ok ? 1 : 0;
    }
    block_add<kB>(c, tmp, kept);
}

// In-edges and wedge checks of every target (the sum of the remaining row
// lengths of its in-edges).  In-edges of one target are consecutive, so each
// wave adds one partial sum per run of equal targets.
__global__ void k_in_work(const uint64_t *key, const uint32_t *pay, uint64_t n_in, int kbits,
                          unsigned long long *work, uint32_t *count)
{
    const unsigned lane = lane_id();
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t base = blockIdx.x * (size_t)blockDim.x + (threadIdx.x & ~(kWave - 1)); base < n_in; base += stride) {
        const size_t i = base + lane;
        const bool ok = i < n_in;
        uint64_t t = ~0ull, len = 0;
        if (ok) {
            t = key[i] >> kbits;
            len = pay[i] & 0xffffffu;
        }
        const uint64_t tprev = __shfl_up(t, 1, kWave);
        const bool head = ok && (lane == 0 || tprev != t);
        const uint64_t heads = __ballot(head);
        const uint64_t incl = wave_incl_scan(len);
        // the lane where this lane's run starts, and the prefix before it
        const uint64_t upto = heads & (lane == 63 ? ~0ull : ((2ull << lane) - 1));
        const int start = 63 - __clzll(upto);
        const uint64_t before = __shfl(incl - len, start, kWave);
        const uint64_t tnext = __shfl_down(t, 1, kWave);
        const bool last = ok && (lane == 63 || i + 1 >= n_in || tnext != t);
        if (last) {
            atomicAdd(&work[t], (unsigned long long)(incl - before));
            atomicAdd(&count[t], lane - (unsigned)start + 1u);
        }
    }
}

// ------------------------------------------------------------ phase 7

__device__ __forceinline__ int class_of(uint64_t dq)
{
    return dq <= kTinyMaxDeg ? kClassTiny
                             : (dq <= kSmallMaxDeg ? kClassSmall : (dq <= kLargeMaxDeg ? kClassLarge : kClassHuge));
}

// Tile caps of each class: records per tile and wedge checks per tile, and the
// records of its work tiles where they are bounded (bounded_cap; else 0).
struct TileCaps {
    uint32_t rec[kNumClasses];
    uint64_t work[kNumClasses];
    uint32_t bound[kNumClasses];
};

// ceil(a / b), in 32 bits where both fit (a 64-bit division is some 100
// instructions)
__device__ __forceinline__ uint64_t div_up(uint64_t a, uint64_t b)
{
    const uint64_t x = a + b - 1;
    return (x | b) >> 32 ? x / b : (uint64_t)((uint32_t)x / (uint32_t)b);
}

__device__ __forceinline__ uint32_t tiles_of(uint64_t cnt, uint64_t work, uint32_t rec_cap, uint64_t work_cap)
{
    if (cnt == 0) return 0;
    const uint64_t a = div_up(cnt, rec_cap);
    const uint64_t b = div_up(work, work_cap);
    uint64_t t = a > b ? a : b;
    if (t > cnt) t = cnt;
    return (uint32_t)t;
}

// The caps of the work tiles (the cut the surveys walk): where a class whose
// cap is the default one has too little work to give every claimer of a full device about 8 tiles (4 in
// the larger two classes) at the plan's cap, its records are cut finer, down to a floor
// below which a tile's table and claim would outweigh its records.  The
// claimers are waves for the tiny class and workgroups for the others, as
// many as the plain survey keeps on kPlanUnits compute units (32 waves, 5 and 1
// workgroups each; the other forms keep fewer).  Without
// it a small graph waits for the one wave or workgroup that walks its largest
// target (scale 13: 1024 records on one wave, 247 us of a 380 us survey).
// 8 tiles against 4: 300-graph batch's tiny class 1.63 against 2.07 ms, 300,007
// vertices' small class 407 against 467 us, scale 22's large class 2.71
// against 2.63 ms.
__host__ __device__ inline uint64_t class_claimers(int c)
{
    return (uint64_t)kPlanUnits * (c == kClassTiny ? 32 : (c == kClassSmall ? 5 : 1));
}

__host__ __device__ inline uint32_t work_rec_cap(int c, uint32_t rec_cap, uint64_t class_records)
{
    const uint64_t share = c == kClassTiny || c == kClassSmall ? 8 : 4;
    const uint64_t claimers = class_claimers(c);
    const uint32_t least = c == kClassTiny ? kWorkRecMinTiny : (c == kClassSmall ? kWorkRecMinSmall : kWorkRecMinLarge);
    const uint64_t want = class_records / (claimers * share);
    const uint64_t cap = want > least ? want : least;
    return cap < rec_cap ? (uint32_t)cap : rec_cap;
}

// The cap of a class's work tiles where that rule would cut it into more than
// four times as many, 0 elsewhere (its records, its wedge checks, its tiles at
// the plan's cap and the finer ones).  That is where few targets hold most of the
// records, hubs of leaves.  Every finer tile costs a claim (17 ns on one counter
// for all) and fills its target's table again (331,000 records of hubs with d+
// of some 700, small class, count: 477 tiles 62 us, 954 59, 10,555 180), and
// since the tiles of a target interleave, each walks the whole range of its
// rows, which the targets walked at the same time share in cache (10e6 records
// of hubs with d+ of 17, tiny class, count and survey: 11,250 tiles 516 and
// 925 us, 21,402 556 and 944, 67,304 1012 and 1397).  So such a class is cut into
// about twice its tiles, the tiny class into two for every wave at least, which
// the forms with more work per triangle want (4.1e6 records of 1000 hubs, tiny
// class, count / survey / extended: 4341 tiles 93 / 197 / 1772 us, 16,341
// 129 / 259 / 1321, 64,240 172 / 259 / 1415).
// The full cut stays where the plan's tiles are fewer than an eighth of the
// claimers; where they hold 2^16 checks and more, whose tail the finer ones fill
// (complete graph of 1500, small class, survey: 1800 tiles of 177,000 checks
// 870 us, 17,509 tiles 752; 2000 vertices at density 0.3, 46,000 checks: 183
// against 211 finer); and in the tiny class, whose tables a wave fills in one
// round, up to 2^20 records (542,000: 128 us in 1140 tiles, 97 in 34,438).
// R-MAT graphs are cut into at most 2.8 (tiny) and 5.2 (small) times as many.
constexpr uint64_t kFinerMost = 4;
constexpr uint64_t kFinerTinyRecords = uint64_t(1) << 20;
constexpr uint64_t kFinerChecks = uint64_t(1) << 16;
uint32_t bounded_cap(int c, uint32_t rec_cap, uint64_t records, uint64_t checks, uint64_t tiles, uint64_t finer)
{
    if (finer <= kFinerMost * tiles || 8 * tiles < class_claimers(c) || checks >= kFinerChecks * tiles) return 0;
    if (c == kClassTiny && records < kFinerTinyRecords) return 0;
    const uint64_t want = std::max(2 * tiles, c == kClassTiny ? 2 * class_claimers(c) : 0);
    return (uint32_t)std::max<uint64_t>(work_rec_cap(c, rec_cap, records), records / want);
}

// Records of piece j of target q (pieces of huge targets; pos[] is the
// exclusive scan of the cut flags, fbase[] the first flag of each target):
// [first, first + count) in the piece record arrays.
__device__ __forceinline__ void piece_records(const uint64_t *fbase, const uint64_t *pos, size_t q, uint32_t j,
                                              uint64_t cnt, uint64_t &first, uint64_t &count)
{
    first = pos[fbase[q] + j * cnt];
    count = pos[fbase[q] + (j + 1) * cnt] - first;
}

// Records of every class (the work tiles' caps follow from them); one atomic
// per block and value.
__global__ __launch_bounds__(kB) void k_plan_records(const uint32_t *incnt, const uint64_t *rowptr, uint32_t n,
                                                     unsigned long long *rec /* [classes] */)
{
    __shared__ unsigned long long tmp[kB / kWave];
    unsigned long long r[kNumClasses] = {};
    for (size_t q = blockIdx.x * (size_t)blockDim.x + threadIdx.x; q < n; q += (size_t)gridDim.x * blockDim.x) {
        const uint32_t cnt = incnt[q];
        if (!cnt) continue;
        const int c = class_of(rowptr[q + 1] - rowptr[q]);
#pragma unroll
        for (int i = 0; i < kNumClasses; ++i) r[i] += i == c ? cnt : 0u;
    }
#pragma unroll
    for (int i = 0; i < kNumClasses; ++i) block_add<kB>(r[i], tmp, &rec[i]);
}

// The plan in two passes over the targets, kPlanChunk consecutive targets to
// a block and kPlanItems consecutive ones to a thread.  k_plan_count leaves
// one column of sums per block (rows below); their exclusive scan, row after
// row, gives every block the places of its tiles and the host the totals;
// k_plan_write computes the same counts again and writes the tiles.
constexpr int kPlanItems = 2;
constexpr size_t kPlanChunk = (size_t)kB * kPlanItems;
// rows: tiles and work tiles of each class (target order), then records,
// staged out-list entries under either cut and wedge checks of each class, then
// all wedge checks and the targets with any
static_assert(6 * kNumClasses + 2 < kWave, "k_plan_heads takes one lane per row");
constexpr int kPlanTiles = 0, kPlanWork = kNumClasses, kPlanRec = 2 * kNumClasses, kPlanStaged = 3 * kNumClasses,
              kPlanWorkStaged = 4 * kNumClasses, kPlanProbes = 5 * kNumClasses, kPlanAll = 6 * kNumClasses,
              kPlanTargets = 6 * kNumClasses + 1, kPlanRows = 6 * kNumClasses + 2;

struct PlanIn {
    const uint64_t *cptr;             // [n + 1] first record of each target
    const unsigned long long *work;   // [n] wedge checks of each target
    const uint64_t *rowptr;
    const uint64_t *fbase, *pos;      // pieces of huge targets (null without any)
    const unsigned long long *rec;    // records of each class
    uint32_t n;
    TileCaps caps;
};

struct PlanTarget {
    int c;             // class
    uint32_t tiles, work_tiles;
    uint64_t cnt, work, dq;
};

// Caps of class c under the plan, and those of its work tiles.
__device__ __forceinline__ void class_caps(const PlanIn &in, int c, uint32_t &rc, uint64_t &wc, uint32_t &frc, uint64_t &fwc)
{
    rc = in.caps.rec[0];
    wc = in.caps.work[0];
#pragma unroll
    for (int i = 1; i < kNumClasses; ++i) {
        if (i == c) {
            rc = in.caps.rec[i];
            wc = in.caps.work[i];
        }
    }
    // (a cap that a caller has chosen is walked as it is)
    frc = rc;
    if (rc == default_tile_records(c)) {
        uint32_t bound = in.caps.bound[0];
#pragma unroll
        for (int i = 1; i < kNumClasses; ++i)
            if (i == c) bound = in.caps.bound[i];
        frc = bound ? bound : work_rec_cap(c, rc, in.rec[c]);
    }
    fwc = min(wc, kTileWorkPerRecord * (uint64_t)frc);
}

__device__ __forceinline__ PlanTarget plan_target(const PlanIn &in, size_t q)
{
    PlanTarget t{};
    if (q >= in.n) return t;
    t.cnt = in.cptr[q + 1] - in.cptr[q];
    if (!t.cnt) return t;
    t.work = in.work[q];
    t.dq = in.rowptr[q + 1] - in.rowptr[q];
    t.c = class_of(t.dq);
    uint32_t rc, frc;
    uint64_t wc, fwc;
    class_caps(in, t.c, rc, wc, frc, fwc);
    if (t.c == kClassHuge) {
        // each piece of Adj+(q) has its own records and tiles; it sees
        // about 1/S of the target's wedge checks
        const uint32_t S = piece_count(t.dq);
        for (uint32_t j = 0; j < S; ++j) {
            uint64_t first, count;
            piece_records(in.fbase, in.pos, q, j, t.cnt, first, count);
            t.tiles += tiles_of(count, (t.work + S - 1) / S, rc, wc);
            t.work_tiles += tiles_of(count, (t.work + S - 1) / S, frc, fwc);
        }
    } else {
        t.tiles = tiles_of(t.cnt, t.work, rc, wc);
        t.work_tiles = tiles_of(t.cnt, t.work, frc, fwc);
    }
    return t;
}

__global__ __launch_bounds__(kB) void k_plan_count(PlanIn in, uint64_t *sums /* [rows][blocks] */)
{
    __shared__ unsigned long long part[kB / kWave][kPlanRows];
    unsigned long long v[kPlanRows] = {};
    const size_t q0 = blockIdx.x * kPlanChunk;
    for (int k = 0; k < kPlanItems; ++k) {
        const size_t q = q0 + (size_t)k * kB + threadIdx.x;
        const PlanTarget t = plan_target(in, q);
        if (!t.cnt) continue;
        // a huge target: the records cut to its pieces, each piece staged by
        // each of its tiles
        uint64_t nrec = t.cnt, staged = (uint64_t)t.tiles * t.dq, work_staged = (uint64_t)t.work_tiles * t.dq;
        if (t.c == kClassHuge) {
            uint32_t rc, frc;
            uint64_t wc, fwc;
            class_caps(in, t.c, rc, wc, frc, fwc);
            const uint32_t S = piece_count(t.dq), psz = piece_size(t.dq);
            nrec = 0;
            staged = 0;
            work_staged = 0;
            for (uint32_t j = 0; j < S; ++j) {
                uint64_t first, count;
                piece_records(in.fbase, in.pos, q, j, t.cnt, first, count);
                nrec += count;
                const uint64_t keys = min((uint64_t)psz, t.dq - (uint64_t)j * psz);
                staged += tiles_of(count, (t.work + S - 1) / S, rc, wc) * keys;
                work_staged += tiles_of(count, (t.work + S - 1) / S, frc, fwc) * keys;
            }
        }
#pragma unroll
        for (int i = 0; i < kNumClasses; ++i) {
            const bool on = i == t.c;
            v[kPlanTiles + i] += on ? t.tiles : 0u;
            v[kPlanWork + i] += on ? t.work_tiles : 0u;
            v[kPlanRec + i] += on && t.tiles ? nrec : 0u;
            v[kPlanStaged + i] += on && t.tiles ? staged : 0u;
            v[kPlanWorkStaged + i] += on && t.tiles ? work_staged : 0u;
            v[kPlanProbes + i] += on && t.tiles ? t.work : 0u;
        }
        v[kPlanAll] += t.work;
        v[kPlanTargets] += t.work ? 1 : 0;
    }
#pragma unroll
    for (int i = 0; i < kPlanRows; ++i) {
        const unsigned long long x = wave_sum(v[i]);
        if (lane_id() == 0) part[threadIdx.x / kWave][i] = x;
    }
    __syncthreads();
    if (threadIdx.x < kPlanRows) {
        unsigned long long x = 0;
        for (int w = 0; w < kB / kWave; ++w) x += part[w][threadIdx.x];
        sums[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = x;
    }
}

// The first place of every row of the scanned sums and, past the last, the end.
__global__ void k_plan_heads(const uint64_t *sums, unsigned blocks, uint64_t *head /* [rows + 1] */)
{
    if (threadIdx.x <= kPlanRows) head[threadIdx.x] = sums[(size_t)threadIdx.x * blocks];
}

struct PlanOut {
    TileDesc *tiles[kNumClasses];  // null: the class has none, or its work tiles are its tiles
    TileDesc *work[kNumClasses];
};

// The tiles of target q, dealing its records round-robin; for a huge target,
// the tiles of each piece in turn over that piece's records.  Places are in
// target order: a block's first place from the scanned sums, a thread's from
// a scan of the block's threads.
__global__ __launch_bounds__(kB) void k_plan_write(PlanIn in, const uint64_t *sums, PlanOut out)
{
    __shared__ uint64_t tmp[kB / kWave];
    PlanTarget t[kPlanItems];
    const size_t q0 = blockIdx.x * kPlanChunk + (size_t)threadIdx.x * kPlanItems;
#pragma unroll
    for (int k = 0; k < kPlanItems; ++k) t[k] = plan_target(in, q0 + k);
    for (int list = 0; list < 2; ++list) {
        for (int c = 0; c < kNumClasses; ++c) {
            TileDesc *dst = list ? out.work[c] : out.tiles[c];
            if (!dst) continue;
            const uint64_t *row = sums + (size_t)((list ? kPlanWork : kPlanTiles) + c) * gridDim.x;
            uint64_t mine = 0;
#pragma unroll
            for (int k = 0; k < kPlanItems; ++k)
                if (t[k].cnt && t[k].c == c) mine += list ? t[k].work_tiles : t[k].tiles;
            uint64_t total;
            uint64_t at = row[blockIdx.x] - row[0] + block_excl_scan<kB>(mine, tmp, total);
            if (!total) continue;
            uint32_t rc, frc;
            uint64_t wc, fwc;
            class_caps(in, c, rc, wc, frc, fwc);
            if (list) {
                rc = frc;
                wc = fwc;
            }
            // a run of tj tiles over `count` records from `first`; a target
            // with many is written by its whole wave
            auto put = [&](uint64_t where, uint32_t i, uint32_t q, uint64_t first, uint32_t each, uint32_t more,
                           uint32_t tj, uint32_t piece) {
                TileDesc d;
                d.q = q;
                d.cnt = each + (i < more ? 1u : 0u);  // records i, i + tj, ...
                d.e0 = first + i;
                d.stride = tj;
                d.piece = piece;
                dst[where + i] = d;
            };
#pragma unroll
            for (int k = 0; k < kPlanItems; ++k) {
                const bool on = t[k].cnt && t[k].c == c;
                const uint32_t nt = on ? (list ? t[k].work_tiles : t[k].tiles) : 0u;
                const uint32_t q = (uint32_t)(q0 + k);
                if (c == kClassHuge) {
                    if (!on) continue;
                    const uint32_t S = piece_count(t[k].dq);
                    for (uint32_t j = 0; j < S; ++j) {
                        uint64_t first, count;
                        piece_records(in.fbase, in.pos, q, j, t[k].cnt, first, count);
                        const uint32_t tj = tiles_of(count, (t[k].work + S - 1) / S, rc, wc);
                        for (uint32_t i = 0; i < tj; ++i)
                            put(at, i, q, first, (uint32_t)(count / tj), (uint32_t)(count % tj), tj, j);
                        at += tj;
                    }
                    continue;
                }
                const uint64_t first = on ? in.cptr[q] : 0;
                // (a target has fewer than 2^32 records: in-edges)
                const uint32_t each = nt ? (uint32_t)t[k].cnt / nt : 0u, more = nt ? (uint32_t)t[k].cnt % nt : 0u;
                const bool many = nt > 8;
                if (!many)
                    for (uint32_t i = 0; i < nt; ++i) put(at, i, q, first, each, more, nt, 0);
                for (uint64_t m = __ballot(many); m; m &= m - 1) {
                    const int l = __ffsll((long long)m) - 1;
                    const uint64_t lat = __shfl(at, l, kWave), lfirst = __shfl(first, l, kWave);
                    const uint32_t ln = __shfl(nt, l, kWave), lq = __shfl(q, l, kWave);
                    const uint32_t leach = __shfl(each, l, kWave), lmore = __shfl(more, l, kWave);
                    for (uint32_t i = lane_id(); i < ln; i += kWave) put(lat, i, lq, lfirst, leach, lmore, ln, 0);
                }
                at += nt;
            }
        }
    }
}

// ---- records of huge targets, cut to the pieces of Adj+(q)

// Number of the `len` sorted ranks at `a` that are below x (binary search).
__device__ __forceinline__ uint32_t count_below(const uint32_t *a, uint32_t len, uint32_t x)
{
    uint32_t lo = 0, hi = len;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Cut flags per target: S * (records) for a huge target with records, else
// none; the huge targets with records are listed (in no particular order;
// at most m / (kLargeMaxDeg + 1) targets have d+ above kLargeMaxDeg).
__global__ void k_piece_slots(const uint64_t *cptr, const uint64_t *rowptr, uint32_t n, uint32_t *slots,
                              uint32_t *list, unsigned long long *n_list)
{
    for (size_t q = blockIdx.x * (size_t)blockDim.x + threadIdx.x; q < n; q += (size_t)gridDim.x * blockDim.x) {
        const uint64_t dq = rowptr[q + 1] - rowptr[q], cnt = cptr[q + 1] - cptr[q];
        const bool huge = class_of(dq) == kClassHuge && cnt > 0;
        slots[q] = huge ? (uint32_t)(piece_count(dq) * cnt) : 0u;
        if (huge) list[atomicAdd(n_list, 1ull)] = (uint32_t)q;
    }
}

// For every record p -> q of a listed huge target (grid row y: targets y,
// y + gridDim.y, ...) and every piece j of Adj+(q): the candidates of the
// record (the rest of p's row, sorted by rank) whose ranks lie in the
// piece's range [first key of piece j, first key of piece j + 1).
// WRITE false: at f = fbase[q] + j cnt + r (r the record's place among q's
// records) flag[f] = (any candidates) and cut[f] = the end of the piece's
// candidates in the record.  WRITE true: the record cut to the piece, from
// cut[], at pos[f].
template <bool WRITE>
__global__ void k_piece_cut(const uint64_t *inkey, const uint32_t *inpay, int kbits, const uint32_t *list,
                            uint64_t n_list, const uint64_t *cptr, const uint64_t *rowptr, const uint32_t *col,
                            const uint64_t *fbase, uint32_t *flag, uint32_t *cut, const uint64_t *pos,
                            uint64_t *pkey, uint32_t *ppay)
{
    const uint64_t kmask = (1ull << kbits) - 1;
    for (uint64_t t = blockIdx.y; t < n_list; t += gridDim.y) {
        const uint64_t q = list[t];
        const uint64_t kq = rowptr[q], dq = rowptr[q + 1] - kq;
        const uint32_t S = piece_count(dq), psz = piece_size(dq);
        const uint64_t c0 = cptr[q], cnt = cptr[q + 1] - c0;
        for (uint64_t r = blockIdx.x * (size_t)blockDim.x + threadIdx.x; r < cnt; r += (size_t)gridDim.x * blockDim.x) {
            const uint64_t key = inkey[c0 + r];
            const uint64_t k = key & kmask;
            const uint32_t pay = inpay[c0 + r], len = pay & 0xffffffu;
            const uint32_t *cand = col + k + 1;
            uint32_t lo = 0;
            for (uint32_t j = 0; j < S; ++j) {
                const uint64_t f = fbase[q] + j * cnt + r;
                uint32_t hi;
                if (!WRITE) {
                    hi = j + 1 < S ? count_below(cand, len, col[kq + (uint64_t)(j + 1) * psz]) : len;
                    flag[f] = hi > lo ? 1u : 0u;
                    cut[f] = hi;
                } else if ((hi = cut[f]) > lo) {
                    // q + lo < 2n fits above bit kbits, as q <= n does
                    pkey[pos[f]] = ((q + lo) << kbits) | k;
                    ppay[pos[f]] = (pay & 0xff000000u) | (hi - lo);
                }
                lo = hi;
            }
        }
    }
}

template <class T>
T read_scalar(const T *dev, hipStream_t s)
{
    T v;
    TP_HIP(hipMemcpyAsync(&v, dev, sizeof(T), hipMemcpyDeviceToHost, s));
    TP_HIP(hipStreamSynchronize(s));
    return v;
}

template <class T>
const T *to_device(const T *p, size_t n, uint32_t space, DArray<T> &hold, hipStream_t s)
{
    if (!p || space == TP_MEM_DEVICE) return p;
    hold.reset(n, s);
    if (n) TP_HIP(hipMemcpyAsync(hold.get(), p, n * sizeof(T), hipMemcpyHostToDevice, s));
    return hold.get();
}

}  // namespace

// ================================================================ plan

uint64_t graph_bytes(const tp_graph *g)
{
    uint64_t b = g->rowptr.bytes() + g->col.bytes() + g->ets.bytes() + g->tlab.bytes() + g->rlab.bytes() +
                 g->perm.bytes() + g->inkey.bytes() + g->inpay.bytes() + g->rank_gid.bytes() +
                 g->dbin_rank.bytes() + g->dbin_slot.bytes() + g->edir.bytes() + g->piece_key.bytes() +
                 g->piece_pay.bytes();
    for (int c = 0; c < kNumClasses; ++c) b += g->tiles[c].bytes() + g->work_tiles[c].bytes();
    return b;
}

namespace {

// A plan that is cut, but not yet its graph's: whatever fails up to the wait
// for its last kernel leaves the graph with the plan that it had.
struct CutPlan {
    PlanCfg cfg{};
    DArray<TileDesc> tiles[kNumClasses], work_tiles[kNumClasses];
    uint64_t n_tiles[kNumClasses] = {}, n_work_tiles[kNumClasses] = {};
    // (empty where the graph has its piece records: they depend on the graph alone)
    uint64_t n_piece_recs = 0;
    DArray<uint64_t> piece_key;
    DArray<uint32_t> piece_pay;
    tp_graph_stats stats{};  // the graph's, with the plan's figures
};

// Cut the tiles of every class with the caps of `cfg`.  The work of each
// target (in-edges and wedge checks) is recomputed from the in-edge index.
// The plan is complete once `s` has been waited for.
CutPlan cut_plan(const tp_graph *g, const PlanCfg &cfg, hipStream_t s)
{
    CutPlan plan;
    plan.cfg = cfg;
    plan.stats = g->stats;
    const uint32_t n = g->n;
    DArray<unsigned long long> work((size_t)n + kNumClasses, s);
    DArray<uint64_t> cptr((size_t)n + 1, s);
    unsigned long long *rec = work.get() + n;  // records of each class
    {
        DArray<uint32_t> incnt(n, s);
        fill<uint32_t>(incnt.get(), 0u, n, s);
        fill<uint64_t>(reinterpret_cast<uint64_t *>(work.get()), 0ull, (size_t)n + kNumClasses, s);
        if (g->n_in) {
            k_in_work<<<grid_for(g->n_in, kB), kB, 0, s>>>(g->inkey.get(), g->inpay.get(), g->n_in, (int)g->kbits,
                                                           work.get(), incnt.get());
            TP_CHECK_LAUNCH();
        }
        k_plan_records<<<stat_grid(n, kB), kB, 0, s>>>(incnt.get(), g->rowptr.get(), n, rec);
        TP_CHECK_LAUNCH();
        scan_u32_to_u64(incnt.get(), cptr.get(), n, s);
    }
    // the records of huge targets cut to the pieces of Adj+(q): a flag per
    // (record, piece), laid out target by target and piece by piece; the
    // scan of the flags places every cut record
    DArray<uint64_t> fbase, pos;
    if (g->n_in && g->stats.dplus_max > kLargeMaxDeg) {
        fbase.reset((size_t)n + 1, s);
        DArray<uint32_t> list(g->m / (kLargeMaxDeg + 1) + 1, s);
        DArray<unsigned long long> n_list(1, s);
        TP_HIP(hipMemsetAsync(n_list.get(), 0, sizeof(unsigned long long), s));
        {
            DArray<uint32_t> slots(n, s);
            k_piece_slots<<<grid_for(n, kB), kB, 0, s>>>(cptr.get(), g->rowptr.get(), n, slots.get(), list.get(),
                                                         n_list.get());
            TP_CHECK_LAUNCH();
            scan_u32_to_u64(slots.get(), fbase.get(), n, s);
        }
        const uint64_t nf = read_scalar(fbase.get() + n, s);
        const uint64_t nh = read_scalar(n_list.get(), s);
        // a grid row per listed target (strided), its records across the row
        const dim3 grid(64, (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(nh, 4096)));
        pos.reset(nf + 1, s);
        DArray<uint32_t> cut(std::max<uint64_t>(nf, 1), s);
        {
            DArray<uint32_t> flag(std::max<uint64_t>(nf, 1), s);
            if (nh) {
                k_piece_cut<false><<<grid, kB, 0, s>>>(g->inkey.get(), g->inpay.get(), (int)g->kbits, list.get(), nh,
                                                       cptr.get(), g->rowptr.get(), g->col.get(), fbase.get(),
                                                       flag.get(), cut.get(), nullptr, nullptr, nullptr);
                TP_CHECK_LAUNCH();
            }
            scan_u32_to_u64(flag.get(), pos.get(), nf, s);
        }
        const uint64_t nr = g->n_piece_recs ? 0 : read_scalar(pos.get() + nf, s);
        if (nr) {
            plan.n_piece_recs = nr;
            plan.piece_key.reset(nr, s);
            plan.piece_pay.reset(nr, s);
            k_piece_cut<true><<<grid, kB, 0, s>>>(g->inkey.get(), g->inpay.get(), (int)g->kbits, list.get(), nh,
                                                  cptr.get(), g->rowptr.get(), g->col.get(), fbase.get(), nullptr,
                                                  cut.get(), pos.get(), plan.piece_key.get(), plan.piece_pay.get());
            TP_CHECK_LAUNCH();
        }
    }
    TileCaps caps{};
    for (int c = 0; c < kNumClasses; ++c) {
        caps.rec[c] = cfg.tile_records[c];
        caps.work[c] = kTileWorkPerRecord * cfg.tile_records[c];
    }
    PlanIn in{cptr.get(), work.get(), g->rowptr.get(), fbase.get(), pos.get(), rec, n, caps};
    const unsigned nb = (unsigned)((n + kPlanChunk - 1) / kPlanChunk);
    DArray<uint64_t> sums((size_t)kPlanRows * nb + 1, s), head(kPlanRows + 1, s);
    uint64_t first[kPlanRows + 1];
    auto total = [&](int row) { return first[row + 1] - first[row]; };
    for (bool bounded = false;;) {
        k_plan_count<<<nb, kB, 0, s>>>(in, sums.get());
        TP_CHECK_LAUNCH();
        scan_u64(sums.get(), sums.get(), (size_t)kPlanRows * nb, true, s);
        k_plan_heads<<<1, kWave, 0, s>>>(sums.get(), nb, head.get());
        TP_CHECK_LAUNCH();
        TP_HIP(hipMemcpyAsync(first, head.get(), sizeof(first), hipMemcpyDeviceToHost, s));
        TP_HIP(hipStreamSynchronize(s));
        if (bounded) break;
        // counted again with a bound on the classes that the rule cuts too fine
        for (int c = 0; c < kNumClasses; ++c) {
            in.caps.bound[c] = bounded_cap(c, caps.rec[c], total(kPlanRec + c), total(kPlanProbes + c),
                                           total(kPlanTiles + c), total(kPlanWork + c));
            bounded = bounded || in.caps.bound[c];
        }
        if (!bounded) break;
    }
    PlanOut out{};
    bool any = false;
    for (int c = 0; c < kNumClasses; ++c) {
        const uint64_t nt = total(kPlanTiles + c), nw = total(kPlanWork + c);
        plan.n_tiles[c] = nt;
        plan.tiles[c].reset(std::max<uint64_t>(nt, 1), s);
        // (a finer cut gives no target fewer tiles: as many in all is the same cut)
        plan.n_work_tiles[c] = nw == nt ? 0 : nw;
        plan.work_tiles[c].reset(plan.n_work_tiles[c], s);
        out.tiles[c] = nt ? plan.tiles[c].get() : nullptr;
        out.work[c] = plan.work_tiles[c].get();
        any = any || nt;
    }
    if (any) {
        k_plan_write<<<nb, kB, 0, s>>>(in, sums.get(), out);
        TP_CHECK_LAUNCH();
    }
    tp_graph_stats &st = plan.stats;
    st.n_tiles = 0;
    for (int c = 0; c < kNumClasses; ++c) {
        st.class_tiles[c] = plan.n_work_tiles[c] ? plan.n_work_tiles[c] : plan.n_tiles[c];
        st.class_records[c] = total(kPlanRec + c);
        st.class_staged[c] = total((plan.n_work_tiles[c] ? kPlanWorkStaged : kPlanStaged) + c);
        st.class_probes[c] = total(kPlanProbes + c);
        st.n_tiles += st.class_tiles[c];
    }
    st.probes = total(kPlanAll);
    st.n_targets = total(kPlanTargets);
    return plan;
}

// Make a complete plan the graph's.  Nothing here can fail.
void adopt_plan(tp_graph *g, CutPlan &plan)
{
    for (int c = 0; c < kNumClasses; ++c) {
        g->tiles[c] = std::move(plan.tiles[c]);
        g->work_tiles[c] = std::move(plan.work_tiles[c]);
        g->n_tiles[c] = plan.n_tiles[c];
        g->n_work_tiles[c] = plan.n_work_tiles[c];
    }
    if (plan.n_piece_recs) {
        g->n_piece_recs = plan.n_piece_recs;
        g->piece_key = std::move(plan.piece_key);
        g->piece_pay = std::move(plan.piece_pay);
    }
    g->plan = plan.cfg;
    g->stats = plan.stats;
    g->stats.device_bytes = graph_bytes(g);
}

}  // namespace

void plan_graph(tp_graph *g, const PlanCfg &cfg, hipStream_t s)
{
    CallScope scope(s);
    CutPlan plan = cut_plan(g, cfg, s);
    TP_HIP(hipStreamSynchronize(s));
    adopt_plan(g, plan);
}

// ================================================================ build

struct HostBatch {
    uint32_t n_graphs = 0;
    std::vector<uint64_t> eoff;  // [n_graphs + 1]
    std::vector<uint32_t> voff;  // [n_graphs + 1]
};

static void build_impl(const tp_edge_list *el, hipStream_t s, tp_graph **out, const HostBatch *hb = nullptr)
{
    if (!el || !out) fail(TP_ERR_INVALID, "tripoll_build: NULL argument");
    if (el->mem_space != TP_MEM_HOST && el->mem_space != TP_MEM_DEVICE)
        fail(TP_ERR_INVALID, "tripoll_build: mem_space must be TP_MEM_HOST or TP_MEM_DEVICE");
    if (el->tie_hash != TP_TIE_MIX && el->tie_hash != TP_TIE_ID)
        fail(TP_ERR_INVALID, "tripoll_build: unknown tie_hash");
    if (el->n_vertices == 0 || el->n_vertices >= 0xffffffffu)
        fail(TP_ERR_INVALID, "tripoll_build: n_vertices must be in [1, 2^32-1)");
    if (el->n_edges > 0 && (!el->src || !el->dst)) fail(TP_ERR_INVALID, "tripoll_build: NULL src/dst");
    if (el->flags & ~TP_EDGES_DIRECTED) fail(TP_ERR_INVALID, "tripoll_build: unknown flags");

    CallScope scope(s);  // temporaries of the build are reused without waiting
    const uint32_t n = el->n_vertices;
    const size_t M = el->n_edges;
    const int nb = std::max(1, bits_for((uint64_t)n - 1));
    // directed inputs carry one direction bit per raw edge through the pair
    // sort and two per oriented edge through the orientation sort
    const bool directed = (el->flags & TP_EDGES_DIRECTED) != 0;
    const int dbit = directed ? 1 : 0, dbit2 = directed ? 2 : 0;
    if (2 * nb + dbit2 > 64) fail(TP_ERR_UNSUPPORTED, "tripoll_build: too many vertices for directed keys");
    // pair keys: a batch keeps its ids local (graph index on top) when that
    // layout is the shorter one
    int kb = 2 * nb;  // bits of a pair key
    int lb = nb;      // bits of one id in it
    bool local_keys = false;
    if (hb && hb->n_graphs > 1) {
        uint32_t vmax = 1;
        for (uint32_t i = 0; i < hb->n_graphs; ++i) vmax = std::max(vmax, hb->voff[i + 1] - hb->voff[i]);
        const int l = std::max(1, bits_for((uint64_t)vmax - 1));
        const int gb = bits_for((uint64_t)hb->n_graphs - 1);
        if (2 * l + gb < kb) {
            local_keys = true;
            lb = l;
            kb = 2 * l + gb;
        }
    }
    const uint64_t sentinel = (kb + dbit >= 64) ? ~0ull : ((1ull << (kb + dbit)) - 1);

    auto g = std::make_unique<tp_graph>();
    TP_HIP(hipGetDevice(&g->device));
    g->n = n;
    g->nbits = (uint32_t)nb;

    hipEvent_t ev[9];
    for (auto &e : ev) TP_HIP(hipEventCreate(&e));
    struct EvGuard {
        hipEvent_t *e;
        ~EvGuard() { for (int i = 0; i < 9; ++i) (void)hipEventDestroy(e[i]); }
    } evg{ev};
    TP_HIP(hipEventRecord(ev[0], s));

    // ---- phase 0: upload and canonicalise
    DArray<uint32_t> h_src, h_dst, h_ts;
    DArray<uint8_t> h_lab;
    const uint32_t *src = to_device(el->src, M, el->mem_space, h_src, s);
    const uint32_t *dst = to_device(el->dst, M, el->mem_space, h_dst, s);
    const uint32_t *ts = to_device(el->edge_time, M, el->mem_space, h_ts, s);
    const uint8_t *vlab = to_device(el->vertex_label, n, el->mem_space, h_lab, s);

    // bad ids, self-loops, d_max, max label, wedges, d+_max, in-edge records
    DArray<unsigned long long> counters(8, s);
    TP_HIP(hipMemsetAsync(counters.get(), 0, 8 * sizeof(unsigned long long), s));
    unsigned long long *c_bad = counters.get(), *c_loop = c_bad + 1, *c_dmax = c_bad + 2, *c_lab = c_bad + 3,
                       *c_wedge = c_bad + 4, *c_dpmax = c_bad + 5, *c_kept = c_bad + 6;

    const size_t Mcap = std::max<size_t>(M, 1);
    DArray<uint64_t> keyA(Mcap, s), keyB(Mcap, s);
    // (the value buffers end with room for the row pad: one of them becomes
    // the graph's edge times)
    DArray<uint32_t> valA(Mcap + kRowPad, s), valB(Mcap + kRowPad, s);
    BatchMap bm{0, nullptr, nullptr};
    DArray<uint64_t> d_eoff;
    DArray<uint32_t> d_voff;
    if (hb) {
        d_eoff.reset(hb->n_graphs + 1, s);
        d_voff.reset(hb->n_graphs + 1, s);
        TP_HIP(hipMemcpyAsync(d_eoff.get(), hb->eoff.data(), (hb->n_graphs + 1) * sizeof(uint64_t),
                              hipMemcpyHostToDevice, s));
        TP_HIP(hipMemcpyAsync(d_voff.get(), hb->voff.data(), (hb->n_graphs + 1) * sizeof(uint32_t),
                              hipMemcpyHostToDevice, s));
        bm = BatchMap{hb->n_graphs, d_eoff.get(), d_voff.get()};
    }
    const PairCode pc{lb, local_keys ? d_voff.get() : nullptr};
    if (M) {
        const unsigned blocks = grid_for(M, kB);
        const size_t per_block = (M + blocks - 1) / blocks;
        k_canon<<<blocks, kB, 0, s>>>(src, dst, ts, M, n, pc, dbit, sentinel, keyA.get(), valA.get(), c_bad, c_loop, bm,
                                      per_block);
        TP_CHECK_LAUNCH();
    }
    // ids out of range refuse the input: where the sort takes longer than a
    // wait (some 10 us; 2^24 edges: 1.0 ms), before it, else with the counts
    // that are read after it
    unsigned long long hc[2];  // bad ids, self-loops
    auto check_ids = [&] {
        TP_HIP(hipMemcpyAsync(hc, counters.get(), sizeof(hc), hipMemcpyDeviceToHost, s));
        TP_HIP(hipStreamSynchronize(s));
        if (hc[0]) fail(TP_ERR_INVALID, "tripoll_build: " + std::to_string(hc[0]) + " edge endpoints >= n_vertices");
    };
    const bool check_first = M >= size_t(1) << 24;
    if (check_first) check_ids();
    h_src.release();
    h_dst.release();
    h_ts.release();
    TP_HIP(hipEventRecord(ev[1], s));

    // ---- phase 1: sort by pair
    const bool sorted_in_b = radix_sort_pairs(keyA.get(), valA.get(), keyB.get(), valB.get(), M, kb + dbit, s);
    uint64_t *skey = sorted_in_b ? keyB.get() : keyA.get();
    uint32_t *sval = sorted_in_b ? valB.get() : valA.get();
    uint64_t *fkey = sorted_in_b ? keyA.get() : keyB.get();  // free buffers
    uint32_t *fval = sorted_in_b ? valA.get() : valB.get();
    TP_HIP(hipEventRecord(ev[2], s));

    // ---- phase 2: dedup keeping the earliest time (and the directions)
    uint64_t m = 0;
    DArray<uint8_t> udir;
    if (directed) udir.reset(Mcap, s);
    {
        const size_t nt = std::max<size_t>(1, (M + kCompTile - 1) / kCompTile);
        DArray<uint64_t> toff(nt + 1, s);
        if (M) {
            k_dedup_count<<<(unsigned)nt, kB, 0, s>>>(skey, c_loop, M, dbit, toff.get());
            TP_CHECK_LAUNCH();
        } else {
            TP_HIP(hipMemsetAsync(toff.get(), 0, sizeof(uint64_t), s));
        }
        scan_u64(toff.get(), toff.get(), nt, true, s);
        TP_HIP(hipMemcpyAsync(&m, toff.get() + nt, sizeof(m), hipMemcpyDeviceToHost, s));
        if (check_first) TP_HIP(hipStreamSynchronize(s));
        else check_ids();
        g->stats.n_raw_edges = M;
        g->stats.n_self_loops = hc[1];
        if (m) {
            k_dedup_write<<<(unsigned)nt, kB, 0, s>>>(skey, sval, c_loop, M, dbit, toff.get(), fkey, fval, udir.get());
            TP_CHECK_LAUNCH();
        }
    }
    uint64_t *ukey = fkey;
    uint32_t *uts = fval;
    g->m = m;
    g->stats.n_edges = m;
    TP_HIP(hipEventRecord(ev[3], s));

    // ---- phase 3: degree and the order <+
    DArray<uint32_t> rank(n, s);
    {
        DArray<uint32_t> deg(n, s);
        fill<uint32_t>(deg.get(), 0u, n, s);
        if (m) {
            // the sorted (pre-dedup) pairs are no longer needed: their buffer
            // holds the two halves of the higher-end sort
            uint32_t *hiA = reinterpret_cast<uint32_t *>(skey), *hiB = hiA + Mcap;
            k_degree_low<<<grid_for(m, kB), kB, 0, s>>>(ukey, m, pc, deg.get(), hiA);
            TP_CHECK_LAUNCH();
            if (degree_by_count(m, n, nb)) {
                const int rb = partition_bits(nb);
                DArray<uint64_t> start(((size_t)1 << rb) + 1, s);
                partition_u32(hiA, hiB, m, nb, start.get(), s);
                const int log_range = nb - rb;
                const size_t lds = sizeof(uint32_t) << std::min(log_range, kCountLog);
                TP_HIP(hipFuncSetAttribute((const void *)k_degree_count, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(sizeof(uint32_t) << kCountLog)));
                // a few workgroups' chunks for every compute unit, of a part or more
                const size_t chunk = std::max<size_t>(m / 2048 + 1, std::min<size_t>((m >> rb) + 1, m / 1024 + 1));
                k_degree_count<<<(unsigned)((m + chunk - 1) / chunk), kCountBlock, lds, s>>>(
                    hiB, m, start.get(), 1u << rb, log_range, chunk, deg.get());
                TP_CHECK_LAUNCH();
            } else {
                const bool hb2 = radix_sort_u32(hiA, hiB, m, nb, s);
                k_degree_runs<<<grid_for(m, kB), kB, 0, s>>>(hb2 ? hiB : hiA, m, deg.get());
                TP_CHECK_LAUNCH();
            }
        }
        k_vertex_max<<<stat_grid(n, kB), kB, 0, s>>>(deg.get(), vlab, n, c_dmax, c_lab);
        TP_CHECK_LAUNCH();
        unsigned long long mx[2];
        TP_HIP(hipMemcpyAsync(mx, c_dmax, 2 * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
        TP_HIP(hipStreamSynchronize(s));
        g->stats.d_max = mx[0];
        g->stats.max_label = (uint32_t)mx[1];
        // sort keys (d(v), hash(v)) with the vertex as value
        DArray<uint64_t> rkeyA(n, s), rkeyB(n, s);
        DArray<uint32_t> rvalA(n, s), rvalB(n, s);
        const int gshift = nb + bits_for(mx[0]);
        const int rbits = gshift + (hb ? bits_for(hb->n_graphs - 1) : 0);
        if (rbits > 64) fail(TP_ERR_INVALID, "tripoll_build_batch: too many graphs and vertices for one order key");
        k_rank_keys<<<grid_for(n, kB), kB, 0, s>>>(deg.get(), n, nb, gshift, hb ? d_voff.get() : nullptr,
                                                   hb ? hb->n_graphs : 0u, el->tie_hash, rkeyA.get(), rvalA.get());
        TP_CHECK_LAUNCH();
        const bool rb = radix_sort_pairs(rkeyA.get(), rvalA.get(), rkeyB.get(), rvalB.get(), n, rbits, s);
        const uint64_t *skey = rb ? rkeyB.get() : rkeyA.get();
        g->perm = rb ? std::move(rvalB) : std::move(rvalA);
        g->rlab.reset(n, s);
        k_rank_scatter<<<grid_for(n, kB), kB, 0, s>>>(g->perm.get(), n, vlab, rank.get(), g->rlab.get());
        TP_CHECK_LAUNCH();
        if (hb) {
            g->n_graphs = hb->n_graphs;
            g->rank_gid.reset(n, s);
            k_rank_graph<<<grid_for(n, kB), kB, 0, s>>>(skey, n, gshift, g->rank_gid.get());
            TP_CHECK_LAUNCH();
        }
        {
            // bins 0 .. bin(d_max) are in use; 32 bounds per graph
            uint32_t top = 0;
            for (uint64_t d = mx[0]; d > 1 && top < 31; ++top) d = (d + 1) / 2;
            g->dbin_values = top + 1;
            const size_t nbins = (size_t)32 * (hb ? hb->n_graphs : 1u);
            g->dbin_rank.reset(nbins, s);
            fill_u32<<<grid_for(nbins, kB), kB, 0, s>>>(g->dbin_rank.get(), nbins, 0xffffffffu);
            TP_CHECK_LAUNCH();
            k_dbin_rank<<<grid_for(n, kB), kB, 0, s>>>(skey, n, nb, gshift, hb != nullptr, g->dbin_rank.get());
            TP_CHECK_LAUNCH();
        }
    }
    h_lab.release();
    TP_HIP(hipEventRecord(ev[4], s));

    // ---- phase 4: orient and sort by (source rank, target rank)
    DArray<uint32_t> dplus(n, s);
    fill<uint32_t>(dplus.get(), 0u, n, s);
    if (m) {
        k_orient<<<grid_for(m, kB), kB, 0, s>>>(ukey, udir.get(), m, pc, rank.get(), skey);
        TP_CHECK_LAUNCH();
    }
    rank.release();
    udir.release();
    // keys from k_orient, values the dedup's times (same order); the
    // dedup's keys and the free value buffer take the other halves
    const bool ob = radix_sort_pairs(skey, uts, ukey, sval, m, kb + dbit2, s);
    uint64_t *okey = ob ? ukey : skey;
    uint32_t *ots = ob ? sval : uts;
    uint32_t *spare_val = ob ? uts : sval;
    TP_HIP(hipEventRecord(ev[5], s));

    // ---- phase 5: CSR with co-located metadata
    // col and ets carry kRowPad zeroed slots past the end: the survey loads a
    // whole wave of slots from any row start.  The sorted times are ets
    // itself: their buffer (sized for that pad) moves into the graph.
    g->col.reset(m + kRowPad, s);
    g->tlab.reset(std::max<uint64_t>(m, 1), s);
    g->ets = std::move(ots == valA.get() ? valA : valB);
    if (directed) {
        g->directed = true;
        g->edir.reset(m + kRowPad * 4, s);
    }
    uint32_t *srow = spare_val;
    k_csr<<<grid_for(m, kB), kB, 0, s>>>(okey, m, pc, g->rlab.get(), g->col.get(), g->ets.get(), g->tlab.get(), srow,
                                         g->edir.get(), dplus.get());
    TP_CHECK_LAUNCH();
    g->rowptr.reset((size_t)n + 1, s);
    scan_u32_to_u64(dplus.get(), g->rowptr.get(), n, s);
    dplus.release();
    k_row_stats<<<stat_grid(n, kB), kB, 0, s>>>(g->rowptr.get(), n, c_wedge, c_dpmax);
    TP_CHECK_LAUNCH();
    if (g->dbin_rank.get()) {
        const size_t nbins = g->dbin_rank.n;
        g->dbin_slot.reset(nbins, s);
        k_dbin_slot<<<grid_for(nbins, 64), 64, 0, s>>>(g->dbin_rank.get(), g->rowptr.get(), nbins, g->dbin_slot.get());
        TP_CHECK_LAUNCH();
    }
    TP_HIP(hipEventRecord(ev[6], s));

    // ---- phase 6: in-edge index, a sort of the oriented edges by target
    {
        int kbits = std::max(1, bits_for(m));
        if (kbits + nb + 1 > 64) fail(TP_ERR_UNSUPPORTED, "tripoll_build: graph too large for the in-edge keys");
        g->kbits = (uint32_t)kbits;
        uint64_t *ikey = keyA.get(), *ikey_alt = keyB.get();
        // the payloads go to a buffer of their own (the sorted times became
        // ets); srow's buffer is free once the keys are written
        DArray<uint32_t> pay(std::max<uint64_t>(m, 1), s);
        uint32_t *ival = pay.get(), *ival_alt = srow;
        DArray<uint64_t> has_out;
        if (m) {
            has_out.reset((n + 63) / 64, s);
            k_has_out<<<grid_for(n, kB), kB, 0, s>>>(g->rowptr.get(), n, has_out.get());
            TP_CHECK_LAUNCH();
            k_in_keys<<<stat_grid(m, kB), kB, 0, s>>>(srow, g->col.get(), g->rowptr.get(), has_out.get(),
                                                     g->rlab.get(), m, kbits, n, ikey, ival, c_kept);
            TP_CHECK_LAUNCH();
        }
        const bool alt = radix_sort_pairs(ikey, ival, ikey_alt, ival_alt, m, nb + 1, s, kbits);
        if (alt) {
            std::swap(ikey, ikey_alt);
            std::swap(ival, ival_alt);
        }
        // keep the sorted buffers as the index; the others go back to the pool
        DArray<uint64_t> &kk = (ikey == keyA.get()) ? keyA : keyB;
        DArray<uint32_t> &vv = (ival == pay.get()) ? pay : ((ival == valA.get()) ? valA : valB);
        g->inkey = std::move(kk);
        g->inpay = std::move(vv);
    }
    keyA.release();
    keyB.release();
    valA.release();
    valB.release();
    TP_HIP(hipEventRecord(ev[7], s));

    // ---- phase 7: work per target and the tile plan per class
    PlanCfg cfg{};
    for (int c = 0; c < kNumClasses; ++c) cfg.tile_records[c] = default_tile_records(c);
    unsigned long long hs[8];
    TP_HIP(hipMemcpyAsync(hs, counters.get(), sizeof(hs), hipMemcpyDeviceToHost, s));
    TP_HIP(hipStreamSynchronize(s));
    g->n_in = hs[6];
    g->stats.dplus_max = hs[5];  // the plan cuts huge targets' records
    CutPlan plan = cut_plan(g.get(), cfg, s);
    TP_HIP(hipEventRecord(ev[8], s));
    TP_HIP(hipStreamSynchronize(s));
    adopt_plan(g.get(), plan);

    g->stats.n_vertices = n;
    g->stats.wedges = hs[4];
    // the survey packs a position in Adj+(q) into 22 bits; d+ <= sqrt(2m) keeps
    // this far away for any graph that fits in memory
    if (hs[5] >= (1ull << 22)) fail(TP_ERR_UNSUPPORTED, "tripoll_build: out-degree above 2^22 in the oriented graph");

    float total = 0.f;
    for (int i = 0; i < 8; ++i) {
        float t = 0.f;
        TP_HIP(hipEventElapsedTime(&t, ev[i], ev[i + 1]));
        g->stats.phase_ms[i] = t;
        total += t;
    }
    g->stats.build_ms = total;
    *out = g.release();
}

extern "C" tp_status tripoll_build(const tp_edge_list *edges, void *stream, tp_graph **out)
{
    return guard([&] { build_impl(edges, (hipStream_t)stream, out); });
}

extern "C" tp_status tripoll_build_batch(const tp_batch_edges *be, void *stream, tp_graph **out)
{
    return guard([&] {
        if (!be || !out || !be->edge_offsets || !be->vertex_counts || be->n_graphs == 0)
            fail(TP_ERR_INVALID, "tripoll_build_batch: NULL argument or no graphs");
        HostBatch hb;
        hb.n_graphs = be->n_graphs;
        hb.eoff.assign(be->edge_offsets, be->edge_offsets + be->n_graphs + 1);
        hb.voff.resize(be->n_graphs + 1);
        uint64_t nv = 0;
        hb.voff[0] = 0;
        for (uint32_t i = 0; i < be->n_graphs; ++i) {
            if (hb.eoff[i + 1] < hb.eoff[i]) fail(TP_ERR_INVALID, "tripoll_build_batch: edge offsets decrease");
            nv += be->vertex_counts[i];
            if (nv >= 0xffffffffull) fail(TP_ERR_INVALID, "tripoll_build_batch: more than 2^32-2 vertices in all");
            hb.voff[i + 1] = (uint32_t)nv;
        }
        if (hb.eoff[0] != 0) fail(TP_ERR_INVALID, "tripoll_build_batch: edge_offsets[0] must be 0");
        if (nv == 0) fail(TP_ERR_INVALID, "tripoll_build_batch: no vertices");
        tp_edge_list el{};
        el.n_vertices = (uint32_t)nv;
        el.mem_space = be->mem_space;
        el.n_edges = hb.eoff[be->n_graphs];
        el.src = be->src;
        el.dst = be->dst;
        el.edge_time = be->edge_time;
        el.vertex_label = be->vertex_label;
        el.tie_hash = be->tie_hash;
        if (be->flags & ~TP_EDGES_DIRECTED) fail(TP_ERR_INVALID, "tripoll_build_batch: unknown flags");
        el.flags = be->flags;
        build_impl(&el, (hipStream_t)stream, out, &hb);
    });
}
