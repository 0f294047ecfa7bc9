// prim.hip -- library runtime pieces and device primitives for gfx950:
// per-thread error state, the caching device allocator, exclusive scans and
// a stable LSD radix sort of (uint64 key, uint32 value) pairs.
#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>

#include "pool.hpp"
#include "tp_internal.hpp"

namespace tp {

// ================================================================ errors

static thread_local std::string g_last_error;

void fail(tp_status st, const std::string &msg) { throw Error{st, msg}; }
void set_last_error(const std::string &msg) { g_last_error = msg; }
void clear_last_error() { g_last_error.clear(); }
const char *last_error_cstr() { return g_last_error.c_str(); }

// ================================================================ allocator

namespace {

struct HipDevice {
    using Stream = hipStream_t;
    void *take(size_t bytes)
    {
        void *p = nullptr;
        const hipError_t e = hipMalloc(&p, bytes);
        if (e == hipSuccess) return p;
        (void)hipGetLastError();
        if (e != hipErrorOutOfMemory && e != hipErrorMemoryAllocation)
            fail(TP_ERR_DEVICE, "device allocation of " + std::to_string(bytes) + " bytes failed: " + hipGetErrorString(e));
        return nullptr;
    }
    void give(void *p) { (void)hipFree(p); }
    void wait(hipStream_t s) { (void)hipStreamSynchronize(s); }
};
using Pool = BlockPool<HipDevice>;

Pool &pool_for_current_device()
{
    static std::mutex m;
    static std::map<int, Pool *> pools;
    int dev = 0;
    TP_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(m);
    Pool *&p = pools[dev];
    if (!p) p = new Pool();  // lives until process exit
    return *p;
}

thread_local Pool::Scope t_scope;

// Fault injection: when non-zero, the allocation that brings it to zero
// fails as if the device were out of memory.
std::atomic<uint64_t> g_fail_countdown{0};

}  // namespace

void dev_fail_after(uint64_t n) { g_fail_countdown.store(n); }

CallScope::CallScope(hipStream_t stream) : outer_(!t_scope.pool)
{
    if (outer_) pool_for_current_device().open(t_scope, stream);
}

CallScope::~CallScope()
{
    if (outer_) t_scope.pool->close(t_scope);
}

void *dev_alloc(size_t bytes, hipStream_t stream)
{
    for (uint64_t c = g_fail_countdown.load(); c;) {
        if (g_fail_countdown.compare_exchange_weak(c, c - 1)) {
            if (c == 1) fail(TP_ERR_OOM, "device allocation of " + std::to_string(bytes) + " bytes failed (injected)");
            break;
        }
    }
    void *p = pool_for_current_device().alloc(bytes, stream, &t_scope);
    if (!p) fail(TP_ERR_OOM, "device allocation of " + std::to_string(bytes) + " bytes failed: out of memory");
    return p;
}

void dev_release(void *ptr, hipStream_t stream)
{
    if (ptr) pool_for_current_device().release(ptr, stream, &t_scope);
}

void dev_trim() { pool_for_current_device().trim(); }

size_t dev_cached_bytes() { return pool_for_current_device().cached(); }

size_t dev_live_bytes() { return pool_for_current_device().live(); }

// ================================================================ fill

template <class T>
__global__ void fill_kernel(T *p, T v, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

template <class T>
void fill(T *p, T v, size_t n, hipStream_t s)
{
    if (!n) return;
    fill_kernel<T><<<grid_for(n, 256), 256, 0, s>>>(p, v, n);
    TP_CHECK_LAUNCH();
}
template void fill<uint32_t>(uint32_t *, uint32_t, size_t, hipStream_t);
template void fill<uint64_t>(uint64_t *, uint64_t, size_t, hipStream_t);
template void fill<uint8_t>(uint8_t *, uint8_t, size_t, hipStream_t);

// ================================================================ scan

namespace {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 16;
constexpr size_t kScanTile = (size_t)kScanBlock * kScanItems;

template <class Tin>
__global__ __launch_bounds__(kScanBlock) void scan_reduce_kernel(const Tin *in, uint64_t *partial, size_t n)
{
    __shared__ uint64_t tmp[kScanBlock / kWave];
    const size_t base = blockIdx.x * kScanTile;
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const size_t i = base + (size_t)j * kScanBlock + threadIdx.x;
        if (i < n) s += (uint64_t)in[i];
    }
    s = wave_sum(s);
    if (lane_id() == 0) tmp[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int w = 0; w < kScanBlock / kWave; ++w) t += tmp[w];
        partial[blockIdx.x] = t;
    }
}

// Each thread owns kScanItems consecutive elements.
template <class Tin>
__global__ __launch_bounds__(kScanBlock) void scan_block_kernel(const Tin *in, uint64_t *out, size_t n,
                                                                 const uint64_t *partial, uint64_t *total_out)
{
    __shared__ uint64_t tmp[kScanBlock / kWave];
    const size_t base = blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    uint64_t v[kScanItems];
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const size_t i = base + j;
        v[j] = i < n ? (uint64_t)in[i] : 0;
        s += v[j];
    }
    uint64_t tot;
    uint64_t pre = block_excl_scan<kScanBlock>(s, tmp, tot);
    pre += partial ? partial[blockIdx.x] : 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const size_t i = base + j;
        if (i < n) out[i] = pre;
        pre += v[j];
    }
    if (total_out && blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanBlock - 1) *total_out = pre;
}

template <class Tin>
void scan_impl(const Tin *in, uint64_t *out, size_t n, uint64_t *total_out, hipStream_t s)
{
    if (n == 0) {
        if (total_out) TP_HIP(hipMemsetAsync(total_out, 0, sizeof(uint64_t), s));
        return;
    }
    const size_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 1) {
        scan_block_kernel<Tin><<<1, kScanBlock, 0, s>>>(in, out, n, nullptr, total_out);
        TP_CHECK_LAUNCH();
        return;
    }
    DArray<uint64_t> partial(nb, s);
    scan_reduce_kernel<Tin><<<(unsigned)nb, kScanBlock, 0, s>>>(in, partial.get(), n);
    TP_CHECK_LAUNCH();
    scan_impl<uint64_t>(partial.get(), partial.get(), nb, nullptr, s);
    scan_block_kernel<Tin><<<(unsigned)nb, kScanBlock, 0, s>>>(in, out, n, partial.get(), total_out);
    TP_CHECK_LAUNCH();
}

}  // namespace

void scan_u64(const uint64_t *in, uint64_t *out, size_t n, bool with_total, hipStream_t s)
{
    scan_impl<uint64_t>(in, out, n, with_total ? out + n : nullptr, s);
}

void scan_u32_to_u64(const uint32_t *in, uint64_t *out, size_t n, hipStream_t s)
{
    scan_impl<uint32_t>(in, out, n, out + n, s);
}

// ================================================================ radix sort
//
// Reduce-then-scan LSD radix sort, 9-bit digits (52-bit pair keys take 6
// passes; 8-bit digits took 7 and were slower overall, 10-bit digits write
// runs too short to coalesce), except that a sort takes some 10-bit digits
// where they save a pass (56-bit keys: 6 passes, two of them 10-bit, not 7).
// At most a fixed number of blocks each own a contiguous chunk of tiles (1024 to 8192
// keys).  Per pass:
//   1. upsweep: digit histogram of each block's chunk -> hist[digit][block]
//   2. exclusive scan of each digit's row of hist, and the rows' totals, from
//      which each (digit, block) has its first output position
//   3. downsweep: per tile, each wave ranks its share of the tile stably
//      with ballot-based digit matching; the tile is reordered in LDS by
//      digit and written out in digit runs, so stores are contiguous.

namespace {

constexpr int kSortBlock = 256;  // threads of a row's scan
constexpr int kMaxRadixBits = 10;
constexpr unsigned kMaxSortBlocks = 2048;

// Shape of a downsweep tile: BLOCK threads of ROUNDS keys each; the upsweep's
// threads, and the blocks of both at most.  The wide shape's downsweep has one
// block per compute unit at a time, so 1024 blocks leave it four turns, and
// half the counts of 2048 to write, scan and read (64e6 pairs: a pass 660 to
// 642 us), with as many waves in the upsweep (1024 blocks of 256 threads took
// 1.93 ms where 2048 took 1.51, 1024 of 1024 now 1.47).
template <int BLOCK, int ROUNDS, int UP, unsigned BLOCKS>
struct SortShape {
    static constexpr int kUpBlock = UP;             // threads of an upsweep block
    static constexpr unsigned kMaxBlocks = BLOCKS;
    static constexpr int kBlock = BLOCK;
    static constexpr int kRounds = ROUNDS;
    static constexpr int kWaves = BLOCK / kWave;
    static constexpr int kTile = BLOCK * ROUNDS;
};
using SortSmall = SortShape<256, 4, 256, kMaxSortBlocks>;
using SortNarrow = SortShape<256, 16, 256, kMaxSortBlocks>;
using SortWide = SortShape<1024, 8, 1024, 1024>;

template <int RB>
__device__ __forceinline__ unsigned digit_of(uint64_t k, int shift)
{
    return (unsigned)(k >> shift) & ((1u << RB) - 1);
}

constexpr int kUpLoads = 8;  // keys in flight per thread of an upsweep

// FEW: at most kFewBlocks blocks, whose counts leave as 32-bit words block by
// block, for the downsweep to add up itself.
template <class K, int RB, int BLOCK, bool FEW>
__global__ __launch_bounds__(BLOCK) void radix_upsweep(const K *keys, size_t n, int shift, size_t chunk,
                                                            uint64_t *hist)
{
    constexpr int kRadix = 1 << RB;
    __shared__ unsigned cnt[kRadix];
    for (int d = threadIdx.x; d < kRadix; d += BLOCK) cnt[d] = 0;
    __syncthreads();
    const size_t lo = blockIdx.x * chunk;
    const size_t hi = std::min(n, lo + chunk);
    size_t i = lo + threadIdx.x;
    for (; i + (size_t)(kUpLoads - 1) * BLOCK < hi; i += (size_t)kUpLoads * BLOCK) {
        K k[kUpLoads];
#pragma unroll
        for (int j = 0; j < kUpLoads; ++j) k[j] = keys[i + (size_t)j * BLOCK];
#pragma unroll
        for (int j = 0; j < kUpLoads; ++j) atomicAdd(&cnt[digit_of<RB>(k[j], shift)], 1u);
    }
    for (; i < hi; i += BLOCK) atomicAdd(&cnt[digit_of<RB>(keys[i], shift)], 1u);
    __syncthreads();
    if (FEW) {
        uint32_t *few = reinterpret_cast<uint32_t *>(hist) + (size_t)blockIdx.x * kRadix;
        for (int d = threadIdx.x; d < kRadix; d += BLOCK) few[d] = cnt[d];
    } else {
        for (int d = threadIdx.x; d < kRadix; d += BLOCK) hist[(size_t)d * gridDim.x + blockIdx.x] = cnt[d];
    }
}

// K: uint64_t or uint32_t keys; VALS: whether 32-bit values travel with
// them; RB: bits of the digit.
template <class K, bool VALS, int RB, class S, bool FEW>
// (the narrow shape: two blocks of 4 waves per compute unit, where 10-bit
// digits with values take 191 of 256 registers and 69,680 of 81,920 bytes of LDS)
__global__ __launch_bounds__(S::kBlock, S::kRounds == 16 ? 2 : 1) void radix_downsweep(const K *keys_in, const uint32_t *vals_in,
                                                              K *keys_out, uint32_t *vals_out, size_t n,
                                                              int shift, size_t tiles_per_block,
                                                              const uint64_t *offsets)
{
    constexpr int kRadix = 1 << RB;
    constexpr int kSortBlock = S::kBlock, kSortWaves = S::kWaves, kSortRounds = S::kRounds, kSortTile = S::kTile;
    constexpr int kDigitsPerThread = kRadix > kSortBlock ? kRadix / kSortBlock : 1;
    constexpr int kDigitThreads = kRadix / kDigitsPerThread;
    __shared__ K skey[kSortTile];
    __shared__ uint32_t sval[VALS ? kSortTile : 1];
    // per-wave running count, then per-wave base within the digit (at most a
    // tile's keys: 16 bits)
    __shared__ uint16_t wcnt[kSortWaves][kRadix];
    __shared__ unsigned tstart[kRadix];
    __shared__ uint64_t grun[kRadix];              // next output position of each digit
    __shared__ unsigned scan_tmp[kSortWaves];

    const int w = threadIdx.x / kWave;
    const unsigned lane = lane_id();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    if (FEW) {
        // the digit's first place: all smaller digits, then this one in the
        // blocks before
        const uint32_t *few = reinterpret_cast<const uint32_t *>(offsets);
        unsigned before[kDigitsPerThread], all[kDigitsPerThread], sum = 0;
        const bool mine = kDigitThreads == kSortBlock || (int)threadIdx.x < kDigitThreads;
#pragma unroll
        for (int j = 0; j < kDigitsPerThread; ++j) before[j] = all[j] = 0;
        if (mine) {
#pragma unroll 8
            for (unsigned b = 0; b < gridDim.x; ++b) {
#pragma unroll
                for (int j = 0; j < kDigitsPerThread; ++j) {
                    const unsigned c = few[(size_t)b * kRadix + threadIdx.x * kDigitsPerThread + j];
                    before[j] += b < blockIdx.x ? c : 0u;
                    all[j] += c;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kDigitsPerThread; ++j) sum += all[j];
        unsigned total;
        unsigned at = block_excl_scan<kSortBlock>(sum, scan_tmp, total);
        if (mine) {
#pragma unroll
            for (int j = 0; j < kDigitsPerThread; ++j) {
                grun[threadIdx.x * kDigitsPerThread + j] = at + before[j];
                at += all[j];
            }
        }
    } else {
        // all smaller digits (their totals follow the rows), then this digit
        // in the blocks before (the scanned row)
        const uint64_t *total = offsets + (size_t)kRadix * gridDim.x;
        uint64_t sum = 0, all[kDigitsPerThread];
        const bool mine = kDigitThreads == kSortBlock || (int)threadIdx.x < kDigitThreads;
#pragma unroll
        for (int j = 0; j < kDigitsPerThread; ++j) {
            all[j] = mine ? total[threadIdx.x * kDigitsPerThread + j] : 0ull;
            sum += all[j];
        }
        __shared__ uint64_t wide_tmp[kSortWaves];
        uint64_t end;
        uint64_t at = block_excl_scan<kSortBlock>(sum, wide_tmp, end);
        if (mine) {
#pragma unroll
            for (int j = 0; j < kDigitsPerThread; ++j) {
                const unsigned d = threadIdx.x * kDigitsPerThread + j;
                grun[d] = at + offsets[(size_t)d * gridDim.x + blockIdx.x];
                at += all[j];
            }
        }
    }
    for (int d = threadIdx.x; d < kRadix; d += kSortBlock)
        for (int i = 0; i < kSortWaves; ++i) wcnt[i][d] = 0;
    __syncthreads();

    const size_t t0 = blockIdx.x * tiles_per_block;
    // the keys and values of the next tile are requested while this one is
    // ranked and written, so that the loads overlap the tile's work
    K kn[kSortRounds];
    uint32_t vn[kSortRounds];
    auto load_tile = [&](size_t t) {
        const size_t wl = t * kSortTile + (size_t)w * (kSortTile / kSortWaves);
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const size_t i = wl + (size_t)r * kWave + lane;
            kn[r] = i < n ? keys_in[i] : 0;
            vn[r] = (VALS && i < n) ? vals_in[i] : 0;
        }
    };
    if (t0 * kSortTile < n) load_tile(t0);
    for (size_t t = t0; t < t0 + tiles_per_block; ++t) {
        const size_t tile_lo = t * kSortTile;
        if (tile_lo >= n) break;
        const size_t wave_lo = tile_lo + (size_t)w * (kSortTile / kSortWaves);

        K k[kSortRounds];
        uint32_t v[kSortRounds];
        unsigned rnk[kSortRounds];
        unsigned dg[kSortRounds];
        bool ok[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const size_t i = wave_lo + (size_t)r * kWave + lane;
            ok[r] = i < n;
            k[r] = kn[r];
            v[r] = vn[r];
            dg[r] = digit_of<RB>(k[r], shift);
        }
        if (t + 1 < t0 + tiles_per_block && (t + 1) * kSortTile < n) load_tile(t + 1);
        // stable rank of every key among equal digits of this wave's share
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            uint64_t peers = __ballot(ok[r]);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const bool bit = (dg[r] >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            unsigned before = 0;
            if (ok[r]) {
                before = wcnt[w][dg[r]];
                rnk[r] = before + (unsigned)__popcll(peers & lt_mask);
            }
            // the lowest lane of each digit group advances the running count;
            // same-wave LDS accesses are performed in program order
            if (ok[r] && (peers & lt_mask) == 0) wcnt[w][dg[r]] = (uint16_t)(before + (unsigned)__popcll(peers));
        }
        __syncthreads();
        // per-digit totals, wave bases and tile starts
        {
            unsigned loc[kDigitsPerThread];
            unsigned sum = 0;
            const bool mine = kDigitThreads == kSortBlock || (int)threadIdx.x < kDigitThreads;
#pragma unroll
            for (int j = 0; j < kDigitsPerThread; ++j) {
                const unsigned d = threadIdx.x * kDigitsPerThread + j;
                unsigned tot = 0;
                if (mine) {
#pragma unroll
                    for (int i = 0; i < kSortWaves; ++i) {
                        const unsigned c = wcnt[i][d];
                        wcnt[i][d] = (uint16_t)tot;
                        tot += c;
                    }
                }
                loc[j] = sum;
                sum += tot;
            }
            unsigned total;
            const unsigned base = block_excl_scan<kSortBlock>(sum, scan_tmp, total);
            if (mine) {
#pragma unroll
                for (int j = 0; j < kDigitsPerThread; ++j) tstart[threadIdx.x * kDigitsPerThread + j] = base + loc[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            if (ok[r]) {
                const unsigned pos = tstart[dg[r]] + wcnt[w][dg[r]] + rnk[r];
                skey[pos] = k[r];
                if (VALS) sval[pos] = v[r];
            }
        }
        __syncthreads();
        const unsigned valid = (unsigned)std::min<size_t>(kSortTile, n - tile_lo);
        for (unsigned i = threadIdx.x; i < valid; i += kSortBlock) {
            const K key = skey[i];
            const unsigned d = digit_of<RB>(key, shift);
            const uint64_t dst = grun[d] + (i - tstart[d]);
            keys_out[dst] = key;
            if (VALS) vals_out[dst] = sval[i];
        }
        __syncthreads();
        for (int d = threadIdx.x; d < kRadix; d += kSortBlock) {
            // the digit's keys in this tile: up to the next digit's start
            grun[d] += (d + 1 < kRadix ? tstart[d + 1] : valid) - tstart[d];
            for (int i = 0; i < kSortWaves; ++i) wcnt[i][d] = 0;
        }
        __syncthreads();
    }
}

// One block per digit: the exclusive scan of its row of block counts, in
// place, and the row's total past the rows.  Each downsweep block scans the
// totals over the digits itself, so that a pass takes three launches where a
// scan of the whole table took five (300,007 vertices, 3.3e6 raw edges, 14
// passes: build and survey 2.32 -> 2.11 ms).
static_assert(kMaxSortBlocks <= kSortBlock * 8, "a row is scanned by one block of 8 counts a thread");
__global__ __launch_bounds__(kSortBlock) void radix_rows(uint64_t *hist, unsigned blocks)
{
    __shared__ uint64_t tmp[kSortBlock / kWave];
    uint64_t *row = hist + (size_t)blockIdx.x * blocks;
    uint64_t v[8], sum = 0;
    const unsigned b0 = threadIdx.x * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = b0 + j < blocks ? row[b0 + j] : 0ull;
        sum += v[j];
    }
    uint64_t total;
    uint64_t at = block_excl_scan<kSortBlock>(sum, tmp, total);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (b0 + j < blocks) row[b0 + j] = at;
        at += v[j];
    }
    if (threadIdx.x == 0) hist[(size_t)gridDim.x * blocks + blockIdx.x] = total;
}

// Up to this many blocks a downsweep adds up the blocks' counts itself (each
// reads all of them): a pass takes 2 launches (65,536 pairs in 16 blocks: about
// 55 -> 21 us a pass with the gaps; in 64 blocks of 1024-key tiles, 14 us).
// Whole builds of 30,000 vertices by the tile of their sorts, 1024 against 4096
// keys: 65,536 edges 500 against 541 us, 100,000 532 against 546, 131,072 548
// against 562, 200,000 616 against 576 (of 256 small blocks each reads 4 times
// the counts): between 65,536 and 200,000 the line gives or takes 3%.
constexpr unsigned kFewBlocks = 64;

// One pass over digit [shift, shift + RB): histograms, their scan, the
// stable scatter (values travel when vi is set, as they always do with 64-bit
// keys).
template <class K, int RB, class S, bool FEW>
void sort_pass(const K *ki, const uint32_t *vi, K *ko, uint32_t *vo, size_t n, int shift, unsigned nb, size_t tpb,
               uint64_t *hist, hipStream_t s)
{
    radix_upsweep<K, RB, S::kUpBlock, FEW><<<nb, S::kUpBlock, 0, s>>>(ki, n, shift, tpb * S::kTile, hist);
    TP_CHECK_LAUNCH();
    if (!FEW) {
        radix_rows<<<1u << RB, kSortBlock, 0, s>>>(hist, nb);
        TP_CHECK_LAUNCH();
    }
    if (sizeof(K) == 8 || vi) {
        radix_downsweep<K, true, RB, S, FEW><<<nb, S::kBlock, 0, s>>>(ki, vi, ko, vo, n, shift, tpb, hist);
    } else if constexpr (sizeof(K) == 4) {
        radix_downsweep<K, false, RB, S, FEW><<<nb, S::kBlock, 0, s>>>(ki, nullptr, ko, nullptr, n, shift, tpb, hist);
    }
    TP_CHECK_LAUNCH();
}

template <class K, class S, bool FEW>
bool radix_sort_shape(K *keys, uint32_t *vals, K *keys_alt, uint32_t *vals_alt, size_t n, int bits, hipStream_t s,
                      int begin_bit)
{
    const size_t tiles = (n + S::kTile - 1) / S::kTile;
    const unsigned nb = (unsigned)std::min<size_t>(tiles, S::kMaxBlocks);
    const size_t tpb = (tiles + nb - 1) / nb;
    DArray<uint64_t> hist((size_t)(1u << kMaxRadixBits) * (nb + 1), s);  // the rows, then their totals
    // 9-bit digits, or as few 10-bit ones as cover `bits` in one pass less
    const int p9 = (bits + 8) / 9, p10 = (bits + 9) / 10;
    const int passes = std::min(p9, p10);
    const int n10 = passes < p9 ? bits - 9 * passes : 0;
    bool in_alt = false;
    int shift = begin_bit;
    for (int pass = 0; pass < passes; ++pass) {
        const K *ki = in_alt ? keys_alt : keys;
        const uint32_t *vi = in_alt ? vals_alt : vals;
        K *ko = in_alt ? keys : keys_alt;
        uint32_t *vo = in_alt ? vals : vals_alt;
        if (pass < n10) sort_pass<K, 10, S, FEW>(ki, vi, ko, vo, n, shift, nb, tpb, hist.get(), s);
        else sort_pass<K, 9, S, FEW>(ki, vi, ko, vo, n, shift, nb, tpb, hist.get(), s);
        shift += pass < n10 ? 10 : 9;
        in_alt = !in_alt;
    }
    return in_alt;
}

// All passes of a sort of at most kOneKeys pairs in one workgroup: keys and
// values stay in registers (wave w's in places [64 r w, 64 r (w + 1)), r rounds)
// and trade places through LDS.  What bounds sorts of this size is the launches
// and a pass's chain of waits: here one launch, 17 us for 4096 keys of 24 bits,
// where the smallest shape takes two launches a pass.  A build of 1000 / 8000
// edges (both its sorts): 395 -> 307 / 451 -> 392 us; of 2^16 edges with 4096
// vertices (the order only), with its survey: 728 -> 698; at 8192 vertices and
// 30,000 edges still 498 -> 453.
constexpr int kOneBlock = 1024;
constexpr int kOneRounds = 8;
constexpr size_t kOneKeys = (size_t)kOneBlock * kOneRounds;

__global__ __launch_bounds__(kOneBlock) void radix_sort_one(uint64_t *keys, uint32_t *vals, unsigned n, int bits,
                                                            int begin_bit)
{
    constexpr int RB = 8, kRadix = 1 << RB, kWaves = kOneBlock / kWave;
    __shared__ uint64_t skey[kOneKeys];
    __shared__ uint32_t sval[kOneKeys];
    __shared__ uint16_t wcnt[kWaves][kRadix];
    __shared__ unsigned tstart[kRadix];
    __shared__ unsigned scan_tmp[kWaves];
    const int w = threadIdx.x / kWave;
    const unsigned lane = lane_id();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int rounds = (int)((n + kOneBlock - 1) / kOneBlock); // of each wave
    const unsigned first = (unsigned)(w * rounds * kWave) + lane;
    uint64_t k[kOneRounds];
    uint32_t v[kOneRounds];
#pragma unroll
    for (int r = 0; r < kOneRounds; ++r) {
        const unsigned i = first + (unsigned)r * kWave;
        const bool ok = r < rounds && i < n;
        k[r] = ok ? keys[i] : 0ull;
        v[r] = ok ? vals[i] : 0u;
    }
    for (int done = 0; done < bits; done += RB) {
        const int shift = begin_bit + done;
        const unsigned mask = bits - done < RB ? (1u << (bits - done)) - 1u : kRadix - 1u;
        for (int d = threadIdx.x; d < kRadix * kWaves; d += kOneBlock) wcnt[d / kRadix][d % kRadix] = 0;
        __syncthreads();
        unsigned rnk[kOneRounds];
#pragma unroll
        for (int r = 0; r < kOneRounds; ++r) {
            if (r >= rounds) break;
            const bool ok = first + (unsigned)r * kWave < n;
            const unsigned d = (unsigned)(k[r] >> shift) & mask;
            uint64_t peers = __ballot(ok);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            unsigned before = 0;
            if (ok) {
                before = wcnt[w][d];
                rnk[r] = before + (unsigned)__popcll(peers & lt_mask);
            }
            // (as in radix_downsweep)
            if (ok && (peers & lt_mask) == 0) wcnt[w][d] = (uint16_t)(before + (unsigned)__popcll(peers));
        }
        __syncthreads();
        unsigned tot = 0;
        if (threadIdx.x < kRadix) {
#pragma unroll
            for (int i = 0; i < kWaves; ++i) {
                const unsigned c = wcnt[i][threadIdx.x];
                wcnt[i][threadIdx.x] = (uint16_t)tot;
                tot += c;
            }
        }
        unsigned total;
        const unsigned base = block_excl_scan<kOneBlock>(tot, scan_tmp, total);
        if (threadIdx.x < kRadix) tstart[threadIdx.x] = base;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kOneRounds; ++r) {
            if (r < rounds && first + (unsigned)r * kWave < n) {
                const unsigned d = (unsigned)(k[r] >> shift) & mask;
                const unsigned pos = tstart[d] + wcnt[w][d] + rnk[r];
                skey[pos] = k[r];
                sval[pos] = v[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kOneRounds; ++r) {
            const unsigned i = first + (unsigned)r * kWave;
            if (r < rounds && i < n) {
                k[r] = skey[i];
                v[r] = sval[i];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < kOneRounds; ++r) {
        const unsigned i = first + (unsigned)r * kWave;
        if (r < rounds && i < n) {
            keys[i] = k[r];
            vals[i] = v[r];
        }
    }
}

// 64-bit keys from kWideKeys on take the wide shape's tiles of 8192 keys, one
// per compute unit: a digit's keys of a tile fill whole lines of the output
// (16 keys, 128 bytes, against 8), and half as many lines are open for writing
// at a time (1.05e9 pairs: a 9-bit downsweep 7.46 -> 6.67 ms, 3.8 TB/s of reads
// and writes where a copy reaches 4.6; 512 threads of 16 keys 6.70 ms; 64e6
// pairs 535 -> 483 us).  32-bit keys alone move a third of the bytes and gain
// more from a second block per compute unit (3.92 against 4.97 ms), and fewer
// keys than that leave compute units without a tile.
constexpr size_t kWideKeys = size_t(1) << 22;

template <class K>
bool radix_sort(K *keys, uint32_t *vals, K *keys_alt, uint32_t *vals_alt, size_t n, int bits, hipStream_t s,
                int begin_bit)
{
    if (n <= 1 || bits <= 0) return false;
    if constexpr (sizeof(K) == 8) {
        if (n >= kWideKeys)
            return radix_sort_shape<K, SortWide, false>(keys, vals, keys_alt, vals_alt, n, bits, s, begin_bit);
    }
    if (n <= (size_t)kFewBlocks * SortSmall::kTile)
        return radix_sort_shape<K, SortSmall, true>(keys, vals, keys_alt, vals_alt, n, bits, s, begin_bit);
    if (n <= (size_t)kFewBlocks * SortNarrow::kTile)
        return radix_sort_shape<K, SortNarrow, true>(keys, vals, keys_alt, vals_alt, n, bits, s, begin_bit);
    return radix_sort_shape<K, SortNarrow, false>(keys, vals, keys_alt, vals_alt, n, bits, s, begin_bit);
}

}  // namespace

bool radix_sort_pairs(uint64_t *keys, uint32_t *vals, uint64_t *keys_alt, uint32_t *vals_alt, size_t n, int bits,
                      hipStream_t s, int begin_bit)
{
    if (n > 1 && n <= kOneKeys && bits > 0) {
        radix_sort_one<<<1, kOneBlock, 0, s>>>(keys, vals, (unsigned)n, bits, begin_bit);
        TP_CHECK_LAUNCH();
        return false;
    }
    return radix_sort<uint64_t>(keys, vals, keys_alt, vals_alt, n, bits, s, begin_bit);
}

bool radix_sort_pairs32(uint32_t *keys, uint32_t *vals, uint32_t *keys_alt, uint32_t *vals_alt, size_t n, int bits,
                        hipStream_t s)
{
    return radix_sort<uint32_t>(keys, vals, keys_alt, vals_alt, n, bits, s, 0);
}

// Partition by the top bits: one pass of the sort.  The blocks' scanned rows
// hold each digit's place only relative to the digit, so the starts are summed
// from the totals here.
namespace {
template <int RB>
__global__ __launch_bounds__(kSortBlock) void partition_starts(const uint64_t *total, uint64_t n, uint64_t *start)
{
    __shared__ uint64_t tmp[kSortBlock / kWave];
    constexpr int kPer = (1 << RB) / kSortBlock;
    uint64_t v[kPer], sum = 0, all;
    for (int j = 0; j < kPer; ++j) {
        v[j] = total[threadIdx.x * kPer + j];
        sum += v[j];
    }
    uint64_t at = block_excl_scan<kSortBlock>(sum, tmp, all);
    for (int j = 0; j < kPer; ++j) {
        start[threadIdx.x * kPer + j] = at;
        at += v[j];
    }
    if (threadIdx.x == 0) start[1 << RB] = n;
}

template <int RB>
void partition(const uint32_t *keys, uint32_t *out, size_t n, int shift, uint64_t *start, hipStream_t s)
{
    using S = SortNarrow;
    const size_t tiles = (n + S::kTile - 1) / S::kTile;
    const unsigned nb = (unsigned)std::min<size_t>(tiles, kMaxSortBlocks);
    const size_t tpb = (tiles + nb - 1) / nb;
    DArray<uint64_t> hist((size_t)(1u << RB) * (nb + 1), s);
    sort_pass<uint32_t, RB, S, false>(keys, nullptr, out, nullptr, n, shift, nb, tpb, hist.get(), s);
    partition_starts<RB><<<1, kSortBlock, 0, s>>>(hist.get() + (size_t)(1u << RB) * nb, n, start);
    TP_CHECK_LAUNCH();
}
}  // namespace

int partition_bits(int bits) { return bits <= 24 ? 9 : 10; }

void partition_u32(const uint32_t *keys, uint32_t *out, size_t n, int bits, uint64_t *start, hipStream_t s)
{
    const int rb = partition_bits(bits);
    if (rb == 9) partition<9>(keys, out, n, bits - rb, start, s);
    else partition<10>(keys, out, n, bits - rb, start, s);
}

bool radix_sort_u32(uint32_t *keys, uint32_t *keys_alt, size_t n, int bits, hipStream_t s, int begin_bit)
{
    return radix_sort<uint32_t>(keys, nullptr, keys_alt, nullptr, n, bits, s, begin_bit);
}

}  // namespace tp
