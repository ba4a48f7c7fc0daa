// Selection (section 4.2, Q3; section 3.2, Q0) and projection (section 4.1,
// Q1 and Q2) kernels, plus the fill kernels used to clear outputs.
#include "block.hpp"
#include "internal.hpp"
#include "variants.hpp"

namespace crystal {

// ------------------------------------------------------------------ fills --
__global__ __launch_bounds__(256) void fill_u64_kernel(uint64_t *__restrict__ p, int64_t n,
                                                       uint64_t value) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        p[i] = value;
}

// zero p[0..n) and one word elsewhere
__global__ __launch_bounds__(256) void zero_and_word_kernel(uint64_t *__restrict__ p, int64_t n, uint64_t *word) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
    if (i == 0) *word = 0;
}

__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t *__restrict__ p, int64_t n,
                                                       uint32_t value) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        p[i] = value;
}

__global__ void zero_pair_kernel(uint64_t *a, uint64_t *b) {
    if (threadIdx.x == 0) *a = 0;
    if (threadIdx.x == 1) *b = 0;
}

hipError_t zero_pair(uint64_t *a, uint64_t *b, hipStream_t s) {
    hipLaunchKernelGGL(zero_pair_kernel, dim3(1), dim3(64), 0, s, a, b);
    return hipGetLastError();
}

static int64_t fill_grid(int64_t n) {
    int64_t g = (n + 255) / 256;
    int64_t cap = (int64_t)device_cu_count() * 16;
    return g < cap ? (g > 0 ? g : 1) : cap;
}

hipError_t fill_u64(uint64_t *p, int64_t n, uint64_t value, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3((unsigned)fill_grid(n)), dim3(256), 0, s, p, n, value);
    return hipGetLastError();
}

hipError_t fill_u32(uint32_t *p, int64_t n, uint32_t value, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)fill_grid(n)), dim3(256), 0, s, p, n, value);
    return hipGetLastError();
}

static hipError_t zero_and_word(uint64_t *p, int64_t n, uint64_t *word, hipStream_t s) {
    hipLaunchKernelGGL(zero_and_word_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, word);
    return hipGetLastError();
}

// Zero several equal-sized slots of one array in one launch: slot slots[i]
// covers base[slots[i] * len, (slots[i] + 1) * len).
struct SlotList {
    int32_t count;
    int32_t slot[kMaxSlots];
};

__global__ __launch_bounds__(256) void zero_slots_kernel(uint64_t *__restrict__ base, int64_t len, SlotList l) {
    const int64_t n = (int64_t)l.count * len;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int64_t k = i / len;
        base[(int64_t)l.slot[k] * len + (i - k * len)] = 0ull;
    }
}

hipError_t zero_slots(uint64_t *base, int64_t len, const int32_t *slots, int count, hipStream_t s) {
    if (count <= 0 || len <= 0) return hipSuccess;
    if (count > kMaxSlots) return hipErrorInvalidValue;
    SlotList l = {};
    l.count = count;
    for (int i = 0; i < count; ++i) l.slot[i] = slots[i];
    hipLaunchKernelGGL(zero_slots_kernel, dim3((unsigned)fill_grid((int64_t)count * len)), dim3(256), 0, s, base, len,
                       l);
    return hipGetLastError();
}

// The results a served step completes, written straight into pinned host
// memory (dst and status_copy).  A copy call per query cost about 10 us each
// on the stream: a step that completes 32 queries went from 33 calls to one
// launch, bound by the 900 KB it sends over PCIe.
__global__ __launch_bounds__(256) void copy_ranges_kernel(const uint64_t *__restrict__ src, uint64_t *__restrict__ dst,
                                                          WordRanges ranges, const int32_t *__restrict__ status,
                                                          int32_t *__restrict__ status_copy) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 == 0) *status_copy = *status;
    for (int k = 0; k < ranges.count; ++k) {
        const int64_t at = ranges.r[k].at;
        for (int64_t i = i0; i < ranges.r[k].len; i += stride) dst[at + i] = src[at + i];
    }
}

hipError_t copy_ranges(const uint64_t *src, uint64_t *dst, const WordRanges &ranges, const int32_t *status,
                       int32_t *status_copy, hipStream_t s) {
    if (ranges.count < 0 || ranges.count > kMaxSlots) return hipErrorInvalidValue;
    int64_t longest = 1;
    for (int k = 0; k < ranges.count; ++k) longest = ranges.r[k].len > longest ? ranges.r[k].len : longest;
    hipLaunchKernelGGL(copy_ranges_kernel, dim3((unsigned)fill_grid(longest)), dim3(256), 0, s, src, dst, ranges,
                       status, status_copy);
    return hipGetLastError();
}

// ------------------------------------------------------------- selection --
// Tile = BlockLoad -> BlockPred -> BlockScan of the match counts -> the tile's
// output offset -> BlockShuffle into LDS (matches in input order within the
// tile) -> BlockStore.
//
// Output offsets, two ways:
//  - unordered (the method of section 3.2): thread 0 reserves the tile's
//    output range with one 64-bit atomic on the global counter, skipped when
//    the tile has no match.  Same-address atomics from the eight XCDs
//    serialise at the memory-side atomic unit (about 12 ns each on MI355X),
//    so tiles are large (the tuned default is 1024 x 16 = 16 Ki items) to
//    keep the reservations well below the time the column takes to stream.
//  - stable: sums on three levels.  A tile publishes its match count; the
//    last tile of a group (64 tiles) also the group's, once it has read the
//    others'; the last tile of a supergroup (64 groups) the supergroup's.  A
//    tile's offset is then at most 63 words of tiles, 63 of groups and the
//    earlier supergroups, read by one wave in one memory round trip once they
//    are there.  Tiles land in input order, so the output is the qualifying
//    values in input order on every run.
//
//    What bounds it is the wait for words that all XCDs see.  With a status
//    word per tile only (decoupled look-back), 1,024 tiles that start together
//    learn their offsets 64 or 512 at a time, one round trip after another,
//    and every poll reads as many words: 64M rows, half of them qualifying,
//    took 161 us (512 words a round, read by the whole workgroup) and 106 us
//    (64, by one wave), 80 us so.  (Sums added up with atomics serialised on
//    their lines: 560 us.)
//
// Words are read and written with agent-scope atomics (coherent across XCDs)
// and are zero before the launch.  There is one tile per workgroup, dispatched
// in order, a tile publishes before it waits, and a group's and a supergroup's
// word need only words of their own tiles and groups, so every wait ends;
// should a predecessor still never publish, the wait gives up after a bounded
// number of polls: the tile writes nothing and the count becomes -1.
static constexpr uint32_t kPublished = 1u << 31;          // a tile's or group's word: this and its count
static constexpr uint64_t kSuperPublished = 1ull << 63;
static constexpr uint32_t kLookbackPolls = 1u << 15;

// The words of n_tiles tiles, in at most 8 bytes per tile: groups are needed
// from 65 tiles on, supergroups from 4,097.
struct TileSums {
    uint64_t *super;
    uint32_t *group, *tile;
    __host__ __device__ TileSums(void *mem, int64_t n_tiles) {
        const int64_t ns = n_tiles > 4096 ? (n_tiles + 4095) / 4096 : 0, ng = n_tiles > 64 ? (n_tiles + 63) / 64 : 0;
        super = (uint64_t *)mem;
        group = (uint32_t *)(super + ns);
        tile = group + ng;
    }
};

template <typename W>
__device__ __forceinline__ W word_load(const W *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename W>
__device__ __forceinline__ void word_store(W *p, W v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by one whole wave after the tile's own word was published: the number
// of matches in all tiles before `tile`, or ~0 if a wait gave up.
__device__ __forceinline__ uint64_t matches_before(const TileSums &w, int64_t tile, int64_t n_tiles, uint32_t count) {
    const uint32_t lane = lane_id();
    const int64_t group = tile / 64, super = tile / 4096;
    bool need_t = lane < (uint32_t)(tile & 63), need_g = lane < (uint32_t)(group & 63);
    bool owe_g = (tile & 63) == 63 && n_tiles > 64, owe_s = (tile & 4095) == 4095 && n_tiles > 4096;
    int64_t s = lane;  // this lane's next supergroup
    uint32_t t = 0, g = 0;
    uint64_t before = 0;
    for (uint32_t polls = 0; polls < kLookbackPolls; ++polls) {
        __builtin_amdgcn_s_sleep(8);  // polls that find nothing slow the stores they wait for
        uint64_t u = 0;
        if (need_t) t = word_load(w.tile + (tile & ~int64_t(63)) + lane);
        if (need_g) g = word_load(w.group + (group & ~int64_t(63)) + lane);
        if (s < super) u = word_load(w.super + s);
        need_t = need_t && !(t & kPublished);
        need_g = need_g && !(g & kPublished);
        if (u & kSuperPublished) {
            before += u & ~kSuperPublished;
            s += kWave;
        }
        const bool tiles_in = ballot(need_t) == 0, groups_in = ballot(need_g) == 0;
        if (owe_g && tiles_in) {
            const uint32_t sum = (uint32_t)wave_sum_u64(t & ~kPublished) + count;  // at most 2^20
            if (lane == 0) word_store(w.group + group, kPublished | sum);
            owe_g = false;
        }
        if (owe_s && tiles_in && groups_in) {
            const uint64_t sum = wave_sum_u64((uint64_t)(t & ~kPublished) + (g & ~kPublished)) + count;
            if (lane == 0) word_store(w.super + super, kSuperPublished | sum);
            owe_s = false;
        }
        if (tiles_in && groups_in && ballot(s < super) == 0)
            return wave_sum_u64(before + (t & ~kPublished) + (g & ~kPublished));
    }
    return ~0ull;
}

// Store n entries of buf (LDS) to dst: scalar stores up to a 16-byte boundary,
// vectors, then the tail.
template <int BLOCK>
__device__ __forceinline__ void store_run(const int32_t *buf, uint32_t n, int32_t *__restrict__ dst) {
    uint32_t head = (uint32_t)(((16u - ((uint32_t)(uintptr_t)dst & 15u)) & 15u) >> 2);
    if (head > n) head = n;
    if (threadIdx.x < head) __builtin_nontemporal_store(buf[threadIdx.x], dst + threadIdx.x);
    const uint32_t nvec = (n - head) >> 2;
    for (uint32_t i = threadIdx.x; i < nvec; i += BLOCK) {
        const uint32_t b = head + 4 * i;
        const v4i x = {buf[b], buf[b + 1], buf[b + 2], buf[b + 3]};
        __builtin_nontemporal_store(x, reinterpret_cast<v4i *>(dst + b));
    }
    for (uint32_t i = head + 4 * nvec + threadIdx.x; i < n; i += BLOCK) __builtin_nontemporal_store(buf[i], dst + i);
}

// Stable selection: one workgroup per tile.  A wave owns 64 * IPT consecutive
// items, chunk by chunk of 64 vectors, so it ranks its own matches and the waves
// exchange one total each.  In a chunk, lane l's items follow lane l - 1's: an
// item's place is the matches of all lanes below (one ballot per item of the
// vector, counted with mbcnt, which also adds) and of the lane's items before
// it.  (With chunks across the workgroup the exchange of every wave's chunk
// totals, and the scan of per-lane counts bit by bit, made the kernel bound by
// its instructions: 103 us for 64M rows, half of them qualifying.)
template <int BLOCK, int IPT>
__global__ __launch_bounds__(BLOCK) void select_kernel(const int32_t *__restrict__ in, int64_t n,
                                                       int32_t lo, int32_t hi, int32_t *__restrict__ out,
                                                       TileSums sums, int64_t *__restrict__ count_out,
                                                       int64_t n_tiles) {
    using T = TileShape<BLOCK, IPT>;
    constexpr int C = T::CHUNKS, W = T::WAVES, V = T::VEC;
    __shared__ int32_t buf[T::ITEMS];
    __shared__ uint32_t wave_tot[W];
    __shared__ uint64_t out_base;
    const int w = threadIdx.x / kWave;
    const uint32_t lane = lane_id();
    const int64_t tile = blockIdx.x;
    const int64_t i0 = tile * T::ITEMS + (int64_t)w * (kWave * IPT) + (int64_t)lane * V;  // chunk 0, item 0
    const bool full = (tile + 1) * T::ITEMS <= n;
    int32_t v[IPT];
    if (full) {
#pragma unroll
        for (int c = 0; c < C; ++c) load_vec<V, true>(in + i0 + c * (kWave * V), &v[c * V]);
    } else {
        // vectors as far as the column goes, then its last items
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int64_t i = i0 + c * (kWave * V);
#pragma unroll
            for (int e = 0; e < V; ++e) v[c * V + e] = 0;
            if (i + V <= n) {
                load_vec<V, true>(in + i, &v[c * V]);
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (i + e < n) v[c * V + e] = in[i + e];
            }
        }
    }
    uint64_t m[IPT];
    uint32_t pos[C], run = 0;  // run: the wave's matches so far (uniform)
#pragma unroll
    for (int c = 0; c < C; ++c) {
        pos[c] = run;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int k = c * V + e;
            bool q = in_range(v[k], lo, hi);
            if (!full) q = q && i0 + c * (kWave * V) + e < n;
            m[k] = ballot(q);
            pos[c] = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], pos[c]));
            run += (uint32_t)__popcll(m[k]);
        }
    }
    if (lane == 0) wave_tot[w] = run;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const uint32_t t = wave_tot[i];
        before = i == w ? total : before;
        total += t;
    }
    if (threadIdx.x == 0 && n_tiles > 1) word_store(sums.tile + tile, kPublished | total);
    // BlockShuffle: matches to their tile positions in LDS
#pragma unroll
    for (int c = 0; c < C; ++c) {
        uint32_t p = before + pos[c];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const bool q = __builtin_amdgcn_inverse_ballot_w64(m[c * V + e]);
            if (q) buf[p] = v[c * V + e];
            p += q ? 1u : 0u;
        }
    }
    // one wave finds the offset, the others wait at the barrier (polling before
    // the matches are placed, while fewer words are there, costs more than the
    // wait it saves: 110 us)
    if (w == W - 1) {
        const uint64_t ob = n_tiles > 1 ? matches_before(sums, tile, n_tiles, total) : 0ull;
        if (lane == 0) out_base = ob;
    }
    __syncthreads();
    const uint64_t ob = out_base;
    if (ob != ~0ull) store_run<BLOCK>(buf, total, out + ob);
    // a single tile's count is stored; otherwise it was zero and becomes the last
    // tile's total, or -1 from any tile that gave up
    if (n_tiles == 1) {
        if (threadIdx.x == 0) *count_out = total;
    } else if (threadIdx.x == 0 && (ob == ~0ull || tile == n_tiles - 1))
        atomicOr((unsigned long long *)count_out, ob == ~0ull ? ~0ull : ob + total);
}

// Unstable selection with buffered reservations.  Persistent workgroups
// stride over the tiles and compact each tile's matches into an LDS buffer of
// two tiles; output space is reserved with one atomic only when the buffer
// could not take another tile, then the whole buffer is written out with
// 16-byte stores.  Fewer reservations than one per tile (they serialise on
// one address), and the loads of the next two tiles are in flight while the
// current one is compacted.
//
// Compaction (BlockScan + BlockShuffle): for every item slot k, a ballot of
// the wave's flags gives each matching lane its rank among the wave's matches
// in that slot (mbcnt), so a wave's matches are laid out slot by slot, lane
// by lane, and each LDS store instruction writes consecutive words.  The
// waves' totals are exchanged once per tile.  Within a tile the order is
// therefore slot-major, not input order; the tile's matches stay contiguous.
// A non-matching item is stored to a per-thread spare word, so the scatter
// has no branches.
template <int BLOCK, int IPT>
__global__ __launch_bounds__(BLOCK) void select_buffered_kernel(const int32_t *__restrict__ in, int64_t n,
                                                                int32_t lo, int32_t hi,
                                                                int32_t *__restrict__ out,
                                                                int64_t *__restrict__ count_out,
                                                                int64_t n_tiles) {
    using T = TileShape<BLOCK, IPT>;
    constexpr int W = T::WAVES;
    constexpr uint32_t CAP = 2 * T::ITEMS;
    extern __shared__ __align__(16) int32_t buf[];  // CAP entries, then one spare word per thread
    __shared__ uint32_t wave_tot[W];
    __shared__ uint64_t flush_off;
    const int w = threadIdx.x / kWave;
    const uint32_t lane = lane_id();
    uint32_t fill = 0;  // entries in buf, equal in every thread

    auto flush = [&]() {
        if (threadIdx.x == 0) flush_off = atomic_add_u64((uint64_t *)count_out, fill);
        __syncthreads();
        store_run<BLOCK>(buf, fill, out + flush_off);
        __syncthreads();  // buf and flush_off are reused
        fill = 0;
    };
    // compact one tile's values (already loaded) into buf
    auto compact = [&](int64_t tile, const int32_t(&v)[IPT]) {
        const int64_t base = tile * T::ITEMS;
        const uint32_t flags = block_pred_range<IPT>(v, valid_mask<BLOCK, IPT>(base, n), lo, hi);
        uint32_t pos[IPT];
        uint32_t wt = 0;  // the wave's matches so far (uniform)
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            const uint64_t m = ballot((flags >> k) & 1u);
            pos[k] = wt + count_below(m);
            wt += (uint32_t)__popcll(m);
        }
        if (lane == 0) wave_tot[w] = wt;
        __syncthreads();
        uint32_t before = 0, total = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const uint32_t t = wave_tot[i];
            before += i < w ? t : 0u;
            total += t;
        }
        const uint32_t b0 = fill + before;
        const uint32_t spare = CAP + threadIdx.x;
#pragma unroll
        for (int k = 0; k < IPT; ++k) buf[((flags >> k) & 1u) ? b0 + pos[k] : spare] = v[k];
        fill += total;
        __syncthreads();  // wave_tot is rewritten by the next tile; buf is complete
        if (fill + T::ITEMS > CAP) flush();
    };

    // three register buffers, rotated so that a buffer receiving loads is never copied
    int32_t va[IPT], vb[IPT], vc[IPT];
    int64_t tile = blockIdx.x;
    const int64_t g = gridDim.x;
    if (tile < n_tiles) block_load<BLOCK, IPT, true>(in, tile * T::ITEMS, n, va);
    if (tile + g < n_tiles) block_load<BLOCK, IPT, true>(in, (tile + g) * T::ITEMS, n, vb);
    while (tile < n_tiles) {
        if (tile + 2 * g < n_tiles) block_load<BLOCK, IPT, true>(in, (tile + 2 * g) * T::ITEMS, n, vc);
        compact(tile, va);
        tile += g;
        if (tile >= n_tiles) break;
        if (tile + 2 * g < n_tiles) block_load<BLOCK, IPT, true>(in, (tile + 2 * g) * T::ITEMS, n, va);
        compact(tile, vb);
        tile += g;
        if (tile >= n_tiles) break;
        if (tile + 2 * g < n_tiles) block_load<BLOCK, IPT, true>(in, (tile + 2 * g) * T::ITEMS, n, vb);
        compact(tile, vc);
        tile += g;
    }
    if (fill) flush();
}

template <int BLOCK, int IPT>
static hipError_t select_t(const LaunchCfg &cfg, const int32_t *in, int64_t n, int32_t lo, int32_t hi,
                           int32_t *out, int64_t *count, uint64_t *st, bool stable, hipStream_t s) {
    using T = TileShape<BLOCK, IPT>;
    const int64_t n_tiles = (n + T::ITEMS - 1) / T::ITEMS;
    // stable: one workgroup per tile, always: a stable tile only waits for
    // lower-numbered tiles, which in-order dispatch has already started;
    // workgroups striding over tiles could wait for a tile whose workgroup is
    // not resident
    hipError_t e;
    if (stable) {
        const TileSums sums(st, n_tiles);
        if (n_tiles > 1) {  // a single tile needs no words: one launch (1,000 rows 7.7 -> 4.2 us)
            const int64_t words = ((const char *)(sums.tile + n_tiles) - (const char *)st + 7) / 8;  // at most n_tiles
            e = zero_and_word(st, words, (uint64_t *)count, s);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL((select_kernel<BLOCK, IPT>), dim3((unsigned)n_tiles), dim3(BLOCK), 0, s, in, n,
                           lo, hi, out, sums, count, n_tiles);
    } else {
        e = fill_u64((uint64_t *)count, 1, 0ull, s);
        if (e != hipSuccess) return e;
        // persistent: as many workgroups per CU as waves and the two-tile LDS buffer allow (or as tuned)
        const size_t lds = ((size_t)2 * T::ITEMS + BLOCK) * sizeof(int32_t);
        int64_t per_cu = cfg.grid_per_cu > 0 ? cfg.grid_per_cu : (2048 / BLOCK > 0 ? 2048 / BLOCK : 1);
        const int64_t lds_cap = device_lds_per_cu() / (int64_t)(lds + 1024);
        if (per_cu > lds_cap) per_cu = lds_cap > 0 ? lds_cap : 1;
        int64_t grid = per_cu * device_cu_count();
        if (grid > n_tiles) grid = n_tiles;
        if (lds > 65536) {
            e = hipFuncSetAttribute((const void *)select_buffered_kernel<BLOCK, IPT>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL((select_buffered_kernel<BLOCK, IPT>), dim3((unsigned)grid), dim3(BLOCK), lds, s, in, n,
                           lo, hi, out, count, n_tiles);
    }
    return hipGetLastError();
}

int64_t select_tile_items(const LaunchCfg &cfg) { return (int64_t)cfg.block * cfg.ipt; }

hipError_t launch_select(const LaunchCfg &cfg, const int32_t *in, int64_t n, int32_t lo, int32_t hi,
                         int32_t *out, int64_t *count, uint64_t *status_words, bool stable, hipStream_t s) {
    if (n == 0 || lo > hi) return fill_u64((uint64_t *)count, 1, 0ull, s);
    switch (CRYSTAL_VARIANT_KEY(cfg.block, cfg.ipt)) {
#define X(B, I) \
    case CRYSTAL_VARIANT_KEY(B, I): return select_t<B, I>(cfg, in, n, lo, hi, out, count, status_words, stable, s);
        CRYSTAL_VARIANTS_ALL(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------ projection --
__device__ __forceinline__ float linear2(float x1, float x2, float a, float b) {
#pragma clang fp contract(off)
    const float p = a * x1;
    const float q = b * x2;
    return p + q;
}

template <bool SIGMOID>
__device__ __forceinline__ float project_one(float x1, float x2, float a, float b) {
    const float t = linear2(x1, x2, a, b);
    if constexpr (SIGMOID) {
        return 1.0f / (1.0f + expf(-t));
    } else {
        return t;
    }
}

// Two BlockLoads, the arithmetic, one BlockStore (streaming, non-temporal).
template <int BLOCK, int IPT, bool SIGMOID>
__global__ __launch_bounds__(BLOCK) void project_kernel(const float *__restrict__ x1,
                                                        const float *__restrict__ x2, int64_t n,
                                                        float a, float b,
                                                        float *__restrict__ out,
                                                        int64_t n_tiles) {
    using T = TileShape<BLOCK, IPT>;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t base = tile * T::ITEMS;
        if (base + T::ITEMS <= n) {
#pragma unroll
            for (int c = 0; c < T::CHUNKS; ++c) {
                const int64_t i = T::index(base, c, 0);
                if constexpr (T::VEC == 4) {
                    v4f p = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(x1 + i));
                    v4f q = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(x2 + i));
                    v4f r;
                    r.x = project_one<SIGMOID>(p.x, q.x, a, b);
                    r.y = project_one<SIGMOID>(p.y, q.y, a, b);
                    r.z = project_one<SIGMOID>(p.z, q.z, a, b);
                    r.w = project_one<SIGMOID>(p.w, q.w, a, b);
                    __builtin_nontemporal_store(r, reinterpret_cast<v4f *>(out + i));
                } else {
#pragma unroll
                    for (int e = 0; e < T::VEC; ++e)
                        __builtin_nontemporal_store(project_one<SIGMOID>(
                            __builtin_nontemporal_load(x1 + i + e),
                            __builtin_nontemporal_load(x2 + i + e), a, b), out + i + e);
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < T::CHUNKS; ++c)
#pragma unroll
                for (int e = 0; e < T::VEC; ++e) {
                    const int64_t i = T::index(base, c, e);
                    if (i < n) out[i] = project_one<SIGMOID>(x1[i], x2[i], a, b);
                }
        }
    }
}

template <int BLOCK, int IPT>
static hipError_t project_t(const LaunchCfg &cfg, const float *x1, const float *x2, int64_t n,
                            float a, float b, float *out, bool sigmoid, hipStream_t s) {
    using T = TileShape<BLOCK, IPT>;
    const int64_t n_tiles = (n + T::ITEMS - 1) / T::ITEMS;
    const int64_t grid = grid_for(n_tiles, cfg);
    if (grid == 0) return hipSuccess;
    if (sigmoid)
        hipLaunchKernelGGL((project_kernel<BLOCK, IPT, true>), dim3((unsigned)grid), dim3(BLOCK), 0,
                           s, x1, x2, n, a, b, out, n_tiles);
    else
        hipLaunchKernelGGL((project_kernel<BLOCK, IPT, false>), dim3((unsigned)grid), dim3(BLOCK),
                           0, s, x1, x2, n, a, b, out, n_tiles);
    return hipGetLastError();
}

hipError_t launch_project(const LaunchCfg &cfg, const float *x1, const float *x2, int64_t n,
                          float a, float b, float *out, bool sigmoid, hipStream_t s) {
    switch (CRYSTAL_VARIANT_KEY(cfg.block, cfg.ipt)) {
#define X(B, I) \
    case CRYSTAL_VARIANT_KEY(B, I): return project_t<B, I>(cfg, x1, x2, n, a, b, out, sigmoid, s);
        CRYSTAL_VARIANTS_VEC(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------ narrow columns --
// out[i] = in[i] - base as an unsigned E; values that do not fit are stored
// truncated and reported.
template <typename E>
__global__ __launch_bounds__(256) void pack_column_kernel(const int32_t *__restrict__ in, int64_t n, int32_t base,
                                                          E *__restrict__ out, int32_t *status) {
    constexpr uint32_t kMax = (uint32_t)(E)~(E)0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t d = (uint32_t)in[i] - (uint32_t)base;
        bad |= in[i] < base || d > kMax;
        out[i] = (E)d;
    }
    if (bad) set_status(status, CRYSTAL_ERANGE);
}

// Bit-packed column: each thread assembles whole output words, so no word is
// written twice and no atomics are needed.  A row's range check is made by
// the word that holds its first bit; the padding words are written as zero.
__global__ __launch_bounds__(256) void pack_bits_kernel(const int32_t *__restrict__ in, int64_t n, int32_t base,
                                                        uint32_t bits, uint32_t *__restrict__ out, int64_t words,
                                                        int32_t *status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const uint32_t mask = (1u << bits) - 1u;  // bits <= 16
    bool bad = false;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < words; w += stride) {
        const int64_t b0 = w * 32;  // the stream bits of word w: [b0, b0 + 32)
        int64_t i0 = b0 / bits, i1 = (b0 + 32 + bits - 1) / bits;
        if (i1 > n) i1 = n;
        uint32_t word = 0;
        for (int64_t i = i0; i < i1; ++i) {
            const uint32_t d = (uint32_t)in[i] - (uint32_t)base;
            const int64_t sh = i * (int64_t)bits - b0;  // > -bits and < 32
            if (sh >= 0) {
                bad |= in[i] < base || d > mask;
                word |= (d & mask) << sh;
            } else {
                word |= (d & mask) >> (-sh);
            }
        }
        out[w] = word;
    }
    if (bad) set_status(status, CRYSTAL_ERANGE);
}

hipError_t launch_pack_column_bits(const int32_t *in, int64_t n, int32_t base, int32_t bits, uint32_t *out,
                                   int64_t words, int32_t *status, hipStream_t s) {
    int64_t grid = (words + 255) / 256;
    const int64_t cap = (int64_t)device_cu_count() * 16;
    if (grid > cap) grid = cap;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(pack_bits_kernel, dim3((unsigned)grid), dim3(256), 0, s, in, n, base, (uint32_t)bits, out,
                       words, status);
    return hipGetLastError();
}

hipError_t launch_pack_column(const int32_t *in, int64_t n, int32_t base, int32_t width, void *out,
                              int32_t *status, hipStream_t s) {
    int64_t grid = (n + 255) / 256;
    const int64_t cap = (int64_t)device_cu_count() * 16;
    if (grid > cap) grid = cap;
    if (width == 2)
        hipLaunchKernelGGL(pack_column_kernel<uint16_t>, dim3((unsigned)grid), dim3(256), 0, s, in, n, base,
                           (uint16_t *)out, status);
    else
        hipLaunchKernelGGL(pack_column_kernel<uint8_t>, dim3((unsigned)grid), dim3(256), 0, s, in, n, base,
                           (uint8_t *)out, status);
    return hipGetLastError();
}

}  // namespace crystal
