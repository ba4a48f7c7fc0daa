// Hash-join build and probe (section 4.3; perfect hashing of section 5.3)
// and the dense group-by aggregate.
#include "block.hpp"
#include "internal.hpp"
#include "stage.hpp"
#include "variants.hpp"

namespace crystal {

static constexpr uint64_t kEmptySlot = (uint64_t)(uint32_t)kEmptyKey;  // {EMPTY, 0}

__host__ __device__ static inline int64_t direct_bitmap_words(int64_t span) {
    int64_t w = (span + 31) / 32;
    return (w + 63) / 64 * 64;
}

static DevTable to_dev(const crystal_ht &ht) {
    DevTable t = {};
    t.kind = ht.kind;
    t.has_payload = ht.has_payload;
    if (ht.kind == CRYSTAL_HT_DIRECT) {
        t.bitmap = (const uint32_t *)ht.mem;
        t.payload = ht.has_payload ? (const int32_t *)ht.mem + direct_bitmap_words(ht.capacity)
                                   : nullptr;
        t.span = ht.capacity;
        t.key_min = ht.key_min;
    } else {
        t.slots = (const v2i *)ht.mem;
        t.mask = (uint32_t)(ht.capacity - 1);
        t.shift = 32 - ht.log2_capacity;
    }
    return t;
}

hipError_t launch_ht_clear(const crystal_ht &ht, hipStream_t s) {
    if (ht.kind == CRYSTAL_HT_DIRECT)
        return fill_u32((uint32_t *)ht.mem, direct_bitmap_words(ht.capacity), 0u, s);
    return fill_u64((uint64_t *)ht.mem, ht.capacity, kEmptySlot, s);
}

// --------------------------------------------------------------- build ----
// One thread per build row: a 64-bit compare-and-swap claims an empty slot
// {EMPTY, 0} -> {key, payload} (linear probing), or an atomic OR sets the
// key's presence bit and the payload is stored (direct table).
template <int KIND>
__device__ __forceinline__ void build_row(const DevTable &t, const int32_t *__restrict__ keys,
                                          const int32_t *__restrict__ payload,
                                          const int32_t *__restrict__ filter_col, int32_t flo, int32_t fhi,
                                          int64_t i, int32_t *status) {
    if (filter_col && !in_range(filter_col[i], flo, fhi)) return;
    const int32_t k = keys[i];
    const int32_t v = payload ? payload[i] : 0;
    if constexpr (KIND == CRYSTAL_HT_DIRECT) {
        const uint32_t off = (uint32_t)k - (uint32_t)t.key_min;
        if ((int64_t)off >= t.span) {
            set_status(status, CRYSTAL_ERANGE);
            return;
        }
        const uint32_t bit = 1u << (off & 31u);
        const uint32_t old = atomicOr(const_cast<uint32_t *>(t.bitmap) + (off >> 5), bit);
        if (old & bit) {
            set_status(status, CRYSTAL_EDUPKEY);
            return;
        }
        if (t.payload) const_cast<int32_t *>(t.payload)[off] = v;
    } else {
        if (k == kEmptyKey) {
            set_status(status, CRYSTAL_EINVAL);
            return;
        }
        unsigned long long *slots = (unsigned long long *)const_cast<v2i *>(t.slots);
        const unsigned long long want = (unsigned long long)(uint32_t)k | ((unsigned long long)(uint32_t)v << 32);
        uint32_t sl = hash_slot(k, t.shift);
        for (uint32_t step = 0; step <= t.mask; ++step) {
            const unsigned long long old = atomicCAS(slots + sl, (unsigned long long)kEmptySlot, want);
            if (old == kEmptySlot) return;
            if ((int32_t)(uint32_t)old == k) {
                set_status(status, CRYSTAL_EDUPKEY);
                return;
            }
            sl = (sl + 1u) & t.mask;
        }
        set_status(status, CRYSTAL_EFULL);
    }
}

template <int KIND>
__global__ __launch_bounds__(256) void ht_build_kernel(DevTable t, const int32_t *__restrict__ keys,
                                                       const int32_t *__restrict__ payload,
                                                       const int32_t *__restrict__ filter_col,
                                                       int32_t flo, int32_t fhi, int64_t n,
                                                       int32_t *status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        build_row<KIND>(t, keys, payload, filter_col, flo, fhi, i, status);
}

// ------------------------------------------------------------ batch build --
// Several tables in two launches: one clear of every table's memory, then
// one build kernel whose workgroups are split between the tables (a range of
// workgroups per table, each striding over that table's rows).
struct ClearRange {
    uint64_t *p;
    int64_t n;        // 64-bit words
    uint64_t value;
};

// up to kMaxBuildBatch tables, and one more range (an output to zero)
struct ClearBatch {
    int32_t count;
    ClearRange r[kMaxBuildBatch + 1];
};

// the clears, spread over `blocks` workgroups of which this is `block`
__device__ __forceinline__ void clear_part(const ClearBatch &b, int64_t block, int64_t blocks) {
    const int64_t stride = blocks * blockDim.x;
    const int64_t g0 = block * blockDim.x + threadIdx.x;
    for (int r = 0; r < b.count; ++r)
        for (int64_t i = g0; i < b.r[r].n; i += stride) b.r[r].p[i] = b.r[r].value;
}

__global__ __launch_bounds__(256) void clear_batch_kernel(ClearBatch b) {
    clear_part(b, blockIdx.x, gridDim.x);
}

// clear memory of a table, as crystal_ht_clear would leave it
ClearRange table_clear_range(const crystal_ht &ht) {
    ClearRange c;
    c.p = (uint64_t *)ht.mem;
    if (ht.kind == CRYSTAL_HT_DIRECT) {
        c.n = direct_bitmap_words(ht.capacity) / 2;  // an even number of 32-bit words
        c.value = 0;
    } else {
        c.n = ht.capacity;
        c.value = kEmptySlot;
    }
    return c;
}

struct BuildItemDev {
    DevTable t;
    const int32_t *keys;
    const int32_t *payload;
    const int32_t *filter;
    int32_t flo, fhi;
    int64_t n;
    int64_t block0, blocks;
};

struct BuildBatch {
    int32_t count;
    BuildItemDev it[kMaxBuildBatch];
};

// workgroup `block` of the build part: its item's range of workgroups strides over that item's rows
__device__ __forceinline__ void build_part(const BuildBatch &b, int64_t block, int32_t *status) {
    int r = 0;
    while (r + 1 < b.count && block >= b.it[r + 1].block0) ++r;
    const BuildItemDev &it = b.it[r];
    const int64_t stride = it.blocks * blockDim.x;
    for (int64_t i = (block - it.block0) * blockDim.x + threadIdx.x; i < it.n; i += stride) {
        if (it.t.kind == CRYSTAL_HT_DIRECT)
            build_row<CRYSTAL_HT_DIRECT>(it.t, it.keys, it.payload, it.filter, it.flo, it.fhi, i, status);
        else
            build_row<CRYSTAL_HT_LINEAR>(it.t, it.keys, it.payload, it.filter, it.flo, it.fhi, i, status);
    }
}

__global__ __launch_bounds__(256) void build_batch_kernel(BuildBatch b, int32_t *status) {
    build_part(b, blockIdx.x, status);
}

// Builds into tables that are already clear, and, in other workgroups of the
// same launch, clears of memory no build touches: the first build_blocks
// workgroups build, the rest clear.
__global__ __launch_bounds__(256) void build_clear_kernel(BuildBatch b, ClearBatch c, int64_t build_blocks,
                                                          int32_t *status) {
    const int64_t block = blockIdx.x;
    if (block < build_blocks)
        build_part(b, block, status);
    else
        clear_part(c, block - build_blocks, (int64_t)gridDim.x - build_blocks);
}

// build items of a batch with their workgroup ranges; returns the workgroups used
static int64_t fill_build_batch(const crystal_ht_build_item *items, int n_items, BuildBatch &bb) {
    int64_t blocks = 0;
    const int64_t cap = (int64_t)device_cu_count() * 32;
    for (int i = 0; i < n_items; ++i) {
        if (items[i].n == 0) continue;
        const crystal_ht &ht = *items[i].ht;
        BuildItemDev &d = bb.it[bb.count++];
        d.t = to_dev(ht);
        d.keys = items[i].keys;
        d.payload = ht.has_payload ? items[i].payload : nullptr;
        d.filter = items[i].filter_col;
        d.flo = items[i].filter.lo;
        d.fhi = items[i].filter.hi;
        d.n = items[i].n;
        int64_t nb = (items[i].n + 255) / 256;
        if (nb > cap) nb = cap;
        d.block0 = blocks;
        d.blocks = nb;
        blocks += nb;
    }
    return blocks;
}

// workgroups for clearing `words` 64-bit words at most per range
static int64_t clear_grid(int64_t words) {
    const int64_t cap = (int64_t)device_cu_count() * 32;
    int64_t g = (words + 255) / 256;
    if (g > cap) g = cap;
    return g < 1 ? 1 : g;
}

hipError_t launch_ht_build_batch(const crystal_ht_build_item *items, int n_items, int32_t *status,
                                 hipStream_t s) {
    ClearBatch cb = {};
    BuildBatch bb = {};
    int64_t clear_words = 0;
    for (int i = 0; i < n_items; ++i) {
        ClearRange &c = cb.r[cb.count++];
        c = table_clear_range(*items[i].ht);
        clear_words = c.n > clear_words ? c.n : clear_words;
    }
    if (cb.count == 0) return hipSuccess;
    const int64_t blocks = fill_build_batch(items, n_items, bb);
    hipLaunchKernelGGL(clear_batch_kernel, dim3((unsigned)clear_grid(clear_words)), dim3(256), 0, s, cb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || bb.count == 0) return e;
    hipLaunchKernelGGL(build_batch_kernel, dim3((unsigned)blocks), dim3(256), 0, s, bb, status);
    return hipGetLastError();
}

hipError_t launch_ht_build_batch_fused(const crystal_ht_build_item *items, int n_items, const crystal_ht *const *clear,
                                       int n_clear, int64_t *zero, int64_t zero_n, int32_t *status, hipStream_t s) {
    ClearBatch cb = {};
    BuildBatch bb = {};
    int64_t clear_words = 0;
    for (int i = 0; i < n_clear; ++i) {
        ClearRange &c = cb.r[cb.count++];
        c = table_clear_range(*clear[i]);
        clear_words = c.n > clear_words ? c.n : clear_words;
    }
    if (zero_n > 0) {
        ClearRange &c = cb.r[cb.count++];
        c.p = (uint64_t *)zero;
        c.n = zero_n;
        c.value = 0;
        clear_words = c.n > clear_words ? c.n : clear_words;
    }
    const int64_t build_blocks = fill_build_batch(items, n_items, bb);
    const int64_t clear_blocks = cb.count ? clear_grid(clear_words) : 0;
    if (build_blocks + clear_blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(build_clear_kernel, dim3((unsigned)(build_blocks + clear_blocks)), dim3(256), 0, s, bb, cb,
                       build_blocks, status);
    return hipGetLastError();
}

hipError_t launch_ht_build(const crystal_ht &ht, const int32_t *keys, const int32_t *payload,
                           const int32_t *filter_col, int32_t flo, int32_t fhi, int64_t n,
                           int32_t *status, hipStream_t s) {
    hipError_t e = launch_ht_clear(ht, s);
    if (e != hipSuccess || n == 0) return e;
    const DevTable t = to_dev(ht);
    int64_t grid = (n + 255) / 256;
    const int64_t cap = (int64_t)device_cu_count() * 32;
    if (grid > cap) grid = cap;
    if (ht.kind == CRYSTAL_HT_DIRECT)
        hipLaunchKernelGGL(ht_build_kernel<CRYSTAL_HT_DIRECT>, dim3((unsigned)grid), dim3(256), 0, s,
                           t, keys, payload, filter_col, flo, fhi, n, status);
    else
        hipLaunchKernelGGL(ht_build_kernel<CRYSTAL_HT_LINEAR>, dim3((unsigned)grid), dim3(256), 0, s,
                           t, keys, payload, filter_col, flo, fhi, n, status);
    return hipGetLastError();
}

// A tile's probe keys (and probe payloads) in registers.
template <int IPT, bool PP>
struct ProbeRegs {
    int32_t key[IPT];
    int32_t pv[PP ? IPT : 1];
};

// --------------------------------------------------------------- probe ----
// Query Q4: BlockLoad a tile of probe keys (and probe payloads), probe every
// item, keep a per-thread sum and match count, BlockAggregate, and add the
// workgroup's totals with two 64-bit atomics.  MODE 0: linear probing in
// global memory; MODE 1: linear probing in a copy of the table staged in LDS
// once per workgroup; MODE 2: direct table; MODE 3: direct table whose bitmap
// is staged, MODE 4: whose payloads are staged too.  A gather from L2 moves a
// 128-byte line to the CU, so 2^27 probes that make one take about 520 us and
// two about 1,000: with the bitmap staged, 2^20 keys went from 1,094 to 620 us
// and 2^16 from 590 to 518; with all of it staged, 2^15 keys from 527 to 95 us
// and 2^10 from 235 to 94 (the keys' own 512 MB take 83).  PP: probe rows carry a payload
// (pp is not null), a separate instance so that the payload registers exist
// only when used.
//
// probe_tiles: every gridDim.x-th tile from the workgroup's own on, added to sum
// and cnt.  slots: the linear table; lds_words: what of a direct table is staged.
template <int BLOCK, int IPT, int MODE, bool PP>
__device__ __forceinline__ void probe_tiles(const DevTable &t, const v2i *slots, const uint32_t *lds_words,
                                            const int32_t *__restrict__ fk, const int32_t *__restrict__ pp, int64_t n,
                                            int64_t n_tiles, uint64_t &sum, uint64_t &cnt) {
    using T = TileShape<BLOCK, IPT>;
    const int bitmap_words = (int)direct_bitmap_words(t.span);
    // one tile: the probes of its (already loaded) keys
    auto probe_tile = [&](int64_t tile, const ProbeRegs<IPT, PP> &r) {
        const int32_t(&key)[IPT] = r.key;
        const int64_t base = tile * T::ITEMS;
        const uint32_t valid = valid_mask<BLOCK, IPT>(base, n);
        uint32_t hit = 0;
        int32_t pay[IPT];
        if constexpr (MODE >= 2) {
            // direct table: every item's presence word at once, then the payloads of the hits
            uint32_t word[IPT], ok = 0;
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint32_t off = (uint32_t)key[k] - (uint32_t)t.key_min;
                const bool in = ((valid >> k) & 1u) && (int64_t)off < t.span;
                ok |= (uint32_t)in << k;
                if constexpr (MODE == 2)
                    word[k] = t.bitmap[in ? (off >> 5) : 0u];
                else
                    word[k] = lds_words[in ? (off >> 5) : 0u];
            }
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint32_t off = (uint32_t)key[k] - (uint32_t)t.key_min;
                hit |= (((word[k] >> (off & 31u)) & 1u) << k) & ok;
            }
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint32_t off = (uint32_t)key[k] - (uint32_t)t.key_min;
                if constexpr (MODE == 4) {
                    const uint32_t x = lds_words[bitmap_words + (((hit >> k) & 1u) ? off : 0u)];
                    pay[k] = ((hit >> k) & 1u) ? (int32_t)x : 0;
                } else {
                    pay[k] = t.has_payload && ((hit >> k) & 1u) ? t.payload[off] : 0;
                }
            }
        } else if constexpr (MODE == 0) {
            // table in global memory: one probe sequence per item (issuing every
            // item's slot at once measured slower when the table sits in the
            // last-level cache, and no faster from HBM)
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                pay[k] = 0;
                if (((valid >> k) & 1u) && key[k] != kEmptyKey && probe_linear(slots, t.mask, t.shift, key[k], pay[k]))
                    hit |= 1u << k;
            }
        } else {
            // table staged in LDS: every item's home slot is read at once and
            // compared without branches; only items whose home slot holds
            // another key continue, in rounds that read the next slot of every
            // item still searching at once (at fill rate 1/2 most items end in
            // the first round)
            uint32_t slot[IPT];
            uint32_t pending = 0;
            {
                v2i e[IPT];
#pragma unroll
                for (int k = 0; k < IPT; ++k) {
                    slot[k] = hash_slot(key[k], t.shift);
                    e[k] = slots[slot[k]];
                }
#pragma unroll
                for (int k = 0; k < IPT; ++k) {
                    const bool ok = ((valid >> k) & 1u) && key[k] != kEmptyKey;
                    const bool h = ok && e[k].x == key[k];
                    hit |= (uint32_t)h << k;
                    pay[k] = h ? e[k].y : 0;
                    pending |= (uint32_t)(ok && !h && e[k].x != kEmptyKey) << k;
                }
            }
            if (pending) {
#pragma unroll
                for (int k = 0; k < IPT; ++k) slot[k] = (slot[k] + 1u) & t.mask;
                for (uint32_t step = 1; pending && step <= t.mask; ++step) {
                    v2i e[IPT];
#pragma unroll
                    for (int k = 0; k < IPT; ++k)
                        if ((pending >> k) & 1u) e[k] = slots[slot[k]];
#pragma unroll
                    for (int k = 0; k < IPT; ++k) {
                        if (!((pending >> k) & 1u)) continue;
                        if (e[k].x == key[k]) {
                            hit |= 1u << k;
                            pay[k] = e[k].y;
                            pending &= ~(1u << k);
                        } else if (e[k].x == kEmptyKey) {
                            pending &= ~(1u << k);
                        } else {
                            slot[k] = (slot[k] + 1u) & t.mask;
                        }
                    }
                }
            }
        }
        if constexpr (MODE != 0) {
            // pay[k] is 0 for misses: the sum needs no per-item branch
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                sum += (uint64_t)(int64_t)pay[k];
                if constexpr (PP) sum += ((hit >> k) & 1u) ? (uint64_t)(int64_t)r.pv[k] : 0ull;
            }
            cnt += (uint64_t)__popc(hit);
            return;
        }
#pragma unroll
        for (int k = 0; k < IPT; ++k)
            if ((hit >> k) & 1u) {
                uint64_t add = (uint64_t)(int64_t)pay[k];
                if constexpr (PP) add += (uint64_t)(int64_t)r.pv[k];
                sum += add;
                cnt += 1;
            }
    };
    auto load = [&](int64_t tile, ProbeRegs<IPT, PP> &r) {
        block_load<BLOCK, IPT, true>(fk, tile * T::ITEMS, n, r.key);
        if constexpr (PP) block_load<BLOCK, IPT, true>(pp, tile * T::ITEMS, n, r.pv);
    };
    int64_t tile = blockIdx.x;
    if constexpr (PP) {
        // probe payloads too: one buffer (a second one would spill at 16 items per thread)
        ProbeRegs<IPT, PP> r;
        for (; tile < n_tiles; tile += gridDim.x) {
            load(tile, r);
            probe_tile(tile, r);
        }
    } else {
    // the next tile's keys are loaded while the current tile is probed, in
    // alternating register buffers so that a buffer receiving loads is never
    // copied
    ProbeRegs<IPT, PP> ra, rb;
    if (tile < n_tiles) load(tile, ra);
    while (tile < n_tiles) {
        int64_t nxt = tile + gridDim.x;
        if (nxt < n_tiles) load(nxt, rb);
        probe_tile(tile, ra);
        tile = nxt;
        if (tile >= n_tiles) break;
        nxt = tile + gridDim.x;
        if (nxt < n_tiles) load(nxt, ra);
        probe_tile(tile, rb);
        tile = nxt;
    }
    }
}

template <int BLOCK, int IPT, int MODE, bool PP>
__global__ __launch_bounds__(BLOCK) void ht_probe_kernel(DevTable t, const int32_t *__restrict__ fk,
                                                         const int32_t *__restrict__ pp, int64_t n,
                                                         uint64_t *__restrict__ out_sum,
                                                         uint64_t *__restrict__ out_cnt,
                                                         int64_t n_tiles) {
    using T = TileShape<BLOCK, IPT>;
    extern __shared__ v4i lds_raw[];
    __shared__ uint64_t red[T::WAVES];
    const v2i *slots = t.slots;
    if constexpr (MODE == 1) {
        // stage the whole table
        copy_to_lds<BLOCK>(reinterpret_cast<const uint32_t *>(t.slots), reinterpret_cast<uint32_t *>(lds_raw),
                           2 * ((int)t.mask + 1));
        __syncthreads();
        slots = reinterpret_cast<const v2i *>(lds_raw);
    }
    const uint32_t *lds_words = reinterpret_cast<const uint32_t *>(lds_raw);
    const int bitmap_words = (int)direct_bitmap_words(t.span);
    if constexpr (MODE == 3 || MODE == 4) {
        // stage the bitmap, and the payloads, which follow it in memory
        copy_to_lds<BLOCK>(t.bitmap, reinterpret_cast<uint32_t *>(lds_raw),
                           bitmap_words + (MODE == 4 ? (int)t.span : 0));
        __syncthreads();
    }
    uint64_t sum = 0, cnt = 0;
    probe_tiles<BLOCK, IPT, MODE, PP>(t, slots, lds_words, fk, pp, n, n_tiles, sum, cnt);
    const uint64_t bs = block_sum_u64<BLOCK>(sum, red);
    __syncthreads();
    const uint64_t bc = block_sum_u64<BLOCK>(cnt, red);
    if (threadIdx.x == 0) {
        if (bs) atomic_add_u64(out_sum, bs);
        if (bc) atomic_add_u64(out_cnt, bc);
    }
}

template <int BLOCK, int IPT, bool PP>
static hipError_t probe_launch(const crystal_ht &ht, const DevTable &t, bool stage, bool all, int64_t table_bytes,
                               int64_t grid, const int32_t *fk, const int32_t *pp, int64_t n, uint64_t *out,
                               uint64_t *cnt, int64_t n_tiles, hipStream_t s) {
    if (ht.kind == CRYSTAL_HT_DIRECT && stage) {
        auto fn = all ? ht_probe_kernel<BLOCK, IPT, 4, PP> : ht_probe_kernel<BLOCK, IPT, 3, PP>;
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)table_bytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(BLOCK), (size_t)table_bytes, s, t, fk, pp, n,
                           out, cnt, n_tiles);
    } else if (ht.kind == CRYSTAL_HT_DIRECT) {
        hipLaunchKernelGGL((ht_probe_kernel<BLOCK, IPT, 2, PP>), dim3((unsigned)grid), dim3(BLOCK), 0, s,
                           t, fk, pp, n, out, cnt, n_tiles);
    } else if (stage) {
        auto fn = ht_probe_kernel<BLOCK, IPT, 1, PP>;
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)table_bytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(BLOCK), (size_t)table_bytes, s, t, fk, pp, n,
                           out, cnt, n_tiles);
    } else {
        hipLaunchKernelGGL((ht_probe_kernel<BLOCK, IPT, 0, PP>), dim3((unsigned)grid), dim3(BLOCK), 0, s,
                           t, fk, pp, n, out, cnt, n_tiles);
    }
    return hipGetLastError();
}

template <int BLOCK, int IPT>
static hipError_t probe_t(const LaunchCfg &cfg_in, const crystal_ht &ht, const int32_t *fk,
                          const int32_t *pp, int64_t n, uint64_t *out, uint64_t *cnt, hipStream_t s) {
    using T = TileShape<BLOCK, IPT>;
    const int64_t n_tiles = (n + T::ITEMS - 1) / T::ITEMS;
    const DevTable t = to_dev(ht);
    LaunchCfg cfg = cfg_in;
    // staged in LDS: a linear table, a direct table, or only its bitmap
    const int64_t lds_max = device_lds_per_block() - 4096;
    int64_t table_bytes = ht.capacity * 8;
    bool all = false;
    if (ht.kind == CRYSTAL_HT_DIRECT) {
        table_bytes = direct_bitmap_words(ht.capacity) * 4;
        const int64_t with_payload = table_bytes + (ht.capacity * 4 + 15) / 16 * 16;
        all = ht.has_payload && with_payload <= lds_max;
        if (all) table_bytes = with_payload;
    }
    // a direct table's copy costs a short probe more than its gathers (38,000 and
    // 2^20 keys, in us, staged / not: 1,000 probes 9.3/8.5 and 9.1/8.4, 4,096
    // 9.6/9.3 and 9.9/9.9, 6,000 10.0/10.4 and 10.7/11.4)
    const bool stage = table_bytes <= lds_max && (ht.kind == CRYSTAL_HT_LINEAR || n >= 5000);
    if (stage && cfg.grid_per_cu <= 0) cfg.grid_per_cu = 1;  // stage once per resident workgroup
    const int64_t grid = grid_for(n_tiles, cfg);
    if (grid == 0) return hipSuccess;
    if (pp)
        return probe_launch<BLOCK, IPT, true>(ht, t, stage, all, table_bytes, grid, fk, pp, n, out, cnt, n_tiles, s);
    return probe_launch<BLOCK, IPT, false>(ht, t, stage, all, table_bytes, grid, fk, pp, n, out, cnt, n_tiles, s);
}

// ----------------------------------------------------------- sliced probe --
// Query Q4 on a table larger than an XCD's 4 MB L2, where a probe costs a
// 128-byte line from the last-level cache (2^20 build keys, a 16 MB table:
// 9 TB/s of lines, 1,767 us for 2^27 probes).
//
// Slices: the table is dealt to 2^LG slices in pieces of at least 8 KB, and a
// workgroup probes only the keys whose home lies in its slice; the workgroups
// of every slice read all the keys.  Consecutive workgroups run on the eight
// XCDs in turn, so an XCD's L2 sees one slice of the table (only speed depends
// on that).  Each wave compacts the keys of its slice into an LDS queue and
// probes them four per lane.  The keys are loaded without the non-temporal
// hint, so that their second and later reads hit the last-level cache.
// Retries (linear probing): a lane reads its home slot and the next with one
// 16-byte load; keys those do not decide wait in a second queue until 64 are
// there, so a wave does not follow its longest chain.
//
// Measured, 2^27 probes without payload, before -> now: 8 MB table 1,218 ->
// 782 us, 16 MB 1,767 -> 962 us, 32 MB 2,110 -> 1,330 us.  What bounds it is
// the line each probe moves from L2 to the CU (a table within L2 takes 600 us)
// and the compaction of the keys, about 45 us per slice.
//
// That holds for keys spread over the table.  When they are not, the gathers
// find their lines in L2 or share them, and a slice's workgroups may get most
// of the keys: keys_are_spread looks at a sample, and if it says no, every
// workgroup probes the keys of its own tiles as ht_probe_kernel does.  2^27
// keys, in us, always sliced / now (unsliced): 16 MB direct sorted 2,161/178
// (179), 90% one key 2,183/304 (302), 8,192-key windows 942/472 (460), Zipf
// 1,105/1,127 (1,152); 32 MB linear sorted 728/286 (289), 90% one key 1,907/326
// (322), half one key 1,419/1,111 (1,108).  Spread keys lose 1% to the sample.

// Whether the probe keys fk[0..n) are spread over the table, from a sample of
// 32 groups of 64 neighbouring keys: at least `percent` of the sample have a
// line of the table of their own.  Groups in ascending order and (direct tables)
// groups within 4 MB of payloads count as not spread, since neighbours in the
// column then share an XCD's L2.  All workgroups read the same sample and come
// to the same answer.  seen: 2^kSeenLg bits of LDS; total: one word.
// Called by the whole workgroup, ends with a barrier.
constexpr uint32_t kSeenLg = 15;

template <int BLOCK, int KIND>
__device__ __forceinline__ bool keys_are_spread(const DevTable &t, const int32_t *__restrict__ fk, int64_t n,
                                                uint32_t percent, uint32_t *seen, uint32_t *total) {
    constexpr int W = BLOCK / kWave, kGroups = 32;
    const int w = (int)threadIdx.x / kWave;
    const uint32_t lane = lane_id();
    const int64_t all = n / kWave;  // whole groups
    const int groups = all < kGroups ? (int)all : kGroups;
    int32_t key[kGroups / W];
#pragma unroll
    for (int i = 0; i < kGroups / W; ++i) {
        const int g = w + i * W;
        key[i] = g < groups ? fk[all * g / groups * kWave + lane] : 0;
    }
    for (uint32_t i = threadIdx.x; i < (1u << kSeenLg) / 32; i += BLOCK) seen[i] = 0u;
    if (threadIdx.x == 0) *total = 0u;
    __syncthreads();
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kGroups / W; ++i) {
        if (w + i * W >= groups) break;
        const int32_t k = key[i], before = __shfl_up(k, 1);
        uint32_t line;
        bool counts = ballot(lane > 0 && k < before) != 0, in = true;
        if constexpr (KIND == CRYSTAL_HT_LINEAR) {
            line = hash_slot(k, t.shift) >> 4;  // 16 slots
            in = k != kEmptyKey;
        } else {
            const uint32_t off = (uint32_t)k - (uint32_t)t.key_min;
            in = (int64_t)off < t.span;
            line = off >> 5;  // 32 payloads
            constexpr uint32_t kReach = 1u << 19;  // payloads
            const uint32_t first = __builtin_amdgcn_readfirstlane(off);
            counts = counts && ballot(in && off - first + kReach > 2 * kReach) != 0;
        }
        if (counts && in) {
            const uint32_t h = line * 2654435761u >> (32 - kSeenLg), bit = 1u << (h & 31u);
            mine += (atomicOr(seen + (h >> 5), bit) & bit) ? 0u : 1u;
        }
    }
    const uint32_t sum = (uint32_t)wave_sum_u64(mine);
    if (lane == 0) atomicAdd(total, sum);
    __syncthreads();
    const bool spread = 100u * *total >= percent * (uint32_t)(groups * kWave);
    __syncthreads();
    return spread;
}

template <int BLOCK, int IPT, int KIND, bool PP, int LG>
__global__ __launch_bounds__(BLOCK) void ht_probe_sliced_kernel(DevTable t, const int32_t *__restrict__ fk,
                                                                const int32_t *__restrict__ pp, int64_t n,
                                                                uint64_t *__restrict__ out_sum,
                                                                uint64_t *__restrict__ out_cnt, int64_t n_tiles) {
    using T = TileShape<BLOCK, IPT>;
    constexpr bool kLinear = KIND == CRYSTAL_HT_LINEAR;
    constexpr int D = 4;                       // keys a lane probes at a time
    constexpr uint32_t kQ = 2 * D * kWave;     // slice queue: fewer than D * 64 left over, then at most D * 64 more
    constexpr uint32_t kR = 2 * kWave;         // retry queue: fewer than 64 left over, then at most 64 more
    constexpr uint32_t kPieceLg = 11;          // direct: 2^11 payloads, 8 KB
    // up to so many keys the table is probed in slices whatever the keys: the
    // sample takes 1.5 us, and a short probe is no slower for them (in us, sliced /
    // unsliced: 2^18 keys 8-13 / 10-40, four slices 2^20 keys 10-16 / 11-40; eight
    // slices, 2^20 times mostly one key 24 / 12)
    constexpr int64_t kSampleFrom = int64_t(1) << (LG == 3 ? 18 : 20);
    // percent of the sample that has to be spread: with a fifth of the keys sorted
    // or equal slices gain, with half of them four slices of a linear table still
    // do (2^27 keys into 16 MB, in us, unsliced / sliced: one key 968/807, sorted
    // 1,121/744, Zipf 887/738; 8 MB 688/733, 788/609, 728/644), but not with probe
    // payloads (1,029/1,156), of a direct table (8 MB sorted 807/982) or eight
    // slices (32 MB one key 1,114/1,422)
    constexpr uint32_t kSpread = kLinear && LG == 2 && !PP ? 45 : 75;
    __shared__ int32_t q_key[T::WAVES][kQ];
    __shared__ int32_t q_pv[PP ? T::WAVES : 1][PP ? kQ : 1];
    __shared__ int32_t r_key[kLinear ? T::WAVES : 1][kR];
    __shared__ uint32_t r_slot[kLinear ? T::WAVES : 1][kR];
    __shared__ int32_t r_pv[kLinear && PP ? T::WAVES : 1][kLinear && PP ? kR : 1];
    __shared__ uint64_t red[2][T::WAVES];
    const int w = (int)threadIdx.x / kWave;
    int32_t *my_key = q_key[w], *my_pv = q_pv[PP ? w : 0];
    int32_t *my_rkey = r_key[kLinear ? w : 0], *my_rpv = r_pv[kLinear && PP ? w : 0];
    uint32_t *my_rslot = r_slot[kLinear ? w : 0];
    const uint32_t lane = lane_id();
    __shared__ uint32_t total;
    const uint32_t slice = blockIdx.x & ((1u << LG) - 1u);
    uint32_t head = 0, tail = 0, rhead = 0, rtail = 0;  // queue cursors, equal in every lane of the wave
    uint64_t sum = 0, cnt = 0;

    // Bits [24 - LG, 24) of the hash product, which the low 24 bits of both
    // factors determine (a full-rate multiply): they are slot bits, the lowest
    // of them bit 24 - LG - shift, at least 10 for the tables of 2^20 slots or
    // more that take this path.
    auto slice_of = [&](int32_t k) -> uint32_t {
        if constexpr (kLinear)
            return __builtin_amdgcn_ubfe(__umul24((uint32_t)k, 2654435761u & 0xffffffu), 24 - LG, LG);
        else
            return __builtin_amdgcn_ubfe((uint32_t)k - (uint32_t)t.key_min, kPieceLg, LG);
    };
    // the oldest `count` (at most 64) retries, one per lane, slot by slot to their end
    auto retry = [&](uint32_t count) {
        if (lane < count) {
            const uint32_t i = (rhead + lane) & (kR - 1u);
            const int32_t k = my_rkey[i];
            uint32_t s = my_rslot[i];
            for (uint32_t step = 0; step <= t.mask; ++step) {
                const v2i e = t.slots[s];
                if (e.x == k) {
                    sum += (uint64_t)(int64_t)e.y;
                    if constexpr (PP) sum += (uint64_t)(int64_t)my_rpv[i];
                    ++cnt;
                    break;
                }
                if (e.x == kEmptyKey) break;
                s = (s + 1u) & t.mask;
            }
        }
        rhead += count;
    };
    // probe the keys of `ok`, D per lane
    auto probe = [&](const int32_t(&key)[D], const int32_t(&pv)[PP ? D : 1], uint32_t ok) {
        if constexpr (kLinear) {
            typedef int32_t v4i_8 __attribute__((ext_vector_type(4), aligned(8)));
            uint32_t slot[D];
            v4i e[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (key[d] == kEmptyKey) ok &= ~(1u << d);
                slot[d] = ((ok >> d) & 1u) ? hash_slot(key[d], t.shift) : 0u;
                // the last slot is read as the second of its pair
                const uint32_t at = slot[d] < t.mask ? slot[d] : t.mask - 1u;
                e[d] = *reinterpret_cast<const v4i_8 *>(t.slots + at);
            }
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const bool valid = (ok >> d) & 1u;
                const bool last = slot[d] == t.mask;
                const int32_t k0 = last ? e[d].z : e[d].x, p0 = last ? e[d].w : e[d].y;
                const bool h0 = k0 == key[d];
                const bool go = !h0 && k0 != kEmptyKey;
                const bool h1 = go && !last && e[d].z == key[d];
                if (valid && (h0 || h1)) {
                    sum += (uint64_t)(int64_t)(h0 ? p0 : e[d].w);
                    if constexpr (PP) sum += (uint64_t)(int64_t)pv[d];
                    ++cnt;
                }
                const bool again = valid && go && !h1 && (last || e[d].z != kEmptyKey);
                const uint64_t m = ballot(again);
                if (again) {
                    const uint32_t i = (rtail + count_below(m)) & (kR - 1u);
                    my_rkey[i] = key[d];
                    my_rslot[i] = (slot[d] + (last ? 1u : 2u)) & t.mask;
                    if constexpr (PP) my_rpv[i] = pv[d];
                }
                rtail += (uint32_t)__popcll(m);
                __builtin_amdgcn_wave_barrier();
                if (rtail - rhead >= (uint32_t)kWave) retry(kWave);
                __builtin_amdgcn_wave_barrier();
            }
        } else {
            uint32_t off[D], word[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                off[d] = (uint32_t)key[d] - (uint32_t)t.key_min;
                if ((int64_t)off[d] >= t.span) ok &= ~(1u << d);
                word[d] = t.bitmap[((ok >> d) & 1u) ? off[d] >> 5 : 0u];
            }
            int32_t pay[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (!((word[d] >> (off[d] & 31u)) & 1u)) ok &= ~(1u << d);
                pay[d] = t.has_payload && ((ok >> d) & 1u) ? t.payload[off[d]] : 0;
            }
#pragma unroll
            for (int d = 0; d < D; ++d) {
                sum += (uint64_t)(int64_t)pay[d];
                if constexpr (PP) sum += ((ok >> d) & 1u) ? (uint64_t)(int64_t)pv[d] : 0ull;
            }
            cnt += (uint64_t)__popc(ok);
        }
    };
    // probe the oldest `count` (at most D * 64) keys of the slice queue
    auto drain = [&](uint32_t count) {
        int32_t key[D], pv[PP ? D : 1];
        uint32_t ok = 0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t j = (uint32_t)d * kWave + lane;
            const uint32_t i = (head + j) & (kQ - 1u);
            key[d] = my_key[i];
            if constexpr (PP) pv[d] = my_pv[i];
            ok |= (uint32_t)(j < count) << d;
        }
        head += count;
        probe(key, pv, ok);
    };
    auto run_tile = [&](int64_t tile, const ProbeRegs<IPT, PP> &r) {
        const bool full = (tile + 1) * T::ITEMS <= n;
        const uint32_t valid = valid_mask<BLOCK, IPT>(tile * T::ITEMS, n);
#pragma unroll
        for (int c = 0; c < IPT; c += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int32_t k = r.key[c + d];
                bool in = slice_of(k) == slice;
                if (!full) in = in && ((valid >> (c + d)) & 1u);
                const uint64_t m = ballot(in);
                if (in) {
                    const uint32_t i = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, tail)) & (kQ - 1u);
                    my_key[i] = k;
                    if constexpr (PP) my_pv[i] = r.pv[c + d];
                }
                tail += (uint32_t)__popcll(m);
            }
            __builtin_amdgcn_wave_barrier();
            if (tail - head >= (uint32_t)(D * kWave)) drain(D * kWave);
            __builtin_amdgcn_wave_barrier();
        }
    };
    auto load = [&](int64_t tile, ProbeRegs<IPT, PP> &r) {
        block_load<BLOCK, IPT, false>(fk, tile * T::ITEMS, n, r.key);
        if constexpr (PP) block_load<BLOCK, IPT, false>(pp, tile * T::ITEMS, n, r.pv);
    };
    const int64_t stride = gridDim.x >> LG;
    static_assert(T::WAVES * kQ * 32 >= 1u << kSeenLg, "the sample's bits lie in the slice queues");
    const bool sliced = n <= kSampleFrom || keys_are_spread<BLOCK, KIND>(t, fk, n, kSpread, (uint32_t *)q_key, &total);
    int64_t tile = sliced ? blockIdx.x >> LG : n_tiles;
    ProbeRegs<IPT, PP> ra, rb;
    if (tile < n_tiles) load(tile, ra);
    while (tile < n_tiles) {
        if (tile + stride < n_tiles) load(tile + stride, rb);
        run_tile(tile, ra);
        tile += stride;
        if (tile >= n_tiles) break;
        if (tile + stride < n_tiles) load(tile + stride, ra);
        run_tile(tile, rb);
        tile += stride;
    }
    if (tail != head) drain(tail - head);
    if (rtail != rhead) retry(rtail - rhead);
    if (!sliced)
        probe_tiles<BLOCK, 16, kLinear ? 0 : 2, PP>(t, t.slots, nullptr, fk, pp, n, (n + 16 * BLOCK - 1) / (16 * BLOCK), sum,
                                                    cnt);
    sum = wave_sum_u64(sum);
    cnt = wave_sum_u64(cnt);
    if (lane == 0) {
        red[0][w] = sum;
        red[1][w] = cnt;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint64_t x = 0;
        for (int i = 0; i < T::WAVES; ++i) x += red[threadIdx.x][i];
        if (x) atomic_add_u64(threadIdx.x ? out_cnt : out_sum, x);
    }
}

template <int KIND, bool PP, int LG>
static hipError_t sliced_launch(const DevTable &t, const int32_t *fk, const int32_t *pp, int64_t n, uint64_t *out,
                                uint64_t *cnt, hipStream_t s) {
    constexpr int B = 1024, I = PP ? 8 : 16;
    const int64_t n_tiles = (n + (int64_t)B * I - 1) / ((int64_t)B * I);
    auto fn = ht_probe_sliced_kernel<B, I, KIND, PP, LG>;
    int64_t per_cu = 0;
    hipError_t e = resident_per_cu((const void *)fn, B, 0, per_cu);
    if (e != hipSuccess) return e;
    int64_t per_slice = (per_cu < 1 ? 1 : per_cu) * device_cu_count() >> LG;
    if (per_slice > n_tiles) per_slice = n_tiles;
    if (per_slice < 1) per_slice = 1;
    hipLaunchKernelGGL(fn, dim3((unsigned)(per_slice << LG)), dim3(B), 0, s, t, fk, pp, n, out, cnt, n_tiles);
    return hipGetLastError();
}

template <int KIND>
static hipError_t sliced_probe(int lg, const DevTable &t, const int32_t *fk, const int32_t *pp, int64_t n,
                               uint64_t *out, uint64_t *cnt, hipStream_t s) {
    if (pp) return sliced_launch<KIND, true, 2>(t, fk, pp, n, out, cnt, s);
    return lg == 2 ? sliced_launch<KIND, false, 2>(t, fk, pp, n, out, cnt, s)
                   : sliced_launch<KIND, false, 3>(t, fk, pp, n, out, cnt, s);
}

// log2 of the slices of a probe (0: not sliced).  `bytes` is what the probes
// gather from: all slots, or a direct table's payloads (its bitmap is 32 times
// smaller).  Up to 4 MB an XCD's L2 holds it; beyond, more slices fit L2 better
// but each reads all keys, and payloads, again.  2^27 probes, in us, unsliced /
// 4 slices / 8 slices:
//   linear 8 MB 1,222/788/928, 16 MB 1,768/957/972, 32 MB 2,102/1,625/1,330,
//   64 MB 2,409/2,214/2,005, 128 MB 2,505/2,976/2,883; with payloads 8 MB
//   1,303/1,006/1,314, 16 MB 1,845/1,325/1,519, 32 MB 2,153/2,009/2,123, 64 MB
//   2,461/2,514/2,746;
//   direct 8 MB 1,399/1,059/1,086, 16 MB 1,865/1,342/1,269, 32 MB
//   2,225/1,686/1,535; with payloads 8 MB 1,508/1,338/1,529, 16 MB
//   1,943/1,568/1,733, 32 MB 2,303/2,031/2,205.
// Short probes gain as well (2^18 into 16 MB: 35 -> 14 us).
static int probe_slices_lg(const crystal_ht &ht, bool pp) {
    const bool linear = ht.kind == CRYSTAL_HT_LINEAR;
    const int64_t mb = int64_t(1) << 20;
    const int64_t bytes = linear ? ht.capacity * 8 : ht.has_payload ? ht.capacity * 4 : 0;
    if (bytes <= 4 * mb || bytes > (linear && !pp ? 64 : 32) * mb) return 0;
    return pp || bytes <= (linear ? 16 : 8) * mb ? 2 : 3;
}

int ht_probe_slices(const crystal_ht &ht, bool with_payload) {
    const int lg = probe_slices_lg(ht, with_payload);
    return lg ? 1 << lg : 0;
}

hipError_t launch_ht_probe(const LaunchCfg &cfg, const crystal_ht &ht, const int32_t *fk,
                           const int32_t *probe_payload, int64_t n, uint64_t *sum, uint64_t *count,
                           hipStream_t s) {
    hipError_t e = zero_pair(sum, count, s);
    if (e != hipSuccess || n == 0) return e;
    if (const int lg = probe_slices_lg(ht, probe_payload != nullptr)) {
        const DevTable t = to_dev(ht);
        return ht.kind == CRYSTAL_HT_LINEAR ? sliced_probe<CRYSTAL_HT_LINEAR>(lg, t, fk, probe_payload, n, sum, count, s)
                                            : sliced_probe<CRYSTAL_HT_DIRECT>(lg, t, fk, probe_payload, n, sum, count, s);
    }
    switch (CRYSTAL_VARIANT_KEY(cfg.block, cfg.ipt)) {
#define X(B, I) \
    case CRYSTAL_VARIANT_KEY(B, I): return probe_t<B, I>(cfg, ht, fk, probe_payload, n, sum, count, s);
        CRYSTAL_VARIANTS_VEC(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

// -------------------------------------------------------------- group-by ---
// LDS_PART: each workgroup accumulates into an LDS copy of the group array
// (ds_add_u64) over the tiles it strides through, then flushes the non-zero
// entries with global 64-bit atomics.  Otherwise every row adds directly.
template <int BLOCK, int IPT, bool LDS_PART>
__global__ __launch_bounds__(BLOCK) void groupby_kernel(const int32_t *__restrict__ g,
                                                        const int32_t *__restrict__ v, int64_t n,
                                                        int64_t n_groups,
                                                        uint64_t *__restrict__ sums,
                                                        int32_t *status, int64_t n_tiles) {
    using T = TileShape<BLOCK, IPT>;
    extern __shared__ __align__(16) uint64_t part[];
    if constexpr (LDS_PART) {
        for (int64_t i = threadIdx.x; i < n_groups; i += BLOCK) part[i] = 0;
        __syncthreads();
    }
    bool bad = false;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t base = tile * T::ITEMS;
        int32_t gk[IPT], vk[IPT];
        block_load<BLOCK, IPT, true>(g, base, n, gk);
        block_load<BLOCK, IPT, true>(v, base, n, vk);
        const uint32_t valid = valid_mask<BLOCK, IPT>(base, n);
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            if (!((valid >> k) & 1u)) continue;
            if ((uint64_t)(int64_t)gk[k] >= (uint64_t)n_groups) {
                bad = true;
                continue;
            }
            const uint64_t add = (uint64_t)(int64_t)vk[k];
            if constexpr (LDS_PART)
                atomicAdd((unsigned long long *)&part[gk[k]], (unsigned long long)add);
            else
                atomic_add_u64(sums + gk[k], add);
        }
    }
    if (bad) set_status(status, CRYSTAL_ERANGE);
    if constexpr (LDS_PART) {
        __syncthreads();
        for (int64_t i = threadIdx.x; i < n_groups; i += BLOCK) {
            const uint64_t x = part[i];
            if (x) atomic_add_u64(sums + i, x);
        }
    }
}

template <int BLOCK, int IPT>
static hipError_t groupby_t(const LaunchCfg &cfg_in, const int32_t *g, const int32_t *v, int64_t n,
                            int64_t n_groups, uint64_t *sums, int32_t *status, hipStream_t s) {
    using T = TileShape<BLOCK, IPT>;
    const int64_t n_tiles = (n + T::ITEMS - 1) / T::ITEMS;
    LaunchCfg cfg = cfg_in;
    const int64_t lds = n_groups * 8;
    // LDS partials cost one flush of n_groups atomics per workgroup instead
    // of one atomic per row: worth it when rows outnumber those flushes
    LaunchCfg pcfg = cfg;
    if (pcfg.grid_per_cu <= 0) pcfg.grid_per_cu = 1;
    const bool part = lds <= device_lds_per_block() / 2 && n >= 4 * grid_for(n_tiles, pcfg) * n_groups;
    if (part) cfg = pcfg;
    const int64_t grid = grid_for(n_tiles, cfg);
    if (grid == 0) return hipSuccess;
    if (part) {
        auto fn = groupby_kernel<BLOCK, IPT, true>;
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(BLOCK), (size_t)lds, s, g, v, n, n_groups,
                           sums, status, n_tiles);
    } else {
        hipLaunchKernelGGL((groupby_kernel<BLOCK, IPT, false>), dim3((unsigned)grid), dim3(BLOCK), 0, s,
                           g, v, n, n_groups, sums, status, n_tiles);
    }
    return hipGetLastError();
}

hipError_t launch_groupby(const LaunchCfg &cfg, const int32_t *group, const int32_t *value,
                          int64_t n, int64_t n_groups, uint64_t *sums, int32_t *status,
                          hipStream_t s) {
    hipError_t e = fill_u64(sums, n_groups, 0ull, s);
    if (e != hipSuccess || n == 0) return e;
    switch (CRYSTAL_VARIANT_KEY(cfg.block, cfg.ipt)) {
#define X(B, I) \
    case CRYSTAL_VARIANT_KEY(B, I): return groupby_t<B, I>(cfg, group, value, n, n_groups, sums, status, s);
        CRYSTAL_VARIANTS_VEC(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

}  // namespace crystal
