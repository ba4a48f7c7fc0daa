// Radix partitioning and radix sort of 32-bit key / 32-bit value pairs
// (section 4.4).  A partition pass on radix r = bits and start bit a = shift
// places every pair into one of 2^r contiguous partitions by the digit
// (key >> a) & (2^r - 1).  It has the two phases of section 4.4:
//
//   histogram  workgroups count the digits of tiles, or of chunks of several
//              tiles; one small kernel turns the digit x column count matrix
//              into exclusive prefixes (digit-major), which are the output
//              offsets of every (digit, column) run; for few tiles the shuffle
//              sums the counts itself;
//   shuffle    each workgroup writes the pairs of its tile, or of its chunk
//              tile by tile, to their partitions (radix_tile.hpp).
//
// The shuffle is stable, also for 8-bit digits.  Within a tile each wave
// ranks its items per digit with ballots: the lanes whose digit equals the
// calling lane's are the AND over the digit's bits of ballot(bit) or its
// complement, so the rank of an item among equal digits is the number of
// such lanes below it plus a per-wave running count in LDS.  The tile is then
// sorted by digit in LDS and written out in that order, so consecutive lanes
// write consecutive addresses of one partition.  The section's GPU designs
// keep per-thread digit counters in registers, which limits a stable pass to
// 7 bits; the wave-level ranking needs no per-thread counters.
#include "block.hpp"
#include "internal.hpp"
#include "radix_tile.hpp"
#include "variants.hpp"

namespace crystal {
namespace {

// Tiles [t0, t1) of the chunk that column `col` of the count matrix covers.
struct Chunk {
    int64_t t0, t1;
};

__device__ __forceinline__ Chunk chunk_of(int64_t col, int sub, int64_t tiles_per_block, int64_t n_tiles) {
    const int64_t b = col / sub, j = col % sub;
    const int64_t per_sub = (tiles_per_block + sub - 1) / sub;
    int64_t end = (b + 1) * tiles_per_block;
    if (end > n_tiles) end = n_tiles;
    int64_t t0 = b * tiles_per_block + j * per_sub;
    int64_t t1 = t0 + per_sub;
    if (t0 > end) t0 = end;
    if (t1 > end) t1 = end;
    return {t0, t1};
}

// ------------------------------------------------------------- histogram --
// Column c of the count matrix counts the digits of sub-chunk c (sub-chunks
// split each shuffle workgroup's chunk `sub` ways, in order; chunks are whole
// shuffle tiles of tile_items items).  MODE kMatrix: write counts[d * cols + c];
// kRows (a tile per column): write 16-bit counts[c * 256 + d]; kTotals: add into
// the global histogram counts[d].  The counting workgroup
// has its own shape: kHistBlock threads reading kHistIpt coalesced words each
// per step, with one LDS digit histogram per wave.
constexpr int kHistBlock = 256;
constexpr int kHistIpt = 16;

enum HistMode { kMatrix, kRows, kTotals };

template <HistMode MODE>
__global__ __launch_bounds__(kHistBlock) void radix_hist_kernel(const uint32_t *__restrict__ keys, int64_t n,
                                                                int shift, uint32_t mask, int64_t tile_items,
                                                                int64_t n_tiles, int64_t tiles_per_block, int sub,
                                                                uint32_t *__restrict__ counts, int64_t cols) {
    constexpr int W = kHistBlock / kWave;
    constexpr int STEP = kHistBlock * kHistIpt;
    __shared__ uint32_t h[W][kBins];
    for (int i = threadIdx.x; i < W * kBins; i += kHistBlock) (&h[0][0])[i] = 0u;
    __syncthreads();
    const int w = threadIdx.x / kWave;
    const int64_t col = xcd_item(blockIdx.x, gridDim.x);
    const Chunk ch = chunk_of(col, sub, tiles_per_block, n_tiles);
    const int64_t i0 = ch.t0 * tile_items;
    int64_t i1 = ch.t1 * tile_items;
    if (i1 > n) i1 = n;
    // full batches of STEP keys, the next batch's loads in flight while the
    // current one is counted (two register buffers, so that the one receiving
    // loads is never copied); then the partial batch
    const int64_t nfull = i1 > i0 ? (i1 - i0) / STEP : 0;
    auto load = [&](int64_t bi, uint32_t(&v)[kHistIpt]) {
        const uint32_t *kb = keys + i0 + bi * STEP;
        asm volatile("" : "+s"(kb));
#pragma unroll
        for (int k = 0; k < kHistIpt; ++k) v[k] = __builtin_nontemporal_load(kb + k * kHistBlock + threadIdx.x);
    };
    auto count = [&](const uint32_t(&v)[kHistIpt]) {
#pragma unroll
        for (int k = 0; k < kHistIpt; ++k) atomicAdd(&h[w][digit_of(v[k], shift, mask)], 1u);
    };
    uint32_t va[kHistIpt], vb[kHistIpt];
    if (nfull > 0) load(0, va);
    for (int64_t bi = 0; bi < nfull;) {
        if (bi + 1 < nfull) load(bi + 1, vb);
        count(va);
        if (++bi >= nfull) break;
        if (bi + 1 < nfull) load(bi + 1, va);
        count(vb);
        ++bi;
    }
    const int64_t b = i0 + nfull * STEP;
    if (b < i1) {
        const uint32_t *kb = keys + b;
        const int64_t left = i1 - b;
#pragma unroll
        for (int k = 0; k < kHistIpt; ++k) {
            const int i = k * kHistBlock + (int)threadIdx.x;
            if (i < left) atomicAdd(&h[w][digit_of(kb[i], shift, mask)], 1u);
        }
    }
    __syncthreads();
    const int d = threadIdx.x;
    if (d < kBins && (uint32_t)d <= mask) {
        uint32_t s = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) s += h[i][d];
        if (MODE == kMatrix)
            counts[(int64_t)d * cols + col] = s;
        else if (MODE == kRows)
            reinterpret_cast<uint16_t *>(counts)[col * kBins + d] = (uint16_t)s;
        else if (s)
            atomicAdd(&counts[d], s);
    } else if (MODE == kRows && d < kBins) {
        reinterpret_cast<uint16_t *>(counts)[col * kBins + d] = 0;
    }
}

// Row d of the count matrix becomes its exclusive prefix; totals[d] = row sum.
constexpr int kScanBlock = 1024;

__global__ __launch_bounds__(kScanBlock) void radix_scan_kernel(uint32_t *__restrict__ counts, int64_t cols,
                                                                uint32_t *__restrict__ totals) {
    __shared__ uint32_t tmp[kScanBlock / kWave];
    // rounds of kScanBlock * kAhead columns, neighbouring threads on neighbouring
    // words (16,384 columns: 51 -> 18 us against a run of columns per thread)
    constexpr int kAhead = 4;
    uint32_t *row = counts + (int64_t)blockIdx.x * cols;
    uint32_t total = 0;
    for (int64_t c0 = 0; c0 < cols; c0 += kScanBlock * kAhead) {
        uint32_t v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int64_t c = c0 + k * kScanBlock + (int64_t)threadIdx.x;
            v[k] = c < cols ? row[c] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int64_t c = c0 + k * kScanBlock + (int64_t)threadIdx.x;
            if (c0 + k * kScanBlock >= cols) break;
            uint32_t sum;
            const uint32_t before = block_exclusive_scan<kScanBlock>(v[k], tmp, sum);
            if (c < cols) row[c] = total + before;
            total += sum;
        }
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

// --------------------------------------------------------------- shuffle --
// One workgroup per chunk of tiles_per_block tiles (the chunks the count
// matrix's columns b * sub .. b * sub + sub - 1 counted).  STABLE: ballot
// ranking in input order; otherwise every item takes its rank from an LDS
// atomic on its wave's digit counter, which orders equal digits of one load
// arbitrarily (the unstable shuffle of section 4.4) for far fewer
// instructions per item.
template <int BLOCK, int IPT, bool VALS, bool STABLE>
__global__ __launch_bounds__(BLOCK, 8) void radix_shuffle_kernel(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals, int64_t n, int shift, uint32_t mask,
    int64_t n_tiles, int64_t tiles_per_block, int sub, const uint32_t *__restrict__ counts, int64_t cols,
    const uint32_t *__restrict__ totals, uint32_t *__restrict__ out_keys, uint32_t *__restrict__ out_vals,
    uint32_t *__restrict__ part_offsets) {
    using RT = RadixTile<BLOCK, IPT>;
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t *s_run = lds + RT::RUN;
    const int tid = threadIdx.x;
    const int64_t block = xcd_item(blockIdx.x, gridDim.x);

    if (totals) {
        // partition starts: exclusive prefix of the digit totals (the stage is free as scratch)
        uint32_t unused;
        const uint32_t tot = (tid < kBins && (uint32_t)tid <= mask) ? totals[tid] : 0u;
        const uint32_t dstart = block_exclusive_scan<BLOCK>(tot, lds, unused);
        if (tid < kBins) {
            s_run[tid] = (uint32_t)tid <= mask ? dstart + counts[(int64_t)tid * cols + block * sub] : 0u;
            if (block == 0 && part_offsets && (uint32_t)tid <= mask) part_offsets[tid] = dstart;
        }
    } else {
        // few tiles: the rows of counts are summed here, each wave every W-th
        // row, a lane four digits (see kRows); no scan launch
        uint32_t *s_tot = lds + RT::GBASE;
        if (tid < kBins) s_run[tid] = s_tot[tid] = 0u;
        __syncthreads();
        const uint2 *rows = reinterpret_cast<const uint2 *>(counts) + lane_id();
        uint32_t tot[4] = {0u, 0u, 0u, 0u}, before[4] = {0u, 0u, 0u, 0u};
        constexpr int kAhead = 8;
        for (int64_t c0 = tid / kWave; c0 < cols; c0 += kAhead * RT::W) {
            uint2 v[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const int64_t c = c0 + k * RT::W;
                v[k] = c < cols ? rows[c * (kBins / 4)] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const uint32_t x[4] = {v[k].x & 0xffffu, v[k].x >> 16, v[k].y & 0xffffu, v[k].y >> 16};
                const bool earlier = c0 + k * RT::W < block;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    tot[i] += x[i];
                    before[i] += earlier ? x[i] : 0u;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            atomicAdd(&s_tot[4 * lane_id() + i], tot[i]);
            atomicAdd(&s_run[4 * lane_id() + i], before[i]);
        }
        __syncthreads();
        if (tid < kWave) {
            const uint4 t = reinterpret_cast<uint4 *>(s_tot)[tid];
            uint32_t at = t.x + t.y + t.z + t.w;
            at = wave_inclusive_scan(at) - at;
            const uint32_t start[4] = {at, at + t.x, at + t.x + t.y, at + t.x + t.y + t.z};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s_run[4 * tid + i] += start[i];
                if (block == 0 && part_offsets && (uint32_t)(4 * tid + i) <= mask) part_offsets[4 * tid + i] = start[i];
            }
        }
    }
    if (block == 0 && part_offsets && tid == 0) part_offsets[mask + 1] = (uint32_t)n;
    __syncthreads();

    const int64_t t0 = block * tiles_per_block;
    int64_t t1 = t0 + tiles_per_block;
    if (t1 > n_tiles) t1 = n_tiles;
    if (t0 >= t1) return;
    const int64_t end = t1 * RT::ITEMS < n ? t1 * RT::ITEMS : n;
    shuffle_range<BLOCK, IPT, VALS, STABLE>(keys, vals, t0 * RT::ITEMS, end, shift, mask, out_keys, out_vals, lds);
}

// ---------------------------------------------------------------- launch --
struct RadixGeom {
    int64_t n_tiles, tiles_per_block, grid, cols;
    int sub;
    bool rows;  // counts as kRows, summed by the shuffle
};

template <int BLOCK, int IPT>
struct RadixKernels {
    template <bool VALS, bool STABLE>
    static hipError_t prepare_one() {
        static bool done = false;
        if (done) return hipSuccess;
        hipError_t e = hipFuncSetAttribute((const void *)radix_shuffle_kernel<BLOCK, IPT, VALS, STABLE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)RadixTile<BLOCK, IPT>::BYTES);
        if (e == hipSuccess) done = true;
        return e;
    }

    template <HistMode MODE>
    static hipError_t histogram(const uint32_t *keys, int64_t n, int shift, uint32_t mask, const RadixGeom &g,
                                uint32_t *counts, hipStream_t s) {
        hipLaunchKernelGGL((radix_hist_kernel<MODE>), dim3((unsigned)(g.grid * g.sub)), dim3(kHistBlock), 0, s, keys,
                           n, shift, mask, (int64_t)BLOCK * IPT, g.n_tiles, g.tiles_per_block, g.sub, counts, g.cols);
        return hipGetLastError();
    }

    template <bool VALS, bool STABLE>
    static hipError_t shuffle_t(const uint32_t *keys, const uint32_t *vals, int64_t n, int shift, uint32_t mask,
                                const RadixGeom &g, const uint32_t *counts, const uint32_t *totals, uint32_t *ok,
                                uint32_t *ov, uint32_t *part_offsets, hipStream_t s) {
        hipError_t e = prepare_one<VALS, STABLE>();
        if (e != hipSuccess) return e;
        const size_t lds = RadixTile<BLOCK, IPT>::BYTES;
        hipLaunchKernelGGL((radix_shuffle_kernel<BLOCK, IPT, VALS, STABLE>), dim3((unsigned)g.grid), dim3(BLOCK),
                           lds, s, keys, vals, n, shift, mask, g.n_tiles, g.tiles_per_block, g.sub, counts, g.cols,
                           totals, ok, ov, part_offsets);
        return hipGetLastError();
    }

    static hipError_t shuffle(const uint32_t *keys, const uint32_t *vals, int64_t n, int shift, uint32_t mask,
                              const RadixGeom &g, const uint32_t *counts, const uint32_t *totals,
                              uint32_t *ok, uint32_t *ov, uint32_t *part_offsets, bool stable, hipStream_t s) {
        if (vals)
            return stable ? shuffle_t<true, true>(keys, vals, n, shift, mask, g, counts, totals, ok, ov, part_offsets, s)
                          : shuffle_t<true, false>(keys, vals, n, shift, mask, g, counts, totals, ok, ov,
                                                   part_offsets, s);
        return stable ? shuffle_t<false, true>(keys, vals, n, shift, mask, g, counts, totals, ok, ov, part_offsets, s)
                      : shuffle_t<false, false>(keys, vals, n, shift, mask, g, counts, totals, ok, ov, part_offsets, s);
    }
};

size_t shuffle_lds_bytes(int block, int ipt) {
    switch (CRYSTAL_VARIANT_KEY(block, ipt)) {
#define X(B, I) \
    case CRYSTAL_VARIANT_KEY(B, I): return RadixTile<B, I>::BYTES;
        CRYSTAL_VARIANTS_RADIX(X)
#undef X
    default: return 0;
    }
}

// Up to so many tiles the shuffle sums the counts of earlier tiles itself,
// which saves the scan launch (four passes over 100,003 pairs 57 -> 45 us;
// 244 tiles 66 -> 62 us; 490 tiles 75 -> 84 us).
constexpr int64_t kRowsMax = 256;

// Scratch of a pass with a count per tile: kRows, or as below.
int64_t rows_bytes(int64_t tiles) { return tiles * kBins * 2; }

// Scratch of a pass under g: the count matrix (kBins rows of cols words,
// 256-byte aligned) and the digit totals.
int64_t pass_bytes(int64_t cols) { return ((int64_t)kBins * cols * 4 + 255) / 256 * 256 + kBins * 4; }

int64_t fine_bytes(int64_t tiles) { return tiles <= kRowsMax ? rows_bytes(tiles) : pass_bytes(tiles); }

// One tile per workgroup when the scratch holds a count per tile and no grid
// was tuned: then neighbouring tiles are written at the same time on one XCD
// (xcd_item).  Shuffle of 2^28 pairs: 1,400 us with 32 tiles per workgroup,
// 1,080 us so.  Else workgroups of several tiles, a tuned number per CU or by the
// LDS (at most 8).
RadixGeom geometry(const LaunchCfg &cfg, int64_t n, int64_t scratch_bytes) {
    RadixGeom g{};
    const int64_t items = (int64_t)cfg.block * cfg.ipt;
    g.n_tiles = (n + items - 1) / items;
    if (cfg.grid_per_cu <= 0 && scratch_bytes >= fine_bytes(g.n_tiles)) {
        g.grid = g.cols = g.n_tiles;
        g.tiles_per_block = 1;
        g.sub = 1;
        g.rows = g.n_tiles <= kRowsMax;
        return g;
    }
    int per_cu = cfg.grid_per_cu;
    if (per_cu <= 0) {
        // half of what the LDS holds (a tile twice, and its counters): chunks
        // gain nothing from more (2^28 pairs 1,628 us, with twice as many 1,643)
        const int64_t waves = cfg.block / kWave;
        per_cu = (int)(device_lds_per_cu() / (4 * (2 * items + waves * (kBins + 1) + 2 * kBins)));
        if (per_cu < 1) per_cu = 1;
        if (per_cu > 8) per_cu = 8;
    }
    const int64_t cus = device_cu_count();
    int64_t grid = (int64_t)per_cu * cus;
    if (grid > g.n_tiles) grid = g.n_tiles;
    if (grid < 1) grid = 1;
    g.tiles_per_block = (g.n_tiles + grid - 1) / grid;
    g.grid = (g.n_tiles + g.tiles_per_block - 1) / g.tiles_per_block;
    if (g.grid < 1) g.grid = 1;
    // the histogram pass splits each chunk so that about 8 workgroups per CU count
    int64_t sub = (8 * cus + g.grid - 1) / g.grid;
    if (sub > g.tiles_per_block) sub = g.tiles_per_block;
    if (sub < 1) sub = 1;
    g.sub = (int)sub;
    g.cols = g.grid * g.sub;
    return g;
}

}  // namespace

int64_t radix_pass_min_scratch_bytes(const LaunchCfg &cfg, int64_t n) {
    return pass_bytes(geometry(cfg, n > 0 ? n : 1, 0).cols);
}

int64_t radix_pass_scratch_bytes(const LaunchCfg &cfg, int64_t n) {
    const int64_t items = (int64_t)cfg.block * cfg.ipt;
    if (cfg.grid_per_cu > 0) return radix_pass_min_scratch_bytes(cfg, n);
    return fine_bytes(((n > 0 ? n : 1) + items - 1) / items);
}

bool radix_variant_fits(int block, int ipt) {
    const size_t b = shuffle_lds_bytes(block, ipt);
    return b > 0 && (int64_t)b <= device_lds_per_block();
}

#define RADIX_DISPATCH(cfg, CALL)                                               \
    switch (CRYSTAL_VARIANT_KEY(cfg.block, cfg.ipt)) {                         \
        CRYSTAL_VARIANTS_RADIX(CALL)                                           \
    default: return hipErrorInvalidValue;                                      \
    }

hipError_t launch_radix_histogram(const LaunchCfg &cfg, const uint32_t *keys, int64_t n, int shift, int bits,
                                  uint32_t *hist, hipStream_t s) {
    const uint32_t mask = (1u << bits) - 1u;
    hipError_t e = fill_u32(hist, (int64_t)mask + 1, 0u, s);
    if (e != hipSuccess || n == 0) return e;
    const RadixGeom g = geometry(cfg, n, 0);
#define X(B, I) \
    case CRYSTAL_VARIANT_KEY(B, I): return RadixKernels<B, I>::template histogram<kTotals>(keys, n, shift, mask, g, hist, s);
    RADIX_DISPATCH(cfg, X)
#undef X
}

hipError_t launch_radix_partition(const LaunchCfg &cfg, const uint32_t *keys, const uint32_t *vals, int64_t n,
                                  int shift, int bits, uint32_t *out_keys, uint32_t *out_vals,
                                  uint32_t *part_offsets, void *scratch, int64_t scratch_bytes, bool stable,
                                  hipStream_t s) {
    const uint32_t mask = (1u << bits) - 1u;
    // With few digits the unstable ranking's atomics meet on few LDS words; the
    // ballots take the same time whatever the digits (2^25 pairs, in us, unstable
    // / stable ranking: 1 bit 246/172, 2 bits 177/151, 3 bits 141/140, 4 bits
    // 126/132; 2^27 keys 1 bit 818/501, 3 bits 378/361, 4 bits 304/325).
    if (bits <= 3) stable = true;
    if (n == 0) return part_offsets ? fill_u32(part_offsets, (int64_t)mask + 2, 0u, s) : hipSuccess;
    const RadixGeom g = geometry(cfg, n, scratch_bytes);
    uint32_t *counts = (uint32_t *)scratch;
    uint32_t *totals = (uint32_t *)((char *)scratch + ((int64_t)kBins * g.cols * 4 + 255) / 256 * 256);
    hipError_t e;
    if (g.rows) {
        totals = nullptr;  // the shuffle sums the rows itself
#define X(B, I)                                                                                         \
    case CRYSTAL_VARIANT_KEY(B, I):                                                                     \
        e = RadixKernels<B, I>::template histogram<kRows>(keys, n, shift, mask, g, counts, s);          \
        break;
        RADIX_DISPATCH(cfg, X)
#undef X
        if (e != hipSuccess) return e;
    } else {
#define X(B, I)                                                                                         \
    case CRYSTAL_VARIANT_KEY(B, I):                                                                     \
        e = RadixKernels<B, I>::template histogram<kMatrix>(keys, n, shift, mask, g, counts, s);        \
        break;
        RADIX_DISPATCH(cfg, X)
#undef X
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(radix_scan_kernel, dim3(mask + 1), dim3(kScanBlock), 0, s, counts, g.cols, totals);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#define X(B, I)                                                                                              \
    case CRYSTAL_VARIANT_KEY(B, I):                                                                          \
        return RadixKernels<B, I>::shuffle(keys, vals, n, shift, mask, g, counts, totals, out_keys, out_vals, \
                                           part_offsets, stable, s);
    RADIX_DISPATCH(cfg, X)
#undef X
}

}  // namespace crystal
