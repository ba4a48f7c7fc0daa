// One tile of a stable radix partition: ranking, digit offsets, and the
// reorder through LDS, shared by the partition pass, the MSB levels and the
// MSB sort's local passes.
//
// Tile layout: BLOCK x IPT items; wave w owns the 64 * IPT consecutive items
// from w * 64 * IPT, and lane l's slot k is item k * 64 + l of them.  Visiting
// slots in order therefore visits a wave's items in input order, which makes
// the ranking stable, and every load of a wave reads 256 consecutive bytes.
//
// A tile's phases (rank, scan, reorder, write) follow one another, so a second
// workgroup per CU has to fill the gaps, and a tile is kept small: keys and
// values go through one LDS buffer in turn, counters and positions are 16 bits
// wide, and the kernels ask for 64 vector registers.  A 16 Ki tile takes 74 KB,
// two per CU; with both buffers and 32-bit counters it took 146 KB, one per CU.
// The ranking, the larger part of the vector instructions, was cut from about
// 75 per 64 items to 42.  On 2^28 pairs the MSB sort's local passes, bound by
// those instructions, went from 1,804 to 1,220 us and a partition's shuffle
// from 1,450 to 1,399 us (keys alone, 10^8: four passes 1,854 -> 1,283 us).
#pragma once

#include "block.hpp"

namespace crystal {

constexpr int kBins = 256;  // digits of at most 8 bits

template <int BLOCK, int IPT>
struct RadixTile {
    static constexpr int W = BLOCK / kWave;
    static constexpr int ITEMS = BLOCK * IPT;
    static_assert(ITEMS <= 16384, "positions and counters are 16 bits");
    // LDS, in 32-bit words
    static constexpr int STAGE = 0;                  // [ITEMS] keys, then values, in digit order
    static constexpr int WC = (ITEMS + 3) / 4 * 4;   // [W][kBins] 16-bit counters, then each wave's digit offsets
    static constexpr int GBASE = WC + W * kBins / 2; // [kBins] output offset of the digit minus its tile offset
    static constexpr int RUN = GBASE + kBins;        // [kBins] next output offset of the digit
    static constexpr int WORDS = RUN + kBins;
    static constexpr size_t BYTES = (size_t)WORDS * 4;

    // tile offset of this lane's slot k
    __device__ static __forceinline__ int offset(int k) {
        return (int)(threadIdx.x / kWave) * (kWave * IPT) + k * kWave + (int)(threadIdx.x % kWave);
    }
};

// Work item of workgroup b of n, such that the workgroups of an XCD (consecutive
// workgroups go round the eight XCDs) get consecutive items.  A tile's run in a
// partition rarely ends at a 128-byte line; the next tile continues the line, and
// when that is on the same XCD at about the same time the line leaves its L2
// whole.  Only speed depends on the placement.
__device__ __forceinline__ int64_t xcd_item(int64_t b, int64_t n) {
    const int64_t q = n / 8, r = n % 8, x = b % 8;
    return x * q + (x < r ? x : r) + b / 8;
}

__device__ __forceinline__ uint32_t digit_of(uint32_t key, int shift, uint32_t mask) { return (key >> shift) & mask; }

// Inclusive prefix over the 64 lanes of a wave.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    const int lane = (int)lane_id();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// Exclusive prefix of x over threads 0 .. BLOCK-1 in thread order; `tmp` holds
// one word per wave.  Every thread calls it; it ends with a barrier, after
// which tmp may be reused.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t *tmp, uint32_t &total) {
    constexpr int W = BLOCK / kWave;
    const uint32_t inc = wave_inclusive_scan(x);
    const int w = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) tmp[w] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        uint32_t t = tmp[i];
        before += i < w ? t : 0u;
        tot += t;
    }
    total = tot;
    __syncthreads();
    return before + inc - x;
}

// Lanes of the wave whose 8-bit digit equals the calling lane's.  Per bit: the
// bit as 0 or -1 (one signed bit-field extract), its ballot (one compare), and
// one three-operand bit operation per half of the mask.
__device__ __forceinline__ uint64_t wave_peers8(uint32_t d) {
    uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const int32_t x = __builtin_amdgcn_sbfe((int32_t)d, b, 1);
        const uint64_t m = ballot(x < 0);
        // mask & ~(ballot ^ bit): truth table 0xF0 & ~(0xCC ^ 0xAA)
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, (uint32_t)x, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), (uint32_t)x, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

// The wave clears its own counter row.
__device__ __forceinline__ void clear_counters(uint16_t *my_wc) {
    reinterpret_cast<uint2 *>(my_wc)[lane_id()] = make_uint2(0u, 0u);
}

// Rank of an item among the wave's items of digit d so far (earlier slots
// through the wave's counter, earlier lanes of this slot through the ballots),
// counting it.
__device__ __forceinline__ uint32_t stable_rank(uint32_t d, uint16_t *my_wc) {
    const uint64_t peers = wave_peers8(d);
    const uint32_t below = count_below(peers);
    const uint32_t same = (uint32_t)__popcll(peers);
    const uint32_t c = my_wc[d];
    if (below + 1 == same) my_wc[d] = (uint16_t)(c + same);
    return c + below;
}

// One wave turns the waves' digit counts into their offsets in the tile (digit
// major, waves in order); starts and counts of the lane's four digits 4 l ..
// 4 l + 3 are returned.  Each lane handles its digits of a row as two packed
// pairs; sums stay below 2^16, so plain 32-bit adds do.
template <int W>
__device__ __forceinline__ void scan_counters(uint16_t *wc, uint32_t (&start)[4], uint32_t (&cnt)[4]) {
    uint2 *rows = reinterpret_cast<uint2 *>(wc) + lane_id();
    constexpr int R = kBins / 4;  // uint2 per row
    uint32_t a = 0, b = 0;
#pragma unroll 4
    for (int i = 0; i < W; ++i) {
        const uint2 t = rows[i * R];
        a += t.x;
        b += t.y;
    }
    cnt[0] = a & 0xffffu;
    cnt[1] = a >> 16;
    cnt[2] = b & 0xffffu;
    cnt[3] = b >> 16;
    const uint32_t tot = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    start[0] = wave_inclusive_scan(tot) - tot;
    start[1] = start[0] + cnt[0];
    start[2] = start[1] + cnt[1];
    start[3] = start[2] + cnt[2];
    a = start[0] | start[1] << 16;
    b = start[2] | start[3] << 16;
#pragma unroll 4
    for (int i = 0; i < W; ++i) {
        const uint2 t = rows[i * R];
        rows[i * R] = make_uint2(a, b);
        a += t.x;
        b += t.y;
    }
}

// One column of the tile at `base`, rem items of it.  Places past the end get
// all ones: the largest digit in every pass and last in input order, so the
// stable ranking treats them like any item and they end up behind the others;
// only loads and stores test for the end.  The tile's base
// pointer is made an opaque scalar, so that every load is one scalar base plus
// one lane offset (global address space: a generic pointer would give flat
// loads).
template <int BLOCK, int IPT, bool NT>
__device__ __forceinline__ void load_tile(const uint32_t *__restrict__ col, int64_t base, int rem, int off0,
                                          uint32_t (&v)[IPT]) {
    typedef const __attribute__((address_space(1))) uint32_t *gptr;
    typedef const __attribute__((address_space(1))) char *gbytes;
    // the address is uniform; readfirstlane states it for the scalar constraint below
    const uint64_t at = (uint64_t)(uintptr_t)(col + base);
    gptr p = (gptr)(((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(at >> 32)) << 32) |
                    (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)at));
    asm volatile("" : "+s"(p), "+v"(off0));  // off0: the items' offsets must not be carried from tile to tile
    if (rem >= BLOCK * IPT) {
#pragma unroll
        for (int k = 0; k < IPT; ++k)
            v[k] = NT ? __builtin_nontemporal_load(&p[off0 + k * kWave]) : p[off0 + k * kWave];
    } else {
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            const int i = off0 + k * kWave;
            const uint32_t x = *(gptr)((gbytes)p + (uint32_t)(i < rem ? i : rem - 1) * 4u);
            v[k] = i < rem ? x : ~0u;
        }
    }
}

// Two 16-bit ranks or positions per word.
template <int IPT>
struct Pos16 {
    uint32_t w[(IPT + 1) / 2];
    __device__ __forceinline__ uint32_t get(int k) const { return k & 1 ? w[k / 2] >> 16 : w[k / 2] & 0xffffu; }
    // slots are first set in order
    __device__ __forceinline__ void init(int k, uint32_t x) {
        w[k / 2] = k & 1 ? w[k / 2] | x << 16 : x;
        asm volatile("" : "+v"(w[k / 2]));  // formed here: its parts must not stay in registers
    }
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int i = 0; i < (IPT + 1) / 2; ++i) asm volatile("" : "+v"(w[i]));
    }
    // no carry leaves the low half: positions are below 2^16
    __device__ __forceinline__ void add(int k, uint32_t x) { w[k / 2] += k & 1 ? x << 16 : x; }
};

// Items of the tile to their places in digit order: rank + the wave's digit offset.
template <int IPT>
__device__ __forceinline__ void place_keys(const uint32_t (&key)[IPT], int shift, uint32_t mask,
                                           const uint16_t *my_wc, Pos16<IPT> &pos, uint32_t *stage) {
    // opaque: the ranking's counter addresses must not stay in registers until here
    asm volatile("" : "+s"(shift));
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
        pos.add(k, my_wc[digit_of(key[k], shift, mask)]);
        stage[pos.get(k)] = key[k];
        if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    pos.opaque();  // the values compute their stage addresses again
}

// Items [begin, end) of a column, a tile at a time, to their output places;
// s_run (RUN) holds each digit's next output offset, complete before the call
// (the caller's barrier).  !STABLE: ranks of a full tile from LDS atomics on
// the wave's counters, which order equal digits of one load arbitrarily; a
// partial tile is ranked stably, so that its places past the end come last.
template <int BLOCK, int IPT, bool VALS, bool STABLE>
__device__ __forceinline__ void shuffle_range(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals,
                                              int64_t begin, int64_t end, int shift, uint32_t mask,
                                              uint32_t *__restrict__ out_keys, uint32_t *__restrict__ out_vals,
                                              uint32_t *lds) {
    using RT = RadixTile<BLOCK, IPT>;
    uint32_t *stage = lds + RT::STAGE;
    uint16_t *wc = reinterpret_cast<uint16_t *>(lds + RT::WC);
    uint32_t *s_gbase = lds + RT::GBASE, *s_run = lds + RT::RUN;
    const int tid = (int)threadIdx.x;
    const int w = tid / kWave;
    uint16_t *my_wc = wc + w * kBins;
    const int off0 = RT::offset(0);
    auto rem_at = [&](int64_t b) { return end - b >= RT::ITEMS ? RT::ITEMS : (int)(end - b); };

    for (int64_t base = begin; base < end; base += RT::ITEMS) {
        const int rem = rem_at(base);
        uint32_t key[IPT], val[IPT];
        load_tile<BLOCK, IPT, true>(keys, base, rem, off0, key);
        Pos16<IPT> pos;
        // 1. ranks.  The counter row was last read before the previous tile's
        //    scatter barrier.
        clear_counters(my_wc);
        __builtin_amdgcn_wave_barrier();
        if (STABLE || rem < RT::ITEMS) {
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                pos.init(k, stable_rank(digit_of(key[k], shift, mask), my_wc));
                // one slot at a time: interleaving slots only raises register pressure,
                // since each slot waits for the previous slot's counter update anyway
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            uint32_t *my_wc32 = reinterpret_cast<uint32_t *>(my_wc);
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint32_t d = digit_of(key[k], shift, mask), sh = (d & 1u) * 16u;
                pos.init(k, (atomicAdd(&my_wc32[d >> 1], 1u << sh) >> sh) & 0xffffu);
            }
        }
        __syncthreads();
        // 2. tile offsets of every wave's digits, and the digits' output bases
        if (w == 0) {
            uint32_t start[4], cnt[4];
            scan_counters<RT::W>(wc, start, cnt);
            const uint4 run = reinterpret_cast<uint4 *>(s_run)[tid];
            reinterpret_cast<uint4 *>(s_gbase)[tid] =
                make_uint4(run.x - start[0], run.y - start[1], run.z - start[2], run.w - start[3]);
            reinterpret_cast<uint4 *>(s_run)[tid] =
                make_uint4(run.x + cnt[0], run.y + cnt[1], run.z + cnt[2], run.w + cnt[3]);
        }
        __syncthreads();
        // the values arrive while the keys are placed and written
        if (VALS) load_tile<BLOCK, IPT, true>(vals, base, rem, off0, val);
        // 3. the keys in digit order
        place_keys<IPT>(key, shift, mask, my_wc, pos, stage);
        __syncthreads();
        // 4. out, consecutive lanes to consecutive places of a partition
        int tidv = tid;  // opaque: keeps per-item offsets out of registers
        asm volatile("" : "+v"(tidv));
        uint32_t digits[(IPT + 3) / 4];  // of the items written, four per word, for the values
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const int p = j * BLOCK + tidv;
            const uint32_t k = stage[p];
            const uint32_t d = digit_of(k, shift, mask);
            if (VALS) digits[j / 4] = j % 4 ? digits[j / 4] | d << (j % 4 * 8) : d;
            const uint32_t g = s_gbase[d] + (uint32_t)p;  // < n < 2^32
            if (p < rem) out_keys[g] = k;
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (VALS) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                stage[pos.get(k)] = val[k];
                if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
        }
        if constexpr (VALS) {
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const int p = j * BLOCK + tidv;
                const uint32_t g = s_gbase[(digits[j / 4] >> (j % 4 * 8)) & 0xffu] + (uint32_t)p;
                if (p < rem) out_vals[g] = stage[p];
                if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        }
        // no barrier: the next tile writes s_gbase, s_run and the stage only
        // after its ranking barrier, which every wave reaches after this write-out
    }
}

// Sort of a tile: the items key (and val), `len` of them in tile layout, by
// their low `bits` key bits with stable 8-bit passes, written to out_k (out_v)
// from `start` on.  (With the sum of the two as a restrict pointer the MSB sort's
// local passes took 1,490 us instead of 1,250.)
template <int BLOCK, int IPT, bool VALS>
__device__ __forceinline__ void sort_in_lds(uint32_t (&key)[IPT], uint32_t (&val)[IPT], int len, uint32_t bits,
                                            uint32_t *out_k, uint32_t *out_v, uint32_t start,
                                            uint32_t *lds) {
    using RT = RadixTile<BLOCK, IPT>;
    uint32_t *stage = lds + RT::STAGE;
    uint16_t *wc = reinterpret_cast<uint16_t *>(lds + RT::WC);
    const int tid = (int)threadIdx.x;
    const int w = tid / kWave;
    uint16_t *my_wc = wc + w * kBins;
    const int off0 = RT::offset(0);
    for (uint32_t sh = 0; sh < bits; sh += 8) {
        const uint32_t left = bits - sh;
        const uint32_t mask = left >= 8 ? 0xFFu : (1u << left) - 1u;
        Pos16<IPT> pos;
        clear_counters(my_wc);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            pos.init(k, stable_rank(digit_of(key[k], (int)sh, mask), my_wc));
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        if (w == 0) {
            uint32_t start[4], cnt[4];
            scan_counters<RT::W>(wc, start, cnt);
        }
        __syncthreads();
        place_keys<IPT>(key, (int)sh, mask, my_wc, pos, stage);
        __syncthreads();
        const bool last = sh + 8 >= bits;
        if (last) {
            for (int i = tid; i < len; i += BLOCK) out_k[start + i] = stage[i];
        } else {
#pragma unroll
            for (int k = 0; k < IPT; ++k) key[k] = stage[off0 + k * kWave];
        }
        if constexpr (VALS) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < IPT; ++k) stage[pos.get(k)] = val[k];
            __syncthreads();
            if (last) {
                for (int i = tid; i < len; i += BLOCK) out_v[start + i] = stage[i];
            } else {
#pragma unroll
                for (int k = 0; k < IPT; ++k) val[k] = stage[off0 + k * kWave];
            }
        }
        // no barrier: the stage is written again only after the next ranking
        // barrier, and a wave's counters were last read by the wave itself
    }
}

}  // namespace crystal
