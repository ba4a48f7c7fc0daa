// The unstable shuffle of radix_tile.hpp on the CPU, one fiber per lane: lanes
// meet at barriers and ballots and otherwise run in an order the test chooses,
// so that LDS atomics of one instruction are served in any lane order.  After a
// ballot they run upwards: a lane's read of a wave's counter comes before the
// last lane's write to it, an instruction later.
// Prints every case whose partitions do not hold exactly the input's pairs.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <algorithm>
#include <random>
#include <utility>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __restrict__ __restrict
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
static uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
static uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }

namespace lanes {

constexpr int kMaxThreads = 1024;
struct Barrier {
    int waiting = 0, generation = 0;
};
static int n_threads, current;
static Barrier block_barrier, wave_barriers[kMaxThreads / 64];
static uint64_t slots[kMaxThreads];
static ucontext_t scheduler, fibers[kMaxThreads];
static bool done[kMaxThreads], after_ballot[kMaxThreads / 64];
static std::vector<char> stacks;
static void (*body)();

static void yield() { swapcontext(&fibers[current], &scheduler); }

// the scheduler opens a full barrier between two rounds of the lanes
static void arrive(Barrier &b) {
    const int g = b.generation;
    ++b.waiting;
    do yield();
    while (b.generation == g);
}

static void open_if_full(Barrier &b, int n) {
    if (b.waiting < n) return;
    b.waiting = 0;
    ++b.generation;
}

static void wave_sync() { arrive(wave_barriers[current / 64]); }

// every lane's x, gathered over the wave
static uint64_t gather(uint64_t x, uint64_t (&all)[64]) {
    slots[current] = x;
    wave_sync();
    std::copy(slots + current / 64 * 64, slots + current / 64 * 64 + 64, all);
    wave_sync();
    return all[current % 64];
}

static void entry() {
    body();
    done[current] = true;
    yield();
}

}  // namespace lanes

static struct { unsigned x; } threadIdx;

static void __syncthreads() {
    lanes::after_ballot[lanes::current / 64] = false;
    lanes::arrive(lanes::block_barrier);
}
static uint32_t atomicAdd(uint32_t *p, uint32_t v) {
    const uint32_t old = *p;
    *p += v;
    lanes::yield();  // the other lanes' atomics of this instruction come before this lane's next one
    return old;
}
static uint32_t __shfl_up(uint32_t x, int o) {
    uint64_t all[64];
    lanes::gather(x, all);
    const int l = lanes::current % 64;
    return (uint32_t)all[l >= o ? l - o : l];
}
#define __builtin_amdgcn_wave_barrier() lanes::wave_sync()
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sbfe(x, b, w) (((x) >> (b)) & 1 ? -1 : 0)
#define __builtin_amdgcn_bitop3_b32(a, b, c, t) ((a) & ~((b) ^ (c)))
#define __popcll(x) __builtin_popcountll(x)
#define asm
#define volatile(...)

namespace crystal {
constexpr int kWave = 64;
static uint64_t ballot(bool p) {
    uint64_t all[64], m = 0;
    lanes::gather(p, all);
    lanes::after_ballot[lanes::current / 64] = true;
    for (int i = 0; i < 64; ++i) m |= (uint64_t)(all[i] != 0) << i;
    return m;
}
static uint32_t lane_id() { return (uint32_t)lanes::current % 64; }
static uint32_t count_below(uint64_t m) { return (uint32_t)__builtin_popcountll(m & ((1ull << lane_id()) - 1)); }
}  // namespace crystal

#include "radix_tile.hpp"

namespace lanes {

// order: the lanes in the order in which they run between meeting points
static void run_block(int threads, void (*fn)(), const std::vector<int> &order) {
    constexpr size_t kStack = 1 << 16;
    n_threads = threads;
    body = fn;
    stacks.resize(kStack * threads);
    block_barrier = Barrier();
    for (auto &b : wave_barriers) b = Barrier();
    for (bool &b : after_ballot) b = false;
    for (int t = 0; t < threads; ++t) {
        done[t] = false;
        getcontext(&fibers[t]);
        fibers[t].uc_stack.ss_sp = stacks.data() + kStack * t;
        fibers[t].uc_stack.ss_size = kStack;
        fibers[t].uc_link = &scheduler;
        makecontext(&fibers[t], entry, 0);
    }
    for (int left = threads; left > 0;) {
        open_if_full(block_barrier, threads);
        for (int w = 0; w < threads / 64; ++w) open_if_full(wave_barriers[w], 64);
        bool upwards[kMaxThreads / 64];
        int next[kMaxThreads / 64];
        for (int w = 0; w < threads / 64; ++w) {
            upwards[w] = after_ballot[w];
            next[w] = w * 64;
        }
        for (int t : order) {
            const int lane = upwards[t / 64] ? next[t / 64]++ : t;
            if (done[lane]) continue;
            current = lane;
            threadIdx.x = (unsigned)lane;
            swapcontext(&scheduler, &fibers[lane]);
            left -= done[lane];
        }
    }
}

}  // namespace lanes

using namespace crystal;

constexpr int kBlock = 256, kIpt = 4;
using RT = RadixTile<kBlock, kIpt>;
static std::vector<uint32_t> keys, vals, out_k, out_v, start;
static int g_shift;
static uint32_t g_mask;
static bool g_vals;
alignas(16) static uint32_t lds[RT::WORDS];

static void shuffle_body() {
    if (threadIdx.x < kBins) lds[RT::RUN + threadIdx.x] = threadIdx.x <= g_mask ? start[threadIdx.x] : 0u;
    __syncthreads();
    const int64_t n = (int64_t)keys.size();
    if (g_vals)
        shuffle_range<kBlock, kIpt, true, false>(keys.data(), vals.data(), 0, n, g_shift, g_mask, out_k.data(),
                                                 out_v.data(), lds);
    else
        shuffle_range<kBlock, kIpt, false, false>(keys.data(), nullptr, 0, n, g_shift, g_mask, out_k.data(), nullptr,
                                                  lds);
}

int main() {
    std::mt19937 rng(7);
    int bad = 0, cases = 0;
    for (int n : {1, 63, 64, 65, 255, 321, 1000, 1023, 1024, 1025, 2 * 1024 + 130})
        for (int bits : {1, 4, 8})
            for (int kind = 0; kind < 3; ++kind)      // all keys of the largest digit, half of them, none in particular
                for (int way = 0; way < 3; ++way)     // lanes upwards, downwards, shuffled
                    for (bool values : {true, false}) {
                        g_vals = values;
                        g_shift = 32 - bits;
                        g_mask = (1u << bits) - 1u;
                        keys.resize(n);
                        vals.resize(n);
                        for (int i = 0; i < n; ++i) {
                            keys[i] = kind == 0 || (kind == 1 && rng() % 2) ? ~0u - (uint32_t)i : (uint32_t)rng();
                            vals[i] = (uint32_t)i;
                        }
                        start.assign(g_mask + 2, 0);
                        for (uint32_t k : keys) ++start[((k >> g_shift) & g_mask) + 1];
                        for (uint32_t d = 0; d <= g_mask; ++d) start[d + 1] += start[d];
                        out_k.assign(n, 0);
                        out_v.assign(n, 0);
                        std::vector<int> order(kBlock);
                        for (int t = 0; t < kBlock; ++t) order[t] = way == 1 ? kBlock - 1 - t : t;
                        if (way == 2) std::shuffle(order.begin(), order.end(), rng);
                        lanes::run_block(kBlock, shuffle_body, order);
                        bool ok = true;
                        std::vector<std::pair<uint32_t, uint32_t>> want, got;
                        for (int i = 0; i < n; ++i) {
                            want.push_back({keys[i], values ? vals[i] : 0u});
                            got.push_back({out_k[i], out_v[i]});
                            const uint32_t d = (out_k[i] >> g_shift) & g_mask;
                            ok = ok && (uint32_t)i >= start[d] && (uint32_t)i < start[d + 1];
                        }
                        std::sort(want.begin(), want.end());
                        std::sort(got.begin(), got.end());
                        ++cases;
                        if (!ok || want != got) {
                            printf("n %d bits %d kind %d way %d values %d\n", n, bits, kind, way, (int)values);
                            ++bad;
                        }
                    }
    printf("%d cases, %d wrong\n", cases, bad);
    return bad != 0;
}
