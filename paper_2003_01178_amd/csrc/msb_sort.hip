// MSB radix sort of 32-bit key / 32-bit value pairs (section 4.4: the GPU
// sort partitions by the most significant 8-bit digit first, then within
// each partition by the next digit).
//
// Level 0 is the plain stable partition pass on the top byte (the whole
// input is one segment).  Level L >= 1 (shift 24 - 8L) partitions every
// "big" segment (more pairs than a workgroup sorts in LDS) by its digit at
// `shift`, stably:
//   chunks    each big segment is cut into chunks of one tile;
//   histogram one workgroup counts the digits of a chunk;
//   scan      one workgroup per segment turns its chunks' counts into output
//             offsets (digit-major within the segment) and classifies the
//             segment's 256 sub-segments: big ones go to the next level,
//             the others become local-sort tasks;
//   shuffle   one workgroup per chunk writes its pairs to their offsets, a
//             tile at a time, ranking equal digits stably with ballots (the
//             tile is sorted by digit in LDS, then written in that order).
// Two final launches sort every task in LDS by its remaining low bits
// (stable 8-bit passes from the low digit up), one workgroup per task, and
// write it to the output: tasks of at most kSmallMax pairs in a small shape
// (eight workgroups per CU), the others in a large one.  Levels alternate
// between the output and a scratch copy; a task reads whichever holds its
// segment.  Uniform keys need two partition levels (256, then
// 65,536 segments of about 4,096 pairs) and the local pass; skewed keys
// simply keep more segments big for more levels.
//
// All work lists live in device memory and every kernel loops over its list
// (persistent workgroups), so the host never waits for the device.
#include "block.hpp"
#include "internal.hpp"
#include "radix_tile.hpp"

namespace crystal {
namespace {

constexpr uint32_t kLocalMax = 8192;  // pairs one local-sort workgroup holds (512 threads x 16)
constexpr uint32_t kSmallSeg = 1024;  // sub-segments shorter than this are grouped into one task
constexpr int kPartBlock = 1024;
constexpr int kPartIpt = 16;
constexpr uint32_t kChunk = kPartBlock * kPartIpt;    // pairs per partition chunk: one tile
constexpr uint32_t kCopy = 65536;     // pairs per copy task
constexpr int kLocBlock = 512, kLocIpt = 16;  // tasks up to kLocalMax pairs
constexpr int kSmlBlock = 256, kSmlIpt = 17;  // tasks up to kSmallMax pairs, eight workgroups per CU
constexpr uint32_t kSmallMax = kSmlBlock * kSmlIpt;
static_assert(kLocBlock * kLocIpt >= (int)kLocalMax, "the large shape holds every sorted task");
constexpr int kAuxBlock = 256;

struct Seg {
    uint32_t start, len, chunk_base, nchunks;
};
struct ChunkD {
    uint32_t seg, start, end, pad;
};
// src: where the segment lives (0 the input, 1 the output, 2 the scratch
// copy); bits: low key bits still to sort (0: copy only)
struct Task {
    uint32_t start, len, bits, src;
};
// two task lists: 0 for tasks of at most kSmallMax pairs, 1 for the others
struct Ctl {
    uint32_t n_big[2];
    uint32_t n_chunks;
    uint32_t n_tasks[2];
    uint32_t taken[8];  // chunks of each XCD's range taken beyond its workgroups' first
};

__device__ __forceinline__ int task_list(uint32_t len, uint32_t bits) { return bits && len <= kSmallMax ? 0 : 1; }

// ------------------------------------------------------------ work lists --
// One workgroup: chunk counts of the level's big segments, their exclusive
// prefix (each segment's first chunk), the level's chunk total; clears the
// next level's big-segment count.
__global__ __launch_bounds__(1024) void msb_chunk_scan_kernel(Ctl *ctl, Seg *big, int cur) {
    __shared__ uint32_t tmp[1024 / kWave];
    const uint32_t nb = ctl->n_big[cur];
    const uint32_t per = (nb + 1023u) / 1024u;
    const uint32_t s0 = threadIdx.x * per;
    uint32_t s1 = s0 + per;
    if (s1 > nb) s1 = nb;
    uint32_t sum = 0;
    for (uint32_t i = s0; i < s1; ++i) sum += (big[i].len + kChunk - 1) / kChunk;
    uint32_t total;
    uint32_t run = block_exclusive_scan<1024>(sum, tmp, total);
    for (uint32_t i = s0; i < s1; ++i) {
        const uint32_t c = (big[i].len + kChunk - 1) / kChunk;
        big[i].chunk_base = run;
        big[i].nchunks = c;
        run += c;
    }
    if (threadIdx.x == 0) {
        ctl->n_chunks = total;
        ctl->n_big[cur ^ 1] = 0;
    }
    if (threadIdx.x < 8) ctl->taken[threadIdx.x] = 0;
}

// Chunk c of the level: its segment (binary search over the segments' first
// chunks) and its pair range.
__global__ __launch_bounds__(kAuxBlock) void msb_chunk_fill_kernel(const Ctl *ctl, const Seg *big, int cur,
                                                                   ChunkD *chunks) {
    const uint32_t nb = ctl->n_big[cur], nc = ctl->n_chunks;
    for (uint32_t c = blockIdx.x * kAuxBlock + threadIdx.x; c < nc; c += gridDim.x * kAuxBlock) {
        uint32_t lo = 0, hi = nb - 1;  // the last segment whose first chunk is <= c
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) / 2;
            if (big[mid].chunk_base <= c)
                lo = mid;
            else
                hi = mid - 1;
        }
        const Seg s = big[lo];
        const uint32_t start = s.start + (c - s.chunk_base) * kChunk;
        const uint32_t seg_end = s.start + s.len;
        chunks[c] = ChunkD{lo, start, (seg_end - start > kChunk) ? start + kChunk : seg_end, 0u};
    }
}

// Digit counts of every chunk: hist[c * 256 + d].
__global__ __launch_bounds__(kAuxBlock) void msb_hist_kernel(const Ctl *ctl, const ChunkD *chunks,
                                                             const uint32_t *__restrict__ keys, int shift,
                                                             uint32_t *__restrict__ hist) {
    constexpr int W = kAuxBlock / kWave;
    __shared__ uint32_t h[W][kBins];
    const int w = threadIdx.x / kWave;
    const uint32_t nc = ctl->n_chunks;
    for (uint32_t c = blockIdx.x; c < nc; c += gridDim.x) {
        for (int i = threadIdx.x; i < W * kBins; i += kAuxBlock) (&h[0][0])[i] = 0u;
        __syncthreads();
        const ChunkD ch = chunks[c];
        // 16 keys per thread in flight at a time, then the tail
        constexpr int B = 16;
        uint32_t i = ch.start;
        for (; i + B * kAuxBlock <= ch.end; i += B * kAuxBlock) {
            uint32_t v[B];
#pragma unroll
            for (int k = 0; k < B; ++k) v[k] = __builtin_nontemporal_load(keys + i + k * kAuxBlock + threadIdx.x);
#pragma unroll
            for (int k = 0; k < B; ++k) atomicAdd(&h[w][(v[k] >> shift) & 0xFFu], 1u);
        }
        for (i += threadIdx.x; i < ch.end; i += kAuxBlock)
            atomicAdd(&h[w][(__builtin_nontemporal_load(keys + i) >> shift) & 0xFFu], 1u);
        __syncthreads();
        const int d = threadIdx.x;  // kAuxBlock == kBins
        uint32_t s = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) s += h[i][d];
        hist[(int64_t)c * kBins + d] = s;
        __syncthreads();
    }
}

// The sub-segments of one big segment, after its partition at `shift`
// (starts st[], lengths tot[], per digit), become next-level big segments or
// local-sort tasks; run by one thread.  Sub-segments of kSmallSeg pairs or
// more are tasks of their own, sorted by the `shift` bits below their digit;
// shorter neighbours are grouped into tasks of at most kLocalMax pairs,
// sorted by their digit too.  At the last digit every sub-segment is final
// where the level wrote it: copy tasks of at most kCopy pairs when that is
// the scratch copy.  Two walks: count and reserve, then write.
__device__ void plan_subsegments(Ctl *ctl, int cur, const uint32_t *st, const uint32_t *tot, uint32_t seg_start,
                                 uint32_t seg_len, int shift, uint32_t dst, Seg *next, Task *tasks,
                                 uint32_t list_stride, uint32_t &base_big, uint32_t *base_task) {
    for (int write = 0; write < 2; ++write) {
        uint32_t nbig = 0, ntask[2] = {0u, 0u};
        auto emit_task = [&](uint32_t a, uint32_t len, uint32_t bits) {
            const int l = task_list(len, bits);
            if (write) tasks[(int64_t)l * list_stride + base_task[l] + ntask[l]] = Task{a, len, bits, dst};
            ++ntask[l];
        };
        if (shift == 0) {
            // copies in pieces of kCopy pairs, so that a long run of one key
            // is copied by many workgroups
            if (dst != 1u)
                for (uint64_t a = 0; a < seg_len; a += kCopy)
                    emit_task(seg_start + (uint32_t)a, seg_len - a < kCopy ? (uint32_t)(seg_len - a) : kCopy, 0u);
        } else {
            uint32_t g_start = 0, g_len = 0, g_digits = 0;
            auto flush = [&]() {
                if (g_len) emit_task(g_start, g_len, g_digits > 1 ? (uint32_t)shift + 8u : (uint32_t)shift);
                g_len = 0;
                g_digits = 0;
            };
            for (int e = 0; e < kBins; ++e) {
                const uint32_t len = tot[e];
                if (!len) continue;
                if (len > kLocalMax) {
                    flush();
                    if (write) next[base_big + nbig] = Seg{st[e], len, 0u, 0u};
                    ++nbig;
                } else if (len >= kSmallSeg) {
                    flush();
                    emit_task(st[e], len, (uint32_t)shift);
                } else {
                    if (g_len && g_len + len > kLocalMax) flush();
                    if (!g_len) g_start = st[e];
                    g_len += len;
                    ++g_digits;
                }
            }
            flush();
        }
        if (!write) {
            base_big = nbig ? atomicAdd(&ctl->n_big[cur ^ 1], nbig) : 0u;
            for (int l = 0; l < 2; ++l) base_task[l] = ntask[l] ? atomicAdd(&ctl->n_tasks[l], ntask[l]) : 0u;
        }
    }
}

// The same by the whole workgroup, thread d for digit d; called by all with
// st and tot written, ends with a barrier.  One thread's two walks over the
// digits took 60 us; when no sub-segment is short enough to be grouped (the
// usual case of a long segment), each thread emits its own.
__device__ __forceinline__ void plan_segment(Ctl *ctl, int cur, const uint32_t *st, const uint32_t *tot,
                                             uint32_t seg_start, uint32_t seg_len, int shift, uint32_t dst, Seg *next,
                                             Task *tasks, uint32_t list_stride, uint32_t &base_big,
                                             uint32_t *base_task) {
    const int d = (int)threadIdx.x;
    __syncthreads();
    const uint32_t len = tot[d];
    if (__syncthreads_or(shift == 0 || (len > 0 && len < kSmallSeg))) {
        if (d == 0)
            plan_subsegments(ctl, cur, st, tot, seg_start, seg_len, shift, dst, next, tasks, list_stride, base_big,
                             base_task);
        __syncthreads();
        return;
    }
    // 2: a big segment of the next level; 0, 1: a task of that list; 3: nothing.
    // Entries keep the digits' order, so that neighbours are sorted at about the
    // same time.
    constexpr int W = kAuxBlock / kWave;
    __shared__ uint32_t count[3][W];
    const int kind = len == 0 ? 3 : len > kLocalMax ? 2 : task_list(len, (uint32_t)shift);
    uint32_t at = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint64_t m = ballot(kind == k);
        if (kind == k) at = count_below(m);
        if (lane_id() == 0) count[k][d / kWave] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    if (d < 3) {
        uint32_t total = 0;
        for (int w = 0; w < W; ++w) {
            const uint32_t c = count[d][w];
            count[d][w] = total;
            total += c;
        }
        const uint32_t base = total ? atomicAdd(d == 2 ? &ctl->n_big[cur ^ 1] : &ctl->n_tasks[d], total) : 0u;
        if (d == 2)
            base_big = base;
        else
            base_task[d] = base;
    }
    __syncthreads();
    if (kind < 3) at += count[kind][d / kWave];
    if (kind == 2)
        next[base_big + at] = Seg{st[d], len, 0u, 0u};
    else if (kind < 2)
        tasks[(int64_t)kind * list_stride + base_task[kind] + at] = Task{st[d], len, (uint32_t)shift, dst};
    __syncthreads();
}

// Level 0 done by the plain partition pass (the whole input is one segment):
// its partition offsets (part[d], part[256] = n) become the first level's
// sub-segments.  One workgroup of 256 threads; also resets the counters.
__global__ __launch_bounds__(kAuxBlock) void msb_level0_kernel(Ctl *ctl, const uint32_t *part, uint32_t n,
                                                               Seg *next, Task *tasks, uint32_t list_stride) {
    __shared__ uint32_t st[kBins], tot[kBins];
    __shared__ uint32_t base_big, base_task[2];
    const int d = threadIdx.x;
    st[d] = part[d];
    tot[d] = part[d + 1] - part[d];
    if (d == 0) {
        ctl->n_big[0] = 0;
        ctl->n_big[1] = 0;
        ctl->n_chunks = 0;
        ctl->n_tasks[0] = ctl->n_tasks[1] = 0;
    }
    __syncthreads();
    // big sub-segments go to list 1, which level 1 reads
    plan_segment(ctl, 0, st, tot, 0u, n, 24, 1u, next, tasks, list_stride, base_big, base_task);
}

// One workgroup per big segment (thread d = digit d): the chunks' counts
// become global output offsets, in place; the segment's sub-segments become
// next-level big segments or tasks.  dst: where this level writes (1 the
// output, 2 the scratch copy).
__global__ __launch_bounds__(kAuxBlock) void msb_scan_kernel(Ctl *ctl, const Seg *big, int cur,
                                                             uint32_t *__restrict__ hist, Seg *next, Task *tasks,
                                                             uint32_t list_stride, int shift, uint32_t dst) {
    __shared__ uint32_t tmp[kAuxBlock / kWave];
    __shared__ uint32_t st[kBins], tot[kBins];
    __shared__ uint32_t base_big, base_task[2];
    const int d = threadIdx.x;
    const uint32_t nb = ctl->n_big[cur];
    for (uint32_t i = blockIdx.x; i < nb; i += gridDim.x) {
        const Seg s = big[i];
        // the chunks' counts of this digit, kAhead loads in flight: their sum, then their prefixes
        constexpr uint32_t kAhead = 16;
        uint32_t *col = hist + (int64_t)s.chunk_base * kBins + d;
        uint32_t run = 0;
        for (uint32_t j = 0; j < s.nchunks; j += kAhead) {
            uint32_t v[kAhead];
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) v[k] = j + k < s.nchunks ? col[(int64_t)(j + k) * kBins] : 0u;
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) run += v[k];
        }
        uint32_t unused;
        const uint32_t dstart = block_exclusive_scan<kAuxBlock>(run, tmp, unused);
        const uint32_t at = s.start + dstart;
        uint32_t next_at = at;
        for (uint32_t j = 0; j < s.nchunks; j += kAhead) {
            uint32_t v[kAhead];
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) v[k] = j + k < s.nchunks ? col[(int64_t)(j + k) * kBins] : 0u;
#pragma unroll
            for (uint32_t k = 0; k < kAhead; ++k) {
                if (j + k < s.nchunks) col[(int64_t)(j + k) * kBins] = next_at;
                next_at += v[k];
            }
        }
        st[d] = at;
        tot[d] = run;
        plan_segment(ctl, cur, st, tot, s.start, s.len, shift, dst, next, tasks, list_stride, base_big, base_task);
    }
}

// ---------------------------------------------------------------- shuffle --
template <bool VALS>
__global__ __launch_bounds__(kPartBlock, 8) void msb_shuffle_kernel(Ctl *ctl, const ChunkD *chunks,
                                                                    const uint32_t *__restrict__ hist,
                                                                    const uint32_t *__restrict__ ik,
                                                                    const uint32_t *__restrict__ iv,
                                                                    uint32_t *__restrict__ ok,
                                                                    uint32_t *__restrict__ ov, int shift) {
    using RT = RadixTile<kPartBlock, kPartIpt>;
    extern __shared__ __align__(16) uint32_t lds[];
    uint32_t *s_run = lds + RT::RUN;
    // the chunks of an XCD's workgroups are consecutive (see xcd_item; the grid
    // is a multiple of 8) and are taken in order, so that neighbours are written
    // at about the same time
    __shared__ uint32_t s_next[2];
    const uint32_t nc = ctl->n_chunks;
    const uint32_t x = blockIdx.x % 8, wgs = gridDim.x / 8;
    const uint32_t first = (uint32_t)((uint64_t)nc * x / 8), last = (uint32_t)((uint64_t)nc * (x + 1) / 8);
    uint32_t c = first + blockIdx.x / 8;
    for (int turn = 0; c < last; turn ^= 1) {
        const ChunkD ch = chunks[c];
        if (threadIdx.x == 0) s_next[turn] = first + wgs + atomicAdd(&ctl->taken[x], 1u);
        // the previous chunk last used s_run before its scatter barrier
        if (threadIdx.x < kBins) s_run[threadIdx.x] = hist[(int64_t)c * kBins + threadIdx.x];
        __syncthreads();
        shuffle_range<kPartBlock, kPartIpt, VALS, true>(ik, iv, ch.start, ch.end, shift, 0xFFu, ok, ov, lds);
        c = s_next[turn];
    }
}

// ------------------------------------------------------------ local sort --
// One task at a time per workgroup: its pairs in registers (the tile layout
// above), sorted by `bits` low key bits with stable 8-bit passes in LDS,
// then written out from LDS.  Two shapes: BLOCK x IPT holds the task list's
// largest task; the small shape fits eight workgroups per CU.
template <bool VALS, int BLOCK, int IPT>
__global__ __launch_bounds__(BLOCK, 8) void msb_local_kernel(const Ctl *ctl, int list, const Task *tasks,
                                                             const uint32_t *__restrict__ in_k,
                                                             const uint32_t *__restrict__ in_v,
                                                             uint32_t *__restrict__ out_k,
                                                             uint32_t *__restrict__ out_v,
                                                             const uint32_t *__restrict__ tmp_k,
                                                             const uint32_t *__restrict__ tmp_v) {
    using RT = RadixTile<BLOCK, IPT>;
    extern __shared__ __align__(16) uint32_t lds[];
    const int tid = threadIdx.x;
    const int off0 = RT::offset(0);
    const uint32_t nt = ctl->n_tasks[list];
    auto src_k = [&](const Task &t) { return t.src == 0 ? in_k : t.src == 1 ? (const uint32_t *)out_k : tmp_k; };
    auto src_v = [&](const Task &t) { return t.src == 0 ? in_v : t.src == 1 ? (const uint32_t *)out_v : tmp_v; };

    for (uint32_t t = blockIdx.x; t < nt; t += gridDim.x) {
        const Task task = tasks[t];
        const int len = (int)task.len;
        if (task.bits == 0) {
            // already in order: copy unless it is in the output already
            if (task.src != 1) {
                const uint32_t *sk = src_k(task), *sv = src_v(task);
                for (uint32_t i = tid; i < task.len; i += BLOCK) {
                    out_k[task.start + i] = sk[task.start + i];
                    if (VALS) out_v[task.start + i] = sv[task.start + i];
                }
            }
            continue;
        }
        uint32_t key[IPT], val[IPT];
        load_tile<BLOCK, IPT, false>(src_k(task) + task.start, 0, len, off0, key);
        if (VALS) load_tile<BLOCK, IPT, false>(src_v(task) + task.start, 0, len, off0, val);
        sort_in_lds<BLOCK, IPT, VALS>(key, val, len, task.bits, out_k, out_v, task.start, lds);
    }
}

// A short input in one workgroup.
template <bool VALS, int BLOCK, int IPT>
__global__ __launch_bounds__(BLOCK) void sort_short_kernel(const uint32_t *__restrict__ in_k,
                                                           const uint32_t *__restrict__ in_v, int n,
                                                           uint32_t *__restrict__ out_k,
                                                           uint32_t *__restrict__ out_v) {
    using RT = RadixTile<BLOCK, IPT>;
    __shared__ __align__(16) uint32_t lds[RT::WORDS];
    uint32_t key[IPT], val[IPT];
    load_tile<BLOCK, IPT, false>(in_k, 0, n, RT::offset(0), key);
    if (VALS) load_tile<BLOCK, IPT, false>(in_v, 0, n, RT::offset(0), val);
    sort_in_lds<BLOCK, IPT, VALS>(key, val, n, 32u, out_k, out_v, 0u, lds);
}

template <bool VALS>
hipError_t sort_short(const uint32_t *keys, const uint32_t *vals, int n, uint32_t *ok, uint32_t *ov, hipStream_t s) {
    if (n <= 2048)
        hipLaunchKernelGGL((sort_short_kernel<VALS, 1024, 2>), dim3(1), dim3(1024), 0, s, keys, vals, n, ok, ov);
    else
        hipLaunchKernelGGL((sort_short_kernel<VALS, 1024, 8>), dim3(1), dim3(1024), 0, s, keys, vals, n, ok, ov);
    return hipGetLastError();
}

int64_t r256(int64_t b) { return (b + 255) / 256 * 256; }

struct MsbLayout {
    int64_t max_big, max_chunks, max_tasks;
    int64_t tmp_k, tmp_v, big0, big1, chunks, hist, tasks, ctl, part, pass, total;
};

MsbLayout msb_layout(int64_t n, bool vals) {
    MsbLayout L{};
    L.max_big = n / (kLocalMax + 1) > 1 ? n / (kLocalMax + 1) : 1;
    // a big segment of up to kChunk = 2 kLocalMax pairs is one chunk, a longer
    // one at most len / kLocalMax: no more than n / kLocalMax chunks
    L.max_chunks = n / kCopy + L.max_big + 1;
    // tasks, per level with a digit left below it: one per sub-segment of
    // kSmallSeg pairs or more (at most n / kSmallSeg), and groups of shorter
    // ones; a group closes above kLocalMax - kSmallSeg pairs, before a longer
    // or a big sub-segment, or at its parent's end, so there are at most
    // n / (kLocalMax - kSmallSeg) + n / kSmallSeg + (big segments of this and
    // the next level) of them.  Then the last level's copies (pieces of at
    // most kCopy pairs of the big segments).
    L.max_tasks = 3 * (2 * (n / kSmallSeg) + n / (kLocalMax - kSmallSeg) + 2 * L.max_big + 2) + n / kCopy +
                  L.max_big + 8;
    int64_t at = 0;
    L.tmp_k = at;
    at += r256(n * 4);
    L.tmp_v = at;
    at += vals ? r256(n * 4) : 0;
    L.big0 = at;
    at += r256(L.max_big * (int64_t)sizeof(Seg));
    L.big1 = at;
    at += r256(L.max_big * (int64_t)sizeof(Seg));
    L.chunks = at;
    at += r256(L.max_chunks * (int64_t)sizeof(ChunkD));
    L.hist = at;
    at += r256(L.max_chunks * kBins * 4);
    L.tasks = at;  // two lists of max_tasks entries
    at += r256(2 * L.max_tasks * (int64_t)sizeof(Task));
    L.ctl = at;
    at += 256;
    L.part = at;
    at += r256((kBins + 1) * 4);
    L.pass = at;
    at += r256(radix_pass_min_scratch_bytes(radix_long_cfg(n), n));
    L.total = at;
    return L;
}

template <bool VALS>
hipError_t msb_run(const uint32_t *keys, const uint32_t *vals, int64_t n, uint32_t *ok, uint32_t *ov, void *scratch,
                   hipStream_t s) {
    const MsbLayout L = msb_layout(n, VALS);
    char *base = (char *)scratch;
    uint32_t *tk = (uint32_t *)(base + L.tmp_k);
    uint32_t *tv = VALS ? (uint32_t *)(base + L.tmp_v) : nullptr;
    Seg *big[2] = {(Seg *)(base + L.big0), (Seg *)(base + L.big1)};
    ChunkD *chunks = (ChunkD *)(base + L.chunks);
    uint32_t *hist = (uint32_t *)(base + L.hist);
    Task *tasks = (Task *)(base + L.tasks);
    Ctl *ctl = (Ctl *)(base + L.ctl);

    const uint32_t stride = (uint32_t)L.max_tasks;
    auto large = msb_local_kernel<VALS, kLocBlock, kLocIpt>;
    auto small = msb_local_kernel<VALS, kSmlBlock, kSmlIpt>;
    const size_t large_lds = RadixTile<kLocBlock, kLocIpt>::BYTES, small_lds = RadixTile<kSmlBlock, kSmlIpt>::BYTES;
    const size_t shuffle_lds = RadixTile<kPartBlock, kPartIpt>::BYTES;
    static bool attrs = false;
    if (!attrs) {
        hipError_t e = hipFuncSetAttribute((const void *)msb_shuffle_kernel<VALS>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)shuffle_lds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)large, hipFuncAttributeMaxDynamicSharedMemorySize, (int)large_lds);
        if (e != hipSuccess) return e;
        attrs = true;
    }
    const int64_t cus = device_cu_count();
    int64_t part_per_cu = 0, large_per_cu = 0, small_per_cu = 0;
    hipError_t e = resident_per_cu((const void *)msb_shuffle_kernel<VALS>, kPartBlock, (int64_t)shuffle_lds,
                                   part_per_cu);
    if (e == hipSuccess) e = resident_per_cu((const void *)large, kLocBlock, (int64_t)large_lds, large_per_cu);
    if (e == hipSuccess) e = resident_per_cu((const void *)small, kSmlBlock, (int64_t)small_lds, small_per_cu);
    if (e != hipSuccess) return e;
    if (part_per_cu < 1) part_per_cu = 1;
    if (large_per_cu < 1) large_per_cu = 1;
    if (small_per_cu < 1) small_per_cu = 1;
    const dim3 aux_grid((unsigned)(cus * 8)), aux(kAuxBlock);
    auto local_sorts = [&](int64_t large_grid, int64_t small_grid) {
        hipLaunchKernelGGL(small, dim3((unsigned)small_grid), dim3(kSmlBlock), small_lds, s, ctl, 0, tasks, keys,
                           vals, ok, ov, tk, tv);
        hipLaunchKernelGGL(large, dim3((unsigned)large_grid), dim3(kLocBlock), large_lds, s, ctl, 1,
                           tasks + stride, keys, vals, ok, ov, tk, tv);
        return hipGetLastError();
    };

    // level 0: the whole input is one segment, so the plain stable partition
    // pass on the top byte does it (input -> output), and its partition
    // offsets give the first level's sub-segments
    const int64_t hist_bytes = L.max_chunks * kBins * 4;
    const LaunchCfg rcfg = radix_cfg(n, VALS, hist_bytes);
    // its counts go where the later levels' will be, if they fit there
    const bool in_hist = hist_bytes >= radix_pass_scratch_bytes(rcfg, n);
    e = launch_radix_partition(rcfg, keys, vals, n, 24, 8, ok, ov, (uint32_t *)(base + L.part),
                               in_hist ? base + L.hist : base + L.pass, in_hist ? hist_bytes : L.total - L.pass, true,
                               s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(msb_level0_kernel, dim3(1), dim3(kAuxBlock), 0, s, ctl, (const uint32_t *)(base + L.part),
                       (uint32_t)n, big[1], tasks, stride);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int level = 1; level < 4; ++level) {
        const int shift = 24 - 8 * level, cur = level & 1;
        const uint32_t *sk = (level & 1) ? ok : tk;
        const uint32_t *sv = (level & 1) ? ov : tv;
        uint32_t *dk = (level & 1) ? tk : ok;
        uint32_t *dv = (level & 1) ? tv : ov;
        const uint32_t dst = (level & 1) ? 2u : 1u;
        hipLaunchKernelGGL(msb_chunk_scan_kernel, dim3(1), dim3(1024), 0, s, ctl, big[cur], cur);
        hipLaunchKernelGGL(msb_chunk_fill_kernel, aux_grid, aux, 0, s, ctl, big[cur], cur, chunks);
        hipLaunchKernelGGL(msb_hist_kernel, aux_grid, aux, 0, s, ctl, chunks, sk, shift, hist);
        hipLaunchKernelGGL(msb_scan_kernel, aux_grid, aux, 0, s, ctl, big[cur], cur, hist, big[cur ^ 1], tasks,
                           stride, shift, dst);
        hipLaunchKernelGGL(msb_shuffle_kernel<VALS>, dim3((unsigned)((cus * part_per_cu + 7) / 8 * 8)), dim3(kPartBlock),
                           shuffle_lds, s, ctl, chunks, hist, sk, sv, dk, dv, shift);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return local_sorts(cus * large_per_cu, cus * small_per_cu);
}

}  // namespace

hipError_t launch_sort_short(const uint32_t *keys, const uint32_t *vals, int64_t n, uint32_t *out_keys,
                             uint32_t *out_vals, hipStream_t s) {
    static_assert(kSortShortMax == 1024 * 8, "the larger shape holds every short input");
    return vals ? sort_short<true>(keys, vals, (int)n, out_keys, out_vals, s)
                : sort_short<false>(keys, nullptr, (int)n, out_keys, nullptr, s);
}

int64_t msb_sort_scratch_bytes(int64_t n, bool with_values) { return msb_layout(n, with_values).total; }

hipError_t launch_msb_sort(const uint32_t *keys, const uint32_t *vals, int64_t n, uint32_t *out_keys,
                           uint32_t *out_vals, void *scratch, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    return vals ? msb_run<true>(keys, vals, n, out_keys, out_vals, scratch, s)
                : msb_run<false>(keys, nullptr, n, out_keys, nullptr, scratch, s);
}

}  // namespace crystal
