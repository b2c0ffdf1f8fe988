// Neighbour sampling of one block on the device (the uniform fan-out sampling of Section 7.1, which the paper runs on
// CPU threads, Section 5): from the nodes of layer l to the block (start, end, columns) and the node list of layer l-1,
// over an in-neighbour CSR held in device-visible memory.
//
// Per node v with degree d and fan-out f: slots 0..d-1 when d <= f; otherwise the row is cut into f disjoint strata
// with integer bounds, stratum j = [floor(j d / f), floor((j + 1) d / f)), draw j takes the slot at offset
// floor(u_j * width_j) of stratum j, and the f slots are moved round the row by a common offset floor(u_f * d) modulo d
// (f distinct slots, every slot of the row with probability f / d); u_j from the counter-based SplitMix64 generator
// keyed by (mini-batch key, layer, v, j); the neighbours at those slots in the order of j, without v and without repeats. The layer
// below is the layer's own nodes followed by the new neighbours in order of first occurrence; columns are positions in
// that list. Everything is a pure function of the inputs: no atomics decide an order, so the result is the same in
// every run.
//
// Launches of one block (sizes from the host-side bound max_rows, the exact count is read on the device):
//   1. draw      a thread per slot of a row: neighbour, repeats removed by comparing within the row. The layer's own nodes go to
//                the head of the list below and enter the hash table with their position, the neighbour at slot k of all rows
//                with the order number max_rows + k; the table keeps the smallest per node, and who is not the smallest any more
//                is marked
//   2. resolve   per slot: a first occurrence, or (marked, one in six as a rule) the order number its entry ended up with; first
//                occurrences are ranked within their workgroup, they and the neighbours kept are counted
//   3. columns   every workgroup adds up the others' counts for itself: rows back to back, columns in row order, first
//                occurrences appended to the list below; every kept neighbour gets the position of its node in that list
// What a block needs clear is cleared for all blocks of a mini-batch by its first launch, and the transpose of a block (below)
// rides in the launches of the next one, on which it does not depend.
// What bounds a large block: every neighbour costs one atomic on the table, and the card takes 27 of those a nanosecond
// whatever their form and the table's size (760 k compare-and-swaps, minima or additions of 32 or 64 bits, with or without
// their result, on 2 to 32 MB: 28 us; plain stores 9, loads 5 to 12). They run beside the draw's own reads, and what a
// colliding neighbour does next counts as much (see smp_insert). 55 k rows x 15 of a graph of 28 M nodes: 80 us in four launches
// (draw 18, insertion 38, lookup 17, columns 7), now 61 (41, 9, 11); a mini-batch of 1024 x 5 x 10 x 15 with its transposes, asked
// for and waited for: 204 us, now 154.
#include "common.h"
#include "scan.h"
#include "stage_queue.h"

namespace {

constexpr int SMP_THREADS = 1024;
constexpr int SMP_LANES = 32;                           // the largest fan-out
constexpr int SMP_PREFIX = 8192;                        // workgroups of candidates whose counts a workgroup adds up for itself
constexpr unsigned long long SMP_EMPTY = ~0ull;
constexpr uint32_t SMP_LINE = 8;                        // entries of the table that are probed together
constexpr uint32_t SMP_LOST = 0x80000000u;              // in `entry`: the slot's node was there with a smaller number
constexpr int SMP_DRAW_THREADS = 256;                   // small workgroups: one that has finished makes room at once

__host__ __device__ inline uint64_t smp_mix(uint64_t x) {
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
__host__ __device__ inline uint64_t smp_word(uint64_t key, uint64_t counter) {
    return smp_mix(key + (counter + 1ull) * 0x9E3779B97F4A7C15ull);
}

struct SmpArgs {
    const int64_t* indptr;
    const int32_t* indices;
    int64_t num_nodes, num_edges;
    const int32_t* ids;
    const int64_t* n_dev;
    int64_t max_rows;
    int32_t fanout;
    int32_t rows_per;     // rows of a workgroup of launches 2 and 3: as many as it has slots for
    int32_t draw_blocks;  // workgroups of launch 1 that draw, then those that enter the layer's own nodes; the others clear
    int32_t own_blocks;
    uint64_t key_l;
    int32_t* row_start;
    int32_t* row_end;
    int32_t* col;
    int32_t* col_ids;     // NULL: the caller wants no ids
    int32_t* below;
    int64_t max_below;
    int64_t* counts;      // [0] nodes of the layer below, [1] edges
    int32_t* nbuf;        // [max_rows * fanout] neighbour of a slot, -1 = none
    uint32_t* entry;      // [max_rows * fanout] its entry of the table (SMP_LOST), then the smallest order number found there
    uint8_t* lost;        // [max_rows * fanout] the slot was the smallest of its node and is not any more; zero before
    uint16_t* rank;       // [max_rows * fanout] rank among the first occurrences of its workgroup
    int32_t* blk_new;     // first occurrences per workgroup
    int32_t* blk_kept;    // neighbours kept per workgroup
    int32_t* new_first;   // [+1] first occurrences and kept neighbours before each workgroup (only where there are more
    int32_t* kept_first;  //      than SMP_PREFIX)
    unsigned long long* table;
    uint32_t mask;        // table entries - 1 (a power of two)
    int shift;            // 32 - log2(entries)
    int32_t* tr_cnt;      // [max_below] edges per source of the block's transpose, zero before; NULL: no transpose
};

__device__ __forceinline__ int64_t smp_rows(const SmpArgs& A) {
    int64_t n = A.n_dev ? *A.n_dev : A.max_rows;
    if (n < 0) n = 0;
    return n < A.max_rows ? n : A.max_rows;
}

__device__ __forceinline__ uint32_t smp_hash(const SmpArgs& A, int32_t node) { return ((uint32_t)node * 0x9E3779B1u) >> A.shift; }

// Whoever brings a node's order number down marks the slot that had the smallest one before (not one of the layer's own nodes,
// whose numbers are below all slots': a layer that names a node twice).
__device__ __forceinline__ bool smp_lower(const SmpArgs& A, uint32_t at, unsigned long long mine) {
    const unsigned long long before = atomicMin(&A.table[at], mine);
    if (before < mine) return false;
    if ((uint32_t)before >= (uint32_t)A.max_rows) A.lost[(uint32_t)before - (uint32_t)A.max_rows] = 1;
    return true;
}

// Keeps the smallest order number seen for `node`, distinct for every call; returns the entry that holds it, with SMP_LOST if a
// smaller number was there already. An entry's node never changes once it is set. The home entry is tried without looking, most
// nodes' case. A node that finds another one there takes the first entry of the home entry's line, cyclically from there
// on, that is its own or empty, then of the lines that follow; a line is read at once (a stale read can only show an entry
// as empty that no longer is). Walking on entry by entry was a chain of two trips to memory for each, and the wavefront waits
// for its longest: 6 k rows x 10 20 us, now 9, 54 k x 15 47, now 40.
__device__ __forceinline__ uint32_t smp_insert(const SmpArgs& A, int32_t node, uint32_t order) {
    const unsigned long long mine = ((unsigned long long)(uint32_t)node << 32) | order;
    const uint32_t home = smp_hash(A, node), from = home & (SMP_LINE - 1);
    uint32_t line = home - from;
    unsigned long long cur = atomicCAS(&A.table[home], SMP_EMPTY, mine);
    if (cur == SMP_EMPTY) return home;
    if ((uint32_t)(cur >> 32) == (uint32_t)node) return cur > mine && smp_lower(A, home, mine) ? home : home | SMP_LOST;
    for (uint32_t probed = 0; probed <= A.mask; probed += SMP_LINE) {
        uint32_t own = 0, empty = 0;      // a bit per entry, the home entry's place first
#pragma unroll
        for (uint32_t q = 0; q < SMP_LINE / 2; ++q) {
            const ulonglong2 e = ((const ulonglong2*)(A.table + line))[q];
            const unsigned long long v[2] = {e.x, e.y};
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) {
                const uint32_t bit = 1u << ((2 * q + u - from) & (SMP_LINE - 1));
                if ((uint32_t)(v[u] >> 32) == (uint32_t)node) own |= bit;
                if (v[u] == SMP_EMPTY) empty |= bit;
            }
        }
        for (uint32_t open = own | empty; open; open &= open - 1) {
            const uint32_t place = (uint32_t)__ffs((int)open) - 1, at = line + ((place + from) & (SMP_LINE - 1));
            if ((empty >> place) & 1u) {
                cur = atomicCAS(&A.table[at], SMP_EMPTY, mine);
                if (cur == SMP_EMPTY) return at;
                if ((uint32_t)(cur >> 32) != (uint32_t)node) continue;
            }
            return smp_lower(A, at, mine) ? at : at | SMP_LOST;
        }
        line = (line + SMP_LINE) & A.mask;
    }
    return SMP_LOST;      // not reached: the table has more entries than a block has nodes
}

// Where in a row of d entries the draws of node v start: the common turn of its strata and the word its draws are derived from.
__device__ __forceinline__ void smp_row(const SmpArgs& A, int32_t v, int64_t d, uint64_t& word, int64_t& turn) {
    word = smp_word(A.key_l, (uint64_t)v);
    const double u = (double)(smp_word(word, (uint64_t)A.fanout) >> 11) * (1.0 / 9007199254740992.0);
    turn = (int64_t)(u * (double)d);
    if (turn > d - 1) turn = d - 1;
}

// Draw j of node v, whose row is [lo, lo + d): the neighbour, or -1 where there is none (a self loop counts as none).
__device__ __forceinline__ int32_t smp_draw(const SmpArgs& A, int32_t v, int64_t lo, int64_t d, uint64_t word, int64_t turn, int j) {
    const int f = A.fanout;
    if (j >= f || j >= d) return -1;
    int64_t slot = j;
    if (d > f) {
        const double u = (double)(smp_word(word, (uint64_t)j) >> 11) * (1.0 / 9007199254740992.0);
        if (d < (1 << 26)) {      // in 32 bits: (j + 1) * d is below 2^31
            const uint32_t a = (uint32_t)j * (uint32_t)d, first = a / (uint32_t)f, width = (a + (uint32_t)d) / (uint32_t)f - first;
            uint32_t inside = (uint32_t)(u * (double)width);
            if (inside > width - 1) inside = width - 1;
            uint32_t at = first + inside + (uint32_t)turn;      // first + inside and turn are both below d
            if (at >= (uint32_t)d) at -= (uint32_t)d;
            slot = at;
        } else {
            const int64_t first = ((int64_t)j * d) / f, width = ((int64_t)(j + 1) * d) / f - first;
            int64_t inside = (int64_t)(u * (double)width);
            if (inside > width - 1) inside = width - 1;
            slot = first + inside + turn;
            if (slot >= d) slot -= d;
        }
    }
    const int64_t at = lo + slot;
    if (at < 0 || at >= A.num_edges) return -1;
    const int32_t nb = A.indices[at];
    return nb != v && nb >= 0 && nb < A.num_nodes ? nb : -1;
}

// Exclusive prefix sums of v[0 .. n) into out[0 .. n) (may be v itself), by one workgroup of FG_SCAN_BLOCK threads; returns the total.
__device__ __forceinline__ int smp_prefix(const int32_t* v, int n, int32_t* out) {
    __shared__ int wave_sum[FG_SCAN_BLOCK / FG_WAVE];
    const int per = (n + FG_SCAN_BLOCK - 1) / FG_SCAN_BLOCK;      // consecutive entries per thread
    const int b = threadIdx.x * per, e = b + per < n ? b + per : n;
    int mine = 0;
    for (int q = b; q < e; ++q) mine += v[q];
    int incl = mine;
    for (int off = 1; off < FG_WAVE; off <<= 1) {
        const int up = __shfl_up(incl, off, FG_WAVE);
        if (fg_lane() >= off) incl += up;
    }
    if (fg_lane() == FG_WAVE - 1) wave_sum[fg_wave()] = incl;
    __syncthreads();
    int earlier = 0, all = 0;
    for (int w = 0; w < FG_SCAN_BLOCK / FG_WAVE; ++w) {
        if (w < fg_wave()) earlier += wave_sum[w];
        all += wave_sum[w];
    }
    int at = earlier + incl - mine;
    for (int q = b; q < e; ++q) {
        const int here = v[q];
        out[q] = at;
        at += here;
    }
    __syncthreads();
    return all;
}

// ---- transpose of a sampled block (what the backward pass walks) ---------------------------------------------------
//
// For every position j of the layer below: the rows that sampled it, ascending, back to back. Stages: count the edges per
// source (a sampled block's last launch does it in passing); exclusive scan (t_start, t_end; a workgroup adds up the counters
// before its own itself, or per-workgroup sums of a stage of their own where there are many); every edge takes a free place
// of its source's list (the order of arrival is arbitrary); every list is sorted (by its length, see tr_sort_lists: a source is sampled by a
// handful of rows; a hub by many), which makes the result independent of that order. Rows are read by groups of lanes: one lane per row
// walked a chain of dependent atomics on a few compute units.
// The stages of a block that was just sampled ride in the launches of the next one (a few dozen workgroups in front of them, which
// leave the chip to it): five launches and 24 us less for 6 k rows x 10 and 54 k sources. By themselves they are a launch each.
constexpr int TR_THREADS = 1024;     // by themselves; a riding stage has workgroups of the size of its launch
constexpr int TR_LANES = 8;          // lanes per row
constexpr int64_t TR_DIRECT = 131072;      // counters up to which a workgroup of the scan adds up those before its own

struct TrArgs {
    const int32_t* row_start;
    const int32_t* row_end;
    const int32_t* col;
    const int64_t* n_dev;
    int64_t max_rows;
    const int64_t* n_src_dev;
    int64_t max_src;
    int64_t max_nnz;
    int32_t* t_start;
    int32_t* t_end;
    int32_t* t_row;
    int32_t* cnt;   // [max_src] edges per source, then the places of its list that are still free
    int32_t* blk;   // per workgroup of the scan
};

enum TrStage { TR_COUNT, TR_SUM, TR_SCAN, TR_SCAN_SUMS, TR_FILL, TR_SORT };
constexpr int TR_MAX_RIDES = 2;

// stages that share a launch with something else: `blocks` workgroups in front of its own, those of ride i up to end[i]
struct TrRides {
    int32_t n, blocks;
    int32_t stage[TR_MAX_RIDES], end[TR_MAX_RIDES];
    TrArgs a[TR_MAX_RIDES];
};

__device__ __forceinline__ int64_t tr_count(const int64_t* dev, int64_t bound) {
    int64_t n = dev ? *dev : bound;
    if (n < 0) n = 0;
    return n < bound ? n : bound;
}

// f(row, source) for every edge of row `i` that names a valid source; the TR_LANES lanes of the row share its edges
template <typename F>
__device__ __forceinline__ void tr_row_edges(const TrArgs& A, int64_t i, int64_t n_src, F f) {
    int64_t b = A.row_start[i], e = A.row_end[i];
    if (b < 0) b = 0;
    if (e > A.max_nnz) e = A.max_nnz;
    for (int64_t k = b + threadIdx.x % TR_LANES; k < e; k += TR_LANES) {
        const int32_t c = A.col[k];
        if (c >= 0 && c < n_src) f((int32_t)i, c);
    }
}

__device__ __forceinline__ void tr_sort(int32_t* list, int64_t b, int64_t e) {  // insertion sort
    for (int64_t k = b + 1; k < e; ++k) {
        const int32_t v = list[k];
        int64_t q = k;
        while (q > b && list[q - 1] > v) {
            list[q] = list[q - 1];
            --q;
        }
        list[q] = v;
    }
}

// Sorts one list of rows per thread, list[b .. e), in place; every thread of the workgroup calls it, b >= e: none. Most sources have a few rows,
// but a hub of a graph with skewed degrees has one for every other row of the block, and a thread that sorts such a list
// by insertion takes n^2 / 4 dependent steps through memory while the launch waits for it. So by length:
//   up to 8 (TR_SHORT)   a thread, in registers: one round of loads, a network of 19 exchanges
//   up to 64             a wavefront, an entry per lane: its place is the number of entries below it
//   more                 a set of rows in LDS, a bit per row, read out in order: by a wavefront for blocks of up to 8192 rows (TR_WORDS),
//                        by the workgroup for up to 128 rows per thread; beyond that, and where a row names a source twice, by insertion
// The longer lists are handed out to the workgroup's wavefronts by a queue. Mini-batches with transposes, the whole call, before and now:
// 988 seeds x 8 x 9 of a graph of 11 k nodes 323 -> 84 us, 598 x 5 x 6 x 9 of 161 k nodes 415 -> 111; 1024 x 5 x 10 x 15 of 28 M nodes, whose lists
// are short, 153 both ways.
constexpr int TR_SHORT = 8, TR_WORDS = 256;
template <int THREADS>
__device__ __forceinline__ void tr_sort_lists(int32_t* list, int64_t b, int64_t e, int64_t max_rows) {
    __shared__ __attribute__((aligned(16))) uint32_t s_rows[THREADS / FG_WAVE * TR_WORDS];
    __shared__ int2 s_queue[THREADS];      // first entry and length
    __shared__ int s_queued, s_odd, s_sum[THREADS / FG_WAVE];
    constexpr int WAVES = THREADS / FG_WAVE, GROUP_WORDS = WAVES * TR_WORDS / THREADS;      // per thread
    static_assert(GROUP_WORDS == 4, "a thread's words are read as one");
    const int t = (int)threadIdx.x, lane = fg_lane(), wave = fg_wave();
    const int n = e > b ? (int)(e - b) : 0;
    const bool by_wave = max_rows <= TR_WORDS * 32, by_group = !by_wave && max_rows <= THREADS * GROUP_WORDS * 32;
    __syncthreads();      // an earlier call's queue is read
    if (t == 0) s_queued = 0;
    __syncthreads();
    if (n > TR_SHORT) {
        if (n <= FG_WAVE || by_wave || by_group)
            s_queue[atomicAdd(&s_queued, 1)] = int2{(int)b, n};
        else
            tr_sort(list, b, e);
    } else if (n > 1) {
        int32_t v[TR_SHORT];
#pragma unroll
        for (int i = 0; i < TR_SHORT; ++i) v[i] = i < n ? list[b + i] : INT32_MAX;
        auto order = [&](int i, int k) {
            const int32_t lo = v[i] < v[k] ? v[i] : v[k];
            v[k] = v[i] < v[k] ? v[k] : v[i];
            v[i] = lo;
        };
        order(0, 1), order(2, 3), order(4, 5), order(6, 7);
        order(0, 2), order(1, 3), order(4, 6), order(5, 7);
        order(1, 2), order(5, 6);
        order(0, 4), order(1, 5), order(2, 6), order(3, 7);
        order(2, 4), order(3, 5);
        order(1, 2), order(3, 4), order(5, 6);
#pragma unroll
        for (int i = 0; i < TR_SHORT; ++i)
            if (i < n) list[b + i] = v[i];
    }
    __syncthreads();
    const int queued = s_queued;
    // Sets the bits of the list's entries; false: an entry is there twice or is no row of the block
    auto set_bits = [&](uint32_t* rows, int first, int len, int from, int step) {
        bool fine = true;
        for (int i = from; i < len; i += step) {
            const uint32_t r = (uint32_t)list[first + i];
            if ((int64_t)r >= max_rows)
                fine = false;
            else
                fine = fine && !((atomicOr(&rows[r >> 5], 1u << (r & 31u)) >> (r & 31u)) & 1u);
        }
        return fine;
    };
    uint32_t* mine = s_rows + wave * TR_WORDS;
    int2 next = wave < queued ? s_queue[wave] : int2{0, 0};
    int32_t next_v = lane < next.y ? list[next.x + lane] : 0;
    for (int q = wave; q < queued; q += WAVES) {      // uniform over the wavefront
        const int first = __builtin_amdgcn_readfirstlane(next.x), len = __builtin_amdgcn_readfirstlane(next.y);
        const int32_t v = next_v;
        next = q + WAVES < queued ? s_queue[q + WAVES] : int2{0, 0};      // the next list's first entries are on their way meanwhile
        next_v = lane < next.y ? list[next.x + lane] : 0;
        if (len <= FG_WAVE) {
            int below = 0;
            for (int i = 0; i < len; ++i) {
                const int32_t x = __builtin_amdgcn_readlane(v, i);
                below += x < v || (x == v && i < lane) ? 1 : 0;
            }
            if (lane < len) list[first + below] = v;
        } else if (by_wave) {
            const int words = (int)((max_rows + 31) >> 5);
            for (int w = lane; w < words; w += FG_WAVE) mine[w] = 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const bool fine = __all(set_bits(mine, first, len, lane, FG_WAVE));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (!fine) {
                if (lane == 0) tr_sort(list, first, (int64_t)first + len);
                continue;
            }
            int at = first;
            for (int w0 = 0; w0 < words; w0 += FG_WAVE) {
                uint32_t bits = w0 + lane < words ? mine[w0 + lane] : 0u;
                const int here = __popc(bits), incl = fg_wave_scan(here);
                int to = at + incl - here;
                for (; bits; bits &= bits - 1) list[to++] = 32 * (w0 + lane) + __ffs((int)bits) - 1;
                at += __builtin_amdgcn_readlane(incl, FG_WAVE - 1);
            }
        }
    }
    if (!by_group) return;      // uniform over the workgroup
    for (int q = 0; q < queued; ++q) {
        const int first = s_queue[q].x, len = s_queue[q].y;
        if (len <= FG_WAVE) continue;
        __syncthreads();      // the bits and sums of the list before are read
        if (t == 0) s_odd = 0;
        ((uint4*)s_rows)[t] = uint4{0, 0, 0, 0};
        __syncthreads();
        if (!set_bits(s_rows, first, len, t, THREADS)) s_odd = 1;
        __syncthreads();
        if (s_odd) {
            if (t == 0) tr_sort(list, first, (int64_t)first + len);
            continue;
        }
        const uint4 set = ((const uint4*)s_rows)[t];
        const uint32_t word[4] = {set.x, set.y, set.z, set.w};
        const int here = __popc(set.x) + __popc(set.y) + __popc(set.z) + __popc(set.w), incl = fg_wave_scan(here);
        if (lane == FG_WAVE - 1) s_sum[wave] = incl;
        __syncthreads();
        int to = first + incl - here;
        for (int w = 0; w < wave; ++w) to += s_sum[w];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (uint32_t bits = word[u]; bits; bits &= bits - 1) list[to++] = 32 * (4 * t + u) + __ffs((int)bits) - 1;
    }
}

// exclusive scan of one value per thread over the workgroup; `total`: their sum
__device__ __forceinline__ int tr_block_scan(int c, int& total) {
    __shared__ int wave_sum[TR_THREADS / FG_WAVE];
    int incl = c;  // inclusive scan over the wavefront, then the wavefronts before this one
    for (int off = 1; off < FG_WAVE; off <<= 1) {
        const int v = __shfl_up(incl, off, FG_WAVE);
        if (fg_lane() >= off) incl += v;
    }
    if (fg_lane() == FG_WAVE - 1) wave_sum[fg_wave()] = incl;
    __syncthreads();
    int earlier = 0;
    total = 0;
    for (int w = 0; w < (int)blockDim.x / FG_WAVE; ++w) {
        if (w < fg_wave()) earlier += wave_sum[w];
        total += wave_sum[w];
    }
    return earlier + incl - c;
}

// one workgroup, of THREADS threads, of a stage
template <int THREADS>
__device__ __forceinline__ void tr_stage(const TrArgs& A, int stage, int block) {
    __shared__ long long red[16];
    constexpr int threads = THREADS;
    const int64_t j = (int64_t)block * threads + threadIdx.x;
    if (stage == TR_COUNT || stage == TR_FILL) {
        const int64_t n = tr_count(A.n_dev, A.max_rows), n_src = tr_count(A.n_src_dev, A.max_src), i = j / TR_LANES;
        if (i >= n) return;
        if (stage == TR_COUNT)
            tr_row_edges(A, i, n_src, [&](int32_t, int32_t c) { atomicAdd(&A.cnt[c], 1); });
        else
            tr_row_edges(A, i, n_src, [&](int32_t row, int32_t c) {
                const int64_t at = (int64_t)A.t_end[c] - atomicSub(&A.cnt[c], 1);      // from the start on: nearly sorted as a rule
                if (at < A.max_nnz) A.t_row[at] = row;
            });
    } else if (stage == TR_SORT) {
        // (sixteen sources in turn to every workgroup: those with long lists are the first ones of the layer below)
        const int64_t blocks = (A.max_src + threads - 1) / threads, s = ((threadIdx.x >> 4) * blocks + block) * 16 + (threadIdx.x & 15);
        int64_t b = 0, e = 0;
        if (s < A.max_src) {
            b = A.t_start[s];
            e = A.t_end[s] < A.max_nnz ? A.t_end[s] : A.max_nnz;
        }
        tr_sort_lists<THREADS>(A.t_row, b, e, A.max_rows);
    } else if (stage == TR_SUM) {
        const int64_t q = (int64_t)block * TR_THREADS + threadIdx.x;      // of TR_THREADS counters in any case
        long long s = 0;
        for (int u = 0; u < TR_THREADS; u += threads) s += q + u < A.max_src ? (long long)A.cnt[q + u] : 0;
        s = fg_block_sum(s, red);
        if (threadIdx.x == 0) A.blk[block] = (int32_t)s;
    } else {
        const int c = j < A.max_src ? A.cnt[j] : 0;
        const int64_t first = (int64_t)block * threads;      // counters ahead of this workgroup's
        long long before = 0;
        if (stage == TR_SCAN_SUMS) {      // whole blocks of TR_THREADS by their sums
            for (int64_t b = threadIdx.x; b < first / TR_THREADS; b += threads) before += A.blk[b];
            for (int64_t b = first / TR_THREADS * TR_THREADS + threadIdx.x; b < first; b += threads) before += A.cnt[b];
        } else {      // `first` is a multiple of 4: sixteen bytes at a time
#pragma unroll 4
            for (int64_t b = threadIdx.x * 4; b < first; b += threads * 4) {
                const int4 v = *(const int4*)(A.cnt + b);
                before += (long long)v.x + v.y + v.z + v.w;
            }
        }
        before = fg_block_sum(before, red);
        int total;
        const long long start = before + tr_block_scan(c, total);
        if (j < A.max_src) {
            A.t_start[j] = (int32_t)start;
            A.t_end[j] = (int32_t)(start + c);
        }
    }
}

// Whether this workgroup belongs to a riding stage (which it then does); `block`: its number among the launch's own, if not.
template <int THREADS = SMP_THREADS>
__device__ __forceinline__ bool tr_rides(const TrRides& T, int& block, int b = (int)blockIdx.x) {
    static_assert(TR_MAX_RIDES == 2, "two rides are told apart here");
    block = b - T.blocks;
    if (block >= 0) return false;
    const int second = b >= T.end[0] ? 1 : 0;
    tr_stage<THREADS>(T.a[second], T.stage[second], b - (second ? T.end[0] : 0));
    return true;
}

__global__ __launch_bounds__(TR_THREADS) void transpose_stage_kernel(TrRides T) {
    int block;
    tr_rides(T, block);
}

// ---- what a mini-batch's first launch clears: hash tables, and the edge counts of the transposes ---------------------------
constexpr int SMP_MAX_LAYERS = 8;
constexpr int64_t SMP_CLEAR_BYTES = 65536;      // per workgroup
struct SmpClear {
    int32_t n;
    uint32_t value[3 * SMP_MAX_LAYERS];
    char* p[3 * SMP_MAX_LAYERS];
    int64_t bytes[3 * SMP_MAX_LAYERS];      // multiples of 16
    void add(char* at, int64_t size, uint32_t v) {
        p[n] = at;
        bytes[n] = size;
        value[n++] = v;
    }
    int64_t total() const {
        int64_t t = 0;
        for (int i = 0; i < n; ++i) t += bytes[i];
        return t;
    }
};
__device__ __forceinline__ void smp_clear(const SmpClear& C, int block, int n_blocks) {
    for (int i = 0; i < C.n; ++i) {
        const uint4 v = {C.value[i], C.value[i], C.value[i], C.value[i]};
        for (int64_t q = (int64_t)block * blockDim.x + threadIdx.x; q < C.bytes[i] >> 4; q += (int64_t)n_blocks * blockDim.x) ((uint4*)C.p[i])[q] = v;
    }
}
__global__ __launch_bounds__(SMP_THREADS) void sample_clear_kernel(SmpClear C) { smp_clear(C, blockIdx.x, gridDim.x); }

// ---- the launches of one block -------------------------------------------------------------------------------------------
//
// Slot k of a block is draw k % fanout of row k / fanout. A workgroup has the slots of whole rows, consecutive ones to
// consecutive threads, then (SLOTS = 4) the next ones to the same threads again.
struct SmpSlot {
    int j;           // draw of the row
    int64_t row, k;
    bool in;         // a slot of the bound
};
__device__ __forceinline__ SmpSlot smp_slot(const SmpArgs& A, int64_t first_row, int rows, int at) {
    SmpSlot s;
    const int g = at / A.fanout;
    s.j = at - g * A.fanout;
    s.row = first_row + g;
    s.k = s.row * A.fanout + s.j;
    s.in = g < rows && s.row < A.max_rows;
    return s;
}

__global__ __launch_bounds__(SMP_DRAW_THREADS) void sample_draw_kernel(SmpArgs A, TrRides T, SmpClear C) {
    __shared__ int32_t s_nb[SMP_DRAW_THREADS];
    int block;
    if (tr_rides<SMP_DRAW_THREADS>(T, block)) return;
    if (block >= A.draw_blocks + A.own_blocks) {
        const int ahead = A.draw_blocks + A.own_blocks;
        smp_clear(C, block - ahead, (int)gridDim.x - T.blocks - ahead);
        return;
    }
    if (block >= A.draw_blocks) {      // the layer's own nodes
        const int64_t row = (int64_t)(block - A.draw_blocks) * SMP_DRAW_THREADS + threadIdx.x;
        const int32_t v = row < A.max_rows ? A.ids[row] : -1;      // asked for together with the count; an entry past it is read and not used
        if (row >= smp_rows(A)) return;
        if (row < A.max_below) A.below[row] = v;
        if (v >= 0 && v < A.num_nodes) smp_insert(A, v, (uint32_t)row);
        return;
    }
    const int rows = SMP_DRAW_THREADS / A.fanout;
    const SmpSlot s = smp_slot(A, (int64_t)block * rows, rows, threadIdx.x);
    const int32_t v = s.in ? A.ids[s.row] : -1;
    const int64_t n = smp_rows(A);
    if ((int64_t)block * rows >= n) return;      // uniform over the workgroup
    const bool there = s.in && s.row < n, valid = there && v >= 0 && v < A.num_nodes;
    int64_t lo = 0, d = 0;
    if (valid) {
        lo = A.indptr[v];
        d = A.indptr[(int64_t)v + 1] - lo;
    }
    uint64_t word;
    int64_t turn;
    smp_row(A, v, d, word, turn);
    const int32_t nb = valid ? smp_draw(A, v, lo, d, word, turn, s.j) : -1;
    s_nb[threadIdx.x] = nb;
    __syncthreads();
    bool keep = nb >= 0;
    for (int b = 1; b <= s.j; ++b)
        if (s_nb[threadIdx.x - b] == nb) keep = false;
    if (!there) return;
    A.nbuf[s.k] = keep ? nb : -1;
    if (keep) A.entry[s.k] = smp_insert(A, nb, (uint32_t)(A.max_rows + s.k));
}

// Exclusive ranks of SLOTS flags per thread, first all threads' flag 0, then all threads' flag 1 ..; the total.
template <int SLOTS>
__device__ __forceinline__ int smp_ranks(const bool (&flag)[SLOTS], int (&rank)[SLOTS]) {
    constexpr int WAVES = SMP_THREADS / FG_WAVE;
    __shared__ int s_wave[SLOTS * WAVES];
    __syncthreads();      // an earlier call's counts are read
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        int total;
        rank[u] = fg_wave_rank(flag[u], total);
        if (fg_lane() == 0) s_wave[u * WAVES + fg_wave()] = total;
    }
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int u = 0; u < SLOTS; ++u)
        for (int w = 0; w < WAVES; ++w) {
            if (w == fg_wave()) rank[u] += all;
            all += s_wave[u * WAVES + w];
        }
    return all;
}

template <int SLOTS>
__global__ __launch_bounds__(SMP_THREADS) void sample_resolve_kernel(SmpArgs A, TrRides T) {
    int block;
    if (tr_rides(T, block)) return;
    const int64_t n = smp_rows(A);
    if ((int64_t)block * A.rows_per >= n) {      // uniform over the workgroup
        if (threadIdx.x == 0) A.blk_new[block] = A.blk_kept[block] = 0;
        return;
    }
    bool kept[SLOTS], is_first[SLOTS];
    int64_t k[SLOTS];
    uint32_t entry[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const SmpSlot s = smp_slot(A, (int64_t)block * A.rows_per, A.rows_per, u * SMP_THREADS + threadIdx.x);
        const bool there = s.in && s.row < n;
        k[u] = there ? s.k : 0;      // (slot 0 exists)
        kept[u] = A.nbuf[k[u]] >= 0 && there;
        entry[u] = A.entry[k[u]];
        is_first[u] = A.lost[k[u]] == 0;
    }
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        is_first[u] = kept[u] && is_first[u] && !(entry[u] & SMP_LOST);
        if (!kept[u]) continue;
        A.entry[k[u]] = is_first[u] ? (uint32_t)(A.max_rows + k[u]) : (uint32_t)A.table[entry[u] & ~SMP_LOST];
    }
    int rank[SLOTS];
    const int n_new = smp_ranks<SLOTS>(is_first, rank);
#pragma unroll
    for (int u = 0; u < SLOTS; ++u)
        if (is_first[u]) A.rank[k[u]] = (uint16_t)rank[u];
    const int n_kept = smp_ranks<SLOTS>(kept, rank);
    if (threadIdx.x == 0) {
        A.blk_new[block] = n_new;
        A.blk_kept[block] = n_kept;
    }
}

// more workgroups than one of the last launch could add up for itself
__global__ __launch_bounds__(FG_SCAN_BLOCK) void sample_prefix_kernel(SmpArgs A, int blocks) {
    const int all = smp_prefix(A.blk_new, blocks, A.new_first);
    const int kept = smp_prefix(A.blk_kept, blocks, A.kept_first);
    if (threadIdx.x == 0) {
        A.new_first[blocks] = all;
        A.kept_first[blocks] = kept;
    }
}

// OWN: the prefix sums of the workgroups' counts are formed by every workgroup (first occurrences in LDS), else read.
template <int SLOTS, bool OWN>
__global__ __launch_bounds__(SMP_THREADS) void sample_columns_kernel(SmpArgs A, TrRides T) {
    extern __shared__ int s_prefix[];
    __shared__ int s_kept[SLOTS * SMP_THREADS + 1];      // neighbours kept by the slots before each
    __shared__ long long red[16];
    int block;
    if (tr_rides(T, block)) return;
    const int64_t n = smp_rows(A);
    bool kept[SLOTS];
    int32_t nb[SLOTS];
    uint32_t m[SLOTS], k[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const SmpSlot s = smp_slot(A, (int64_t)block * A.rows_per, A.rows_per, u * SMP_THREADS + threadIdx.x);
        const bool there = s.in && s.row < n;
        k[u] = there ? (uint32_t)s.k : 0u;
        nb[u] = A.nbuf[k[u]];
        m[u] = A.entry[k[u]];
        kept[u] = there && nb[u] >= 0;
    }
    const int used = (int)((n + A.rows_per - 1) / A.rows_per), last = (int)gridDim.x - T.blocks - 1;
    int all;
    long long before;
    if constexpr (OWN) {
        long long mine = 0;
        for (int b = threadIdx.x; b < used && b < block; b += SMP_THREADS) mine += A.blk_kept[b];
        before = fg_block_sum(mine, red);
        all = smp_prefix(A.blk_new, used, s_prefix);
    } else {
        all = A.new_first[last + 1];
        before = A.kept_first[block];
    }
    const int* prefix = OWN ? s_prefix : A.new_first;
    int rank[SLOTS];
    const int total = smp_ranks<SLOTS>(kept, rank);
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) s_kept[u * SMP_THREADS + threadIdx.x] = rank[u];
    if (threadIdx.x == 0) s_kept[SLOTS * SMP_THREADS] = total;
    __syncthreads();
    for (int g = threadIdx.x; g < A.rows_per; g += SMP_THREADS) {
        const int64_t row = (int64_t)block * A.rows_per + g;
        if (row >= A.max_rows) break;
        A.row_start[row] = (int32_t)(before + s_kept[g * A.fanout]);
        A.row_end[row] = (int32_t)(before + s_kept[(g + 1) * A.fanout]);
    }
    if (threadIdx.x == 0) {
        if (block == 0) A.counts[0] = n + all;
        if (block == last) A.counts[1] = before + total;
    }
    int64_t at[SLOTS];
    bool is_first[SLOTS];
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        at[u] = m[u];      // one of the layer's own nodes, or the slot of the first occurrence of this neighbour
        const uint32_t q = m[u] - (uint32_t)A.max_rows;
        const bool own_node = m[u] < (uint32_t)A.max_rows;
        is_first[u] = kept[u] && q == k[u];
        if (kept[u] && !own_node) at[u] = n + prefix[q / (uint32_t)(A.rows_per * A.fanout)] + A.rank[q];
    }
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        if (!kept[u]) continue;
        A.col[before + rank[u]] = (int32_t)at[u];
        if (A.col_ids) A.col_ids[before + rank[u]] = nb[u];
        if (is_first[u] && at[u] < A.max_below) A.below[at[u]] = nb[u];
        if (A.tr_cnt && at[u] < A.max_below) atomicAdd(&A.tr_cnt[at[u]], 1);
    }
}

// A layer of few draws (the seeds) in one workgroup and one launch: the candidates, the table
// (order numbers only: the node of an order number is in LDS too) and the ranks stay in LDS. Reads from memory are three
// rounds: ids, row ranges, neighbours. One compute unit does all the arithmetic, so what belongs to a row is computed once
// per row and no lane is left idle beside a row's draws. Whole mini-batches of two blocks with their transpose, graph of 2 M nodes, the
// first block so / in three launches behind one that clears, us: 256 seeds x 5 40 / 47, 400 x 5 42 / 50, 700 x 5 45 / 50, 512 x 8
// 48 / 51, 1024 x 5 55 / 52, both blocks 64 x 10 and 704 x 10 54 / 49: up to 4096 draws.
constexpr int SMP_SMALL_ROWS = 1024, SMP_SMALL_FANOUT = 11, SMP_SMALL_DRAWS = 4096;
constexpr int SMP_SMALL_ITEMS = SMP_SMALL_ROWS + SMP_SMALL_DRAWS;      // own nodes and candidates
constexpr int SMP_SMALL_TABLE = 16384;
constexpr size_t SMP_SMALL_ROW_BYTES = 36;                             // what a row keeps while its neighbours are drawn
constexpr size_t SMP_SMALL_NODES = SMP_SMALL_ITEMS * 4 > SMP_SMALL_ROWS * SMP_SMALL_ROW_BYTES ? SMP_SMALL_ITEMS * 4 : SMP_SMALL_ROWS * SMP_SMALL_ROW_BYTES;
constexpr size_t SMP_SMALL_LDS = (size_t)SMP_SMALL_TABLE * 4 + SMP_SMALL_NODES + SMP_SMALL_ITEMS * 2;

__global__ __launch_bounds__(SMP_THREADS) void sample_small_kernel(SmpArgs A, TrRides T, SmpClear C) {
    extern __shared__ __attribute__((aligned(16))) int smem[];
    if (blockIdx.x > 0) {      // beside the one workgroup that samples: riding stages, and what the later launches find clear
        int block;
        if (!tr_rides(T, block, (int)blockIdx.x - 1)) smp_clear(C, block, (int)gridDim.x - 1 - T.blocks);
        return;
    }
    __shared__ int wave_sum[SMP_THREADS / FG_WAVE];
    int* table = smem;                                             // order number of the first item with the node
    int* nodes = table + SMP_SMALL_TABLE;                          // node of an order number
    unsigned short* found = (unsigned short*)((char*)nodes + SMP_SMALL_NODES);
    // before they are needed their space holds what the draws read and write: per row the range, the derived word and turn
    uint64_t* r_word = (uint64_t*)nodes;                           // [1024]
    int64_t* r_lo = (int64_t*)(r_word + SMP_SMALL_ROWS);
    int64_t* r_deg = r_lo + SMP_SMALL_ROWS;
    int64_t* r_turn = r_deg + SMP_SMALL_ROWS;
    int32_t* r_node = (int32_t*)(r_turn + SMP_SMALL_ROWS);
    int32_t* raw = table;                                          // [SMP_SMALL_DRAWS]
    static_assert(SMP_SMALL_DRAWS <= SMP_SMALL_TABLE && SMP_SMALL_ITEMS < SMP_SMALL_TABLE, "the table is never full");
    static_assert(SMP_SMALL_ITEMS < 0x8000, "an order number leaves the top bit of `found` free");
    const int n = (int)smp_rows(A), f = A.fanout, t = threadIdx.x;
    int32_t v = -1;
    if (t < n) {
        v = A.ids[t];
        int64_t lo = 0, d = 0;
        if (v >= 0 && v < A.num_nodes) {
            lo = A.indptr[v];
            d = A.indptr[(int64_t)v + 1] - lo;
        }
        uint64_t word;
        int64_t turn;
        smp_row(A, v, d, word, turn);
        r_word[t] = word;
        r_lo[t] = lo;
        r_deg[t] = d;
        r_turn[t] = turn;
        r_node[t] = v;
        if (t < A.max_below) A.below[t] = v;
    }
    __syncthreads();
    for (int q0 = t; q0 < n * f; q0 += 4 * SMP_THREADS) {      // four neighbours per thread in flight together
        int32_t nb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = q0 + u * SMP_THREADS;
            const int row = q < n * f ? q / f : 0;
            nb[u] = smp_draw(A, r_node[row], r_lo[row], r_deg[row], r_word[row], r_turn[row], q < n * f ? q - row * f : f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (q0 + u * SMP_THREADS < n * f) raw[q0 + u * SMP_THREADS] = nb[u];
    }
    __syncthreads();
    // a thread per row: its distinct neighbours move to the front of its draws
    int c = 0;
    if (t < n) {
        for (int j = 0; j < f; ++j) {
            const int32_t nb = raw[t * f + j];
            bool keep = nb >= 0;
            for (int b = 0; b < c; ++b) keep = keep && raw[t * f + b] != nb;
            if (keep) raw[t * f + c++] = nb;
        }
        nodes[t] = v;      // (the rows' values are not needed any more: all draws are behind the barrier)
    }
    // rows back to back
    int incl = c;
    for (int off = 1; off < FG_WAVE; off <<= 1) {
        const int up = __shfl_up(incl, off, FG_WAVE);
        if (fg_lane() >= off) incl += up;
    }
    if (fg_lane() == FG_WAVE - 1) wave_sum[fg_wave()] = incl;
    __syncthreads();
    int earlier = 0, nnz = 0;
    for (int w = 0; w < SMP_THREADS / FG_WAVE; ++w) {
        if (w < fg_wave()) earlier += wave_sum[w];
        nnz += wave_sum[w];
    }
    const int first = earlier + incl - c;
    if (t < A.max_rows) {
        A.row_start[t] = first;
        A.row_end[t] = first + c;
    }
    for (int b = 0; b < c; ++b) nodes[n + first + b] = raw[t * f + b];
    __syncthreads();
    for (int q = t; q < SMP_SMALL_TABLE; q += SMP_THREADS) table[q] = -1;
    __syncthreads();
    constexpr int SHIFT = 32 - 14;
    static_assert(SMP_SMALL_TABLE == 1 << (32 - SHIFT), "hash width");
    for (int o = t; o < n + nnz; o += SMP_THREADS) {
        const int32_t node = nodes[o];
        if (node < 0) continue;
        uint32_t h = ((uint32_t)node * 0x9E3779B1u) >> SHIFT;
        for (;;) {
            const int cur = atomicCAS(&table[h], -1, o);
            if (cur == -1) break;
            if (nodes[cur] == node) {      // an entry's node never changes once it is set
                atomicMin(&table[h], o);
                break;
            }
            h = (h + 1) & (SMP_SMALL_TABLE - 1);
        }
    }
    // found[k]: the rank among the first occurrences of its 64 candidates (top bit set), or the order number of the first
    // occurrence; s_new: first occurrences per 64 candidates, then before each
    constexpr int GROUPS = SMP_SMALL_DRAWS / FG_WAVE;
    __shared__ int s_new[GROUPS];
    if (t < GROUPS) s_new[t] = 0;
    __syncthreads();      // (also behind the last insertion)
    for (int k0 = 0; k0 < nnz; k0 += SMP_THREADS) {
        const int k = k0 + t;
        int m = -1;
        if (k < nnz) {
            const int32_t node = nodes[n + k];
            uint32_t h = ((uint32_t)node * 0x9E3779B1u) >> SHIFT;
            for (;;) {
                m = table[h];
                if (nodes[m] == node) break;      // it was inserted
                h = (h + 1) & (SMP_SMALL_TABLE - 1);
            }
        }
        const bool is_first = m == n + k;
        int total;
        const int r = fg_wave_rank(is_first, total);
        if (k < nnz) found[k] = (unsigned short)(is_first ? 0x8000 | r : m);
        if (fg_lane() == 0 && k < nnz) s_new[k / FG_WAVE] = total;
    }
    __syncthreads();
    int* source = table;      // the table is not needed any more: edges per source of the transpose
    if (A.tr_cnt)
        for (int j = t; j < SMP_SMALL_ITEMS; j += SMP_THREADS) source[j] = 0;
    const int ranked = smp_prefix(s_new, GROUPS, s_new);      // (its barriers also end the clearing)
    for (int k = t; k < nnz; k += SMP_THREADS) {
        const int x = found[k];
        const int q = (x & 0x8000) ? k : x - n;      // the first occurrence, negative: one of the layer's own nodes
        const int at = q < 0 ? x : n + s_new[q / FG_WAVE] + (found[q] & 0x7FFF);
        A.col[k] = at;
        if (A.col_ids) A.col_ids[k] = nodes[n + k];
        if (q == k && at < A.max_below) A.below[at] = nodes[n + k];
        if (A.tr_cnt) atomicAdd(&source[at], 1);
    }
    if (t == 0) {
        A.counts[0] = n + ranked;
        A.counts[1] = nnz;
    }
    if (A.tr_cnt) {      // uniform
        __syncthreads();
        for (int64_t j = t; j < A.max_below; j += SMP_THREADS) A.tr_cnt[j] = j < SMP_SMALL_ITEMS ? source[j] : 0;
    }
}

// ---- transpose of a block by one workgroup (fg_transpose_block by itself) ------------------------------------------------
//
// Sources, edges and rows up to what fits its LDS: level with the five launches at about half of that on the device (rows x draws
// 1024 x 5 11 us against 13, 1024 x 11 22 against 15), but those also cost the gaps between them and the host's time.
constexpr int TR_SMALL = 12288;

__global__ __launch_bounds__(FG_SCAN_BLOCK) void transpose_small_kernel(TrArgs A) {
    extern __shared__ int tr_lds[];
    int* cnt = tr_lds;                                   // [max_src]
    int32_t* list = tr_lds + A.max_src;                  // [max_nnz]
    const int64_t n = tr_count(A.n_dev, A.max_rows), n_src = tr_count(A.n_src_dev, A.max_src);
    const int src = (int)A.max_src, nnz = (int)A.max_nnz, t = threadIdx.x;
    for (int j = t; j < src; j += FG_SCAN_BLOCK) cnt[j] = 0;
    __syncthreads();
    // f(row, source) for every edge: the ranges of up to 1024 rows at a time, then four rows per group of lanes in flight
    __shared__ int s_begin[FG_SCAN_BLOCK], s_end[FG_SCAN_BLOCK];
    auto each_edge = [&](auto f) {
        constexpr int ROWS = FG_SCAN_BLOCK / TR_LANES, TOGETHER = 4;
        const int g = t / TR_LANES, lane = t % TR_LANES;
        for (int r0 = 0; r0 < (int)n; r0 += FG_SCAN_BLOCK) {
            int rb = 0, re = 0;
            if (r0 + t < (int)n) {
                rb = A.row_start[r0 + t] > 0 ? A.row_start[r0 + t] : 0;
                re = A.row_end[r0 + t] < nnz ? A.row_end[r0 + t] : nnz;
            }
            __syncthreads();
            s_begin[t] = rb;
            s_end[t] = re;
            __syncthreads();
            for (int q = 0; q < FG_SCAN_BLOCK && r0 + q < (int)n; q += ROWS * TOGETHER) {
                int k[TOGETHER], c[TOGETHER];
#pragma unroll
                for (int u = 0; u < TOGETHER; ++u) {
                    k[u] = s_begin[q + u * ROWS + g] + lane;
                    c[u] = k[u] < s_end[q + u * ROWS + g] ? A.col[k[u]] : -1;
                }
#pragma unroll
                for (int u = 0; u < TOGETHER; ++u) {
                    const int row = q + u * ROWS + g;
                    for (;;) {
                        if (c[u] >= 0 && c[u] < n_src) f(r0 + row, c[u]);
                        k[u] += TR_LANES;
                        if (k[u] >= s_end[row]) break;
                        c[u] = A.col[k[u]];
                    }
                }
            }
        }
        __syncthreads();
    };
    each_edge([&](int, int c) { atomicAdd(&cnt[c], 1); });
    // a thread's counters are consecutive, and stay with it until they are the starts of their lists
    const int per = (src + FG_SCAN_BLOCK - 1) / FG_SCAN_BLOCK, b = t * per < src ? t * per : src, e = b + per < src ? b + per : src;
    int mine = 0, total;
    for (int j = b; j < e; ++j) mine += cnt[j];
    int at = tr_block_scan(mine, total);
    for (int j = b; j < e; ++j) {
        const int c = cnt[j];
        A.t_start[j] = at;
        cnt[j] = at;
        at += c;
        A.t_end[j] = at;
    }
    __syncthreads();
    each_edge([&](int row, int c) {
        const int to = atomicAdd(&cnt[c], 1);
        if (to < nnz) list[to] = row;
    });      // cnt[j]: now the end of list j
    for (int j0 = 0; j0 < src; j0 += FG_SCAN_BLOCK) {
        const int j = j0 + t;
        tr_sort_lists<FG_SCAN_BLOCK>(list, j > 0 && j < src ? cnt[j - 1] : 0, j < src ? (cnt[j] < nnz ? cnt[j] : nnz) : 0, A.max_rows);
    }
    __syncthreads();
    const int stored = total < nnz ? total : nnz;
    for (int k = t; k < stored; k += FG_SCAN_BLOCK) A.t_row[k] = list[k];
}


// ---- workspace and launches ----------------------------------------------------------------------------------------------
struct SmpWs {
    size_t nbuf, entry, rank, blk_new, blk_kept, new_first, kept_first;      // one block at a time
    size_t table[SMP_MAX_LAYERS], lost[SMP_MAX_LAYERS], cnt[SMP_MAX_LAYERS], blk[SMP_MAX_LAYERS];  // of every block
    uint32_t entries[SMP_MAX_LAYERS];
    size_t total;
};

bool smp_is_small(int64_t max_rows, int64_t fanout) {
    return max_rows <= SMP_SMALL_ROWS && fanout <= SMP_SMALL_FANOUT && max_rows * fanout <= SMP_SMALL_DRAWS;
}

// Slots per thread of launches 2 and 3: four where one would be more workgroups than the chip holds at a time (two per compute unit)
constexpr int64_t SMP_ONE_SLOT = 512;
int smp_slots(int64_t max_rows, int32_t fanout) { return fg_ceil_div(max_rows, SMP_THREADS / fanout) > SMP_ONE_SLOT ? 4 : 1; }
int64_t smp_blocks(int64_t max_rows, int32_t fanout) { return fg_ceil_div(max_rows, smp_slots(max_rows, fanout) * SMP_THREADS / fanout); }
// ... and the most workgroups of any number of rows up to max_rows: a workspace serves every call of fewer rows, where one slot per thread may
// be four times as many workgroups
int64_t smp_most_blocks(int64_t max_rows, int32_t fanout) {
    const int64_t one_slot = fg_ceil_div(max_rows, SMP_THREADS / fanout), now = smp_blocks(max_rows, fanout);
    const int64_t most = one_slot < SMP_ONE_SLOT ? one_slot : SMP_ONE_SLOT;
    return now > most ? now : most;
}

size_t tr_layout(int64_t max_src, size_t* blk_at) {
    const size_t src = (size_t)(max_src > 0 ? max_src : 1);
    *blk_at = fg_align_up(src * 4, 256);
    return *blk_at + fg_align_up((size_t)fg_ceil_div((int64_t)src, FG_SCAN_BLOCK) * 4, 256);
}

// `bound`: for every call of up to as many rows, else for a call of just these
SmpWs smp_layout(int32_t n_layers, const fg_sample_layer_t* layers, bool bound) {
    SmpWs w{};
    size_t at = 0, cands = 1, blocks = 1;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at += fg_align_up(bytes, 256);
        return here;
    };
    for (int i = 0; i < n_layers; ++i) {
        const size_t rows = (size_t)(layers[i].max_rows > 0 ? layers[i].max_rows : 1), c = rows * (size_t)layers[i].fanout;
        const size_t b = (size_t)(bound ? smp_most_blocks : smp_blocks)((int64_t)rows, layers[i].fanout);
        if (!smp_is_small(layers[i].max_rows, layers[i].fanout)) {
            cands = c > cands ? c : cands;
            blocks = b > blocks ? b : blocks;
            uint32_t entries = 1024;      // at most half full (at most two thirds: 54 k rows x 15 44 us instead of 40)
            while ((size_t)entries < 2 * (rows + c) && entries < (1u << 31)) entries <<= 1;
            w.entries[i] = entries;
            w.table[i] = take((size_t)entries * 8);
            w.lost[i] = take(c);
        }
        if (layers[i].t_start_dev) {
            size_t blk_at;
            const size_t bytes = tr_layout(layers[i].max_below, &blk_at);
            w.cnt[i] = take(bytes);
            w.blk[i] = w.cnt[i] + blk_at;
        }
    }
    w.nbuf = take(cands * 4);
    w.entry = take(cands * 4);
    w.rank = take(cands * 2);
    w.blk_new = take(blocks * 4);
    w.blk_kept = take(blocks * 4);
    w.new_first = take((blocks + 1) * 4);
    w.kept_first = take((blocks + 1) * 4);
    w.total = at;
    return w;
}

// The stages of the transposes that are still to be done. Every launch of the sampler takes the next stage of the first
// TR_MAX_RIDES of them along.
struct TrQueue {
    FgStageQueue<TrArgs, SMP_MAX_LAYERS, 4> q;

    bool empty() const { return q.empty(); }
    static int64_t blocks_of(const TrArgs& a, int stage, int threads) {
        if (stage == TR_COUNT || stage == TR_FILL) return fg_ceil_div(a.max_rows, threads / TR_LANES);
        return fg_ceil_div(a.max_src, stage == TR_SUM ? TR_THREADS : threads);
    }
    void add(const TrArgs& a) {      // the edges are counted
        if (a.max_src == 0) return;
        auto& e = q.add(a);
        const bool direct = a.max_src <= TR_DIRECT;
        if (!direct) e.then(TR_SUM);
        e.then(direct ? TR_SCAN : TR_SCAN_SUMS);
        if (a.max_rows > 0) {
            e.then(TR_FILL);
            e.then(TR_SORT);
        }
    }
    TrRides take(int threads) {      // for a launch with workgroups of that size
        TrRides r{};
        q.take(TR_MAX_RIDES, [&](const TrArgs& a, int stage) {
            r.a[r.n] = a;
            r.stage[r.n] = stage;
            r.blocks += (int32_t)blocks_of(a, stage, threads);
            r.end[r.n++] = r.blocks;
        });
        return r;
    }
};

fg_status_t tr_launch(const TrRides& r, hipStream_t st) {
    if (r.blocks == 0) return FG_OK;
    hipLaunchKernelGGL(transpose_stage_kernel, dim3((unsigned)r.blocks), dim3(TR_THREADS), 0, st, r);
    FG_LAUNCH_CHECK("transpose_stage_kernel");
    return FG_OK;
}

fg_status_t smp_check(const char* who, int64_t num_nodes, int64_t num_edges, const int64_t* indptr, const int32_t* indices, const int32_t* ids,
                      const fg_sample_layer_t& y) {
    if (y.max_rows < 0 || num_nodes <= 0 || num_edges < 0 || y.max_below < 0)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: bad size (max_rows %lld, num_nodes %lld, num_edges %lld, max_below %lld)", who,
                (long long)y.max_rows, (long long)num_nodes, (long long)num_edges, (long long)y.max_below);
    if (num_nodes > INT32_MAX) FG_FAIL(FG_ERR_INVALID_ARG, "%s: node ids are 32-bit", who);
    if (y.fanout < 1 || y.fanout > SMP_LANES) FG_FAIL(FG_ERR_INVALID_ARG, "%s: fanout = %d outside 1..%d", who, y.fanout, SMP_LANES);
    if (y.max_rows > (int64_t)INT32_MAX / SMP_LANES) FG_FAIL(FG_ERR_SHAPE, "%s: max_rows = %lld: edge numbers are 32-bit", who, (long long)y.max_rows);
    if (y.layer < 1) FG_FAIL(FG_ERR_INVALID_ARG, "%s: layer = %d, blocks are numbered from 1", who, y.layer);
    if (!y.counts_dev) FG_FAIL(FG_ERR_INVALID_ARG, "%s: counts_dev is NULL", who);
    if (y.max_rows > 0 && (!indptr || !ids || !y.row_start_dev || !y.row_end_dev || !y.col_dev || !y.ids_below_dev || (num_edges > 0 && !indices)))
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    if (y.max_below < y.max_rows) FG_FAIL(FG_ERR_SHAPE, "%s: max_below = %lld smaller than max_rows = %lld (the layer below starts with this layer)", who, (long long)y.max_below, (long long)y.max_rows);
    if (!y.t_start_dev != !y.t_end_dev || !y.t_start_dev != !y.t_row_dev)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: a transpose needs t_start_dev, t_end_dev and t_row_dev together", who);
    if (y.t_start_dev && y.max_below > INT32_MAX) FG_FAIL(FG_ERR_SHAPE, "%s: max_below = %lld: a transpose has 32-bit positions", who, (long long)y.max_below);
    return FG_OK;
}

fg_status_t smp_launch(const char* who, const int64_t* indptr, const int32_t* indices, int64_t num_nodes, int64_t num_edges, const int32_t* ids,
                       const int64_t* n_dev, int32_t n_layers, const fg_sample_layer_t* layers, uint64_t key, void* ws_dev, size_t ws_bytes, hipStream_t st) {
    for (int i = 0; i < n_layers; ++i) {
        fg_status_t rc = smp_check(who, num_nodes, num_edges, indptr, indices, i ? layers[i - 1].ids_below_dev : ids, layers[i]);
        if (rc != FG_OK) return rc;
        if (i && layers[i].max_rows > layers[i - 1].max_below)
            FG_FAIL(FG_ERR_SHAPE, "%s: layers[%d].max_rows = %lld exceeds the list of layers[%d], %lld", who, i, (long long)layers[i].max_rows, i - 1,
                    (long long)layers[i - 1].max_below);
    }
    const SmpWs w = smp_layout(n_layers, layers, false);
    bool any = false;
    for (int i = 0; i < n_layers; ++i) any = any || layers[i].max_rows > 0 || layers[i].t_start_dev;
    if (any && (!ws_dev || ws_bytes < w.total)) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, w.total);
    if ((uintptr_t)ws_dev & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: workspace must be 16-byte aligned", who);
    fg_clear_error();
    char* ws = (char*)ws_dev;
    // What has to be clear before a block starts: of the first one by a launch of its own (a block of few draws needs nothing),
    // of the others beside the first block's draws, which leave most of the chip idle.
    SmpClear first{}, later{};
    for (int i = 0; i < n_layers; ++i) {
        const fg_sample_layer_t& y = layers[i];
        SmpClear& clear = i == 0 ? first : later;
        if (y.max_rows > 0 && !smp_is_small(y.max_rows, y.fanout)) {
            clear.add(ws + w.table[i], (int64_t)w.entries[i] * 8, ~0u);
            clear.add(ws + w.lost[i], (int64_t)fg_align_up((size_t)y.max_rows * y.fanout, 16), 0u);
        }
        if (y.t_start_dev && (y.max_rows == 0 || !smp_is_small(y.max_rows, y.fanout)))
            clear.add(ws + w.cnt[i], (int64_t)fg_align_up((size_t)y.max_below * 4, 16), 0u);
    }
    if (layers[0].max_rows == 0) {      // nothing to be beside
        for (int i = 0; i < later.n; ++i) first.add(later.p[i], later.bytes[i], later.value[i]);
        later.n = 0;
    }
    auto clear_blocks = [](const SmpClear& c, int64_t most) {
        const int64_t blocks = fg_ceil_div(c.total(), SMP_CLEAR_BYTES);
        return blocks < most ? blocks : most;
    };
    TrQueue queue;
    for (int i = 0; i < n_layers; ++i) {
        const fg_sample_layer_t& y = layers[i];
        const bool small = y.max_rows > 0 && smp_is_small(y.max_rows, y.fanout);
        if (i == 0 && first.n > 0) {
            hipLaunchKernelGGL(sample_clear_kernel, dim3((unsigned)clear_blocks(first, 2048)), dim3(SMP_THREADS), 0, st, first);
            FG_LAUNCH_CHECK("sample_clear_kernel");
        }
        const int64_t* rows_dev = i ? layers[i - 1].counts_dev : n_dev;
        if (y.max_rows == 0) {
            fg_status_t rc = fg_launch_fill_i32((int32_t*)y.counts_dev, 4, 0, st);
            if (rc != FG_OK) return rc;
        } else {
            SmpArgs A{};
            A.indptr = indptr;
            A.indices = indices;
            A.num_nodes = num_nodes;
            A.num_edges = num_edges;
            A.ids = i ? layers[i - 1].ids_below_dev : ids;
            A.n_dev = rows_dev;
            A.max_rows = y.max_rows;
            A.fanout = y.fanout;
            A.rows_per = smp_slots(y.max_rows, y.fanout) * SMP_THREADS / y.fanout;
            A.draw_blocks = (int32_t)fg_ceil_div(y.max_rows, SMP_DRAW_THREADS / y.fanout);
            A.own_blocks = (int32_t)fg_ceil_div(y.max_rows, SMP_DRAW_THREADS);
            A.key_l = smp_word(smp_mix(key), (uint64_t)y.layer);
            A.row_start = y.row_start_dev;
            A.row_end = y.row_end_dev;
            A.col = y.col_dev;
            A.col_ids = y.col_ids_dev;
            A.below = y.ids_below_dev;
            A.max_below = y.max_below;
            A.counts = y.counts_dev;
            A.tr_cnt = y.t_start_dev ? (int32_t*)(ws + w.cnt[i]) : nullptr;
            if (small) {
                const TrRides r = queue.take(SMP_THREADS);
                const int64_t extra = i == 0 ? clear_blocks(later, 255) : 0;      // one per compute unit: each has the launch's LDS
                hipLaunchKernelGGL(sample_small_kernel, dim3((unsigned)(1 + r.blocks + extra)), dim3(SMP_THREADS), SMP_SMALL_LDS, st, A, r, later);
                FG_LAUNCH_CHECK("sample_small_kernel");
            } else {
                A.nbuf = (int32_t*)(ws + w.nbuf);
                A.entry = (uint32_t*)(ws + w.entry);
                A.lost = (uint8_t*)(ws + w.lost[i]);
                A.rank = (uint16_t*)(ws + w.rank);
                A.blk_new = (int32_t*)(ws + w.blk_new);
                A.blk_kept = (int32_t*)(ws + w.blk_kept);
                A.new_first = (int32_t*)(ws + w.new_first);
                A.kept_first = (int32_t*)(ws + w.kept_first);
                A.table = (unsigned long long*)(ws + w.table[i]);
                A.mask = w.entries[i] - 1;
                int lg = 0;
                while ((1u << lg) < w.entries[i]) ++lg;
                A.shift = 32 - lg;
                const int64_t blocks = smp_blocks(y.max_rows, y.fanout);
                TrRides r = queue.take(SMP_DRAW_THREADS);
                const int64_t extra = i == 0 ? clear_blocks(later, 1024) : 0;
                hipLaunchKernelGGL(sample_draw_kernel, dim3((unsigned)(r.blocks + A.draw_blocks + A.own_blocks + extra)), dim3(SMP_DRAW_THREADS), 0, st, A, r,
                                   later);
                FG_LAUNCH_CHECK("sample_draw_kernel");
                const bool one = smp_slots(y.max_rows, y.fanout) == 1, own = blocks <= SMP_PREFIX;
                r = queue.take(SMP_THREADS);
                hipLaunchKernelGGL(one ? sample_resolve_kernel<1> : sample_resolve_kernel<4>, dim3((unsigned)(blocks + r.blocks)), dim3(SMP_THREADS),
                                   0, st, A, r);
                FG_LAUNCH_CHECK("sample_resolve_kernel");
                if (!own) {
                    hipLaunchKernelGGL(sample_prefix_kernel, dim3(1), dim3(FG_SCAN_BLOCK), 0, st, A, (int)blocks);
                    FG_LAUNCH_CHECK("sample_prefix_kernel");
                }
                r = queue.take(SMP_THREADS);
                auto columns = one ? sample_columns_kernel<1, true> : (own ? sample_columns_kernel<4, true> : sample_columns_kernel<4, false>);
                hipLaunchKernelGGL(columns, dim3((unsigned)(blocks + r.blocks)), dim3(SMP_THREADS), own ? (size_t)blocks * 4 : 0, st, A, r);
                FG_LAUNCH_CHECK("sample_columns_kernel");
            }
        }
        if (y.t_start_dev)
            queue.add(TrArgs{y.row_start_dev, y.row_end_dev, y.col_dev, rows_dev, y.max_rows, y.counts_dev, y.max_below,
                             y.max_rows * y.fanout, y.t_start_dev, y.t_end_dev, y.t_row_dev, (int32_t*)(ws + w.cnt[i]), (int32_t*)(ws + w.blk[i])});
    }
    while (!queue.empty()) {      // the last block's transpose has nothing left to ride in
        fg_status_t rc = tr_launch(queue.take(TR_THREADS), st);
        if (rc != FG_OK) return rc;
    }
    return FG_OK;
}

}  // namespace

extern "C" size_t fg_sample_minibatch_workspace_bytes(int32_t n_layers, const fg_sample_layer_t* layers) {
    if (n_layers < 1 || n_layers > SMP_MAX_LAYERS || !layers) return 0;
    for (int i = 0; i < n_layers; ++i)
        if (layers[i].max_rows < 0 || layers[i].fanout < 1 || layers[i].fanout > SMP_LANES || layers[i].max_rows > (int64_t)INT32_MAX / SMP_LANES ||
            layers[i].max_below < 0 || (layers[i].t_start_dev && layers[i].max_below > INT32_MAX))
            return 0;
    return smp_layout(n_layers, layers, true).total;
}

extern "C" fg_status_t fg_sample_minibatch(const int64_t* indptr_dev, const int32_t* indices_dev, int64_t num_nodes, int64_t num_edges,
                                           const int32_t* ids_dev, const int64_t* n_dev, int32_t n_layers, const fg_sample_layer_t* layers,
                                           uint64_t key, void* ws_dev, size_t ws_bytes, void* stream) {
    const char* who = "fg_sample_minibatch";
    if (n_layers < 1 || n_layers > SMP_MAX_LAYERS || !layers)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: n_layers = %d must be in 1..%d and layers non-NULL", who, n_layers, SMP_MAX_LAYERS);
    return smp_launch(who, indptr_dev, indices_dev, num_nodes, num_edges, ids_dev, n_dev, n_layers, layers, key, ws_dev, ws_bytes, (hipStream_t)stream);
}

extern "C" size_t fg_sample_block_workspace_bytes(int64_t max_rows, int32_t fanout) {
    if (max_rows < 0 || fanout < 1 || fanout > SMP_LANES || max_rows > (int64_t)INT32_MAX / SMP_LANES) return 0;
    fg_sample_layer_t y{};
    y.max_rows = max_rows;
    y.fanout = fanout;
    return smp_layout(1, &y, true).total;
}

extern "C" fg_status_t fg_sample_block(const int64_t* indptr_dev, const int32_t* indices_dev, int64_t num_nodes, int64_t num_edges,
                                       const int32_t* ids_dev, const int64_t* n_dev, int64_t max_rows, int32_t fanout, uint64_t key,
                                       int32_t layer, int32_t* row_start_dev, int32_t* row_end_dev, int32_t* col_dev,
                                       int32_t* col_ids_dev, int32_t* ids_below_dev, int64_t max_below, int64_t* counts_dev,
                                       void* ws_dev, size_t ws_bytes, void* stream) {
    const fg_sample_layer_t y = {layer, fanout, max_rows, row_start_dev, row_end_dev, col_dev, col_ids_dev, ids_below_dev, max_below, counts_dev,
                                 nullptr, nullptr, nullptr};
    return smp_launch("fg_sample_block", indptr_dev, indices_dev, num_nodes, num_edges, ids_dev, n_dev, 1, &y, key, ws_dev, ws_bytes, (hipStream_t)stream);
}

extern "C" size_t fg_transpose_block_workspace_bytes(int64_t max_src) {
    if (max_src < 0 || max_src > INT32_MAX) return 0;
    size_t at;
    return tr_layout(max_src, &at);
}

extern "C" fg_status_t fg_transpose_block(const int32_t* row_start_dev, const int32_t* row_end_dev, const int32_t* col_dev,
                                          const int64_t* n_dev, int64_t max_rows, const int64_t* n_src_dev, int64_t max_src,
                                          int64_t max_nnz, int32_t* t_start_dev, int32_t* t_end_dev, int32_t* t_row_dev,
                                          void* ws_dev, size_t ws_bytes, void* stream) {
    const char* who = "fg_transpose_block";
    if (max_rows < 0 || max_src < 0 || max_nnz < 0 || max_rows > INT32_MAX || max_src > INT32_MAX || max_nnz > INT32_MAX)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: bad size (max_rows %lld, max_src %lld, max_nnz %lld)", who, (long long)max_rows,
                (long long)max_src, (long long)max_nnz);
    if (max_rows > 0 && (!row_start_dev || !row_end_dev || (max_nnz > 0 && !col_dev))) FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL block", who);
    if (max_src > 0 && (!t_start_dev || !t_end_dev)) FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL output", who);
    if (max_nnz > 0 && !t_row_dev) FG_FAIL(FG_ERR_INVALID_ARG, "%s: t_row_dev is NULL", who);
    size_t blk_at;
    const size_t need = tr_layout(max_src, &blk_at);
    if (max_src > 0 && (!ws_dev || ws_bytes < need)) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, need);
    if ((uintptr_t)ws_dev & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: workspace must be 16-byte aligned", who);
    fg_clear_error();
    if (max_src == 0) return FG_OK;
    hipStream_t st = (hipStream_t)stream;
    TrArgs A{row_start_dev, row_end_dev, col_dev, n_dev, max_rows, n_src_dev, max_src, max_nnz, t_start_dev, t_end_dev, t_row_dev,
             (int32_t*)ws_dev, (int32_t*)((char*)ws_dev + blk_at)};
    if (max_src <= TR_SMALL && max_nnz <= TR_SMALL && max_rows <= TR_SMALL) {
        hipLaunchKernelGGL(transpose_small_kernel, dim3(1), dim3(FG_SCAN_BLOCK), (size_t)(max_src + max_nnz) * 4, st, A);
        FG_LAUNCH_CHECK("transpose_small_kernel");
        return FG_OK;
    }
    fg_status_t rc = fg_launch_fill_i32(A.cnt, max_src, 0, st);
    if (rc != FG_OK) return rc;
    TrRides count{};
    count.n = 1;
    count.stage[0] = TR_COUNT;
    count.a[0] = A;
    count.blocks = count.end[0] = (int32_t)TrQueue::blocks_of(A, TR_COUNT, TR_THREADS);
    rc = tr_launch(count, st);
    TrQueue queue;
    queue.add(A);
    while (rc == FG_OK && !queue.empty()) rc = tr_launch(queue.take(TR_THREADS), st);
    return rc;
}
