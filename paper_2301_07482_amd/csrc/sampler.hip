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
// Launches (sizes from the host-side bound max_rows, the exact count is read on the device):
//   1. draw      8, 16 or 32 lanes per row: slot, neighbour, repeats removed by comparing within the row; per-row and
//                per-workgroup counts; the layer's own nodes go to the head of the list below; the hash table is cleared
//   2. compact   rows back to back (start/end), candidates in row order; the layer's own nodes enter the table with their
//                position, every candidate k with its order number n + k; the table keeps the smallest per node
//   3. resolve   per candidate: the smallest order number of its node; it is a first occurrence iff that is its own;
//                first occurrences are ranked within their workgroup
//   4. columns   every workgroup adds up the workgroups' first occurrences for itself; first occurrences are appended to
//                the list below, and every candidate gets the position of its node in that list
// Each launch is a chain of three to five dependent reads per element with little else to do, so what counts is how many
// rows are in flight and how many launches there are: with 32 lanes for 15 slots, a launch for clearing and one for
// numbering, 54 k rows x 15 took 102 us (draw 25, compact 40, resolve 16, the rest 21), now 80 (18, 38, 17, 7).
// A layer of few rows (the seeds) runs in one workgroup instead, see sample_small_kernel.
#include "common.h"
#include "scan.h"

namespace {

constexpr int SMP_THREADS = 1024;
constexpr int SMP_LANES = 32;                           // the largest fan-out, and the most lanes per row
constexpr int SMP_PREFIX = 8192;                        // workgroups of candidates whose counts a workgroup adds up for itself
constexpr unsigned long long SMP_EMPTY = ~0ull;

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
    uint64_t key_l;
    int32_t* row_start;
    int32_t* row_end;
    int32_t* col;
    int32_t* col_ids;     // candidates in row order (a workspace array when the caller wants no ids)
    int32_t* below;
    int64_t max_below;
    int64_t* counts;      // [0] nodes of the layer below, [1] edges
    int32_t* nbuf;        // [max_rows * fanout] raw candidates, -1 = none
    int32_t* cnt;         // [max_rows]
    int32_t* blk_rows;    // candidates per workgroup of launch 1
    int32_t* first;       // [max_rows * fanout] smallest order number of the candidate's node
    int32_t* rank;        // [max_rows * fanout] rank among the first occurrences of its workgroup
    int32_t* blk_new;     // first occurrences per workgroup of launch 3
    int32_t* blk_first;   // [+1] first occurrences before each workgroup (only where there are more than SMP_PREFIX)
    unsigned long long* table;
    uint32_t mask;        // table entries - 1 (a power of two)
    int shift;            // 32 - log2(entries)
};

__device__ __forceinline__ int64_t smp_rows(const SmpArgs& A) {
    int64_t n = A.n_dev ? *A.n_dev : A.max_rows;
    if (n < 0) n = 0;
    return n < A.max_rows ? n : A.max_rows;
}

__device__ __forceinline__ uint32_t smp_hash(const SmpArgs& A, int32_t node) { return ((uint32_t)node * 0x9E3779B1u) >> A.shift; }

// Keeps the smallest order number seen for `node`. An entry's node never changes once it is set. Atomics on memory that all
// XCDs share are what the insertion costs, so there are as few as possible: one for an empty entry, most nodes' case; entries
// further on are read first (a stale read can only show an entry as empty that no longer is), and a node that is there
// with a smaller number is left alone.
__device__ __forceinline__ void smp_insert(const SmpArgs& A, int32_t node, uint32_t order) {
    const unsigned long long mine = ((unsigned long long)(uint32_t)node << 32) | order;
    uint32_t h = smp_hash(A, node);
    unsigned long long cur = SMP_EMPTY;      // what the entry is expected to hold
    for (uint32_t probe = 0; probe <= A.mask; ++probe) {
        if (cur == SMP_EMPTY) cur = atomicCAS(&A.table[h], SMP_EMPTY, mine);
        if (cur == SMP_EMPTY) return;
        if ((uint32_t)(cur >> 32) == (uint32_t)node) {
            if (cur > mine) atomicMin(&A.table[h], mine);
            return;
        }
        h = (h + 1) & A.mask;
        cur = A.table[h];
    }
}

__device__ __forceinline__ int64_t smp_lookup(const SmpArgs& A, int32_t node) {
    uint32_t h = smp_hash(A, node);
    for (uint32_t probe = 0; probe <= A.mask; ++probe) {
        const unsigned long long cur = A.table[h];
        if (cur == SMP_EMPTY) return -1;
        if ((uint32_t)(cur >> 32) == (uint32_t)node) return (int64_t)(uint32_t)cur;
        h = (h + 1) & A.mask;
    }
    return -1;
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

// Whether lane j of a group of LANES keeps its neighbour: no earlier draw of the row has it.
template <int LANES>
__device__ __forceinline__ bool smp_keep(int32_t nb, int j, int f) {
    bool keep = nb >= 0;
    for (int b = 0; b < f - 1; ++b) {
        const int32_t other = __shfl(nb, b, LANES);
        if (b < j && other == nb) keep = false;
    }
    return keep;
}

// the group's part of a ballot
template <int LANES>
__device__ __forceinline__ uint32_t smp_group_mask(bool flag) {
    const unsigned long long all = __ballot(flag);
    return (uint32_t)(all >> ((threadIdx.x & 63) / LANES * LANES)) & (LANES == 32 ? ~0u : (1u << (LANES & 31)) - 1u);
}

template <int LANES>
__global__ __launch_bounds__(SMP_THREADS) void sample_draw_kernel(SmpArgs A) {
    constexpr int ROWS = SMP_THREADS / LANES;       // rows per workgroup
    __shared__ int s_cnt[ROWS];
    const int64_t n = smp_rows(A);
    const int g = threadIdx.x / LANES, j = threadIdx.x % LANES;
    const int64_t row = (int64_t)blockIdx.x * ROWS + g;
    const int f = A.fanout;
    int32_t v = -1, nb = -1;
    int64_t lo = 0, d = 0;
    if (row < n) {
        v = A.ids[row];
        if (v >= 0 && v < A.num_nodes) {
            lo = A.indptr[v];
            d = A.indptr[(int64_t)v + 1] - lo;
        }
    }
    // the table of the next launch is cleared while those reads are on their way (an even number of entries)
    const ulonglong2 empty = {SMP_EMPTY, SMP_EMPTY};
    for (int64_t q = (int64_t)blockIdx.x * SMP_THREADS + threadIdx.x; q <= (int64_t)(A.mask >> 1); q += (int64_t)gridDim.x * SMP_THREADS)
        ((ulonglong2*)A.table)[q] = empty;
    uint64_t word;
    int64_t turn;
    smp_row(A, v, d, word, turn);
    nb = smp_draw(A, v, lo, d, word, turn, j);
    const bool keep = smp_keep<LANES>(nb, j, f);
    const uint32_t mine = smp_group_mask<LANES>(keep);
    if (row < A.max_rows) {
        if (j < f) A.nbuf[row * f + j] = keep ? nb : -1;
        if (j == 0) {
            A.cnt[row] = __popc(mine);      // 0 for a row past the count: nothing was drawn
            if (row < n && row < A.max_below) A.below[row] = v;
        }
    }
    if (j == 0) s_cnt[g] = __popc(mine);
    __syncthreads();
    if (threadIdx.x < 64) {
        int t = 0;
        for (int q = threadIdx.x; q < ROWS; q += 64) t += s_cnt[q];
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
        if (threadIdx.x == 0) A.blk_rows[blockIdx.x] = t;
    }
}

template <int LANES>
__global__ __launch_bounds__(SMP_THREADS) void sample_compact_kernel(SmpArgs A) {
    constexpr int ROWS = SMP_THREADS / LANES;
    __shared__ long long red[16];
    __shared__ int s_first[ROWS];
    const int64_t n = smp_rows(A);
    const int g = threadIdx.x / LANES, j = threadIdx.x % LANES;
    const int64_t row = (int64_t)blockIdx.x * ROWS + g;
    const int f = A.fanout;
    // everything this workgroup reads is asked for before the first of it is used
    const int32_t nb = (row < A.max_rows && j < f) ? A.nbuf[row * f + j] : -1;
    const int64_t my_row = (int64_t)blockIdx.x * ROWS + threadIdx.x;      // the first threads: one row of the workgroup each
    const bool has_row = threadIdx.x < ROWS && my_row < A.max_rows;
    const int c = has_row ? A.cnt[my_row] : 0;
    const int32_t v = has_row && my_row < n ? A.ids[my_row] : -1;
    long long before = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += SMP_THREADS) before += A.blk_rows[b];
    if (v >= 0) smp_insert(A, v, (uint32_t)my_row);
    before = fg_block_sum(before, red);
    // exclusive scan of the rows' counts (at most 128 rows: two wavefronts)
    int incl = c;
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off, 64);
        if (fg_lane() >= off) incl += up;
    }
    __shared__ int s_wave;
    if (threadIdx.x == 63) s_wave = incl;
    __syncthreads();
    const int earlier = threadIdx.x >= 64 ? s_wave : 0;
    if (threadIdx.x < ROWS) s_first[threadIdx.x] = earlier + incl - c;
    if (has_row) {
        A.row_start[my_row] = (int32_t)(before + earlier + incl - c);
        A.row_end[my_row] = (int32_t)(before + earlier + incl);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == ROWS - 1) A.counts[1] = before + earlier + incl;
    __syncthreads();
    const uint32_t mine = smp_group_mask<LANES>(nb >= 0);
    if (nb >= 0) {
        const long long k = before + s_first[g] + __popc(mine & ((1u << j) - 1u));
        A.col_ids[k] = nb;
        smp_insert(A, nb, (uint32_t)(n + k));
    }
}

// One thread per candidate. The number of candidates is the end of the last row.
__device__ __forceinline__ int64_t smp_edges(const SmpArgs& A, int64_t n) { return n > 0 ? (int64_t)A.row_end[n - 1] : 0; }

__global__ __launch_bounds__(FG_SCAN_BLOCK) void sample_resolve_kernel(SmpArgs A) {
    __shared__ int sc[17];
    const int64_t n = smp_rows(A);
    const int64_t nnz = smp_edges(A, n);
    const int64_t k = (int64_t)blockIdx.x * FG_SCAN_BLOCK + threadIdx.x;
    if ((int64_t)blockIdx.x * FG_SCAN_BLOCK >= nnz) {      // uniform over the workgroup
        if (threadIdx.x == 0) A.blk_new[blockIdx.x] = 0;
        return;
    }
    bool is_first = false;
    if (k < nnz) {
        const int64_t m = smp_lookup(A, A.col_ids[k]);
        A.first[k] = (int32_t)m;
        is_first = m == n + k;
    }
    int total;
    const int r = fg_block_rank(is_first, total, sc);
    if (is_first) A.rank[k] = r;
    if (threadIdx.x == 0) A.blk_new[blockIdx.x] = total;
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

// more candidates than a workgroup of the last launch could add up for itself
__global__ __launch_bounds__(FG_SCAN_BLOCK) void sample_prefix_kernel(SmpArgs A) {
    const int blocks = (int)((A.max_rows * A.fanout + FG_SCAN_BLOCK - 1) / FG_SCAN_BLOCK);
    const int all = smp_prefix(A.blk_new, blocks, A.blk_first);
    if (threadIdx.x == 0) A.blk_first[blocks] = all;
}

// OWN: the prefix sums of the workgroups' first occurrences are formed in LDS by every workgroup, else read.
template <bool OWN>
__global__ __launch_bounds__(FG_SCAN_BLOCK) void sample_columns_kernel(SmpArgs A) {
    extern __shared__ int s_prefix[];
    const int64_t n = smp_rows(A);
    const int64_t nnz = smp_edges(A, n);
    const int64_t k = (int64_t)blockIdx.x * FG_SCAN_BLOCK + threadIdx.x;
    const int64_t k0 = (int64_t)blockIdx.x * FG_SCAN_BLOCK;
    if (k0 >= nnz && blockIdx.x != 0) return;      // uniform over the workgroup
    const int32_t m32 = k < nnz ? A.first[k] : 0;
    const int blocks = OWN ? (int)((nnz + FG_SCAN_BLOCK - 1) / FG_SCAN_BLOCK) : (int)((A.max_rows * A.fanout + FG_SCAN_BLOCK - 1) / FG_SCAN_BLOCK);
    const int all = OWN ? smp_prefix(A.blk_new, blocks, s_prefix) : A.blk_first[blocks];
    const int* prefix = OWN ? s_prefix : A.blk_first;
    if (blockIdx.x == 0 && threadIdx.x == 0) A.counts[0] = n + all;
    if (k >= nnz) return;
    const int64_t m = m32;
    if (m < n) {
        A.col[k] = (int32_t)m;
        return;
    }
    const int64_t q = m - n;      // the first occurrence of this candidate's node
    const int64_t at = n + prefix[q / FG_SCAN_BLOCK] + A.rank[q];
    A.col[k] = (int32_t)at;
    if (q == k && at < A.max_below) A.below[at] = A.col_ids[k];
}

// A layer of few draws (the seeds) in one workgroup and one launch: the candidates, the table
// (order numbers only: the node of an order number is in LDS too) and the ranks stay in LDS. Reads from memory are three
// rounds: ids, row ranges, neighbours. One compute unit does all the arithmetic, so what belongs to a row is computed once
// per row and no lane is left idle beside a row's draws. Against the four launches, by themselves, graph of 2 M nodes: 256 rows x 5
// 11 us (29), 1024 x 5 24 (27), 512 x 11 27 (29), 640 x 10 32 (29), 777 x 8 33 (33), 1024 x 8 44 (28), 1024 x 11 111 (31).
// In a mini-batch, where launches also cost their gaps and host time: 1024 seeds x 6 x 10 105 us (110), x 7 114 to 116 (116 to 118), 777 x 9
// 114 (114), 1024 x 8 115 (106), x 11 138 (115): up to 7168 draws.
constexpr int SMP_SMALL_ROWS = 1024, SMP_SMALL_FANOUT = 11, SMP_SMALL_DRAWS = 7168;
constexpr int SMP_SMALL_ITEMS = SMP_SMALL_ROWS + SMP_SMALL_DRAWS;      // own nodes and candidates
constexpr int SMP_SMALL_TABLE = 16384;
constexpr size_t SMP_SMALL_ROW_BYTES = 36;                             // what a row keeps while its neighbours are drawn
constexpr size_t SMP_SMALL_NODES = SMP_SMALL_ITEMS * 4 > SMP_SMALL_ROWS * SMP_SMALL_ROW_BYTES ? SMP_SMALL_ITEMS * 4 : SMP_SMALL_ROWS * SMP_SMALL_ROW_BYTES;
constexpr size_t SMP_SMALL_LDS = (size_t)SMP_SMALL_TABLE * 4 + SMP_SMALL_NODES + SMP_SMALL_ITEMS * 2;

__global__ __launch_bounds__(SMP_THREADS) void sample_small_kernel(SmpArgs A) {
    extern __shared__ __attribute__((aligned(16))) int smem[];
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
        if (o >= n) A.col_ids[o - n] = node;
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
    const int ranked = smp_prefix(s_new, GROUPS, s_new);
    for (int k = t; k < nnz; k += SMP_THREADS) {
        const int x = found[k];
        const int q = (x & 0x8000) ? k : x - n;      // the first occurrence, negative: one of the layer's own nodes
        const int at = q < 0 ? x : n + s_new[q / FG_WAVE] + (found[q] & 0x7FFF);
        A.col[k] = at;
        if (q == k && at < A.max_below) A.below[at] = nodes[n + k];
    }
    if (t == 0) {
        A.counts[0] = n + ranked;
        A.counts[1] = nnz;
    }
}

struct SmpWs {
    size_t nbuf, cnt, blk_rows, first, rank, blk_new, blk_first, cand, table, total;
    uint32_t entries;
};
SmpWs smp_layout(int64_t max_rows, int32_t fanout) {
    SmpWs w;
    const size_t rows = (size_t)(max_rows > 0 ? max_rows : 1), cands = rows * (size_t)fanout;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at += fg_align_up(bytes, 256);
        return here;
    };
    w.nbuf = take(cands * 4);
    w.cnt = take(rows * 4);
    w.blk_rows = take((size_t)fg_ceil_div((int64_t)rows, SMP_THREADS / SMP_LANES) * 4);
    w.first = take(cands * 4);
    w.rank = take(cands * 4);
    w.blk_new = take((size_t)fg_ceil_div((int64_t)cands, FG_SCAN_BLOCK) * 4);
    w.blk_first = take((size_t)(fg_ceil_div((int64_t)cands, FG_SCAN_BLOCK) + 1) * 4);
    w.cand = take(cands * 4);
    uint32_t entries = 1024;
    while ((size_t)entries < 2 * (rows + cands) && entries < (1u << 31)) entries <<= 1;
    w.entries = entries;
    w.table = take((size_t)entries * 8);
    w.total = at;
    return w;
}

}  // namespace

extern "C" size_t fg_sample_block_workspace_bytes(int64_t max_rows, int32_t fanout) {
    if (max_rows < 0 || fanout < 1 || fanout > SMP_LANES || max_rows > (int64_t)INT32_MAX / SMP_LANES) return 0;
    return smp_layout(max_rows, fanout).total;
}

extern "C" fg_status_t fg_sample_block(const int64_t* indptr_dev, const int32_t* indices_dev, int64_t num_nodes, int64_t num_edges,
                                       const int32_t* ids_dev, const int64_t* n_dev, int64_t max_rows, int32_t fanout, uint64_t key,
                                       int32_t layer, int32_t* row_start_dev, int32_t* row_end_dev, int32_t* col_dev,
                                       int32_t* col_ids_dev, int32_t* ids_below_dev, int64_t max_below, int64_t* counts_dev,
                                       void* ws_dev, size_t ws_bytes, void* stream) {
    const char* who = "fg_sample_block";
    if (max_rows < 0 || num_nodes <= 0 || num_edges < 0 || max_below < 0)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: bad size (max_rows %lld, num_nodes %lld, num_edges %lld, max_below %lld)", who,
                (long long)max_rows, (long long)num_nodes, (long long)num_edges, (long long)max_below);
    if (num_nodes > INT32_MAX) FG_FAIL(FG_ERR_INVALID_ARG, "%s: node ids are 32-bit", who);
    if (fanout < 1 || fanout > SMP_LANES) FG_FAIL(FG_ERR_INVALID_ARG, "%s: fanout = %d outside 1..%d", who, fanout, SMP_LANES);
    if (max_rows > (int64_t)INT32_MAX / SMP_LANES) FG_FAIL(FG_ERR_SHAPE, "%s: max_rows = %lld: edge numbers are 32-bit", who, (long long)max_rows);
    if (layer < 1) FG_FAIL(FG_ERR_INVALID_ARG, "%s: layer = %d, blocks are numbered from 1", who, layer);
    if (!counts_dev) FG_FAIL(FG_ERR_INVALID_ARG, "%s: counts_dev is NULL", who);
    if (max_rows > 0 && (!indptr_dev || !ids_dev || !row_start_dev || !row_end_dev || !col_dev || !ids_below_dev || (num_edges > 0 && !indices_dev)))
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    if (max_below < max_rows) FG_FAIL(FG_ERR_SHAPE, "%s: max_below = %lld smaller than max_rows = %lld (the layer below starts with this layer)", who, (long long)max_below, (long long)max_rows);
    const SmpWs w = smp_layout(max_rows, fanout);
    if (max_rows > 0 && (!ws_dev || ws_bytes < w.total)) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, w.total);
    if ((uintptr_t)ws_dev & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: workspace must be 16-byte aligned", who);
    fg_clear_error();
    hipStream_t st = (hipStream_t)stream;
    if (max_rows == 0) {
        fg_status_t rc = fg_launch_fill_i32((int32_t*)counts_dev, 4, 0, st);
        return rc;
    }
    char* ws = (char*)ws_dev;
    SmpArgs A;
    A.indptr = indptr_dev;
    A.indices = indices_dev;
    A.num_nodes = num_nodes;
    A.num_edges = num_edges;
    A.ids = ids_dev;
    A.n_dev = n_dev;
    A.max_rows = max_rows;
    A.fanout = fanout;
    A.key_l = smp_word(smp_mix(key), (uint64_t)layer);
    A.row_start = row_start_dev;
    A.row_end = row_end_dev;
    A.col = col_dev;
    A.col_ids = col_ids_dev ? col_ids_dev : (int32_t*)(ws + w.cand);
    A.below = ids_below_dev;
    A.max_below = max_below;
    A.counts = counts_dev;
    A.nbuf = (int32_t*)(ws + w.nbuf);
    A.cnt = (int32_t*)(ws + w.cnt);
    A.blk_rows = (int32_t*)(ws + w.blk_rows);
    A.first = (int32_t*)(ws + w.first);
    A.rank = (int32_t*)(ws + w.rank);
    A.blk_new = (int32_t*)(ws + w.blk_new);
    A.blk_first = (int32_t*)(ws + w.blk_first);
    A.table = (unsigned long long*)(ws + w.table);
    A.mask = w.entries - 1;
    int lg = 0;
    while ((1u << lg) < w.entries) ++lg;
    A.shift = 32 - lg;
    if (max_rows <= SMP_SMALL_ROWS && fanout <= SMP_SMALL_FANOUT && max_rows * fanout <= SMP_SMALL_DRAWS) {
        hipLaunchKernelGGL(sample_small_kernel, dim3(1), dim3(SMP_THREADS), SMP_SMALL_LDS, st, A);
        FG_LAUNCH_CHECK("sample_small_kernel");
        return FG_OK;
    }
    const int lanes = fanout <= 8 ? 8 : (fanout <= 16 ? 16 : 32);
    const unsigned row_blocks = (unsigned)fg_ceil_div(max_rows, SMP_THREADS / lanes);
    const unsigned cand_blocks = (unsigned)fg_ceil_div(max_rows * fanout, FG_SCAN_BLOCK);
#define FG_SMP(kernel)                                                                                   \
    do {                                                                                                 \
        if (lanes == 8)                                                                                  \
            hipLaunchKernelGGL(kernel<8>, dim3(row_blocks), dim3(SMP_THREADS), 0, st, A);                \
        else if (lanes == 16)                                                                            \
            hipLaunchKernelGGL(kernel<16>, dim3(row_blocks), dim3(SMP_THREADS), 0, st, A);               \
        else                                                                                             \
            hipLaunchKernelGGL(kernel<32>, dim3(row_blocks), dim3(SMP_THREADS), 0, st, A);               \
        FG_LAUNCH_CHECK(#kernel);                                                                        \
    } while (0)
    FG_SMP(sample_draw_kernel);
    FG_SMP(sample_compact_kernel);
#undef FG_SMP
    hipLaunchKernelGGL(sample_resolve_kernel, dim3(cand_blocks), dim3(FG_SCAN_BLOCK), 0, st, A);
    FG_LAUNCH_CHECK("sample_resolve_kernel");
    if (cand_blocks <= (unsigned)SMP_PREFIX) {
        hipLaunchKernelGGL(sample_columns_kernel<true>, dim3(cand_blocks), dim3(FG_SCAN_BLOCK), (size_t)cand_blocks * 4, st, A);
    } else {
        hipLaunchKernelGGL(sample_prefix_kernel, dim3(1), dim3(FG_SCAN_BLOCK), 0, st, A);
        FG_LAUNCH_CHECK("sample_prefix_kernel");
        hipLaunchKernelGGL(sample_columns_kernel<false>, dim3(cand_blocks), dim3(FG_SCAN_BLOCK), 0, st, A);
    }
    FG_LAUNCH_CHECK("sample_columns_kernel");
    return FG_OK;
}

// ---- transpose of a sampled block (what the backward pass walks) ---------------------------------------------------
//
// For every position j of the layer below: the rows that sampled it, ascending, back to back. Launches: clear the
// counters; count the edges per source; exclusive scan (t_start, t_end; a workgroup adds up the counters before its own
// itself, or per-workgroup sums of a launch of their own where there are many); every edge takes a free place of its
// source's list (the order of arrival is arbitrary); every list is sorted (lists are short: a source is sampled by a
// handful of rows), which makes the result independent of that order. Rows are read by groups of lanes: one lane per row
// walked a chain of dependent atomics on a few compute units. A small block runs in one workgroup with everything in LDS.
// 6 k rows x 10 and 54 k sources: 32 us in six launches, now 24 in five; 1 k rows x 5: 25 us in six, now 10 in one.
namespace {

constexpr int TR_THREADS = 256;
constexpr int TR_LANES = 8;          // lanes per row
constexpr int TR_DIRECT = 128;       // workgroups of counters that are added up directly
// Sources, edges and rows of a block that one workgroup transposes: what fits its LDS. By itself it is level with the five launches
// at about half of that (rows x draws 1024 x 5 11 us against 13, 1024 x 7 18 against 14, 1024 x 11 22 against 15, 3000 x 2 22
// against 14), but five launches also cost the gaps between them and the host's time. A whole mini-batch, one workgroup / five
// launches for its block: 600 seeds x 3 x 4 x 5, the block of 2400 rows x 4, 146 us / 177; 1024 x 8 x 10 106 / 132; 1024 x 11 x 10 x 15,
// where the device is the bound, 742 / 752.
constexpr int TR_SMALL = 12288;

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

__global__ __launch_bounds__(TR_THREADS) void transpose_count_kernel(TrArgs A) {
    const int64_t n = tr_count(A.n_dev, A.max_rows), n_src = tr_count(A.n_src_dev, A.max_src);
    const int64_t i = ((int64_t)blockIdx.x * TR_THREADS + threadIdx.x) / TR_LANES;
    if (i < n) tr_row_edges(A, i, n_src, [&](int32_t, int32_t c) { atomicAdd(&A.cnt[c], 1); });
}

__global__ __launch_bounds__(FG_SCAN_BLOCK) void transpose_sum_kernel(TrArgs A) {
    __shared__ long long red[16];
    const int64_t j = (int64_t)blockIdx.x * FG_SCAN_BLOCK + threadIdx.x;
    const long long s = fg_block_sum(j < A.max_src ? (long long)A.cnt[j] : 0, red);
    if (threadIdx.x == 0) A.blk[blockIdx.x] = (int32_t)s;
}

// exclusive scan of one value per thread over the workgroup; `total`: their sum
__device__ __forceinline__ int tr_block_scan(int c, int& total) {
    __shared__ int wave_sum[FG_SCAN_BLOCK / FG_WAVE];
    int incl = c;  // inclusive scan over the wavefront, then the wavefronts before this one
    for (int off = 1; off < FG_WAVE; off <<= 1) {
        const int v = __shfl_up(incl, off, FG_WAVE);
        if (fg_lane() >= off) incl += v;
    }
    if (fg_lane() == FG_WAVE - 1) wave_sum[fg_wave()] = incl;
    __syncthreads();
    int earlier = 0;
    total = 0;
    for (int w = 0; w < FG_SCAN_BLOCK / FG_WAVE; ++w) {
        if (w < fg_wave()) earlier += wave_sum[w];
        total += wave_sum[w];
    }
    return earlier + incl - c;
}

// DIRECT: the counters of the workgroups before this one are added up here, else their sums
template <bool DIRECT>
__global__ __launch_bounds__(FG_SCAN_BLOCK) void transpose_scan_kernel(TrArgs A) {
    __shared__ long long red[16];
    const int64_t j = (int64_t)blockIdx.x * FG_SCAN_BLOCK + threadIdx.x;
    const int c = j < A.max_src ? A.cnt[j] : 0;
    long long before = 0;
    if (DIRECT) {
        const int ahead = (int)blockIdx.x * FG_SCAN_BLOCK;      // a multiple of 4: sixteen bytes at a time
#pragma unroll 4
        for (int b = threadIdx.x * 4; b < ahead; b += FG_SCAN_BLOCK * 4) {
            const int4 v = *(const int4*)(A.cnt + b);
            before += (long long)v.x + v.y + v.z + v.w;
        }
    } else {
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += FG_SCAN_BLOCK) before += A.blk[b];
    }
    before = fg_block_sum(before, red);
    int total;
    const long long first = before + tr_block_scan(c, total);
    if (j < A.max_src) {
        A.t_start[j] = (int32_t)first;
        A.t_end[j] = (int32_t)(first + c);
    }
}

__global__ __launch_bounds__(TR_THREADS) void transpose_fill_kernel(TrArgs A) {
    const int64_t n = tr_count(A.n_dev, A.max_rows), n_src = tr_count(A.n_src_dev, A.max_src);
    const int64_t i = ((int64_t)blockIdx.x * TR_THREADS + threadIdx.x) / TR_LANES;
    if (i < n)
        tr_row_edges(A, i, n_src, [&](int32_t row, int32_t c) {
            const int64_t at = (int64_t)A.t_end[c] - atomicSub(&A.cnt[c], 1);      // from the start on: nearly sorted as a rule
            if (at < A.max_nnz) A.t_row[at] = row;
        });
}

__global__ __launch_bounds__(TR_THREADS) void transpose_sort_kernel(TrArgs A) {
    const int64_t j = (int64_t)blockIdx.x * TR_THREADS + threadIdx.x;
    if (j >= A.max_src) return;
    tr_sort(A.t_row, A.t_start[j], A.t_end[j] < A.max_nnz ? A.t_end[j] : A.max_nnz);
}

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
    for (int j = t; j < src; j += FG_SCAN_BLOCK) tr_sort(list, j ? cnt[j - 1] : 0, cnt[j] < nnz ? cnt[j] : nnz);
    __syncthreads();
    const int stored = total < nnz ? total : nnz;
    for (int k = t; k < stored; k += FG_SCAN_BLOCK) A.t_row[k] = list[k];
}

size_t tr_layout(int64_t max_src, size_t* blk_at) {
    const size_t src = (size_t)(max_src > 0 ? max_src : 1);
    *blk_at = fg_align_up(src * 4, 256);
    return *blk_at + fg_align_up((size_t)fg_ceil_div((int64_t)src, FG_SCAN_BLOCK) * 4, 256);
}

}  // namespace

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
    const unsigned row_blocks = (unsigned)fg_ceil_div(max_rows > 0 ? max_rows : 1, TR_THREADS / TR_LANES);
    const unsigned scan_blocks = (unsigned)fg_ceil_div(max_src, FG_SCAN_BLOCK);
    if (max_rows > 0) {
        hipLaunchKernelGGL(transpose_count_kernel, dim3(row_blocks), dim3(TR_THREADS), 0, st, A);
        FG_LAUNCH_CHECK("transpose_count_kernel");
    }
    if (scan_blocks <= TR_DIRECT) {
        hipLaunchKernelGGL(transpose_scan_kernel<true>, dim3(scan_blocks), dim3(FG_SCAN_BLOCK), 0, st, A);
    } else {
        hipLaunchKernelGGL(transpose_sum_kernel, dim3(scan_blocks), dim3(FG_SCAN_BLOCK), 0, st, A);
        FG_LAUNCH_CHECK("transpose_sum_kernel");
        hipLaunchKernelGGL(transpose_scan_kernel<false>, dim3(scan_blocks), dim3(FG_SCAN_BLOCK), 0, st, A);
    }
    FG_LAUNCH_CHECK("transpose_scan_kernel");
    if (max_rows > 0) {
        hipLaunchKernelGGL(transpose_fill_kernel, dim3(row_blocks), dim3(TR_THREADS), 0, st, A);
        FG_LAUNCH_CHECK("transpose_fill_kernel");
        hipLaunchKernelGGL(transpose_sort_kernel, dim3((unsigned)fg_ceil_div(max_src, TR_THREADS)), dim3(TR_THREADS), 0, st, A);
        FG_LAUNCH_CHECK("transpose_sort_kernel");
    }
    return FG_OK;
}
