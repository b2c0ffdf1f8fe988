// The update of the caches: what its launches are told (cache.hip), and the one launch that decides it where a layer's positions are
// held in registers by workgroups that wait for each other. The same code runs as workgroups of the weight gradients' launch
// (backward.hip), which a training iteration's update depends on as little as they on it.
#pragma once
#include "common.h"
#include "meeting.h"
#include "scan.h"

struct UpdHeader {        // lives at the start of a layer's update workspace
    uint32_t tau_key;     // order-preserving key of tau, or its leading digits where no smaller key shares them
    int32_t mode;         // 0: nothing is below tau, 1: compare with tau_key, 2: everything is below tau
    int64_t n_admit;      // rows to copy (<= capacity)
    int64_t m_live;
    int64_t n_cand;       // access-aware policy: admissible nodes, and how many of those whose estimate equals the
    int64_t tie_room;     //   threshold estimate still fit (-1: every admissible node fits)
};

__device__ __forceinline__ int clamp_saving(int32_t a) { return a < 0 ? 0 : (a > 2047 ? 2047 : a); }

__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int SEL_THREADS = 1024;
constexpr int SEL_BINS = 2048;
constexpr int SEL_BPT = SEL_BINS / SEL_THREADS;  // bins owned by a thread in the scan
constexpr int SEL_CHUNK = 4 * SEL_THREADS;       // keys per workgroup in the histogram launches
constexpr int FG_MAX_UPD_LAYERS = 8;

// Selection scratch of a layer, owned by the cache. All-zero between updates: launch 4, or the last of the group, clears it again.
struct SelState {
    unsigned int hist0[SEL_BINS];
    unsigned int hist1[SEL_BINS];
    unsigned int n_surv;
    unsigned int arrived[3];       // workgroups that have counted their keys' digit (update_group_kernel)
    unsigned int done;             // ... and that have left the scratch alone
    unsigned int admits[64];       // a workgroup's admissible nodes, published (meeting.h)
    unsigned int hist2[SEL_BINS];  // estimates of saved accesses of the admissible nodes (access-aware policy), or the third digit
};

static_assert(SEL_BINS == 2048, "clamp_saving saturates the estimates at the last bin");

struct CacheRW {
    int32_t* map;
    int32_t* slot_node;
    int32_t* slot_stamp;
    const int64_t* head;  // current ring header
    int64_t* head_next;   // where an update leaves the advanced header (the two swap roles after every update)
    int64_t* used;        // slots written at least once (what the ring has overwritten of the shared buffer)
    int64_t capacity;
    int64_t num_nodes;
    int64_t iter;
    int32_t t_stale;
};

struct UpdLayer {
    CacheRW c;
    const int32_t* ids;
    const uint8_t* live;
    const uint8_t* hit;
    const float* gnorm;
    int64_t* stats;
    SelState* sel;
    UpdHeader* hdr;
    uint8_t* flag;       // per position: 0 not admitted, 1 admissible (in position order while there is room), 2 in for sure
    int32_t* blk;        // flag-1 nodes per workgroup of launch 3
    int32_t* blk_sure;   // flag-2 nodes per workgroup (access-aware policy)
    const int32_t* saving;  // estimates of saved accesses by position, or NULL
    int64_t room;        // rows this update may admit (<= capacity)
    int32_t* apos;       // admitted positions; before launch 4 the same memory holds the survivor keys
    int32_t* aslot;      // their slots
    const char* h;
    int64_t h_stride;
    char* table;
    int64_t row_bytes;
    int32_t n;           // positions of the layer: the caller's bound ...
    const int64_t* n_dev;  // ... and, if non-null, the count in device memory (positions at or beyond it are not live)
    float p_grad;
};

// positions of the layer that exist: the device-side count where the caller gave one, never above the bound
__device__ __forceinline__ int upd_count(const UpdLayer& L) {
    if (!L.n_dev) return L.n;
    const int64_t c = *L.n_dev;
    return c < 0 ? 0 : (c < (int64_t)L.n ? (int)c : L.n);
}

struct UpdBatch {
    int32_t n_layers;
    int32_t polls;                              // before a workgroup that waits for others gives up
    int32_t sel_first[FG_MAX_UPD_LAYERS + 1];   // first workgroup of each layer in launches 1 and 2
    int32_t scan_first[FG_MAX_UPD_LAYERS + 1];  // the same for launches 3 and 4
    UpdLayer l[FG_MAX_UPD_LAYERS];
};

// leaves the number of admitted rows, the advanced ring header and how far the ring has ever been written
__device__ __forceinline__ void finish_header(const UpdLayer& L, int64_t head, int64_t used, int64_t in) {
    const CacheRW& c = L.c;
    L.hdr->n_admit = in;
    const int64_t reach = head + in;  // the ring fills slots upwards until it first wraps (head < capacity, in <= capacity)
    *c.head_next = reach < c.capacity ? reach : reach - c.capacity;
    if (reach >= c.capacity)
        *c.used = c.capacity;
    else if (reach > used)
        *c.used = reach;
}

__device__ __forceinline__ int layer_of_block(const int32_t* first, int n_layers, int b, int& local) {
    int l = 0;
    while (l + 1 < n_layers && b >= first[l + 1]) ++l;
    local = b - first[l];
    return l;
}

// ---- launches 1 to 4 as one: a layer by one workgroup per 4096 positions --------------------------------------------------------
//
// What bounds the four launches is not their work but their chain: each is a few dependent reads, barriers
// and scans long (6 + 9 + 13 + 6 us at 1.2 k positions, hardly more at 54 k), and workgroups of 1024 threads wait for room beside the
// weight gradients (the third launch, 72 of them at 67 k positions, 33 us there). A workgroup of 1024 threads holds the keys of
// 4096 positions in registers (four per thread), so it reads them once, finds tau by up to three digits,
// classifies, ranks the admissible nodes and hands out their slots. By itself it finds the digits in LDS; the workgroups of a larger
// layer meet up to four times: behind the histogram of each digit, and behind the check-outs, with the numbers of admissible nodes. (The keys that
// carry the first digit as a list, from which each workgroup finds the other two for itself: a meeting less, but up to a third of
// a layer's norms share a digit, and at 67 k positions the list took 5 + 6 us, 5 + 11 in a GCN, for 9 of two meetings.) The
// histograms are kept four times (by lane mod 4): norms share their leading digits, and equal bins of a wavefront are
// added one after the other.
// Who waits needs no more than that the other workgroups start: they are at most 64 in all, so that they are all there together on a chip
// with room for 512 of their size (for 256 where they share the weight gradients' launch: they are its first), and a launch they
// have to wait behind ends without them. The polls are bounded all the same: a workgroup
// that gives up takes its whole layer along (meeting.h), which then admits nothing and says so in its statistics; what it has checked
// out until then stays out.
// Between the barriers the chain is kept short: prefix sums inside the vector registers, a wavefront's place among the others' totals from
// four wide LDS reads, each thread clearing the counters it read, no division (with shuffles, a loop over the wavefronts and 64-bit
// remainders 17.6 us at 1.2 k positions, 14.2 so, 12.9 with two digits where they decide; a third of what is left is the row copy and the first reads).
// Measured, the four launches and now: 28 k positions 36 us and their gaps, 24; 74 k beside the weight gradients of 55 k rows 66, 27; 1.2 k with
// its row copy 31, 13 (one workgroup).
constexpr int ONE_COPIES = 4;
constexpr int GRP_CHUNK = SEL_CHUNK;            // positions of a workgroup
constexpr int GRP_MAX = 64;                     // workgroups of a launch

static __device__ __attribute__((aligned(16))) uint32_t upd_spare[4];      // what is read where a layer has no quad

// LDS of a workgroup of WAVES wavefronts
template <int WAVES>
struct GrpShared {
    __attribute__((aligned(16))) uint32_t hist[SEL_BINS * ONE_COPIES];
    __attribute__((aligned(16))) int wave_count[WAVES];
    __attribute__((aligned(16))) uint32_t red[2][WAVES];      // alternating: read while the next pass writes
    uint2 found[3];      // by digit: its value, and the rank of tau among the keys that carry it and those before
    int evicted, over, ok, before, all;
};

// Place of a thread's BPT of 2048 counters: the sum of those of the threads before it, and of all. `red` needs WAVES words and is read
// until the next barrier.
template <int WAVES, int BPT>
__device__ __forceinline__ uint32_t grp_scan(const uint32_t (&c)[BPT], uint32_t* red, uint32_t& all) {
    uint32_t own = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) own += c[q];
    const uint32_t incl = (uint32_t)fg_wave_scan((int)own);
    if (fg_lane() == FG_WAVE - 1) red[fg_wave()] = incl;
    __syncthreads();
    uint32_t before;
    fg_wave_totals<WAVES>((const int*)red, (int&)before, (int&)all);
    return before + incl - own;
}

// The thread whose bins hold the key of rank `rank` leaves the bin and the rank within it; c and lo as grp_scan has them.
template <int BPT>
__device__ __forceinline__ void grp_find(const uint32_t (&c)[BPT], uint32_t lo, uint32_t rank, uint2* out) {
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
        if (rank >= lo && rank < lo + c[q]) *out = uint2{BPT * threadIdx.x + q, rank - lo};
        lo += c[q];
    }
}

// This thread's counters of hist[bin * ONE_COPIES + copy], which are zero again afterwards
template <int BPT>
__device__ __forceinline__ void grp_take(uint32_t* hist, uint32_t (&c)[BPT]) {
    static_assert(ONE_COPIES == 4, "four counters per bin");
    uint4* mine = (uint4*)hist + BPT * threadIdx.x;
    uint4 a[BPT];
#pragma unroll
    for (int q = 0; q < BPT; ++q) a[q] = mine[q];
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
        mine[q] = uint4{0, 0, 0, 0};
        c[q] = a[q].x + a[q].y + a[q].z + a[q].w;
    }
}

// What the workgroups of a layer tell each other goes past the caches of their XCDs, word by word (atomics of agent scope); before a
// workgroup says that it is there, each of its wavefronts waits until its own have arrived. (Release and acquire fences instead
// write back and invalidate whole L2s: some 3 us more for each meeting, 15 beside the weight gradients.)
template <typename T>
__device__ __forceinline__ T grp_load(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void grp_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void grp_arrive() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// All `n` workgroups of a layer have come here and none has given up.
__device__ __forceinline__ bool grp_meet(unsigned int* arrived, unsigned int n, int polls, int* s_ok) {
    grp_arrive();
    if (threadIdx.x == 0) *s_ok = fg_meet(FgAgentMem{}, arrived, n, polls);
    __syncthreads();
    return *s_ok != 0;
}

// COPY (every layer has one workgroup): the admitted rows are copied here as well (a launch less) instead of by the row copy behind it.
// QUADS: four positions each, of a thread. block: which of the group's workgroups this is.
template <int THREADS, int QUADS, bool COPY>
__device__ __forceinline__ void update_group(const UpdBatch& B, const int block, GrpShared<THREADS / FG_WAVE>& S) {
    constexpr int EL = 4 * QUADS, BPT = SEL_BINS / THREADS, WAVES = THREADS / FG_WAVE;
    constexpr int CHUNK = THREADS * EL;      // positions of a workgroup: B.sel_first counts such chunks
    uint32_t* const hist = S.hist;
    int part;
    const int layer = layer_of_block(B.sel_first, B.n_layers, block, part);
    const UpdLayer& L = B.l[layer];
    const CacheRW& c = L.c;
    const unsigned int parts = (unsigned int)(B.sel_first[layer + 1] - B.sel_first[layer]);
    const int t = threadIdx.x, lane = fg_lane(), wave = fg_wave();
    const int n_all = upd_count(L), base = part * CHUNK;
    const int n = n_all - base < 0 ? 0 : (n_all - base < CHUNK ? n_all - base : CHUNK);      // positions of this workgroup
    const int64_t head = *c.head, used = *c.used;
    // Position of element e: base + EL * t + e. Every read is unconditional (the first quad, or 16 bytes of the
    // library's own, where a quad is not wholly there) so that they are in flight together; the one quad that the end of the layer
    // cuts is read one by one by the thread that owns it, and joins below.
    const int n_quads = n >> 2;
    uint32_t key[EL], is_live = 0, is_hit = 0;      // a bit per element
    int32_t id[EL];
    {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const bool any = n_quads > 0;
        const char* none = (const char*)upd_spare;
        const char* hit_base = any ? (const char*)L.hit + base : none;
        f4 g[QUADS];
        uint32_t l4[QUADS], h4[QUADS];
        int4 v4[QUADS];
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            const uint32_t at = QUADS * t + q < n_quads ? (uint32_t)(QUADS * t + q) : 0u;
            g[q] = *(const f4*)((any ? (const char*)L.gnorm + 4 * (int64_t)base : none) + 16u * at);
            l4[q] = *(const uint32_t*)((any && L.live ? (const char*)L.live + base : hit_base) + 4u * at) | (L.live ? 0u : 0x01010101u);
            h4[q] = *(const uint32_t*)(hit_base + 4u * at);
            v4[q] = *(const int4*)((any ? (const char*)L.ids + 4 * (int64_t)base : none) + 16u * at);
        }
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            id[4 * q] = v4[q].x;
            id[4 * q + 1] = v4[q].y;
            id[4 * q + 2] = v4[q].z;
            id[4 * q + 3] = v4[q].w;
            const bool whole = QUADS * t + q < n_quads;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                key[4 * q + e] = order_key(g[q][e]);
                is_live |= whole && ((l4[q] >> (8 * e)) & 0xFFu) ? 1u << (4 * q + e) : 0u;
                is_hit |= whole && ((h4[q] >> (8 * e)) & 0xFFu) ? 1u << (4 * q + e) : 0u;
            }
            if ((n & 3) != 0 && n_quads == QUADS * t + q)
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const int j = base + 4 * n_quads + e;
                    if (j >= n_all) continue;
                    key[4 * q + e] = order_key(L.gnorm[j]);
                    id[4 * q + e] = L.ids[j];
                    if (L.live ? L.live[j] != 0 : true) is_live |= 1u << (4 * q + e);
                    if (L.hit[j] != 0) is_hit |= 1u << (4 * q + e);
                }
        }
    }
    auto count_key = [&](uint32_t bin) { atomicAdd(&hist[bin * ONE_COPIES + (lane & (ONE_COPIES - 1))], 1u); };
    if (t == 0) S.evicted = S.over = 0;
    for (int b = t; b < SEL_BINS * ONE_COPIES / 4; b += THREADS) ((uint4*)hist)[b] = uint4{0, 0, 0, 0};
    bool lost = false;
    uint32_t m = 0, tau_key = 0;
    int mode = 1;
    if (parts > 1 && part == 0 && t < 4 && L.stats) grp_store(&L.stats[t], (int64_t)0);
    __syncthreads();
    // tau is the key of rank k, found digit by digit (11 + 11 + 10 bits); mode is the same for all workgroups of the layer. A key that is the
    // smallest of those with its digits so far divides the others as these digits with zeros behind them do: of a few thousand norms
    // two digits are as good as always enough.
    bool exact = false;
#pragma unroll 1
    for (int pass = 0; pass < 3 && mode == 1 && !exact; ++pass) {
        const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
        const uint32_t bins = pass == 2 ? 1023u : 2047u;
        const uint32_t above = pass == 0 ? 0u : (pass == 1 ? 0xFFE00000u : 0xFFFFFC00u);      // the digits found so far
#pragma unroll
        for (int e = 0; e < EL; ++e)
            if (((is_live >> e) & 1u) && (key[e] & above) == tau_key) count_key((key[e] >> shift) & bins);
        __syncthreads();
        uint32_t c[BPT], all;
        grp_take(hist, c);
        if (parts > 1) {
            unsigned int* shared = pass == 0 ? L.sel->hist0 : (pass == 1 ? L.sel->hist1 : L.sel->hist2);
#pragma unroll
            for (int q = 0; q < BPT; ++q)
                if (c[q]) atomicAdd(&shared[BPT * t + q], c[q]);
            lost = !grp_meet(&L.sel->arrived[pass], parts, B.polls, &S.ok);
#pragma unroll
            for (int q = 0; q < BPT; ++q) c[q] = grp_load(&shared[BPT * t + q]);
        }
        const uint32_t lo = grp_scan<WAVES>(c, S.red[pass & 1], all);
        uint32_t rank;
        if (pass == 0) {
            m = all;
            const long long k = (long long)floor((double)L.p_grad * (double)m);
            mode = k <= 0 ? 0 : (k >= (long long)m ? 2 : 1);
            rank = (uint32_t)k;
        } else {
            rank = S.found[pass - 1].y;
        }
        if (lost) {
            mode = 0;
            if (t == 0)
                for (int p = pass + 1; p < 3; ++p) fg_lost_ahead(FgAgentMem{}, &L.sel->arrived[p]);
        }
        if (mode == 1) {
            grp_find(c, lo, rank, &S.found[pass]);
            __syncthreads();
            tau_key |= S.found[pass].x << shift;
            exact = S.found[pass].y == 0;
        }
    }
    // check-outs and admissible nodes
    uint32_t admit_bits = 0;
    int evicted = 0;
#pragma unroll
    for (int e = 0; e < EL; ++e) {
        const bool low = mode == 2 || (mode == 1 && key[e] < tau_key);
        if (lost || !((is_live >> e) & 1u) || id[e] < 0 || id[e] >= c.num_nodes || (((is_hit >> e) & 1u) != 0) == low) continue;
        if (low) {
            admit_bits |= 1u << e;
        } else {
            grp_store(&c.map[id[e]], -1);
            ++evicted;
        }
    }
    // ranks in position order: workgroups first, then threads, then a thread's elements
    const int own = __popc(admit_bits);
    const int both = fg_wave_scan(own | evicted << 16), incl = both & 0xFFFF;      // (at most 1024 of each in a wavefront)
    if (lane == FG_WAVE - 1) {
        S.wave_count[wave] = incl;
        if (both >> 16) atomicAdd(&S.evicted, both >> 16);
    }
    __syncthreads();
    int before, total;
    fg_wave_totals<WAVES>(S.wave_count, before, total);
    before += incl - own;
    if (parts > 1) {      // what the other workgroups admit, behind all check-outs
        grp_arrive();
        if (wave == 0) {
            uint32_t w = FG_PUBLISHED;
            if (t == 0) fg_publish(FgAgentMem{}, &L.sel->admits[part], lost ? FG_GIVEN_UP : (uint32_t)total);
            if (t < (int)parts && !lost) w = fg_settled(FgAgentMem{}, &L.sel->admits[t], B.polls);
            int there = (int)(w & ~(FG_PUBLISHED | FG_GIVEN_UP)), ahead = t < part ? there : 0;
            for (int off = FG_WAVE / 2; off > 0; off >>= 1) {
                there += __shfl_xor(there, off, FG_WAVE);
                ahead += __shfl_xor(ahead, off, FG_WAVE);
            }
            const bool all_there = __all((w & FG_GIVEN_UP) == 0) && !lost;
            if (t == 0) {
                S.before = ahead;
                S.all = there;
                S.ok = all_there;
            }
        }
        __syncthreads();
        before += S.before;
        total = S.all;
        if (!S.ok) lost = true;
    }
    if (lost) admit_bits = 0;
    int over = 0;
    {
        int32_t slot[EL], old[EL], old_map[EL], old_stamp[EL];
        int rank[EL];
        bool in[EL];
        // the chains slot -> owner -> its map entry side by side (reads of slot 0 / node 0 where there is nothing to do)
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            rank[e] = before + __popc(admit_bits & ((1u << e) - 1u));
            in[e] = ((admit_bits >> e) & 1u) != 0 && rank[e] < L.room;
            const int64_t at = head + rank[e];      // head < capacity, rank < room <= capacity
            slot[e] = in[e] ? (int32_t)(at < c.capacity ? at : at - c.capacity) : 0;
            old[e] = c.slot_node[slot[e]];
            old_stamp[e] = c.slot_stamp[slot[e]];
        }
#pragma unroll
        for (int e = 0; e < EL; ++e) old_map[e] = grp_load(&c.map[old[e] >= 0 && old[e] < c.num_nodes ? old[e] : 0]);
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            if (!in[e]) continue;
            if (old[e] >= 0 && old[e] < c.num_nodes && old_map[e] == slot[e]) {
                const int64_t age = c.iter + 1 - (int64_t)old_stamp[e];
                over += age >= 1 && age <= (int64_t)c.t_stale ? 1 : 0;
            }
            c.slot_node[slot[e]] = id[e];
            c.slot_stamp[slot[e]] = (int32_t)c.iter;
            c.map[id[e]] = slot[e];
            L.apos[rank[e]] = base + EL * t + e;
            L.aslot[rank[e]] = slot[e];
            if (COPY) ((int2*)hist)[rank[e]] = int2{EL * t + e, slot[e]};      // (the histograms are not needed any more)
        }
    }
    over = fg_wave_scan(over);
    if (lane == FG_WAVE - 1 && over) atomicAdd(&S.over, over);
    __syncthreads();
    if (t == 0) {
        const int64_t in = lost ? 0 : (total < L.room ? total : L.room);
        if (part == 0) {
            L.hdr->mode = mode;
            L.hdr->tau_key = tau_key;
            L.hdr->m_live = m;
            finish_header(L, head, used, in);
        }
        if (L.stats) {
            if (part == 0) {
                L.stats[0] = lost ? -1 : in;
                L.stats[3] = lost ? -1 : total - in;
            }
            if (parts == 1) {
                L.stats[1] = S.evicted;
                L.stats[2] = S.over;
            } else {
                if (S.evicted) atomicAdd((unsigned long long*)&L.stats[1], (unsigned long long)S.evicted);
                if (S.over) atomicAdd((unsigned long long*)&L.stats[2], (unsigned long long)S.over);
            }
        }
        // the last to come here clears the scratch: nobody reads it any more
        if (parts > 1) S.ok = __hip_atomic_fetch_add(&L.sel->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
    }
    if (parts > 1) {
        __syncthreads();
        if (S.ok) {
            for (int b = t; b < SEL_BINS; b += THREADS) L.sel->hist0[b] = L.sel->hist1[b] = L.sel->hist2[b] = 0;
            if (t < 64) L.sel->admits[t] = 0;
            if (t < 3) L.sel->arrived[t] = 0;
            if (t == 0) L.sel->done = 0;
        }
    }
    if constexpr (COPY) {
        static_assert(sizeof(S.hist) >= CHUNK * sizeof(int2), "every position may be admitted");
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const int pieces = (int)(L.row_bytes >> 4), items = (int)(total < L.room ? total : L.room) * pieces;
        constexpr int TOGETHER = 8;
        for (int i0 = t; i0 < items; i0 += TOGETHER * THREADS) {
            u32x4 v[TOGETHER];
#pragma unroll
            for (int u = 0; u < TOGETHER; ++u) {
                const int i = i0 + u * THREADS < items ? i0 + u * THREADS : i0, r = i / pieces;
                v[u] = *((const u32x4*)(L.h + (int64_t)((const int2*)hist)[r].x * L.h_stride) + (i - r * pieces));
            }
#pragma unroll
            for (int u = 0; u < TOGETHER; ++u) {
                const int i = i0 + u * THREADS, r = i / pieces;
                if (i < items) *((u32x4*)(L.table + (int64_t)((const int2*)hist)[r].y * L.row_bytes) + (i - r * pieces)) = v[u];
            }
        }
    }
}

// ---- an update that rides along with another launch -----------------------------------------------------------------------------
struct fg_update_call {
    fg_cache_t* cache;
    int64_t iter;
    float p_grad;
    int32_t n_layers;
    const fg_update_layer_t* layers;
    void* ws;
    size_t ws_bytes;
};
// Checks the call as fg_cache_update_all does and describes it. *rides: its group may be the first sel_first[n_layers] workgroups of another launch
// (512 threads, 2 quads each), and the row copies part of the one behind it; else B says nothing and fg_cache_update_all is to be called.
fg_status_t fg_update_describe(const char* who, const fg_update_call& call, UpdBatch* B, bool* rides);
void fg_update_row_copies(const UpdBatch& B, fg_row_copy_batch* copies);
void fg_update_queued(const fg_update_call& call);      // both are queued: the cache's state moves on ...
void fg_update_selected(const fg_update_call& call);    // ... or in two steps: the group is queued (until the other step the next update is refused)
void fg_update_committed(const fg_update_call& call);   // ... and the row copies,
// or they are queued, some of them on another stream: fg_cache_update_commit then waits for this event in their place
void fg_update_rows_queued(const fg_update_call& call, void* event);
bool fg_update_rows_are_queued(const fg_cache_t* cache, int64_t iter);
// fg_backward_weights_all with an update that rides along (NULL: none)
fg_status_t fg_backward_weights_with(fg_dtype_t compute_dtype, int32_t n_layers, const fg_weight_grad_layer_t* layers, void* ws_dev, size_t ws_bytes,
                                     const UpdBatch* update, void* stream);
// fg_gather_aggregate_ids with an update's selection that rides along, if the launch is one for it (*rode; the row copies are then still due)
fg_status_t fg_gather_aggregate_ids_with(const int32_t* row_start_dev, const int32_t* row_end_dev, const int32_t* col_ids_dev, int64_t nnz,
                                         int32_t n_block_rows, const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                         const int32_t* row_ids_dev, const void* table, int64_t table_rows, int64_t src_stride, int32_t dim,
                                         fg_dtype_t in_dtype, void* agg, int64_t agg_stride, fg_dtype_t out_dtype, void* h_self_out, int64_t h_self_stride,
                                         int32_t n_self_rows, const fg_cache_t* cache, int32_t n_fetch_layers, const fg_fetch_layer_t* fetch_layers,
                                         const UpdBatch* update, bool* rode, void* stream);
// whether that launch is one for a loader of `max_rows` rows with at most most_hits cached rows of a layer to fetch
bool fg_loader_takes_update(int64_t max_rows, int32_t dim, fg_dtype_t dtype, int64_t most_hits, int update_blocks);
// fg_gather_aggregate_linear_ids likewise, for at most so many chunks of 4096 positions: two of them to a workgroup, which takes a compute unit from the
// loader. Steps beside a second stream, against own launches for the selection: 9 to 16 chunks 0.965, 17 to 32 0.99; with all riding 33 to 48 0.99, 49 to 64
// 0.997 (medians of 93 steps; up to 4.5 % longer there). On one stream 33 to 64 would be 0.95 to 0.97 of what they are.
constexpr int fg_load_linear_update_chunks = 32;
fg_status_t fg_gather_aggregate_linear_ids_with(const int32_t* row_start_dev, const int32_t* row_end_dev, const int32_t* col_ids_dev, int64_t nnz,
                                                int32_t n_block_rows, const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                                const int32_t* row_ids_dev, const float* table, int64_t table_rows, int64_t src_stride, int32_t d_in,
                                                int32_t d_out, const float* W, const float* bias, int32_t relu, float* agg_ws, int64_t agg_stride,
                                                float* h_out, int32_t n_out, int64_t out_stride, const fg_cache_t* cache, int32_t n_fetch_layers,
                                                const fg_fetch_layer_t* fetch_layers, const UpdBatch* update, bool* rode, void* stream);
