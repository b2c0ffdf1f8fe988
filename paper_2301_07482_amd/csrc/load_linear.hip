// The loader and the dense update of the lowest layer as one launch: h_out[r, :] = act([x_r ‖ mean of the sampled neighbours' x] . W + bias),
// x the raw features, straight from the table (fg_gather_aggregate_ids and fg_linear_ids in one).
//
// What bounds the two launches is not the same: the loader waits for memory (54 k rows x 13.1 random 512-byte rows of the table, 67 us at
// 5.5 TB/s) with the matrix cores idle, and the dense update (54 k x 256 x 256, 46 to 54 us) is bound by its instructions with the memory idle. Here
// a workgroup of 8 wavefronts, one on each compute unit, does both for blocks of 32 rows: every wavefront gathers 4 rows of a block, sums them in
// double in the order of the two launches, splits them into LDS, and multiplies the block by the 32 columns of W that it holds in registers, split.
// 96 KB of table rows a compute unit stay under way, over the multiplication too. Workgroups that start together would all gather and then all
// multiply: half of them start half a block later, so that one half reads while the other multiplies (54 k rows: 109 us without, 102 with). Cached
// rows that are fetched beside it are copied by the later half, in place of waiting.
// One launch against two, us: 17 k rows x (128 + 128) x 256, fan-out 15: 47 / 51.5; 41 k 82 / 95; 54 k 102 / 116; 82 k 149 / 171; fan-out 7 73 / 80;
// 57 k x (100 + 100) x 256 108 / 127; 54 k x (64 + 64) x 128 55 / 59; 31 k x (52 + 52) x 88 33 / 37. The matrix instructions of 54 k rows take
// 22 us, the rows 62 at the rate of a copy; what is above is the first block's chain of reads and W's split (5 us), the multiplication's waits for
// LDS and the part of it that the other half's reads do not cover.
#include "update_group.h"

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef f32x4 f32x4a __attribute__((aligned(4)));      // 16 bytes from an address that is a multiple of 4

constexpr int LL_THREADS = 512, LL_WAVES = LL_THREADS / 64;
constexpr int LL_SEG = 33;                    // 16-byte units a half-wavefront's fragment takes in LDS: 32 rows and one of padding
constexpr int LL_UNIT = 4;                    // loads of 1 KB that are waited for together
constexpr int LL_RING = 3;                    // such units of a wavefront that are under way
constexpr int LL_LIST = 16;                   // row blocks whose rows a workgroup lists ahead (two halves, one filled while the other is used)
constexpr int LL_UPD_CHUNK = 8192;            // positions of a workgroup of an update that rides along
constexpr int LL_GROUPS = 256;                // workgroups: one on each compute unit, by its LDS
constexpr size_t ll_lds_bytes(int ks) {
    return (size_t)ks * 6 * LL_SEG * 16 + (size_t)LL_WAVES * LL_RING * LL_UNIT * 1024 + (size_t)LL_WAVES * 2 * 64 * 8 + (size_t)2 * LL_LIST * 32 * 4 +
           LL_WAVES * 32 * 4;
}
static_assert(ll_lds_bytes(16) <= 160 * 1024 && LL_GROUPS % 16 == 0, "LDS of a compute unit; two halves");

__device__ __attribute__((aligned(16))) float ll_zero[128];      // what is read where there is no row

// 16 bytes from memory to LDS, a lane's at dst + 16 * lane (dst uniform over the wavefront); the table's rows are read once (nt)
__device__ __forceinline__ void load_lds16(const void* src, void* dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 2);
}
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// all but the last N of this wavefront's accesses to memory are done
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory"); }

__device__ __forceinline__ f32x16 mfma_bf16(const u32x4& a, const u32x4& b, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// the next of the three bf16 terms of two values (x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2), nearest even); x keeps what is left
__device__ __forceinline__ unsigned int next_term(float& a, float& b) {
    const f32x2 x = {a, b};
    const unsigned int u = __builtin_bit_cast(unsigned int, __builtin_convertvector(x, bf16x2));
    a -= __uint_as_float(u << 16);
    b -= __uint_as_float(u & 0xFFFF0000u);
    return u;
}

// the value of lane `lane ^ N`
template <int N>
__device__ __forceinline__ double other_half(double v) {
    const unsigned int lo = (unsigned int)__double2loint(v), hi = (unsigned int)__double2hiint(v);
    const bool upper = (threadIdx.x & N) != 0;
    const auto l = N == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false) : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = N == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false) : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)(upper ? h[0] : h[1]), (int)(upper ? l[0] : l[1]));
}

struct LoadLinear {
    const int32_t *row_start, *row_end, *col_ids, *rows, *row_ids;
    const int64_t* n_rows_dev;
    int64_t nnz, max_rows;
    int n_block_rows, d_in, d_out;
    const char* table;
    int64_t table_rows;
    uint32_t src_stride;
    const float *W, *bias;
    char* h_out;
    int64_t out_stride;
    int n_out, relu, groups;           // groups: workgroups, a multiple of 8
    fg_row_copy_batch copies;          // cached rows that are fetched beside it
};

// U: the selection of the iteration's cache update (n_layers 0: none), as the first workgroups, a compute unit each, which the loader then has
// fewer of (large step with 16 fewer 194.4 us, 193.7 with all); hence twice the positions of the update's own workgroups
// (with 4096 of them large 182.4 us, medium 188.9). On a second stream the selection found no compute unit before this launch ended, and the next
// step waited for it and the top-down pass behind it: large step 194.5 -> 179.3 us, with the paper's thresholds 178.4 -> 166.5, medium 182.7 -> 179.0.
// W's split columns are 192 registers of a lane at KS 16. What is left does not hold the gather too: 6 vector registers are spilled (28 bytes of
// scratch a lane), and since the selection is part of the kernel 29 scalar ones; KS 8 takes 208 registers and spills no vector register.
// KS: steps of 16 of the contraction; SLOTS: rows of the table a block's row is given (its own and SLOTS - 1 neighbours; what is beyond is read in a
// loop of its own); LP: lanes a table row takes.
template <int KS, int SLOTS, int LP>
__global__ __launch_bounds__(LL_THREADS, 2) void load_linear_kernel(LoadLinear A, UpdBatch U) {
    const int beside = U.n_layers ? U.sel_first[U.n_layers] : 0, block = (int)blockIdx.x - beside;
    if (block < 0) {
        extern __shared__ __attribute__((aligned(16))) char group_lds[];
        update_group<LL_THREADS, LL_UPD_CHUNK / 4 / LL_THREADS, false>(U, (int)blockIdx.x, *(GrpShared<LL_WAVES>*)group_lds);
        return;
    }
    constexpr int RPI = 64 / LP;                    // table rows of a load instruction
    constexpr int IPR = SLOTS / RPI;                // load instructions of a block's row
    constexpr int RPW = 32 / LL_WAVES;              // rows of a block a wavefront gathers
    constexpr int NU = RPW * IPR / LL_UNIT;         // units of a block
    static_assert(NU > LL_RING && RPW * 16 == 64, "what is under way belongs to this block or the next; a lane per row and neighbour");
    extern __shared__ __attribute__((aligned(16))) u32x4 frags[];      // the block's operand: [KS][term][half-wavefront][row]
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    char* const raw = (char*)(frags + KS * 6 * LL_SEG) + wave * (LL_RING * LL_UNIT * 1024);
    char* const behind = (char*)(frags + KS * 6 * LL_SEG) + LL_WAVES * (LL_RING * LL_UNIT * 1024);
    uint64_t* const addr = (uint64_t*)behind + wave * (2 * 64);      // [block, mod 2][row][slot]: where the row of the table starts
    int32_t* const rowlist = (int32_t*)((uint64_t*)behind + LL_WAVES * (2 * 64));
    int32_t* const srclist = rowlist + LL_LIST * 32;
    float* const bias_lds = (float*)(srclist + LL_LIST * 32);
    // Workgroups 8 .. 15 of every 16 (one and the other half of each die's compute units) are the later half: they start half a block later and
    // come last when blocks are given out, so where these do not come out even it is they who have one less.
    const int K = 2 * A.d_in, pieces = A.d_in >> 2;
    const bool later = (block & 8) != 0;
    const int earlier = (A.groups + 8) / 16 * 8;      // workgroups of the earlier half: half of them, or eight more than of the other
    const int group = (block >> 4 << 3 | (block & 7)) + (later ? earlier : 0);
    int64_t n_rows = A.n_rows_dev ? *A.n_rows_dev : A.max_rows;
    if (n_rows > A.max_rows) n_rows = A.max_rows;
    uint64_t spent = __builtin_readcyclecounter();
    if (later)
        for (int c = 0; c < A.copies.n; ++c)
            fg_copy_rows_part(A.copies.c[c], (int64_t)(group - earlier) * LL_WAVES + wave, (int64_t)(A.groups - earlier) * LL_WAVES, lane);
    spent = __builtin_readcyclecounter() - spent;
    const int n_blocks = (int)((n_rows + 31) >> 5);
    if (group >= n_blocks) return;                    // uniform over the workgroup, before any barrier
    const int n_tasks = (n_blocks - group + A.groups - 1) / A.groups;

    // Rows of task first + t / 32 (a task is one row block) and where their own features are: -1 past the end or out of range
    auto list_rows = [&](int first) {
        const int task = first + (t >> 5), at = (task % LL_LIST) * 32 + (t & 31);
        const int64_t g = ((int64_t)group + (int64_t)task * A.groups) * 32 + (t & 31);
        int32_t r = -1, s = -1;
        if (g < n_rows) {
            r = A.rows ? A.rows[g] : (int32_t)g;
            if (r < 0 || r >= A.n_block_rows) r = -1;
            if (r >= 0) s = A.row_ids[r];
            if (s < 0 || s >= A.table_rows) s = -1;
        }
        rowlist[at] = r;
        srclist[at] = s;
    };
    static_assert(LL_LIST * 32 == LL_THREADS, "an entry per thread");
    list_rows(0);
    if (t < LL_WAVES * 32) bias_lds[t] = A.bias && t < A.d_out ? A.bias[t] : 0.f;
    for (int i = t; i < KS * 6 * LL_SEG; i += LL_THREADS) frags[i] = u32x4{0, 0, 0, 0};      // (k from K up stays so)
    // this wavefront's part of W: column block `wave`, three terms. Columns from d_out up hold another column's values (their results are not
    // stored), k from K up zeros.
    const int n0 = wave * 32;
    u32x4 w[KS][3];
    {
        const uint32_t c = n0 + l32 < A.d_out ? n0 + l32 : 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k0 = ks * 16 + 8 * half;
            float v[8];
            const uint32_t off = (k0 < K ? (uint32_t)k0 * (uint32_t)A.d_out : 0u) + c;      // K is a multiple of 8: eight values exist together
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (A.W + (int64_t)e * A.d_out)[off];
            if ((ks + 1) * 16 > K)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = k0 < K ? v[e] : 0.f;
#pragma unroll
            for (int term = 0; term < 3; ++term)
#pragma unroll
                for (int p = 0; p < 4; ++p) w[ks][term][p] = next_term(v[2 * p], v[2 * p + 1]);
        }
    }
    lds_barrier();

    // A wavefront gathers rows 4 * wave .. + 3 of a block. Lane 16 * i + e stands for slot e of row i: the row itself, then its neighbours.
    const int my_row = RPW * wave + (lane >> 4), my_slot = lane & 15;
    struct Range {
        int32_t first, deg, own;      // first neighbour's place in col_ids, their number, the row's own table row
    };
    auto range_of = [&](int task) {
        Range R{0, 0, -1};
        if (task < n_tasks) {
            const int at = (task % LL_LIST) * 32 + my_row;
            const int32_t r = rowlist[at];
            R.own = srclist[at];
            const int32_t rr = r >= 0 ? r : 0;
            const int32_t s0 = A.row_start[rr], e0 = A.row_end[rr];
            if (r >= 0 && s0 >= 0 && e0 >= s0 && (int64_t)e0 <= A.nnz) {
                R.first = s0;
                R.deg = e0 - s0;
            }
        }
        return R;
    };
    auto slot_of = [&](const Range& R) -> int32_t {      // the table row of this lane's slot, or -1
        const bool there = my_slot > 0 && my_slot <= R.deg;
        const int32_t c = A.nnz > 0 ? A.col_ids[there ? R.first + my_slot - 1 : 0] : -1;
        return my_slot == 0 ? R.own : (there ? c : -1);
    };
    auto address = [&](int32_t c, int parity) {
        const bool ok = c >= 0 && c < A.table_rows;
        addr[parity * 64 + lane] = ok ? (uint64_t)A.table + (uint64_t)(uint32_t)c * A.src_stride : (uint64_t)ll_zero;
    };
    const int sub = lane / LP, piece = lane % LP;
    const bool has_piece = piece < pieces;
    // Every lane's 16 bytes of a row, or 16 zeros where there is no row (ll_zero is as long as a row) or no such piece
    const uint32_t my_bytes = has_piece ? 16u * piece : 0u;
    auto issue = [&](int u, int ring_at, int parity) {      // unit u (a constant) of a block
        uint64_t at[LL_UNIT];
#pragma unroll
        for (int q = 0; q < LL_UNIT; ++q) {
            const int i = u * LL_UNIT + q, row = i / IPR, s0 = i % IPR * RPI;
            at[q] = addr[parity * 64 + row * 16 + s0 + sub];
        }
#pragma unroll
        for (int q = 0; q < LL_UNIT; ++q) load_lds16((const char*)(at[q] + my_bytes), raw + (ring_at * LL_UNIT + q) * 1024);
    };
    const char* const lane_table = A.table + my_bytes;

    int ring_at = 0;      // unit of the ring that is read next
    Range now = range_of(0), next = range_of(1);
    address(slot_of(now), 0);
#pragma unroll
    for (int u = 0; u < LL_RING; ++u) issue(u, u, 0);

    // where this lane's four values of a row go: the own row's from lanes 0 .. LP - 1, the mean's from the next LP
    const int kk = 4 * piece + (sub == 1 ? A.d_in : 0);
    u32x2* const to_frag = (u32x2*)(frags + ((kk >> 4) * 6 + ((kk >> 3) & 1)) * LL_SEG + RPW * wave) + ((kk >> 2) & 1);
    const u32x4* const frag = frags + half * LL_SEG + l32;

    // Half a block of KS steps is about 768 * KS cycles: 12800 measured best at 16 steps (6400 and 15360: 105.2 and 102.8 us against 101.9), 6400 at
    // 8 (12800: 65.9 us against 60.8).
    if (later)
        for (; spent < 768 * KS; spent += 64 * KS) __builtin_amdgcn_s_sleep(KS);
    for (int task = 0; task < n_tasks; ++task) {
        // ---- gather: the means and the own rows, split into the operand
        const int32_t next_slot = slot_of(next);
        const double my_deg = (double)now.deg;
        const double my_scale = now.deg > 0 ? 1.0 / my_deg : 0.0;
        double acc[4];
        f32x4 own;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            wait_loads<LL_UNIT*(LL_RING - 1)>();
            u32x4 v[LL_UNIT];
#pragma unroll
            for (int q = 0; q < LL_UNIT; ++q) v[q] = *(const u32x4*)(raw + (ring_at * LL_UNIT + q) * 1024 + lane * 16);
#pragma unroll
            for (int q = 0; q < LL_UNIT; ++q) {
                const int i = u * LL_UNIT + q, row = i / IPR;
                const f32x4 x = __builtin_bit_cast(f32x4, v[q]);
                if (i % IPR == 0) {      // a row's first load: its own features in the first LP lanes
                    own = x;
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = sub == 0 ? 0.0 : (double)x[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] += (double)x[e];
                }
                if (i % IPR == IPR - 1) {      // its last
                    const int deg = __builtin_amdgcn_readlane(now.deg, row * 16);
                    if (deg > SLOTS - 1) {      // uniform; neighbours that have no slot
                        const int first = __builtin_amdgcn_readlane(now.first, row * 16);
                        for (int e = SLOTS - 1; e < deg; e += RPI) {
                            const int32_t c = e + sub < deg ? A.col_ids[first + e + sub] : -1;
                            const bool ok = c >= 0 && c < A.table_rows;
                            const f32x4 y = *(const f32x4*)(ok ? lane_table + (uint64_t)(uint32_t)c * A.src_stride : (const char*)ll_zero);
#pragma unroll
                            for (int k = 0; k < 4; ++k) acc[k] += (double)y[k];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (LP == 16) acc[e] += other_half<16>(acc[e]);
                        acc[e] += other_half<32>(acc[e]);
                    }
                    const double scale = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(my_scale), row * 16),
                                                          __builtin_amdgcn_readlane(__double2loint(my_scale), row * 16));
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = sub == 0 ? own[e] : (float)(acc[e] * scale);
                    if (has_piece && sub < 2) {
#pragma unroll
                        for (int term = 0; term < 3; ++term) {
                            u32x2 p;
                            p[0] = next_term(y[0], y[1]);
                            p[1] = next_term(y[2], y[3]);
                            to_frag[term * 4 * LL_SEG + 2 * row] = p;
                        }
                    }
                }
            }
            lds_done();      // the unit has been read: its place takes a later one
            if (u + LL_RING == NU) address(next_slot, (task + 1) & 1);
            if (u + LL_RING < NU)
                issue(u + LL_RING, ring_at, task & 1);
            else
                issue(u + LL_RING - NU, ring_at, (task + 1) & 1);
            ring_at = ring_at == LL_RING - 1 ? 0 : ring_at + 1;
        }
        now = next;
        lds_barrier();
        // ---- multiply, with the next block's first rows under way and the range of the one behind it asked for
        next = range_of(task + 2);
        const int32_t r = rowlist[(task % LL_LIST) * 32 + l32], s_ok = srclist[(task % LL_LIST) * 32 + l32];
        if (n0 < A.d_out) {
            f32x16 big, small;
#pragma unroll
            for (int i = 0; i < 16; ++i) big[i] = small[i] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const u32x4 a1 = frag[(ks * 6 + 0) * LL_SEG], a2 = frag[(ks * 6 + 2) * LL_SEG], a3 = frag[(ks * 6 + 4) * LL_SEG];
                big = mfma_bf16(w[ks][0], a1, big);
                small = mfma_bf16(w[ks][0], a3, small);
                small = mfma_bf16(w[ks][2], a1, small);
                small = mfma_bf16(w[ks][1], a2, small);
                small = mfma_bf16(w[ks][0], a2, small);
                small = mfma_bf16(w[ks][1], a1, small);
            }
            // lane l32's row; element i of the accumulators is column 8 * (i / 4) + 4 * half + i % 4 of the block
            if (r >= 0 && s_ok >= 0 && r < A.n_out) {
                float* o = (float*)(A.h_out + (int64_t)r * A.out_stride) + n0 + 4 * half;
                const float* bl = bias_lds + n0 + 4 * half;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (n0 + 8 * q + 4 * half >= A.d_out) continue;      // (d_out is a multiple of 4)
                    const f32x4 b4 = *(const f32x4*)(bl + 8 * q);
                    f32x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        y[e] = (float)((double)big[4 * q + e] + (double)small[4 * q + e] + (double)b4[e]);
                        if (A.relu) y[e] = fmaxf(y[e], 0.f);
                    }
                    *(f32x4a*)(o + 8 * q) = y;
                }
            }
        }
        lds_barrier();
        if (task % (LL_LIST / 2) == LL_LIST / 2 - 1 && task + 1 + LL_LIST / 2 < n_tasks && t < LL_THREADS / 2) list_rows(task + 1 + LL_LIST / 2);
    }
    wait_loads<0>();      // what was asked for past the last block has arrived before the workgroup's LDS is given away
}

}  // namespace

// Whether one launch takes a layer of this shape: the weights' 2 * d_in values per column fit a wavefront's registers for 32 columns, the
// columns its 8 wavefronts, and a row with its neighbours (nnz / max_rows of them on average) the slots of a block's row. From 16384 rows, two
// blocks for every workgroup: with one there is no other block's reading to multiply beside.
extern "C" int32_t fg_one_launch_load(int64_t nnz, int64_t max_rows, int32_t d_in, int32_t d_out) {
    return d_in > 0 && d_in % 4 == 0 && d_in <= 128 && d_out > 0 && d_out % 4 == 0 && d_out <= 32 * LL_WAVES && max_rows >= 16384 && nnz <= 15 * max_rows;
}

extern "C" fg_status_t fg_gather_aggregate_linear_ids(const int32_t* row_start_dev, const int32_t* row_end_dev, const int32_t* col_ids_dev, int64_t nnz,
                                                      int32_t n_block_rows, const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                                      const int32_t* row_ids_dev, const float* table, int64_t table_rows, int64_t src_stride,
                                                      int32_t d_in, int32_t d_out, const float* W, const float* bias, int32_t relu, float* agg_ws,
                                                      int64_t agg_stride, float* h_out, int32_t n_out, int64_t out_stride, const fg_cache_t* cache,
                                                      int32_t n_fetch_layers, const fg_fetch_layer_t* fetch_layers, void* stream) {
    return fg_gather_aggregate_linear_ids_with(row_start_dev, row_end_dev, col_ids_dev, nnz, n_block_rows, rows_dev, n_rows_dev, max_rows, row_ids_dev, table,
                                               table_rows, src_stride, d_in, d_out, W, bias, relu, agg_ws, agg_stride, h_out, n_out, out_stride, cache,
                                               n_fetch_layers, fetch_layers, nullptr, nullptr, stream);
}

fg_status_t fg_gather_aggregate_linear_ids_with(const int32_t* row_start_dev, const int32_t* row_end_dev, const int32_t* col_ids_dev, int64_t nnz,
                                                int32_t n_block_rows, const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                                const int32_t* row_ids_dev, const float* table, int64_t table_rows, int64_t src_stride, int32_t d_in,
                                                int32_t d_out, const float* W, const float* bias, int32_t relu, float* agg_ws, int64_t agg_stride,
                                                float* h_out, int32_t n_out, int64_t out_stride, const fg_cache_t* cache, int32_t n_fetch_layers,
                                                const fg_fetch_layer_t* fetch_layers, const UpdBatch* update, bool* rode, void* stream) {
    const char* who = "fg_gather_aggregate_linear_ids";
    if (rode) *rode = false;
    if (max_rows > 0 && !agg_ws) FG_FAIL(FG_ERR_INVALID_ARG, "%s: agg_ws is NULL", who);
    if (table_rows > 0x7FFFFFFFll) FG_FAIL(FG_ERR_SHAPE, "%s: table_rows = %lld exceeds 2^31 - 1", who, (long long)table_rows);
    // the other checks are those of the two calls it stands for
    const bool one = fg_one_launch_load(nnz, max_rows, d_in, d_out) && n_block_rows > 0 && src_stride < (1ll << 31) && fg_tuning(FG_TUNE_LINEAR_TILE) == 0;
    const int64_t rows = one ? 0 : max_rows;
    if (one && (!row_start_dev || !row_end_dev || (nnz > 0 && !col_ids_dev) || !row_ids_dev || !table || !W || !h_out))
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    fg_status_t rc = fg_gather_aggregate_ids(row_start_dev, row_end_dev, col_ids_dev, nnz, n_block_rows, rows_dev, n_rows_dev, rows, row_ids_dev, table, table_rows,
                                             src_stride, d_in, FG_F32, agg_ws, agg_stride, FG_F32, nullptr, 0, 0, one ? nullptr : cache,
                                             one ? 0 : n_fetch_layers, one ? nullptr : fetch_layers, stream);
    if (rc != FG_OK) return rc;
    rc = fg_linear_ids(table, (int32_t)table_rows, src_stride, FG_F32, row_ids_dev, agg_ws, agg_stride, rows_dev, n_rows_dev, rows, d_in, d_out, W, FG_F32, bias, relu,
                       h_out, n_out, out_stride, FG_F32, stream);
    if (rc != FG_OK || !one) return rc;
    LoadLinear A{};
    if (n_fetch_layers) {
        rc = fg_build_fetch_batch(who, cache, n_fetch_layers, fetch_layers, &A.copies);
        if (rc != FG_OK) return rc;
    }
    A.row_start = row_start_dev;
    A.row_end = row_end_dev;
    A.col_ids = col_ids_dev;
    A.rows = rows_dev;
    A.row_ids = row_ids_dev;
    A.n_rows_dev = n_rows_dev;
    A.nnz = nnz;
    A.max_rows = max_rows;
    A.n_block_rows = n_block_rows;
    A.d_in = d_in;
    A.d_out = d_out;
    A.table = (const char*)table;
    A.table_rows = table_rows;
    A.src_stride = (uint32_t)src_stride;
    A.W = W;
    A.bias = bias;
    A.h_out = (char*)h_out;
    A.out_stride = out_stride;
    A.n_out = n_out;
    A.relu = relu;
    hipStream_t st = (hipStream_t)stream;
    UpdBatch U;
    U.n_layers = 0;
    if (update && update->sel_first[update->n_layers] <= fg_load_linear_update_chunks) {
        U = *update;
        for (int i = 0; i < U.n_layers; ++i) U.sel_first[i + 1] = U.sel_first[i] + (int)fg_ceil_div(U.l[i].n > 0 ? U.l[i].n : 1, LL_UPD_CHUNK);
    }
    const int beside = U.n_layers ? U.sel_first[U.n_layers] : 0;
    A.groups = (LL_GROUPS - beside) / 8 * 8;
#define FG_LL(KS, SLOTS, LP) hipLaunchKernelGGL((load_linear_kernel<KS, SLOTS, LP>), dim3(beside + A.groups), dim3(LL_THREADS), ll_lds_bytes(KS), st, A, U)
    if (d_in <= 64)
        FG_LL(8, 16, 16);
    else if (nnz <= 7 * max_rows)
        FG_LL(16, 8, 32);
    else
        FG_LL(16, 16, 32);
#undef FG_LL
    FG_LAUNCH_CHECK("load_linear_kernel");
    if (beside) *rode = true;
    return FG_OK;
}
