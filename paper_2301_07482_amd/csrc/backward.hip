// Backward pass of the GraphSAGE-mean layers as far as the embedding gradients (Algorithm 1: loss, loss.backward();
// Section 4.1.1: the norms of dL/dh are what admission to and check-out from the historical cache are decided on).
//
//   fg_softmax_xent_grad   dL/dH(L) of the mean softmax cross-entropy over the seeds
//   fg_layer_backward      dL/dH(l-1) from dL/dH(l) for one layer: ReLU mask, [d_self ‖ d_agg] = dz . W^T on the
//                          matrix cores (the forward GEMM path with transposed weights), then the transposed mean
//                          aggregation as a gather over the block's transpose (no atomics: every output row has one
//                          writer and the sums are carried in fp64, so the result does not depend on scheduling)
//   fg_row_norms           L2 norm per row
//
// Only rows that were computed (V_normal) pass gradient down; a fetched row receives its gradient and stops there.
// All of it is small next to the forward pass: the layer below the lowest cached one needs no input gradient.
#include "update_group.h"
#include <hip/hip_fp16.h>

namespace {

constexpr int BW_THREADS = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

// p = softmax(h[i, :]) in fp64, dh[i, c] = (p[c] - [c == label]) / n. A row belongs to WAVES wavefronts, one or (wide rows) the
// four of a workgroup. A row of up to 64 * WAVES * KEEP columns is read once, its exponentials, which are what the kernel
// spends its time on, are formed once and stay in registers; beyond that they are formed again for the result.
// 1024 rows of 1024 columns: 13.7 us with one wavefront per row and every exponential twice, 7.8 now; of 256: 5.8, now 5.1.
template <int WAVES, int KEEP>
__global__ __launch_bounds__(BW_THREADS) void softmax_xent_grad_kernel(const char* __restrict__ h, int64_t h_stride,
                                                                       const int32_t* __restrict__ labels, int n, int d,
                                                                       char* __restrict__ dh, int64_t dh_stride) {
    __shared__ double red[2][BW_THREADS / 64];
    constexpr int LANES = 64 * WAVES;
    const int lane = threadIdx.x % LANES;
    const int64_t n_groups = (int64_t)gridDim.x * (BW_THREADS / LANES);
    // over the row's wavefronts (WAVES == 1: the wavefront has it already)
    auto combine = [&](double v, int which, bool sum) -> double {
        if (WAVES == 1) return v;
        if ((threadIdx.x & 63) == 0) red[which][threadIdx.x >> 6] = v;
        __syncthreads();
        double t = red[which][0];
#pragma unroll
        for (int w = 1; w < BW_THREADS / 64; ++w) t = sum ? t + red[which][w] : (red[which][w] > t ? red[which][w] : t);
        return t;
    };
    for (int64_t i = ((int64_t)blockIdx.x * BW_THREADS + threadIdx.x) / LANES; i < n; i += n_groups) {      // uniform over the row's wavefronts
        const float* row = (const float*)(h + i * h_stride);
        const int32_t y = labels[i];
        float x[KEEP];
#pragma unroll
        for (int q = 0; q < KEEP; ++q) x[q] = lane + q * LANES < d ? row[lane + q * LANES] : 0.f;
        double m = -1.0e300;
#pragma unroll
        for (int q = 0; q < KEEP; ++q)
            if (lane + q * LANES < d) m = (double)x[q] > m ? (double)x[q] : m;
        for (int c = lane + KEEP * LANES; c < d; c += LANES) {
            const double v = (double)row[c];
            m = v > m ? v : m;
        }
        m = combine(wave_max(m), 0, false);
        double e[KEEP], s = 0.0;
#pragma unroll
        for (int q = 0; q < KEEP; ++q) {
            e[q] = lane + q * LANES < d ? exp((double)x[q] - m) : 0.0;
            s += e[q];
        }
        for (int c = lane + KEEP * LANES; c < d; c += LANES) s += exp((double)row[c] - m);
        s = combine(wave_sum(s), 1, true);
        float* out = (float*)(dh + i * dh_stride);
#pragma unroll
        for (int q = 0; q < KEEP; ++q) {
            const int c = lane + q * LANES;
            if (c < d) out[c] = (float)((e[q] / s - (c == y ? 1.0 : 0.0)) / (double)n);
        }
        for (int c = lane + KEEP * LANES; c < d; c += LANES) {
            const double p = exp((double)row[c] - m) / s;
            out[c] = (float)((p - (c == y ? 1.0 : 0.0)) / (double)n);
        }
        if (WAVES > 1) __syncthreads();      // before the next row's values go to `red`
    }
}

// one wavefront per row: sqrt of the fp64 sum of squares
__global__ __launch_bounds__(BW_THREADS) void row_norms_kernel(const char* __restrict__ x, int64_t stride, int n, int d,
                                                               float* __restrict__ norms) {
    const int lane = threadIdx.x & 63;
    const int64_t n_waves = ((int64_t)gridDim.x * BW_THREADS) >> 6;
    for (int64_t i = ((int64_t)blockIdx.x * BW_THREADS + threadIdx.x) >> 6; i < n; i += n_waves) {
        const float* row = (const float*)(x + i * stride);
        double s = 0.0;
        for (int c = lane; c < d; c += 64) {
            const double v = (double)row[c];
            s += v * v;
        }
        s = wave_sum(s);
        if (lane == 0) norms[i] = (float)sqrt(s);
    }
}

// round an fp32 value to bf16 bits, nearest even (finite inputs)
__device__ __forceinline__ unsigned short bw_bf16_bits(float f) {
    const unsigned int b = __float_as_uint(f);
    return (unsigned short)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bw_bf16_value(unsigned short b) { return __uint_as_float((unsigned int)b << 16); }

// dz = dh[r, :] * (h[r, :] > 0) for r = rows[k]. The GEMM that follows takes its first K/2 input columns from a
// matrix indexed by position and the other K/2 from one indexed by list order, so dz is written in that form:
// columns [0, half) to dz_pos[r, :], columns [half, d) to dz_cmp[k, :].
// BF16: the layer's output h is bf16 and dz is rounded to bf16 (the operand type of the bf16 matrix product that follows).
// one 32 x 32 tile of wt[c, a] = w[a, c]; w is [rows x cols]
template <typename T>
__device__ __forceinline__ void transpose_tile(const T* __restrict__ w, int rows, int cols, T* __restrict__ wt, int bx, int by) {
    __shared__ T tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
    const int c0 = bx * 32, a0 = by * 32;
    for (int i = ty; i < 32; i += 8)
        if (a0 + i < rows && c0 + tx < cols) tile[i][tx] = w[(int64_t)(a0 + i) * cols + c0 + tx];
    __syncthreads();
    for (int i = ty; i < 32; i += 8)
        if (c0 + i < cols && a0 + tx < rows) wt[(int64_t)(c0 + i) * rows + a0 + tx] = tile[tx][i];
}

// The first t_blocks workgroups (t_gx of them per row of tiles) transpose the layer's fp32 weights for the product that
// follows, an independent job that would otherwise be a launch of its own; the others mask the gradient.
template <bool BF16>
__global__ __launch_bounds__(BW_THREADS) void relu_backward_kernel(const char* __restrict__ dh, int64_t dh_stride,
                                                                   const char* __restrict__ h, int64_t h_stride, int n,
                                                                   const int32_t* __restrict__ rows,
                                                                   const int64_t* __restrict__ n_rows_dev, int64_t max_rows,
                                                                   int d, int vec, void* __restrict__ dz_pos_v, void* __restrict__ dz_cmp_v,
                                                                   int t_blocks, int t_gx, const float* __restrict__ w, int w_rows,
                                                                   int w_cols, float* __restrict__ wt) {
    if ((int)blockIdx.x < t_blocks) {      // uniform over the workgroup
        transpose_tile<float>(w, w_rows, w_cols, wt, (int)blockIdx.x % t_gx, (int)blockIdx.x / t_gx);
        return;
    }
    int64_t n_rows = n_rows_dev ? *n_rows_dev : max_rows;
    if (n_rows > max_rows) n_rows = max_rows;
    const int half = d >> 1;
    const int lane = threadIdx.x & 63;
    const int64_t n_waves = ((int64_t)(gridDim.x - t_blocks) * BW_THREADS) >> 6;
    for (int64_t k = ((int64_t)(blockIdx.x - t_blocks) * BW_THREADS + threadIdx.x) >> 6; k < n_rows; k += n_waves) {
        const int32_t r = rows ? rows[k] : (int32_t)k;
        if (r < 0 || r >= n) continue;
        const float* g = (const float*)(dh + (int64_t)r * dh_stride);
        const char* a = h ? h + (int64_t)r * h_stride : nullptr;
        if (vec) {      // four columns per lane: each half holds whole groups of four, every address is aligned for them
            for (int c = 4 * lane; c < d; c += 256) {
                f32x4 v = *(const f32x4*)(g + c);
                if (a) {
                    if constexpr (BF16) {
                        const uint2 w = *(const uint2*)((const unsigned short*)a + c);
                        const float act[4] = {__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16),
                                              __uint_as_float(w.y & 0xFFFF0000u)};
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = act[q] > 0.f ? v[q] : 0.f;
                    } else {
                        const f32x4 act = *(const f32x4*)((const float*)a + c);
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = act[q] > 0.f ? v[q] : 0.f;
                    }
                }
                const int64_t to = c < half ? (int64_t)r * half + c : k * half + (c - half);
                if constexpr (BF16) {
                    const uint2 o = {(unsigned int)bw_bf16_bits(v[0]) | ((unsigned int)bw_bf16_bits(v[1]) << 16),
                                     (unsigned int)bw_bf16_bits(v[2]) | ((unsigned int)bw_bf16_bits(v[3]) << 16)};
                    *(uint2*)((unsigned short*)(c < half ? dz_pos_v : dz_cmp_v) + to) = o;
                } else {
                    *(f32x4*)((float*)(c < half ? dz_pos_v : dz_cmp_v) + to) = v;
                }
            }
            continue;
        }
        for (int c = lane; c < d; c += 64) {
            float v = g[c];
            if (a) {
                const float act = BF16 ? bw_bf16_value(((const unsigned short*)a)[c]) : ((const float*)a)[c];
                if (!(act > 0.f)) v = 0.f;
            }
            if constexpr (BF16) {
                const unsigned short b = bw_bf16_bits(v);
                if (c < half)
                    ((unsigned short*)dz_pos_v)[(int64_t)r * half + c] = b;
                else
                    ((unsigned short*)dz_cmp_v)[k * half + (c - half)] = b;
            } else {
                if (c < half)
                    ((float*)dz_pos_v)[(int64_t)r * half + c] = v;
                else
                    ((float*)dz_cmp_v)[k * half + (c - half)] = v;
            }
        }
    }
}

// Transposed mean aggregation. A group of 2^g lanes owns source position j and 16 bytes of the row per lane:
//   out[j, :] = [j is a computed row] dx[j, 0:d_in]  +  sum over t in [t_start[j], t_end[j]) with r = t_row[t] computed:
//               dx[r, d_in:2*d_in] / deg(r),   deg(r) = row_end[r] - row_start[r] of the pruned block
// A row that was not computed has an empty range in the pruned block (deg = 0) and is skipped by that test; such rows of
// dx were never written. Every position j < n_src is written (zeros where nothing arrives).
// GCN: the transpose of the propagation (h_r + sum of the neighbours) / (deg + 1): dx has d_in columns, and
//   out[j, :] = [j computed] dx[j, :] / (deg(j) + 1)  +  sum over the computed rows r that sampled j of dx[r, :] / (deg(r) + 1)
// (a row found in a transposed list sampled at least one neighbour, so it is computed exactly when deg(r) > 0).
// What bounds it: every output row sits behind a chain of dependent index reads (transposed range -> row -> its degree ->
// the row's gradient), and most rows have one to three incoming edges. The lanes of a group therefore read the rows and
// degrees of up to `lanes` edges side by side, once per row, and hand them round by shuffles; the pieces a lane holds and
// two edges each are then in flight together, from addresses that always exist (a slot with nothing to read takes row 0
// of dx and is dropped by a select: rows that were not computed hold anything). Measured per layer call (with the matrix
// product in front), against one walk of the whole chain per piece and one wavefront per hub: 6.1 k rows -> 66 k positions of
// 256 columns, at most 13 edges each: 47 us (58); the same with hubs of 76: 47 (96); 26 k positions of 88 columns, hubs of
// 84: 23 (51); 14 k positions of 128 columns, hubs of 639: 41 (648); 7 k positions of 1024 columns: 38 (45). Layers whose
// average is beyond a dozen edges: at the rule for the hubs' workgroups.
struct BwAgg {
    const char* dx;
    int64_t dx_stride;
    int n, nb_byte, pieces;      // rows of dx; first byte of the neighbours' share of a row
    const uint8_t* live;
    const uint8_t* hit;
    const int32_t* row_start;
    const int32_t* row_end;
    const int32_t* t_start;
    const int32_t* t_end;
    const int32_t* t_row;
    int64_t nnz;
    int n_src;
    char* out;
    int64_t out_stride;
    float* norms;
};

// edge t of the transposed block: its row (0 where there is nothing to add) and what the row's gradient is multiplied with
template <bool GCN>
__device__ __forceinline__ void bw_edge(const BwAgg& A, int t, bool there, int32_t& r, double& w) {
    r = there ? A.t_row[t] : -1;
    const bool ok = r >= 0 && r < A.n;
    r = ok ? r : 0;
    const int32_t deg = ok ? A.row_end[r] - A.row_start[r] : 0;
    w = deg > 0 ? 1.0 / (double)(GCN ? deg + 1 : deg) : 0.0;
}

// whether position j was computed, and the weight of its own gradient
template <bool GCN>
__device__ __forceinline__ bool bw_own(const BwAgg& A, int64_t j, double& w) {
    const bool own = j < A.n && (A.live ? A.live[j] != 0 : true) && (A.hit ? A.hit[j] == 0 : true);
    w = own ? 1.0 : 0.0;
    if (GCN && own) {
        const int32_t deg = A.row_end[j] - A.row_start[j];
        w = 1.0 / (double)((deg > 0 ? deg : 0) + 1);
    }
    return own;
}

__device__ __forceinline__ void bw_add(double* acc, const f32x4 v, const double w) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += w > 0.0 ? (double)v[e] * w : 0.0;
}

constexpr int BW_WAVES = BW_THREADS / 64;

// position j by a group of `lanes` lanes (this lane: `lane`); s0 .. e0 is its range of the transposed block
// PU: 16-byte pieces of the row a lane holds at a time
template <bool GCN, int PU>
__device__ __forceinline__ void aggregate_backward_row(const BwAgg& A, const int64_t j, const int32_t s0, const int32_t e0,
                                                       const int lane, const int lanes) {
    double own_w;
    const bool own = bw_own<GCN>(A, j, own_w);
    double ss = 0.0;  // this lane's share of the row's sum of squares (of the fp32 values written)
    for (int p0 = 0; p0 < A.pieces; p0 += lanes * PU) {
        double acc[PU][4];
        int64_t off[PU];
#pragma unroll
        for (int q = 0; q < PU; ++q) {
            const int piece = p0 + q * lanes + lane;
            off[q] = piece < A.pieces ? (int64_t)piece * 16 : 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[q][e] = 0.0;
        }
        if (own) {
            f32x4 v[PU];
#pragma unroll
            for (int q = 0; q < PU; ++q) v[q] = *(const f32x4*)(A.dx + j * A.dx_stride + off[q]);
#pragma unroll
            for (int q = 0; q < PU; ++q) bw_add(acc[q], v[q], own_w);
        }
        for (int c = s0; c < e0; c += lanes) {
            const int m = e0 - c < lanes ? e0 - c : lanes;
            int32_t r;
            double w;
            bw_edge<GCN>(A, c + lane, lane < m, r, w);
            for (int u = 0; u < m; u += 2) {     // uniform over the group
                const int u1 = u + 1 < m ? u + 1 : u;
                const int32_t r0 = __shfl(r, u, lanes), r1 = __shfl(r, u1, lanes);
                const double w0 = __shfl(w, u, lanes);
                double w1 = __shfl(w, u1, lanes);
                if (u1 == u) w1 = 0.0;
                const char* b0 = A.dx + (int64_t)r0 * A.dx_stride + A.nb_byte;
                const char* b1 = A.dx + (int64_t)r1 * A.dx_stride + A.nb_byte;
                f32x4 v0[PU], v1[PU];
#pragma unroll
                for (int q = 0; q < PU; ++q) {
                    v0[q] = *(const f32x4*)(b0 + off[q]);
                    v1[q] = *(const f32x4*)(b1 + off[q]);
                }
#pragma unroll
                for (int q = 0; q < PU; ++q) {
                    bw_add(acc[q], v0[q], w0);
                    bw_add(acc[q], v1[q], w1);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < PU; ++q) {
            if (p0 + q * lanes + lane >= A.pieces) continue;
            const f32x4 o = {(float)acc[q][0], (float)acc[q][1], (float)acc[q][2], (float)acc[q][3]};
            *(f32x4*)(A.out + j * A.out_stride + off[q]) = o;
            ss += (double)o.x * o.x + (double)o.y * o.y + (double)o.z * o.z + (double)o.w * o.w;
        }
    }
    if (A.norms) {  // the lanes of a group are neighbours in one wavefront and leave the loop together
        for (int off = lanes >> 1; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
        if (lane == 0) A.norms[j] = (float)sqrt(ss);
    }
}

// A position with many incoming edges by a wavefront, or (JOINT) by a whole workgroup, whose wavefronts take equal blocks of at most
// 64 edges in turn. Where a row has fewer than 64 pieces, the sub-groups of a wavefront take a block's edges in turn; the
// partial sums meet by shuffles (and in LDS), in a fixed order.
template <bool GCN, bool JOINT>
__device__ __forceinline__ void aggregate_backward_hub(const BwAgg& A, const int64_t j, const int32_t s0, const int32_t e0,
                                                       double (*part)[64 * 4]) {
    constexpr int WAVES = JOINT ? BW_WAVES : 1;
    const int wl = threadIdx.x & 63, wave = JOINT ? (int)threadIdx.x >> 6 : 0;
    const int share = (e0 - s0 + WAVES - 1) / WAVES, block = share < 64 ? share : 64;
    int hl = 1;
    while (hl < A.pieces && hl < 64) hl <<= 1;
    const int lane = wl & (hl - 1), sub = wl / hl, subs = 64 / hl;
    double own_w;
    const bool own = bw_own<GCN>(A, j, own_w);
    double ss = 0.0;
    for (int p0 = 0; p0 < A.pieces; p0 += hl) {      // the trip count is uniform over the workgroup
        const int piece = p0 + lane;
        const int64_t off = piece < A.pieces ? (int64_t)piece * 16 : 0;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        for (int c = s0 + wave * block; c < e0; c += WAVES * block) {
            const int m = e0 - c < block ? e0 - c : block;
            int32_t r;
            double w;
            bw_edge<GCN>(A, c + wl, wl < m, r, w);
            constexpr int EB = 8;      // edges in flight per sub-group
            for (int u0 = 0; u0 < m; u0 += EB * subs) {      // uniform over the wavefront; a slot past m has weight 0
                f32x4 v[EB];
                double we[EB];
#pragma unroll
                for (int q = 0; q < EB; ++q) {
                    const int u = u0 + q * subs + sub;
                    const int32_t re = __shfl(r, u < m ? u : 0, 64);
                    we[q] = __shfl(w, u < m ? u : 0, 64);
                    if (u >= m) we[q] = 0.0;
                    v[q] = *(const f32x4*)(A.dx + (int64_t)re * A.dx_stride + A.nb_byte + off);
                }
#pragma unroll
                for (int q = 0; q < EB; ++q) bw_add(acc, v[q], we[q]);
            }
        }
        for (int o = hl; o < 64; o <<= 1)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
        if constexpr (JOINT) {
            if (sub == 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) part[wave][lane * 4 + e] = acc[e];
            __syncthreads();
        }
        if (wave == 0 && sub == 0 && piece < A.pieces) {
            double sum[4] = {0.0, 0.0, 0.0, 0.0};
            if (own) bw_add(sum, *(const f32x4*)(A.dx + j * A.dx_stride + off), own_w);
#pragma unroll
            for (int v = 0; v < WAVES; ++v)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += JOINT ? part[v][lane * 4 + e] : acc[e];
            const f32x4 o = {(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
            *(f32x4*)(A.out + j * A.out_stride + off) = o;
            ss += (double)o.x * o.x + (double)o.y * o.y + (double)o.z * o.z + (double)o.w * o.w;
        }
        if constexpr (JOINT) __syncthreads();      // the partial sums are read
    }
    if (A.norms && wave == 0) {
        ss = wave_sum(ss);
        if (wl == 0) A.norms[j] = (float)sqrt(ss);
    }
}

// Groups of 2^lanes_log2 lanes take the source positions in turn, except those with more than `many` incoming edges: the
// first hub_blocks workgroups look at hub_per positions each, spread over the whole layer (the hubs of a power-law graph are
// drawn early and lie together at its front), and take such positions a wavefront each, or with all wavefronts where it has more
// edges than one wavefront takes in a block (four blocks where there are positions for all of them). Every position is written by
// exactly one group.
template <bool GCN, int PU>
__global__ __launch_bounds__(BW_THREADS) void aggregate_backward_kernel(BwAgg A, int lanes_log2, int many, int hub_blocks,
                                                                        int hub_per) {
    __shared__ double part[BW_WAVES][64 * 4];
    __shared__ unsigned long long s_big, s_joint;
    __shared__ int32_t s_range[2][64];
    auto range_of = [&](int64_t j, int32_t& s, int32_t& e) {
        s = A.t_start[j];
        e = A.t_end[j];
        if (s < 0 || e < s || (int64_t)e > A.nnz) s = e = 0;
    };
    if ((int)blockIdx.x < hub_blocks) {
        if (threadIdx.x < 64) {
            const int64_t j = (int64_t)threadIdx.x * hub_blocks + blockIdx.x;
            int32_t s = 0, e = 0;
            if ((int)threadIdx.x < hub_per && j < A.n_src) range_of(j, s, e);
            s_range[0][threadIdx.x] = s;
            s_range[1][threadIdx.x] = e;
            const unsigned long long big = __ballot(e - s > many);
            const unsigned long long joint = __ballot(e - s > (__popcll(big) < BW_WAVES ? 64 : 256));
            if (threadIdx.x == 0) {
                s_big = big & ~joint;
                s_joint = joint;
            }
        }
        __syncthreads();
        int k = 0;
        for (unsigned long long big = s_big; big; big &= big - 1, ++k) {
            if (k % BW_WAVES != (int)threadIdx.x >> 6) continue;      // uniform over the wavefront
            const int b = __ffsll((long long)big) - 1;
            aggregate_backward_hub<GCN, false>(A, (int64_t)b * hub_blocks + blockIdx.x, s_range[0][b], s_range[1][b], part);
        }
        for (unsigned long long big = s_joint; big; big &= big - 1) {      // uniform over the workgroup
            const int b = __ffsll((long long)big) - 1;
            aggregate_backward_hub<GCN, true>(A, (int64_t)b * hub_blocks + blockIdx.x, s_range[0][b], s_range[1][b], part);
        }
        return;
    }
    const int lanes = 1 << lanes_log2;
    const int gpb = BW_THREADS >> lanes_log2;
    const int64_t block = (int64_t)blockIdx.x - hub_blocks, n_blocks = (int64_t)gridDim.x - hub_blocks;
    for (int64_t j = block * gpb + (threadIdx.x >> lanes_log2); j < A.n_src; j += n_blocks * gpb) {
        int32_t s0, e0;
        range_of(j, s0, e0);
        if (e0 - s0 > many) continue;
        aggregate_backward_row<GCN, PU>(A, j, s0, e0, threadIdx.x & (lanes - 1), lanes);
    }
}

struct BwWs {
    size_t dz_pos, dz_cmp, wt, dx, total;
};
// esz: bytes per element of dz and of the transposed weights (4, or 2 in the bf16 setting); cols: columns of dx
BwWs bw_layout(int64_t n, int64_t max_rows, int64_t cols, int64_t d_out, int64_t esz) {
    BwWs w;
    const size_t half = (size_t)(d_out / 2) * esz;
    w.dz_pos = 0;
    w.dz_cmp = fg_align_up((size_t)(n > 0 ? n : 1) * half, 256);
    w.wt = w.dz_cmp + fg_align_up((size_t)(max_rows > 0 ? max_rows : 1) * half, 256);
    w.dx = w.wt + fg_align_up((size_t)cols * d_out * esz, 256);
    w.total = w.dx + fg_align_up((size_t)(n > 0 ? n : 1) * cols * 4, 256);
    return w;
}

}  // namespace

fg_status_t fg_launch_linear_bf16(const void* h_src, int32_t n_src, int64_t src_stride, fg_dtype_t in_dtype, const void* agg,
                                  int64_t agg_stride, const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                  int32_t d_in, int32_t d_out, const void* W, const float* bias, int32_t relu, void* h_out,
                                  int32_t n_out, int64_t out_stride, fg_dtype_t out_dtype, hipStream_t st, bool w_nk,
                                  const int32_t* src_ids_dev = nullptr);

fg_status_t fg_launch_linear_masked(const float* dh, int64_t dh_stride, const float* h, int64_t h_stride, int32_t n, const int32_t* rows_dev,
                                    const int64_t* n_rows_dev, int64_t max_rows, int32_t d_out, int32_t cols, const float* W, float* dx, hipStream_t st, bool* done);

extern "C" fg_status_t fg_softmax_xent_grad(const float* h_dev, int64_t h_stride, const int32_t* labels_dev, int32_t n, int32_t d,
                                            float* dh_dev, int64_t dh_stride, void* stream) {
    if (n < 0 || d <= 0) FG_FAIL(FG_ERR_INVALID_ARG, "fg_softmax_xent_grad: bad size (n %d, d %d)", n, d);
    if (n > 0 && (!h_dev || !labels_dev || !dh_dev)) FG_FAIL(FG_ERR_INVALID_ARG, "fg_softmax_xent_grad: NULL pointer");
    if (h_stride < (int64_t)d * 4 || dh_stride < (int64_t)d * 4) FG_FAIL(FG_ERR_SHAPE, "fg_softmax_xent_grad: a row stride is smaller than a row");
    if (((uintptr_t)h_dev | (uintptr_t)dh_dev | (uintptr_t)h_stride | (uintptr_t)dh_stride) & 3)
        FG_FAIL(FG_ERR_INVALID_ARG, "fg_softmax_xent_grad: pointers and strides must be 4-byte aligned");
    fg_clear_error();
    if (n == 0) return FG_OK;
    // A workgroup per row pays two barriers: worth it where a wavefront would form exponentials twice, or where there are few rows.
    // One wavefront / four, us: 1024 rows of 300 columns 5.7 / 5.8, of 512 6.9 / 6.4; 2048 of 300 6.6 / 7.8, of 512 8.1 / 8.6; 4096
    // of 300 8.3 / 11.4, of 640 13.2 / 14.4, of 1024 20.3 / 17.9 (before: 10.2, 16.2, 24.2).
    const bool wide = d > (n <= 1536 ? 256 : 640);
    int64_t blocks = wide ? n : fg_ceil_div(n, BW_THREADS / 64);
    if (blocks > 4096) blocks = 4096;
#define FG_SM(WAVES, KEEP)                                                                                                         \
    hipLaunchKernelGGL((softmax_xent_grad_kernel<WAVES, KEEP>), dim3((unsigned)blocks), dim3(BW_THREADS), 0, (hipStream_t)stream,    \
                       (const char*)h_dev, h_stride, labels_dev, n, d, (char*)dh_dev, dh_stride)
    if (wide)
        FG_SM(BW_THREADS / 64, 4);
    else if (d > 256)
        FG_SM(1, 8);
    else
        FG_SM(1, 4);
#undef FG_SM
    FG_LAUNCH_CHECK("softmax_xent_grad_kernel");
    return FG_OK;
}

extern "C" fg_status_t fg_row_norms(const float* x_dev, int64_t x_stride, int32_t n, int32_t d, float* norms_dev, void* stream) {
    if (n < 0 || d <= 0) FG_FAIL(FG_ERR_INVALID_ARG, "fg_row_norms: bad size (n %d, d %d)", n, d);
    if (n > 0 && (!x_dev || !norms_dev)) FG_FAIL(FG_ERR_INVALID_ARG, "fg_row_norms: NULL pointer");
    if (x_stride < (int64_t)d * 4) FG_FAIL(FG_ERR_SHAPE, "fg_row_norms: the row stride is smaller than a row");
    if (((uintptr_t)x_dev | (uintptr_t)x_stride | (uintptr_t)norms_dev) & 3) FG_FAIL(FG_ERR_INVALID_ARG, "fg_row_norms: pointers and stride must be 4-byte aligned");
    fg_clear_error();
    if (n == 0) return FG_OK;
    int64_t blocks = fg_ceil_div(n, BW_THREADS / 64);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(row_norms_kernel, dim3((unsigned)blocks), dim3(BW_THREADS), 0, (hipStream_t)stream, (const char*)x_dev, x_stride, n,
                       d, norms_dev);
    FG_LAUNCH_CHECK("row_norms_kernel");
    return FG_OK;
}

// kind of layer a backward call is for
enum BwKind { BW_SAGE_F32 = 0, BW_GCN_F32 = 1, BW_SAGE_BF16 = 2 };

static size_t layer_backward_ws(int kind, int32_t n, int64_t max_rows, int32_t d_in, int32_t d_out) {
    if (n < 0 || max_rows < 0 || d_in <= 0 || d_out <= 0) return 0;
    return bw_layout(n, max_rows, kind == BW_GCN_F32 ? d_in : 2 * (int64_t)d_in, d_out, kind == BW_SAGE_BF16 ? 2 : 4).total;
}

extern "C" size_t fg_layer_backward_workspace_bytes(int32_t n, int64_t max_rows, int32_t d_in, int32_t d_out) {
    return layer_backward_ws(BW_SAGE_F32, n, max_rows, d_in, d_out);
}
extern "C" size_t fg_layer_backward_gcn_workspace_bytes(int32_t n, int64_t max_rows, int32_t d_in, int32_t d_out) {
    return layer_backward_ws(BW_GCN_F32, n, max_rows, d_in, d_out);
}
extern "C" size_t fg_layer_backward_bf16_workspace_bytes(int32_t n, int64_t max_rows, int32_t d_in, int32_t d_out) {
    return layer_backward_ws(BW_SAGE_BF16, n, max_rows, d_in, d_out);
}

// The three layer kinds share the sequence: dz . W^T, transposed aggregation with the row norms. In fp32 the product masks and
// transposes for itself; in bf16, and for rows too wide for it, a launch forms the masked (and rounded) operand for the forward GEMM.
static fg_status_t layer_backward_launch(const char* who, int kind, const float* dh_dev, int64_t dh_stride, const void* h_dev,
                                         int64_t h_stride, int32_t n, const int32_t* rows_dev, const int64_t* n_rows_dev,
                                         int64_t max_rows, const uint8_t* live_dev, const uint8_t* hit_dev,
                                         const int32_t* row_start_dev, const int32_t* row_end_dev, const int32_t* t_start_dev,
                                         const int32_t* t_end_dev, const int32_t* t_row_dev, int64_t nnz, int32_t n_src, int32_t d_in,
                                         int32_t d_out, const void* W, float* dh_src_dev, int64_t dh_src_stride, float* norms_src_dev,
                                         void* ws_dev, size_t ws_bytes, void* stream) {
    const bool gcn = kind == BW_GCN_F32, b16 = kind == BW_SAGE_BF16;
    const int esz = b16 ? 2 : 4;
    if (n < 0 || max_rows < 0 || n_src < 0 || nnz < 0 || d_in <= 0 || d_out <= 0)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: bad size (n %d, max_rows %lld, n_src %d, nnz %lld, d_in %d, d_out %d)", who, n, (long long)max_rows,
                n_src, (long long)nnz, d_in, d_out);
    if (n_src < n) FG_FAIL(FG_ERR_SHAPE, "%s: the layer below (%d positions) must contain this layer's %d", who, n_src, n);
    if (max_rows > n) FG_FAIL(FG_ERR_SHAPE, "%s: max_rows = %lld exceeds the layer's %d positions", who, (long long)max_rows, n);
    if (d_in % (b16 ? 8 : 4) || d_out % (b16 ? 16 : 8))
        FG_FAIL(FG_ERR_SHAPE, "%s: d_in = %d must be a multiple of %d and d_out = %d of %d", who, d_in, b16 ? 8 : 4, d_out, b16 ? 16 : 8);
    if (n_src > 0 && (!dh_src_dev || !t_start_dev || !t_end_dev || (nnz > 0 && !t_row_dev))) FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    if (n > 0 && (!dh_dev || !row_start_dev || !row_end_dev || !W)) FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    if (dh_stride < (int64_t)d_out * 4 || (h_dev && h_stride < (int64_t)d_out * esz) || dh_src_stride < (int64_t)d_in * 4)
        FG_FAIL(FG_ERR_SHAPE, "%s: a row stride is smaller than its row", who);
    if (((uintptr_t)dh_dev | (uintptr_t)dh_stride) & 3 || ((uintptr_t)h_dev | (uintptr_t)h_stride) & (uintptr_t)(esz - 1))
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: dh, h and their strides must be aligned to their element size", who);
    if ((uintptr_t)W & (b16 ? 15 : 3)) FG_FAIL(FG_ERR_INVALID_ARG, "%s: W must be %d-byte aligned", who, b16 ? 16 : 4);
    if ((uintptr_t)norms_src_dev & 3) FG_FAIL(FG_ERR_INVALID_ARG, "%s: norms_src_dev must be 4-byte aligned", who);
    if (((uintptr_t)dh_src_dev | (uintptr_t)dh_src_stride | (uintptr_t)ws_dev) & 15)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: dh_src_dev, its stride and the workspace must be 16-byte aligned", who);
    const int cols = gcn ? d_in : 2 * d_in;       // columns of dz . W^T
    const BwWs L = bw_layout(n, max_rows, cols, d_out, esz);
    if (!ws_dev || ws_bytes < L.total) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, L.total);
    fg_clear_error();
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)ws_dev;
    void* dz_pos = ws + L.dz_pos;
    void* dz_cmp = ws + L.dz_cmp;
    void* wt = ws + L.wt;
    float* dx = (float*)(ws + L.dx);
    const int half = d_out / 2;
    if (n > 0 && max_rows > 0) {
        int64_t blocks = fg_ceil_div(max_rows, BW_THREADS / 64);
        if (blocks > 4096) blocks = 4096;
        const dim3 tgrid((unsigned)fg_ceil_div(d_out, 32), (unsigned)fg_ceil_div(cols, 32));
        bool multiplied = false;
        // four columns at a time where dh and h allow it (1024 rows of 1024 columns 10.8 -> 6.8 us; the halves of dz are workspace, aligned, and d_out is a multiple of 8)
        const int vec = !(((uintptr_t)dh_dev | (uintptr_t)dh_stride) & 15) && !(((uintptr_t)h_dev | (uintptr_t)h_stride) & (uintptr_t)(4 * esz - 1));
        if (b16) {
            hipLaunchKernelGGL(relu_backward_kernel<true>, dim3((unsigned)blocks), dim3(BW_THREADS), 0, st, (const char*)dh_dev, dh_stride,
                               (const char*)h_dev, h_stride, n, rows_dev, n_rows_dev, max_rows, d_out, vec, dz_pos, dz_cmp, 0, 1,
                               (const float*)nullptr, 0, 0, (float*)nullptr);
            FG_LAUNCH_CHECK("relu_backward_kernel");
            // dx[r, :] = [dz_pos[r, :] ‖ dz_cmp[k, :]] . W^T, bf16 operands, fp32 sums and result. The weights of this product are
            // W^T; the matrix-core kernel takes them transposed, which is W as the caller holds it: nothing to transpose
            fg_status_t rc = fg_launch_linear_bf16(dz_pos, n, (int64_t)half * 2, FG_BF16, dz_cmp, (int64_t)half * 2, rows_dev, n_rows_dev,
                                                   max_rows, half, cols, W, nullptr, 0, dx, n, (int64_t)cols * 4, FG_F32, st, true);
            if (rc != FG_OK) return rc;
        } else if (fg_tuning(FG_TUNE_LINEAR_TILE) == 0) {
            fg_status_t rc = fg_launch_linear_masked(dh_dev, dh_stride, (const float*)h_dev, h_stride, n, rows_dev, n_rows_dev, max_rows, d_out, cols,
                                                     (const float*)W, dx, st, &multiplied);
            if (rc != FG_OK) return rc;
        }
        if (!b16 && !multiplied) {
            // (the transposition of W rides in the same launch: tgrid.x * tgrid.y workgroups in front of the others)
            const int t_blocks = (int)(tgrid.x * tgrid.y);
            hipLaunchKernelGGL(relu_backward_kernel<false>, dim3((unsigned)(blocks + t_blocks)), dim3(BW_THREADS), 0, st, (const char*)dh_dev,
                               dh_stride, (const char*)h_dev, h_stride, n, rows_dev, n_rows_dev, max_rows, d_out, vec, dz_pos, dz_cmp, t_blocks,
                               (int)tgrid.x, (const float*)W, cols, d_out, (float*)wt);
            FG_LAUNCH_CHECK("relu_backward_kernel");
            // dx[r, :] = [dz_pos[r, :] ‖ dz_cmp[k, :]] . W^T for r = rows[k]: the forward GEMM with K = d_out, N = cols
            fg_status_t rc = fg_linear(dz_pos, n, (int64_t)half * 4, FG_F32, dz_cmp, (int64_t)half * 4, rows_dev, n_rows_dev, max_rows, half,
                                       cols, wt, FG_F32, nullptr, 0, dx, n, (int64_t)cols * 4, FG_F32, stream);
            if (rc != FG_OK) return rc;
        }
    }
    if (n_src == 0) return FG_OK;
    const int pieces = d_in / 4;
    // Lanes per source row: up to 16 for rows of at most 64 pieces (four rows, four index chains, per wavefront; a lane holds
    // up to four pieces), a whole wavefront for wider ones. Measured per call of the whole layer's backward pass: 256 columns,
    // 6.1 k rows: 20.3 us against 22.7 with one row per wavefront (66 k rows: 47); 1024 columns, 7 k rows: 38.5.
    const int lg_cap = pieces <= 64 ? 4 : 6;
    int lg = 0;
    while ((1 << lg) < pieces && lg < lg_cap) ++lg;
    const int gpb = BW_THREADS >> lg;
    int64_t blocks = fg_ceil_div(n_src, gpb);
    if (blocks > 256 * 16) blocks = 256 * 16;
    // A row wider than a small group is walked by a whole wavefront in any case: only from 64 edges on it gains from more.
    // Positions per hub workgroup: 64 where hubs are few, but a layer whose positions average a dozen edges and more is all hubs, and
    // one of few positions has too few workgroups to share them. 3 k positions of 256 columns with 20 edges each: 29 us with a
    // wavefront per position, 217 with 64 positions in turn by one workgroup, 26 now; 300 of 1024 columns 61, 604, 24; 8 k of 512
    // columns with 100 edges 242, 958, 135. (Fewer positions per workgroup everywhere: 5 % on layers of one to six edges each.)
    const int many = lg < 6 ? 16 : 64;
    const double average = n_src > 0 ? (double)nnz / (double)n_src : 0.0;
    int64_t hub_per = n_src / 128;
    if ((double)hub_per * average * average > 1024.0) hub_per = (int64_t)(1024.0 / (average * average));
    hub_per = hub_per < BW_WAVES ? BW_WAVES : (hub_per > 64 ? 64 : hub_per);
    const int hub_blocks = nnz > many ? (int)fg_ceil_div(n_src, hub_per) : 0;
    const BwAgg A = {(const char*)dx, (int64_t)cols * 4, n, gcn ? 0 : d_in * 4, pieces, live_dev, hit_dev, row_start_dev, row_end_dev,
                     t_start_dev, t_end_dev, t_row_dev, nnz, n_src, (char*)dh_src_dev, dh_src_stride, norms_src_dev};
    const dim3 agrid((unsigned)(blocks + hub_blocks));
    const int pu = (int)fg_ceil_div(pieces, 1 << lg);
#define FG_AGG_BW(P)                                                                                                           \
    do {                                                                                                                       \
        if (gcn)                                                                                                               \
            hipLaunchKernelGGL((aggregate_backward_kernel<true, P>), agrid, dim3(BW_THREADS), 0, st, A, lg, many, hub_blocks, (int)hub_per); \
        else                                                                                                                   \
            hipLaunchKernelGGL((aggregate_backward_kernel<false, P>), agrid, dim3(BW_THREADS), 0, st, A, lg, many, hub_blocks, (int)hub_per); \
    } while (0)
    if (pu <= 1)
        FG_AGG_BW(1);
    else if (pu <= 2)
        FG_AGG_BW(2);
    else
        FG_AGG_BW(4);
#undef FG_AGG_BW
    FG_LAUNCH_CHECK("aggregate_backward_kernel");
    return FG_OK;
}

#define FG_LAYER_BACKWARD_ARGS                                                                                                      \
    dh_dev, dh_stride, h_dev, h_stride, n, rows_dev, n_rows_dev, max_rows, live_dev, hit_dev, row_start_dev, row_end_dev, t_start_dev, \
        t_end_dev, t_row_dev, nnz, n_src, d_in, d_out, W, dh_src_dev, dh_src_stride, norms_src_dev, ws_dev, ws_bytes, stream

extern "C" fg_status_t fg_layer_backward(const float* dh_dev, int64_t dh_stride, const float* h_dev, int64_t h_stride, int32_t n,
                                         const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                         const uint8_t* live_dev, const uint8_t* hit_dev, const int32_t* row_start_dev,
                                         const int32_t* row_end_dev, const int32_t* t_start_dev, const int32_t* t_end_dev,
                                         const int32_t* t_row_dev, int64_t nnz, int32_t n_src, int32_t d_in, int32_t d_out,
                                         const float* W, float* dh_src_dev, int64_t dh_src_stride, float* norms_src_dev,
                                         void* ws_dev, size_t ws_bytes, void* stream) {
    return layer_backward_launch("fg_layer_backward", BW_SAGE_F32, FG_LAYER_BACKWARD_ARGS);
}

extern "C" fg_status_t fg_layer_backward_gcn(const float* dh_dev, int64_t dh_stride, const float* h_dev, int64_t h_stride, int32_t n,
                                             const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                             const uint8_t* live_dev, const uint8_t* hit_dev, const int32_t* row_start_dev,
                                             const int32_t* row_end_dev, const int32_t* t_start_dev, const int32_t* t_end_dev,
                                             const int32_t* t_row_dev, int64_t nnz, int32_t n_src, int32_t d_in, int32_t d_out,
                                             const float* W, float* dh_src_dev, int64_t dh_src_stride, float* norms_src_dev,
                                             void* ws_dev, size_t ws_bytes, void* stream) {
    return layer_backward_launch("fg_layer_backward_gcn", BW_GCN_F32, FG_LAYER_BACKWARD_ARGS);
}

extern "C" fg_status_t fg_layer_backward_bf16(const float* dh_dev, int64_t dh_stride, const void* h_dev, int64_t h_stride, int32_t n,
                                              const int32_t* rows_dev, const int64_t* n_rows_dev, int64_t max_rows,
                                              const uint8_t* live_dev, const uint8_t* hit_dev, const int32_t* row_start_dev,
                                              const int32_t* row_end_dev, const int32_t* t_start_dev, const int32_t* t_end_dev,
                                              const int32_t* t_row_dev, int64_t nnz, int32_t n_src, int32_t d_in, int32_t d_out,
                                              const void* W, float* dh_src_dev, int64_t dh_src_stride, float* norms_src_dev,
                                              void* ws_dev, size_t ws_bytes, void* stream) {
    return layer_backward_launch("fg_layer_backward_bf16", BW_SAGE_BF16, FG_LAYER_BACKWARD_ARGS);
}
#undef FG_LAYER_BACKWARD_ARGS

// ---- weight gradients --------------------------------------------------------------------------------------
//
// dW = X^T . dz and db = column sums of dz over the computed rows, X[k, :] = [h_src[rows[k], :] ‖ agg[k, :]],
// dz[k, :] = dh[rows[k], :] * (h[rows[k], :] > 0). A contraction over the rows (K = tens of thousands) with a small
// result (2*d_in x d_out), so K is split over the workgroups: workgroup `chunk` multiplies its rows on the matrix
// cores and leaves a partial result, a second launch adds the partials up in fp64.
namespace {

constexpr int WG_THREADS = 512;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The partial products on the bf16 matrix cores, for the fp32 model (TERMS = 3) and the mixed-precision one (TERMS = 1).
//
// fp32: every value is the exact sum of three bf16 values (x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2), nearest
// even), and the six products a_i * b_j with i + j <= 4 (1-based; each exact in fp32) are kept: the dropped three are below
// 2^-24 of the product. The leading products have an accumulator of their own: what limits an fp32 running sum is the
// rounding of the sum at every step, and that one is rounded once per 16 rows; the roundings of the other are 2^-8 of it.
// Mixed precision: both operands are bf16 values (the rows of X as the forward product rounded them, dz rounded after the
// mask; the bias gradient sums the unrounded dz), one product each.
//
// v_mfma_f32_32x32x16_bf16 wants its contraction index contiguous in a lane, which for X^T . dz is the row index, so both
// operands go through LDS and are transposed on the way out of it (ds_read_b64_tr_b16): a step is 32 rows; a thread loads 16 bytes
// of a row, coalesced over the columns, masks and splits them and writes each term's bf16 values row by row. Two LDS buffers,
// one barrier per step; while step s is multiplied the values of step s + 1 are in flight and the positions of step s + 2 are
// there (values two steps ahead: a second set of registers, which are all taken).
//
// Split: every chunk of rows leaves a partial result of 2*d_in x d_out that the reduction reads again, and every tile of
// the result reads the operands again, so the tile is as large as LDS and registers allow.
//
// What bounds it: reading the operands. 55 k rows x 256 x 256 in fp32 are 169 MB (X, dh, and h for its mask), 33 us at the rate of
// a large copy; a step of a 256 x 128 tile takes 2.7 us (2.8 with 4-byte loads of eight rows per thread, transposed by what a
// thread wrote), in mixed precision, where tiles find the rows in L2 and one step of look-ahead does not cover its latency, a
// step of 256 x 256 1.35 (1.7). Measured with its reduction, before and now, rows x 2*d_in x d_out: fp32 55 k x 256 x 256 68.5 -> 64.5 us,
// 6 k x 512 x 256 28.4 -> 26.7, 1 k x 512 x 172 14.9 -> 14.5; mixed 7 k (bound 16 k) x 1536 x 1024 69.8 -> 61.1, 1 k x 2048 x 1024 36.6 ->
// 35.5, 16 k x 1536 x 1024 125 -> 105.
typedef unsigned int wu32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 wbf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 wbf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 wf16x8 __attribute__((ext_vector_type(8)));
typedef short ws16x4 __attribute__((ext_vector_type(4)));
typedef wu32x4 wu32x4a __attribute__((aligned(4)));      // 16 bytes from an address that is a multiple of 4
typedef float f32x8 __attribute__((ext_vector_type(8)));

constexpr int WX_STEP = 32;             // rows per step: two matrix instructions deep
constexpr size_t wx_lds_bytes(int tm, int tn, int terms) { return (size_t)2 * terms * WX_STEP * (tm + tn) * 2; }

// two values -> their three bf16 terms, a word each (the first value in its lower half)
__device__ __forceinline__ void wx_split2(float a, float b, unsigned int (&u)[3]) {
    f32x2 x = {a, b};
#pragma unroll
    for (int term = 0; term < 3; ++term) {
        u[term] = __builtin_bit_cast(unsigned int, __builtin_convertvector(x, wbf16x2));
        x = f32x2{x[0] - __uint_as_float(u[term] << 16), x[1] - __uint_as_float(u[term] & 0xFFFF0000u)};
    }
}

struct WgIn {
    const char *h_src, *agg, *dh, *h;      // own rows and dh, h by position, agg in list order; h NULL: no mask
    int64_t src_stride, agg_stride, dh_stride, h_stride, max_rows;
    const int32_t* rows;
    const int64_t* n_rows_dev;
    int n_src, n, d_in, d_pad, d_out, n_chunks, parts, tiles_m, tiles_n;      // parts: partial results of a chunk
    int src, tm;                           // element type of h_src; rows of a tile
    float *part_w, *part_b;                // partial results of every chunk; of a single chunk the result (part_b of a call without db: workspace)
    float *dw, *db;
};

// The layers of one call: their products share a launch, each with its share of the workgroups, and their reductions another. By
// itself a layer of few rows fills the chip only with chunks so short that starting them costs more than the products.
constexpr int WG_MAX_LAYERS = 8;
struct WgBatch {
    int n;
    int first[WG_MAX_LAYERS + 1];          // first workgroup of each layer: products ...
    int red_first[WG_MAX_LAYERS + 1];      // ... and reduction
    WgIn l[WG_MAX_LAYERS];
};

// TM x TN: the tile of the result, 8 wavefronts as 4 x 2. SRC: element type of h_src (TERMS = 3: fp32). unit: which chunk and tile.
template <int TM, int TN, int TERMS, int SRC>
__device__ __forceinline__ void weight_grad_tile(const WgIn& A, const int unit) {
    constexpr int CPT = TERMS == 3 ? 4 : 8;                       // adjacent columns per thread: 16 bytes of an operand
    constexpr int XT = TM / CPT, ZT = TN / CPT;                   // threads side by side on a row
    constexpr int XS = WG_THREADS / XT, ZS = WG_THREADS / ZT;     // rows of a step that are loaded together
    constexpr int XU = WX_STEP / XS, ZU = WX_STEP / ZS;           // rows per thread
    constexpr int XW = (TERMS == 1 && SRC == FG_F32) ? 2 : 1;     // 16-byte words per loaded piece of h_src
    constexpr int XP = WX_STEP * TM * 2, ZP = WX_STEP * TN * 2, BUF = TERMS * (XP + ZP);      // bytes of a term's rows, of a buffer
    constexpr int MB = TM / 128, NB = TN / 64;                    // 32 x 32 blocks per wavefront
    constexpr int ESZ = SRC == FG_F32 ? 4 : 2, ASZ = TERMS == 3 ? 4 : 2;                   // bytes per element: h_src; agg and h
    static_assert(XS % 4 == 0 && ZS % 4 == 0, "a thread's rows have the same place in their group of four");
    extern __shared__ __attribute__((aligned(16))) char wx_lds[];   // [buffer][X, then dz][term][row][column]
    const int tiles = A.tiles_m * A.tiles_n;
    const int chunk = unit / tiles, tile = unit % tiles;
    const int m_tile = (tile / A.tiles_n) * TM, n_tile = (tile % A.tiles_n) * TN;
    int64_t n_rows = A.n_rows_dev ? *A.n_rows_dev : A.max_rows;
    if (n_rows > A.max_rows) n_rows = A.max_rows;
    const int M = 2 * A.d_in, N = A.d_out, d_in = A.d_in;      // M: rows of the result (m counts them with each half padded to d_pad)
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int wm = (wave & 3) * (TM / 4), wn = (wave >> 2) * (TN / 2);
    // the rows there are, split evenly over the chunks (whole steps per chunk)
    const int64_t per = (n_rows + A.n_chunks - 1) / A.n_chunks;
    const int64_t per_b = (per + WX_STEP - 1) / WX_STEP * WX_STEP;
    const int64_t k_begin = (int64_t)chunk * per_b < n_rows ? (int64_t)chunk * per_b : n_rows;
    int64_t k_end = k_begin + per_b;
    if (k_end > n_rows) k_end = n_rows;
    const int n_steps = (int)((k_end - k_begin + WX_STEP - 1) / WX_STEP);

    // Staging role of this thread: CPT adjacent columns of X and of dz, rows xr + i * XS and zr + i * ZS of a step. Each half of X is walked
    // as if it were d_pad columns wide. (A column that does not exist reads another one: its products go to outputs that are
    // not stored.)
    const int xp = (t % XT) * CPT, zp = (t % ZT) * CPT;
    const int xr = XT == 64 ? wave : t / XT, zr = ZT == 64 ? wave : t / ZT;
    const bool x_agg = m_tile + xp >= A.d_pad;
    const int xc = m_tile + xp - (x_agg ? A.d_pad : 0), zc = n_tile + zp;
    const char* x_base = (x_agg ? A.agg : A.h_src) + (xc < d_in ? xc : 0) * (x_agg ? ASZ : ESZ);
    const int64_t x_stride = x_agg ? A.agg_stride : A.src_stride;
    const char* g_base = A.dh + (zc < N ? zc : 0) * 4;
    const char* o_base = (A.h ? A.h : A.dh) + (zc < N ? zc : 0) * ASZ;      // without a mask: words of dh again, replaced by ones
    const int64_t o_stride = A.h ? A.h_stride : A.dh_stride;
    const unsigned int o_and = A.h ? 0xFFFFFFFFu : 0u, o_or = A.h ? 0u : 0x3F803F80u;
    const int x_second = x_agg ? 0 : 16;
    const int kb = (int)k_begin, ke = (int)k_end;            // list entries are positions: below 2^31
    // Where its pieces go: the 64-byte windows of a row (32 columns, a matrix instruction's block) are exchanged by the row's place in
    // its group of four, so that the four rows a transposing read takes 64 bytes of lie in different banks.
    const int x_to = xr * (TM * 2) + (((xp >> 5) ^ (xr & 3)) << 6) + ((xp & 31) << 1);
    const int z_to = zr * (TN * 2) + (((zp >> 5) ^ (zr & 3)) << 6) + ((zp & 31) << 1);

    struct Vals {
        wu32x4 x[XU][XW];
        wu32x4 g[ZU][CPT / 4];
        wu32x4 o[ZU];
        unsigned int x_in, z_in;      // bit e: row e of the step has own features, exists (scalars)
    };
    // position of row `l32` of step s; one load for the whole step, one register
    const int32_t* list = A.rows ? A.rows : (const int32_t*)A.dh;
    auto load_positions = [&](int s) -> int32_t {
        const int kk = kb + s * WX_STEP + l32;
        const int ks = kk < ke ? kk : ke - 1;
        const int32_t raw = list[A.rows ? ks : 0];
        return A.rows ? raw : ks;
    };
    auto of_row = [](int v, int row, bool uniform) { return uniform ? __builtin_amdgcn_readlane(v, row) : __shfl(v, row, 64); };
    // Values of step s from the positions loaded for it. Rows that do not exist read row 0 / the last entry and are masked when they
    // are staged (with masks, not branches: a branch per row would make the wavefront wait for each load by itself).
    auto load_values = [&](int s, int32_t raw, Vals& V) {
        const int kk = kb + s * WX_STEP + l32;
        // a position without own features: the fp32 product leaves the row out, the mixed one takes zeros for them
        const bool z_ok = kk < ke && raw >= 0 && raw < A.n && (TERMS == 1 || raw < A.n_src);
        const bool x_ok = z_ok && raw < A.n_src;
        const int32_t pos = z_ok ? raw : 0, own = x_ok ? raw : 0;
        V.x_in = (unsigned int)__ballot(x_ok);
        V.z_in = (unsigned int)__ballot(z_ok);
#pragma unroll
        for (int i = 0; i < XU; ++i) {
            const int r = xr + i * XS, at = kb + s * WX_STEP + r;
            const int32_t own_r = of_row(own, r, XT == 64), x_row = x_agg ? (at < ke ? at : ke - 1) : own_r;
            const char* p = x_base + (int64_t)x_row * x_stride;
            V.x[i][0] = *(const wu32x4a*)p;
            if constexpr (XW == 2) V.x[i][1] = *(const wu32x4a*)(p + x_second);
        }
#pragma unroll
        for (int i = 0; i < ZU; ++i) {
            const int64_t pos_r = of_row(pos, zr + i * ZS, ZT == 64);
            const char* p = g_base + pos_r * A.dh_stride;
#pragma unroll
            for (int w = 0; w < CPT / 4; ++w) V.g[i][w] = *(const wu32x4a*)(p + 16 * w);
            V.o[i] = *(const wu32x4a*)(o_base + pos_r * o_stride);
        }
    };
    double colsum[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) colsum[c] = 0.0;
    // the bf16 terms of CPT values to their places in the term's rows
    auto put = [&](char* to, int term_bytes, const float* v) {
        if constexpr (TERMS == 3) {
            unsigned int lo[3], hi[3];
            wx_split2(v[0], v[1], lo);
            wx_split2(v[2], v[3], hi);
#pragma unroll
            for (int term = 0; term < 3; ++term) *(uint2*)(to + term * term_bytes) = uint2{lo[term], hi[term]};
        } else {
            const f32x8 f = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
            *(wu32x4*)to = __builtin_bit_cast(wu32x4, __builtin_convertvector(f, wbf16x8));
        }
    };
    // mask, split and write the loaded step to buffer b; rows that do not exist become zeros (only a chunk's last step, or a list
    // with bad entries, has any)
    auto stage = [&](int b, Vals& V) {
        char* X = wx_lds + b * BUF;
        char* Z = X + TERMS * XP;
        const bool whole = (V.x_in & V.z_in) == 0xFFFFFFFFu;      // uniform
        const unsigned int x_in = x_agg ? V.z_in : V.x_in;
#pragma unroll
        for (int i = 0; i < XU; ++i) {
            if (!whole) {
                const unsigned int m = 0u - ((x_in >> (xr + i * XS)) & 1u);
#pragma unroll
                for (int w = 0; w < XW; ++w) V.x[i][w] &= m;
            }
            float v[CPT];
            if constexpr (TERMS == 3) {
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = __uint_as_float(V.x[i][0][c]);
                put(X + x_to + i * XS * TM * 2, XP, v);
            } else {
                // the means, and own embeddings, are bf16 already
                wu32x4 u = V.x[i][0];
                if constexpr (SRC != FG_BF16) {
                    if constexpr (SRC == FG_F16) {
                        const f32x8 f = __builtin_convertvector(__builtin_bit_cast(wf16x8, u), f32x8);
#pragma unroll
                        for (int c = 0; c < 8; ++c) v[c] = f[c];
                    } else {
#pragma unroll
                        for (int c = 0; c < 8; ++c) v[c] = __uint_as_float(V.x[i][c / 4][c % 4]);
                    }
                    const f32x8 f = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
                    const wu32x4 own = __builtin_bit_cast(wu32x4, __builtin_convertvector(f, wbf16x8));
#pragma unroll
                    for (int q = 0; q < 4; ++q) u[q] = x_agg ? u[q] : own[q];
                }
                *(wu32x4*)(X + x_to + i * XS * TM * 2) = u;
            }
        }
#pragma unroll
        for (int i = 0; i < ZU; ++i) {
            if (!whole) {
                const unsigned int m = 0u - ((V.z_in >> (zr + i * ZS)) & 1u);
#pragma unroll
                for (int w = 0; w < CPT / 4; ++w) V.g[i][w] &= m;
            }
            float v[CPT];
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const unsigned int raw = (V.o[i][TERMS == 3 ? c : c / 2] & o_and) | o_or;
                const float act = __uint_as_float(TERMS == 3 ? raw : (c & 1 ? raw & 0xFFFF0000u : raw << 16));
                v[c] = act > 0.f ? __uint_as_float(V.g[i][c / 4][c % 4]) : 0.f;
            }
            if (m_tile == 0)      // uniform: the bias gradient is summed by the tiles of the first rows
#pragma unroll
                for (int c = 0; c < CPT; ++c) colsum[c] += (double)v[c];
            put(Z + z_to + i * ZS * TN * 2, ZP, v);
        }
    };

    // `lead` takes the products of the leading terms, `rest` the others (TERMS = 3 only)
    f32x16 lead[MB][NB], rest[TERMS == 3 ? MB : 1][TERMS == 3 ? NB : 1];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                lead[i][j][e] = 0.f;
                if constexpr (TERMS == 3) rest[i][j][e] = 0.f;
            }
    // A fragment (column l32 of a block, 8 rows from 8 * half on) is two transposing reads: of the 16 lanes of a group, lane 4 * j + c reads
    // columns 4 c .. 4 c + 3 of row j, and lane i gets column i of the four rows.
    const int place = (lane >> 2) & 3, row_from = 8 * half + place, in_window = ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    int x_from[MB], z_from[NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) x_from[mb] = row_from * (TM * 2) + ((((wm >> 5) + mb) ^ place) << 6) + in_window;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) z_from[nb] = TERMS * XP + row_from * (TN * 2) + ((((wn >> 5) + nb) ^ place) << 6) + in_window;
    auto fragment = [&](int at, int row_bytes) -> wbf16x8 {
        typedef __attribute__((address_space(3))) ws16x4* lds_s16x4;
        const ws16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(wx_lds + at));
        const ws16x4 c = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(wx_lds + at + 4 * row_bytes));
        return __builtin_bit_cast(wbf16x8, __builtin_shufflevector(a, c, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto multiply = [&](int b) {
#pragma unroll
        for (int ph = 0; ph < WX_STEP / 16; ++ph) {
            wbf16x8 ax[MB][TERMS];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int term = 0; term < TERMS; ++term) ax[mb][term] = fragment(b * BUF + x_from[mb] + term * XP + ph * 16 * TM * 2, TM * 2);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                wbf16x8 bz[TERMS];
#pragma unroll
                for (int term = 0; term < TERMS; ++term) bz[term] = fragment(b * BUF + z_from[nb] + term * ZP + ph * 16 * TN * 2, TN * 2);
                if constexpr (TERMS == 3) {      // (X term, dz term) pairs, smallest products first
                    constexpr int TA[5] = {2, 0, 1, 1, 0};
                    constexpr int TZ[5] = {0, 2, 1, 0, 1};
#pragma unroll
                    for (int e = 0; e < 5; ++e)
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
                            rest[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax[mb][TA[e]], bz[TZ[e]], rest[mb][nb], 0, 0, 0);
                }
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) lead[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax[mb][0], bz[0], lead[mb][nb], 0, 0, 0);
            }
        }
    };

    // A partial result: accumulator element e of a block is its row 8 * (e / 4) + 4 * half + e % 4, column l32. (The addresses are formed
    // on the spot: hoisted out of the loop over the steps they would take registers the loop has not got.)
    auto store_part = [&](int part) {
        int m0 = m_tile + wm + 4 * half, c0 = n_tile + wn + l32;
        asm volatile("" : "+v"(m0), "+v"(c0));
        float* pw = A.part_w + ((int64_t)chunk * A.parts + part) * M * N;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int mp = m0 + mb * 32 + 8 * (e >> 2) + (e & 3);
                const int m = mp < A.d_pad ? (mp < d_in ? mp : M) : d_in + mp - A.d_pad;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int c = c0 + nb * 32;
                    float v = lead[mb][nb][e];
                    if constexpr (TERMS == 3) v += rest[mb][nb][e];
                    if (m < M && c < N) pw[(int64_t)m * N + c] = v;
                    lead[mb][nb][e] = 0.f;
                    if constexpr (TERMS == 3) rest[mb][nb][e] = 0.f;
                }
            }
    };
    const int part_steps = (n_steps + A.parts - 1) / A.parts;
    int part = 0;

    if (n_steps > 0) {      // uniform over the workgroup
        Vals V;
        int32_t p0 = load_positions(0), p1 = load_positions(1), p2 = load_positions(2);
        load_values(0, p0, V);
        stage(0, V);
        load_values(1, p1, V);
        __syncthreads();
        for (int s = 0; s < n_steps; ++s) {
            const int b = s & 1;
            // Step s is multiplied with the loads of step s + 1 in flight; then that one goes to the other buffer (last read a step
            // ago, before the previous barrier) and the registers take step s + 2 (past the chunk: rows that count as zero)
            multiply(b);
            stage(b ^ 1, V);
            load_values(s + 2, p2, V);
            p2 = load_positions(s + 3);
            __syncthreads();
            if (s + 1 == (part + 1) * part_steps || s + 1 == n_steps) store_part(part++);      // uniform
        }
    }
    for (; part < A.parts; ++part) {      // zeros for those without rows
        float* pw = A.part_w + ((int64_t)chunk * A.parts + part) * M * N;
        for (int q = t; q < TM * TN; q += WG_THREADS) {
            const int mp = m_tile + q / TN, m = mp < A.d_pad ? (mp < d_in ? mp : M) : d_in + mp - A.d_pad, c = n_tile + q % TN;
            if (m < M && c < N) pw[(int64_t)m * N + c] = 0.f;
        }
    }
    if (m_tile == 0) {      // column sums of dz: the threads of a column meet in LDS
        double* red = (double*)wx_lds;
#pragma unroll
        for (int c = 0; c < CPT; ++c) red[t * CPT + c] = colsum[c];
        __syncthreads();
        if (t < TN && n_tile + t < N) {
            double sum = 0.0;
            for (int j = 0; j < ZS; ++j) sum += red[(t / CPT + j * ZT) * CPT + t % CPT];
            A.part_b[(int64_t)chunk * N + n_tile + t] = (float)sum;
        }
    }
}

// SRC: element type of a layer's h_src; TERMS = 1: that or bf16 (a model's input layer has the features' type, the others bf16)
//
// U: the cache update of the same iteration (n_layers 0: none), which needs the norms of the embedding gradients as this launch needs the
// gradients. It is a chain of reads, scans and meetings by a few workgroups that leaves the chip idle; behind the weight gradients it was 14 us
// of a small training iteration, and on a second stream it cost two waits for events (5 us each), its row copy (28 us beside the products, 9
// by itself) taking memory time from the products. Its workgroups come first: they are the longer chain where there are few rows, and wait
// for each other. A compute unit holds one workgroup of either kind, so a chunk of positions is 512 threads with twice the positions of
// the update's own launch. Training iteration, own launches / here, us: 1.5 k positions 70.5 / 62.0, 28 k 168.5 / 150.0, 74 k 369 / 356 (runs of one side
// 1 to 5 % apart), GCN 320 / 293, mixed 288.5 / 279; the loop with a sampler beside it 410 / 411. 1433 iterations of random sizes, fp32, GCN and mixed: 0.87 of
// the time on average, none slower.
template <int TERMS, int SRC>
__global__ __launch_bounds__(WG_THREADS, 2) void weight_grad_kernel(WgBatch B, UpdBatch U) {
    const int beside = U.n_layers ? U.sel_first[U.n_layers] : 0, block = (int)blockIdx.x - beside;
    if (block < 0) {
        extern __shared__ __attribute__((aligned(16))) char wx_lds[];
        update_group<WG_THREADS, GRP_CHUNK / 4 / WG_THREADS, false>(U, (int)blockIdx.x, *(GrpShared<WG_THREADS / FG_WAVE>*)wx_lds);
        return;
    }
    // A chunk's tiles read the same rows: the workgroups of one XCD (ids congruent mod 8) take consecutive (chunk, tile) pairs
    const int at = (block & 7) * ((int)(gridDim.x - beside) >> 3) + (block >> 3);
    if (at >= B.first[B.n]) return;       // uniform over the workgroup, before any barrier
    int i = 0;
    while (at >= B.first[i + 1]) ++i;
    const WgIn& A = B.l[i];
    const int unit = at - B.first[i];
    if constexpr (TERMS == 3) {
        if (A.tm == 256)
            weight_grad_tile<256, 128, 3, SRC>(A, unit);
        else
            weight_grad_tile<128, 128, 3, SRC>(A, unit);
    } else if (A.src == SRC) {
        if (A.tm == 256)
            weight_grad_tile<256, 256, 1, SRC>(A, unit);
        else
            weight_grad_tile<128, 128, 1, SRC>(A, unit);
    } else if constexpr (SRC != FG_BF16) {
        if (A.tm == 256)
            weight_grad_tile<256, 256, 1, FG_BF16>(A, unit);
        else
            weight_grad_tile<128, 128, 1, FG_BF16>(A, unit);
    }
}

// dw[i] = sum over the chunks of part_w[chunk][i] in fp64. A workgroup owns 128 consecutive elements (32 lanes x 4) and
// splits the chunks over its 8 wavefront halves; db (the last workgroups) likewise.
// C: the rows that the update beside the products has admitted, copy_blocks workgroups for each of its layers, first in the grid.
constexpr int RED_GROUPS = BW_THREADS / 32;
__global__ __launch_bounds__(BW_THREADS) void weight_grad_reduce_kernel(WgBatch B, fg_row_copy_batch C, int copy_blocks) {
    __shared__ double red[RED_GROUPS][32][4];
    const int at = (int)blockIdx.x - C.n * copy_blocks;
    if (at < 0) {
        const int part = (int)blockIdx.x % copy_blocks;
        fg_copy_rows_part(C.c[blockIdx.x / copy_blocks], ((int64_t)part * BW_THREADS + threadIdx.x) >> 6, ((int64_t)copy_blocks * BW_THREADS) >> 6, threadIdx.x & 63);
        return;
    }
    int layer = 0;
    while (at >= B.red_first[layer + 1]) ++layer;
    const WgIn& A = B.l[layer];
    const int64_t mn = (int64_t)2 * A.d_in * A.d_out;
    const int block = at - B.red_first[layer], w_blocks = (int)((mn + 127) / 128);
    const int tx = threadIdx.x & 31, g = threadIdx.x >> 5;
    const bool is_w = block < w_blocks;
    const int n_chunks = is_w ? A.n_chunks * A.parts : A.n_chunks;
    const float* part = is_w ? A.part_w : A.part_b;
    const int64_t len = is_w ? mn : A.d_out;  // both multiples of 4
    float* out = is_w ? A.dw : A.db;
    const int64_t i = ((int64_t)(is_w ? block : block - w_blocks) * 32 + tx) * 4;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < len) {
        for (int c = g; c < n_chunks; c += 4 * RED_GROUPS) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int cc = c + u * RED_GROUPS;
                v[u] = cc < n_chunks ? *(const f32x4*)(part + (int64_t)cc * len + i) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                s[0] += (double)v[u].x;
                s[1] += (double)v[u].y;
                s[2] += (double)v[u].z;
                s[3] += (double)v[u].w;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) red[g][tx][q] = s[q];
    __syncthreads();
    if (g == 0 && i < len && out) {
        double t[4] = {0.0, 0.0, 0.0, 0.0};
        for (int gg = 0; gg < RED_GROUPS; ++gg)
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] += red[gg][tx][q];
        const f32x4 o = {(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
        *(f32x4*)(out + i) = o;
    }
}

// How a contraction is split: tiles of the result, times chunks of rows.
struct WgPlan {
    int tm, tn, d_pad, n_chunks, parts, tiles_m, tiles_n;
    size_t part_b, total;
    void set_bytes(int64_t d_in, int64_t d_out) {
        part_b = fg_align_up((size_t)n_chunks * parts * 2 * d_in * d_out * 4, 256);
        total = part_b + fg_align_up((size_t)n_chunks * d_out * 4, 256);
    }
};
// of a step of 32 rows, by tile
double wg_step_us(bool mixed, bool large) { return mixed ? (large ? 1.7 : 1.15) : (large ? 2.75 : 1.9); }
// One chunk writes the result itself. Several save it steps but leave partial results, which are
// written, read and added up by a second launch: few rows of a wide layer are better off as one chunk. Mixed precision, one /
// several: 300 rows x 2048 x 1024 19 / 29 us, 700 32 / 34, 1024 42 / 37; 300 x 1024 x 1024 18 / 21, 700 31 / 25.
bool wg_worth_splitting(int64_t max_rows, int64_t d_in, int64_t d_out, int64_t chunks, double step_us) {
    const double saved = (double)fg_ceil_div(max_rows > 0 ? max_rows : 1, WX_STEP) * (1.0 - 1.0 / (double)chunks) * step_us;
    return saved >= 5.0 + (double)(2 * chunks + 1) * (double)(2 * d_in * d_out * 4) / 4.5e6;
}
WgPlan wg_plan(int64_t max_rows, int64_t d_in, int64_t d_out, bool mixed) {
    WgPlan p;
    // Large tiles halve the reads of the operands; small ones fill the chip with fewer chunks, whose partial results have to be
    // written and read. What counts is rows x 128-wide tiles. fp32, large / small: 4 k rows x 16 tiles 33.0 / 32.7 us, 8 tiles 28.8 / 26.1,
    // 33 k x 2 31.7 = 31.7, 4 k x 32 46 / 51, 33 k x 8 72 / 85, 1 k x 128 47 / 51, 33 k x 128 816 / 1030. Mixed precision: 42 / 58 at
    // 240 k, 30 = 30 at 84 k, 30 / 24 at 33 k.
    const int64_t tiles128 = fg_ceil_div(2 * fg_ceil_div(d_in, 64) * 64, 128) * fg_ceil_div(d_out, 128);
    const bool large = mixed ? d_in > 64 && d_out > 128 && tiles128 * max_rows >= 98304 : d_in > 64 && tiles128 * max_rows >= 73728;
    p.tm = large ? 256 : 128;
    p.tn = large && mixed ? 256 : 128;
    const int wide = mixed && p.tm == 256 ? 128 : 64;      // columns of a wavefront
    p.d_pad = (int)fg_ceil_div(d_in, wide) * wide;
    p.tiles_m = (int)fg_ceil_div(2 * p.d_pad, p.tm);
    p.tiles_n = (int)fg_ceil_div(d_out, p.tn);
    // One workgroup fills a compute unit. 32 of them are left to the launches this one runs beside: with all 256 taken the cache
    // update waited for the whole product (its second launch 63 us instead of 9; large SAGE iteration 453 -> 441 us). Not where that
    // leaves a quarter of the chip idle (64 tiles, 4 k rows: 118 us with four chunks, 141 with three) nor in a product of 150 us and more,
    // whose eighth is worth more than what waits (33 k x 1024 x 512 212 us, 232 with 224 workgroups; 100 k 625 and 678). In fp32 a
    // chunk has at most 4096 rows if 512 workgroups suffice for that: its sums are fp32, and with all-positive operands 33 k x 2048 x
    // 1024 is off by 8.4e-7 in one chunk, 1.1e-7 in eight (816 us, four chunks 798).
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    auto fill = [&](int64_t workgroups) { return workgroups / tiles > 1 ? workgroups / tiles : 1; };
    int64_t chunks = fill(tiles > 32 || max_rows > 2048 * fill(224) ? 256 : 224);
    if (!mixed && max_rows > 4096 * chunks) chunks = fill(512);
    // at least two steps per chunk, one where there are few tiles and rows (64 / 32 rows: 1024 rows x 512 x 256 17 / 22 us,
    // 777 rows x 176 x 88 13 / 11 us); more rows never make fewer chunks: a workspace for them serves fewer rows too
    const int64_t some = max_rows > 0 ? max_rows : 1;
    int64_t by_rows = fg_ceil_div(some, 2 * WX_STEP);
    if (p.tiles_m * p.tiles_n <= 2) {
        const int64_t by_step = fg_ceil_div(some, WX_STEP) < 64 ? fg_ceil_div(some, WX_STEP) : 64;
        if (by_rows < by_step) by_rows = by_step;
    }
    if (chunks > by_rows) chunks = by_rows;
    p.n_chunks = wg_worth_splitting(max_rows, d_in, d_out, chunks, wg_step_us(mixed, large)) ? (int)chunks : 1;
    p.parts = 1;
    p.set_bytes(d_in, d_out);
    return p;
}

// Chunks of several layers that share a launch: 224 workgroups in all (32 compute units are left to what runs beside, as above), 256 from
// 150 us on, handed out one chunk at a time to the layer whose workgroups take longest, never more than the layer would have by
// itself. A chunk that is longer than by itself leaves several partial results, so that an fp32 sum has no more rows than there
// (relative error of 6 k rows x 512 x 256 8.7e-8 by itself, 1.9e-7 with one sum per chunk of the shared launch, 8.6e-8 so).
// The three fp32 layers above: 106 us behind each other, 84.5 together; of 24 k x 104 x 88, 4 k x 176 x 88 and 777 x 176 x 48 rows 49 and 28.
// beside: workgroups of an update in the same launch, a compute unit each as well. Up to 32 have the ones left free.
void wg_share(WgPlan* p, const fg_weight_grad_layer_t* y, int n, bool mixed, int beside) {
    int64_t steps[WG_MAX_LAYERS], most[WG_MAX_LAYERS], total = 0;
    double step_us[WG_MAX_LAYERS], work = 0.0;
    for (int i = 0; i < n; ++i) {
        steps[i] = fg_ceil_div(y[i].max_rows > 0 ? y[i].max_rows : 1, WX_STEP);
        step_us[i] = wg_step_us(mixed, p[i].tm == 256);
        most[i] = p[i].n_chunks;
        p[i].n_chunks = 1;
        total += (int64_t)p[i].tiles_m * p[i].tiles_n;
        work += (double)(steps[i] * p[i].tiles_m * p[i].tiles_n) * step_us[i];
    }
    const int64_t free = 256 - beside, target = work < 224.0 * 150.0 && free > 224 ? 224 : free;
    // a workgroup's steps and the partial results it leaves on the way (3 or 5 us each)
    auto time_of = [&](int i) {
        return (double)fg_ceil_div(steps[i], p[i].n_chunks) * step_us[i] + (double)fg_ceil_div(most[i], p[i].n_chunks) * (p[i].tm == 256 ? 5.0 : 3.0);
    };
    for (;;) {
        int longest = 0;
        for (int i = 1; i < n; ++i)
            if (time_of(i) > time_of(longest)) longest = i;
        const int64_t tiles = (int64_t)p[longest].tiles_m * p[longest].tiles_n;
        if (p[longest].n_chunks >= most[longest] || total + tiles > target) break;
        ++p[longest].n_chunks;
        total += tiles;
    }
    for (int i = 0; i < n; ++i) {
        p[i].parts = (int)fg_ceil_div(most[i], p[i].n_chunks);
        p[i].set_bytes(y[i].d_in, y[i].d_out);
    }
}

// What the partial results of a layer take at most there, for up to max_rows rows: fewer than twice those of its own call.
size_t wg_share_bytes(const fg_weight_grad_layer_t& y, bool mixed) {
    WgPlan p = wg_plan(y.max_rows, y.d_in, y.d_out, mixed);
    p.parts = p.n_chunks == 1 ? 1 : 2;
    p.set_bytes(y.d_in, y.d_out);
    return p.total;
}


// Partial products of every chunk of every layer, then their sums; of one chunk the sums themselves. The layers' workspaces lie
// behind each other in ws.
fg_status_t wg_launch(WgIn* in, const WgPlan* p, int n, bool mixed, char* ws, hipStream_t st, const UpdBatch* update = nullptr) {
    WgBatch B{};
    B.n = n;
    UpdBatch U;
    U.n_layers = 0;
    if (update) U = *update;
    size_t lds = update ? sizeof(GrpShared<WG_THREADS / FG_WAVE>) : 0;
    int order[WG_MAX_LAYERS];
    double time[WG_MAX_LAYERS];
    for (int i = 0; i < n; ++i) {
        WgIn& A = in[i];
        A.part_w = (float*)ws;
        A.part_b = (float*)(ws + p[i].part_b);
        ws += p[i].total;
        A.d_pad = p[i].d_pad;
        A.n_chunks = p[i].n_chunks;
        A.parts = p[i].parts;
        A.tiles_m = p[i].tiles_m;
        A.tiles_n = p[i].tiles_n;
        A.tm = p[i].tm;
        if (p[i].n_chunks * p[i].parts == 1) {
            A.part_w = A.dw;
            if (A.db) A.part_b = A.db;
        }
        // without rows (or without anything they could index) every chunk is empty and the partials are zeros
        time[i] = (double)(A.max_rows / p[i].n_chunks) * wg_step_us(mixed, p[i].tm == 256);
        if (A.n <= 0 || A.n_src <= 0) A.max_rows = 0;
        const size_t need = wx_lds_bytes(p[i].tm, p[i].tn, mixed ? 1 : 3);
        lds = need > lds ? need : lds;
        int at = i;      // the longest first
        for (; at > 0 && time[order[at - 1]] < time[i]; --at) order[at] = order[at - 1];
        order[at] = i;
    }
    int src = FG_BF16;
    for (int q = 0; q < n; ++q) {
        const WgIn& A = B.l[q] = in[order[q]];
        if (A.src != FG_BF16) src = A.src;
        B.first[q + 1] = B.first[q] + A.n_chunks * A.tiles_m * A.tiles_n;
        B.red_first[q + 1] = B.red_first[q] + (A.n_chunks * A.parts > 1 ? (int)(fg_ceil_div((int64_t)2 * A.d_in * A.d_out, 128) + fg_ceil_div(A.d_out, 128)) : 0);
    }
    const dim3 grid((unsigned)(fg_ceil_div(B.first[n], 8) * 8 + (update ? U.sel_first[U.n_layers] : 0)));
    if (!mixed)
        hipLaunchKernelGGL((weight_grad_kernel<3, FG_F32>), grid, dim3(WG_THREADS), lds, st, B, U);
    else if (src == FG_F32)
        hipLaunchKernelGGL((weight_grad_kernel<1, FG_F32>), grid, dim3(WG_THREADS), lds, st, B, U);
    else if (src == FG_F16)
        hipLaunchKernelGGL((weight_grad_kernel<1, FG_F16>), grid, dim3(WG_THREADS), lds, st, B, U);
    else
        hipLaunchKernelGGL((weight_grad_kernel<1, FG_BF16>), grid, dim3(WG_THREADS), lds, st, B, U);
    FG_LAUNCH_CHECK("weight_grad_kernel");
    fg_row_copy_batch copies;
    copies.n = 0;
    if (update) fg_update_row_copies(U, &copies);
    if (B.red_first[n] == 0) return fg_launch_row_copies(copies, st);
    // Two workgroups per compute unit and layer copy rows, so that those that add run beside them: with as many as a launch of copies
    // has (2048) they come one after the other (28 k positions 150.5 us, 148.5 so; GCN 295, 291.5, large 365, 361, within what their runs differ by), and with
    // one the launch takes longer (23.4 us, 19.3 so)
    const int row_blocks = update ? fg_row_copy_blocks(copies) : 0, copy_blocks = row_blocks < 512 ? row_blocks : 512;
    if (copy_blocks == 0) copies.n = 0;
    hipLaunchKernelGGL(weight_grad_reduce_kernel, dim3((unsigned)(B.red_first[n] + copies.n * copy_blocks)), dim3(BW_THREADS), 0, st, B, copies, copy_blocks);
    FG_LAUNCH_CHECK("weight_grad_reduce_kernel");
    return FG_OK;
}

}  // namespace

static fg_status_t wg_check_f32(const char* who, const float* h_src_dev, int32_t n_src, int64_t src_stride, const float* agg_dev, int64_t agg_stride,
                                const float* dh_dev, int64_t dh_stride, const float* h_dev, int64_t h_stride, int32_t n, int64_t max_rows, int32_t d_in,
                                int32_t d_out, const float* dw_dev, const float* db_dev) {
    if (n < 0 || n_src < 0 || max_rows < 0 || d_in <= 0 || d_out <= 0)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: bad size (n %d, n_src %d, max_rows %lld, d_in %d, d_out %d)", who, n, n_src, (long long)max_rows, d_in, d_out);
    if (!dw_dev) FG_FAIL(FG_ERR_INVALID_ARG, "%s: dw_dev is NULL", who);
    if (d_out % 4) FG_FAIL(FG_ERR_SHAPE, "%s: d_out = %d must be a multiple of 4", who, d_out);
    if (((uintptr_t)dw_dev | (uintptr_t)db_dev) & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: dw_dev and db_dev must be 16-byte aligned", who);
    if (max_rows > 0 && n > 0 && n_src > 0 && (!h_src_dev || !agg_dev || !dh_dev)) FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    if (src_stride < (int64_t)d_in * 4 || agg_stride < (int64_t)d_in * 4 || dh_stride < (int64_t)d_out * 4 || (h_dev && h_stride < (int64_t)d_out * 4))
        FG_FAIL(FG_ERR_SHAPE, "%s: a row stride is smaller than its row", who);
    if (d_in % 4) FG_FAIL(FG_ERR_SHAPE, "%s: d_in = %d must be a multiple of 4", who, d_in);
    if (((uintptr_t)h_src_dev | (uintptr_t)agg_dev | (uintptr_t)dh_dev | (uintptr_t)h_dev | (uintptr_t)src_stride | (uintptr_t)agg_stride |
         (uintptr_t)dh_stride | (uintptr_t)h_stride) & 15)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: h_src, agg, dh, h and their strides must be 16-byte aligned", who);
    return FG_OK;
}

static fg_status_t wg_check_bf16(const char* who, const void* h_src_dev, int32_t n_src, int64_t src_stride, fg_dtype_t src_dtype, const void* agg_dev,
                                 int64_t agg_stride, const float* dh_dev, int64_t dh_stride, const void* h_dev, int64_t h_stride, int32_t n,
                                 int64_t max_rows, int32_t d_in, int32_t d_out, const float* dw_dev, const float* db_dev) {
    if (n < 0 || n_src < 0 || max_rows < 0 || d_in <= 0 || d_out <= 0)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: bad size (n %d, n_src %d, max_rows %lld, d_in %d, d_out %d)", who, n, n_src, (long long)max_rows, d_in, d_out);
    if (!dw_dev) FG_FAIL(FG_ERR_INVALID_ARG, "%s: dw_dev is NULL", who);
    if (src_dtype != FG_F32 && src_dtype != FG_F16 && src_dtype != FG_BF16) FG_FAIL(FG_ERR_DTYPE, "%s: h_src must be fp32, fp16 or bf16", who);
    const int64_t src_esz = src_dtype == FG_F32 ? 4 : 2;
    if (d_in % 8 || d_out % 8) FG_FAIL(FG_ERR_SHAPE, "%s: d_in = %d and d_out = %d must be multiples of 8", who, d_in, d_out);
    if (((uintptr_t)dw_dev | (uintptr_t)db_dev) & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: dw_dev and db_dev must be 16-byte aligned", who);
    if (max_rows > 0 && n > 0 && n_src > 0 && (!h_src_dev || !agg_dev || !dh_dev)) FG_FAIL(FG_ERR_INVALID_ARG, "%s: NULL pointer", who);
    if (src_stride < (int64_t)d_in * src_esz || agg_stride < (int64_t)d_in * 2 || dh_stride < (int64_t)d_out * 4 || (h_dev && h_stride < (int64_t)d_out * 2))
        FG_FAIL(FG_ERR_SHAPE, "%s: a row stride is smaller than its row", who);
    if (((uintptr_t)h_src_dev | (uintptr_t)agg_dev | (uintptr_t)dh_dev | (uintptr_t)h_dev | (uintptr_t)src_stride | (uintptr_t)agg_stride |
         (uintptr_t)dh_stride | (uintptr_t)h_stride) & 3)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: h_src, agg, dh, h and their strides must be 4-byte aligned", who);
    return FG_OK;
}

extern "C" size_t fg_layer_backward_weights_workspace_bytes(int64_t max_rows, int32_t d_in, int32_t d_out) {
    if (max_rows < 0 || d_in <= 0 || d_out <= 0) return 0;
    return wg_plan(max_rows, d_in, d_out, false).total;
}

extern "C" fg_status_t fg_layer_backward_weights(const float* h_src_dev, int32_t n_src, int64_t src_stride, const float* agg_dev,
                                                 int64_t agg_stride, const float* dh_dev, int64_t dh_stride, const float* h_dev,
                                                 int64_t h_stride, int32_t n, const int32_t* rows_dev, const int64_t* n_rows_dev,
                                                 int64_t max_rows, int32_t d_in, int32_t d_out, float* dw_dev, float* db_dev,
                                                 void* ws_dev, size_t ws_bytes, void* stream) {
    const char* who = "fg_layer_backward_weights";
    const fg_status_t rc = wg_check_f32(who, h_src_dev, n_src, src_stride, agg_dev, agg_stride, dh_dev, dh_stride, h_dev, h_stride, n, max_rows, d_in, d_out,
                                        dw_dev, db_dev);
    if (rc != FG_OK) return rc;
    const WgPlan P = wg_plan(max_rows, d_in, d_out, false);
    if (!ws_dev || ws_bytes < P.total) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, P.total);
    if ((uintptr_t)ws_dev & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: the workspace must be 16-byte aligned", who);
    fg_clear_error();
    WgIn A = {(const char*)h_src_dev, (const char*)agg_dev, (const char*)dh_dev, (const char*)h_dev, src_stride, agg_stride, dh_stride,
              h_stride, max_rows, rows_dev, n_rows_dev, n_src, n, d_in, 0, d_out, 0, 0, 0, 0, FG_F32, 0, nullptr, nullptr, dw_dev, db_dev};
    return wg_launch(&A, &P, 1, false, (char*)ws_dev, (hipStream_t)stream);
}

extern "C" size_t fg_layer_backward_weights_bf16_workspace_bytes(int64_t max_rows, int32_t d_in, int32_t d_out) {
    if (max_rows < 0 || d_in <= 0 || d_out <= 0) return 0;
    return wg_plan(max_rows, d_in, d_out, true).total;
}

extern "C" fg_status_t fg_layer_backward_weights_bf16(const void* h_src_dev, int32_t n_src, int64_t src_stride, fg_dtype_t src_dtype,
                                                      const void* agg_dev, int64_t agg_stride, const float* dh_dev, int64_t dh_stride,
                                                      const void* h_dev, int64_t h_stride, int32_t n, const int32_t* rows_dev,
                                                      const int64_t* n_rows_dev, int64_t max_rows, int32_t d_in, int32_t d_out,
                                                      float* dw_dev, float* db_dev, void* ws_dev, size_t ws_bytes, void* stream) {
    const char* who = "fg_layer_backward_weights_bf16";
    const fg_status_t rc = wg_check_bf16(who, h_src_dev, n_src, src_stride, src_dtype, agg_dev, agg_stride, dh_dev, dh_stride, h_dev, h_stride, n, max_rows,
                                         d_in, d_out, dw_dev, db_dev);
    if (rc != FG_OK) return rc;
    const WgPlan P = wg_plan(max_rows, d_in, d_out, true);
    if (!ws_dev || ws_bytes < P.total) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, P.total);
    if ((uintptr_t)ws_dev & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: the workspace must be 16-byte aligned", who);
    fg_clear_error();
    WgIn A = {(const char*)h_src_dev, (const char*)agg_dev, (const char*)dh_dev, (const char*)h_dev, src_stride, agg_stride, dh_stride,
              h_stride, max_rows, rows_dev, n_rows_dev, n_src, n, d_in, 0, d_out, 0, 0, 0, 0, (int)src_dtype, 0, nullptr, nullptr, dw_dev, db_dev};
    return wg_launch(&A, &P, 1, true, (char*)ws_dev, (hipStream_t)stream);
}

static fg_status_t wg_check(const char* who, const fg_weight_grad_layer_t& y, bool mixed) {
    if (mixed)
        return wg_check_bf16(who, y.h_src_dev, y.n_src, y.src_stride, y.src_dtype, y.agg_dev, y.agg_stride, y.dh_dev, y.dh_stride, y.h_dev, y.h_stride,
                             y.n, y.max_rows, y.d_in, y.d_out, y.dw_dev, y.db_dev);
    if (y.src_dtype != FG_F32) FG_FAIL(FG_ERR_DTYPE, "%s: h_src must be fp32", who);
    return wg_check_f32(who, (const float*)y.h_src_dev, y.n_src, y.src_stride, (const float*)y.agg_dev, y.agg_stride, y.dh_dev, y.dh_stride,
                        (const float*)y.h_dev, y.h_stride, y.n, y.max_rows, y.d_in, y.d_out, y.dw_dev, y.db_dev);
}

extern "C" size_t fg_backward_weights_all_workspace_bytes(fg_dtype_t compute_dtype, int32_t n_layers, const fg_weight_grad_layer_t* layers) {
    if ((compute_dtype != FG_F32 && compute_dtype != FG_BF16) || n_layers < 1 || n_layers > WG_MAX_LAYERS || !layers) return 0;
    size_t total = 0;
    for (int i = 0; i < n_layers; ++i) {
        if (layers[i].max_rows < 0 || layers[i].d_in <= 0 || layers[i].d_out <= 0) return 0;
        total += wg_share_bytes(layers[i], compute_dtype == FG_BF16);
    }
    return total;
}

extern "C" fg_status_t fg_backward_weights_all(fg_dtype_t compute_dtype, int32_t n_layers, const fg_weight_grad_layer_t* layers, void* ws_dev,
                                               size_t ws_bytes, void* stream) {
    return fg_backward_weights_with(compute_dtype, n_layers, layers, ws_dev, ws_bytes, nullptr, stream);
}

fg_status_t fg_backward_weights_with(fg_dtype_t compute_dtype, int32_t n_layers, const fg_weight_grad_layer_t* layers, void* ws_dev, size_t ws_bytes,
                                     const UpdBatch* update, void* stream) {
    const char* who = "fg_backward_weights_all";
    if (compute_dtype != FG_F32 && compute_dtype != FG_BF16) FG_FAIL(FG_ERR_DTYPE, "%s: compute_dtype must be F32 or BF16", who);
    if (n_layers < 1 || n_layers > WG_MAX_LAYERS || !layers)
        FG_FAIL(FG_ERR_INVALID_ARG, "%s: n_layers = %d must be in 1..%d and layers non-NULL", who, n_layers, WG_MAX_LAYERS);
    const bool mixed = compute_dtype == FG_BF16;
    WgIn in[WG_MAX_LAYERS];
    WgPlan p[WG_MAX_LAYERS];
    int src = FG_BF16;      // the one type besides it
    for (int i = 0; i < n_layers; ++i) {
        const fg_weight_grad_layer_t& y = layers[i];
        fg_status_t rc = wg_check(who, y, mixed);
        if (rc != FG_OK) return rc;
        if (mixed && y.src_dtype != FG_BF16 && src != FG_BF16 && y.src_dtype != src)
            FG_FAIL(FG_ERR_DTYPE, "%s: the layers' h_src have more than one type besides bf16", who);
        if (y.src_dtype != FG_BF16) src = (int)y.src_dtype;
        p[i] = wg_plan(y.max_rows, y.d_in, y.d_out, mixed);
        in[i] = {(const char*)y.h_src_dev, (const char*)y.agg_dev, (const char*)y.dh_dev, (const char*)y.h_dev, y.src_stride, y.agg_stride, y.dh_stride,
                 y.h_stride, y.max_rows, y.rows_dev, y.n_rows_dev, y.n_src, y.n, y.d_in, 0, y.d_out, 0, 0, 0, 0, (int)y.src_dtype, 0, nullptr, nullptr,
                 y.dw_dev, y.db_dev};
    }
    const size_t need = fg_backward_weights_all_workspace_bytes(compute_dtype, n_layers, layers);
    if (!ws_dev || ws_bytes < need) FG_FAIL(FG_ERR_SHAPE, "%s: workspace of %zu bytes given, %zu needed", who, ws_bytes, need);
    if ((uintptr_t)ws_dev & 15) FG_FAIL(FG_ERR_INVALID_ARG, "%s: the workspace must be 16-byte aligned", who);
    fg_clear_error();
    wg_share(p, layers, n_layers, mixed, update ? update->sel_first[update->n_layers] : 0);
    return wg_launch(in, p, n_layers, mixed, (char*)ws_dev, (hipStream_t)stream, update);
}
