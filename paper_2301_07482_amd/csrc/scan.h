// Device helpers for order-preserving compaction with 64-lane wavefronts.
//
// A list is compacted in two launches with no waiting between workgroups: the first launch leaves one
// count per workgroup, the second lets every workgroup add up the counts of the workgroups before it
// (a few KB from L2) and then ranks its own elements with wavefront ballots.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int FG_WAVE = 64;

__device__ __forceinline__ int fg_lane() { return threadIdx.x & (FG_WAVE - 1); }
__device__ __forceinline__ int fg_wave() { return threadIdx.x >> 6; }

// Inclusive prefix sum over a wavefront, all 64 lanes active. The lanes' values move inside the vector registers (DPP: shifts by 1, 2, 4, 8
// within rows of 16 lanes, then a row's last lane to the next row and the last of the lower half to the upper), where a shuffle
// goes through the LDS unit: six dependent additions instead of six round trips.
__device__ __forceinline__ int fg_wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Of the totals that WAVES wavefronts left in `totals` (16-byte aligned): the sum of those before this one, and of all.
template <int WAVES>
__device__ __forceinline__ void fg_wave_totals(const int* totals, int& before, int& all) {
    static_assert(WAVES % 4 == 0, "read four at a time");
    before = all = 0;
    const int wave = fg_wave();
#pragma unroll
    for (int w = 0; w < WAVES; w += 4) {
        const int4 v = *(const int4*)(totals + w);
        all += v.x + v.y + v.z + v.w;
        before += (w < wave ? v.x : 0) + (w + 1 < wave ? v.y : 0) + (w + 2 < wave ? v.z : 0) + (w + 3 < wave ? v.w : 0);
    }
}

// Number of lanes below this one for which `flag` holds; `total` = lanes of the wave for which it holds.
__device__ __forceinline__ int fg_wave_rank(bool flag, int& total) {
    const unsigned long long m = __ballot(flag);
    total = __popcll(m);
    return __popcll(m & ((1ull << fg_lane()) - 1ull));
}

// Exclusive rank of `flag` within a workgroup of up to 1024 threads (blockDim.x a multiple of 64) and the
// workgroup total. `lds` needs 17 ints and may be reused after the call returns.
__device__ __forceinline__ int fg_block_rank(bool flag, int& block_total, int* lds) {
    int wave_total;
    const int r = fg_wave_rank(flag, wave_total);
    const int nw = blockDim.x >> 6;
    __syncthreads();  // protects a previous use of lds
    if (fg_lane() == 0) lds[fg_wave()] = wave_total;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < nw; ++w) {
        const int t = lds[w];
        if (w < fg_wave()) before += t;
        all += t;
    }
    block_total = all;
    return before + r;
}

// Sum over the workgroup of a per-thread int64 value; every thread gets the result. `lds64` needs 16 entries.
__device__ __forceinline__ long long fg_block_sum(long long v, long long* lds64) {
    for (int off = FG_WAVE / 2; off > 0; off >>= 1) v += __shfl_down(v, off, FG_WAVE);
    const int nw = blockDim.x >> 6;
    __syncthreads();
    if (fg_lane() == 0) lds64[fg_wave()] = v;
    __syncthreads();
    long long s = 0;
    for (int w = 0; w < nw; ++w) s += lds64[w];
    return s;
}
