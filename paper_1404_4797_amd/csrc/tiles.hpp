// Slot tiles for slot-parallel kernels over a CSR: each workgroup takes
// kTile consecutive adjacency slots and recovers the source row of every
// slot in LDS (row starts scattered into the tile, then a max-scan), so rows
// of any length are split evenly over the grid without a per-slot search.
#pragma once

#include "common.hpp"

namespace sclap {
namespace {

constexpr int kTileThreads = 256;
constexpr int kTilePer = 8;
constexpr int kTile = kTileThreads * kTilePer;

__device__ int32_t upper_node(const int64_t* __restrict__ xadj, int32_t n, int64_t slot) {
    // largest u in [0, n) with xadj[u] <= slot
    int32_t lo = 0, hi = n;  // invariant: xadj[lo] <= slot, answer in [lo, hi)
    while (hi - lo > 1) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (xadj[mid] <= slot) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Source row of the first slot of every tile, and at [ntiles] the row of the
// last slot: tile t then holds the row starts of rows trow[t]+1 .. trow[t+1]
// (those that start inside it).  One search per tile, all in parallel, once
// per graph, instead of two dependent searches at the start of every tile.
__global__ void tile_rows_kernel(const int64_t* __restrict__ xadj, int32_t n, int64_t S, int64_t ntiles,
                                 int32_t* __restrict__ trow) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t > ntiles) return;
    const int64_t slot = t * kTile < S ? t * kTile : S - 1;
    trow[t] = upper_node(xadj, n, slot);
}

// Tiles of the S slots over the rows [0, n) of xadj (offsets monotone; no
// tiles when S = 0).
struct TileRows {
    int64_t ntiles = 0;
    DBuf<int32_t> trow;
    TileRows(const int64_t* xadj, int32_t n, int64_t S, hipStream_t s) {
        ntiles = S > 0 ? (S + kTile - 1) / kTile : 0;
        trow.alloc(static_cast<size_t>(ntiles) + 1, s);
        if (ntiles == 0) return;
        tile_rows_kernel<<<grid_for(ntiles + 1, 256), 256, 0, s>>>(xadj, n, S, ntiles, trow.get());
        LAUNCHCHK();
    }
};

// Fills owner[0 .. i1-i0) with the source node of each slot of tile `tile`
// ([i0, i1)), from the tile's first row trow[tile].
__device__ void tile_owners(const int64_t* __restrict__ xadj, const int32_t* __restrict__ trow, int64_t tile,
                            int64_t i0, int64_t i1, int32_t* owner) {
    __shared__ int32_t s_carry[kTileThreads / kWave];
    const int tid = threadIdx.x;
    for (int j = tid; j < kTile; j += kTileThreads) owner[j] = -1;
    const int32_t u0 = trow[tile], u1 = trow[tile + 1];
    __syncthreads();
    if (tid == 0) atomicMax(&owner[0], u0);
    for (int64_t u = static_cast<int64_t>(u0) + 1 + tid; u <= u1; u += kTileThreads) {
        const int64_t st = xadj[u];
        if (st >= i0 && st < i1) atomicMax(&owner[st - i0], static_cast<int32_t>(u));
    }
    __syncthreads();
    // inclusive max-scan over the tile: 8 consecutive entries per thread
    int32_t loc[kTilePer];
    int32_t m = -1;
#pragma unroll
    for (int j = 0; j < kTilePer; ++j) {
        loc[j] = owner[tid * kTilePer + j];
        m = loc[j] > m ? loc[j] : m;
    }
    int32_t incl = m;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, 64);
        if (lane_id() >= o) incl = t > incl ? t : incl;
    }
    if (lane_id() == kWave - 1) s_carry[tid / kWave] = incl;
    __syncthreads();
    int32_t run = __shfl_up(incl, 1, 64);
    if (lane_id() == 0) run = -1;
    for (int w = 0; w < tid / kWave; ++w) run = s_carry[w] > run ? s_carry[w] : run;
#pragma unroll
    for (int j = 0; j < kTilePer; ++j) {
        run = loc[j] > run ? loc[j] : run;
        owner[tid * kTilePer + j] = run;
    }
    __syncthreads();
}

// The same for the kTilePer consecutive slots i0 + kTilePer * threadIdx.x ..
// of each thread, in registers (entries past i1 repeat the last row): no
// second trip through LDS, and the thread reads its slots' ids and weights 16
// bytes at a time.  mark: kTile entries of LDS, 16-byte aligned.
__device__ __forceinline__ void tile_rows(const int64_t* __restrict__ xadj, const int32_t* __restrict__ trow,
                                          int64_t tile, int64_t i0, int64_t i1, int32_t* mark,
                                          int32_t (&row)[kTilePer]) {
    static_assert(kTilePer == 8, "two 16-byte words per thread");
    __shared__ int32_t s_carry[kTileThreads / kWave];
    const int tid = threadIdx.x;
    int4* own = reinterpret_cast<int4*>(mark) + 2 * tid;
    own[0] = make_int4(-1, -1, -1, -1);
    own[1] = make_int4(-1, -1, -1, -1);
    const int32_t u0 = trow[tile], u1 = trow[tile + 1];
    __syncthreads();
    for (int64_t u = static_cast<int64_t>(u0) + 1 + tid; u <= u1; u += kTileThreads) {
        const int64_t st = xadj[u];
        if (st >= i0 && st < i1) atomicMax(&mark[st - i0], static_cast<int32_t>(u));
    }
    __syncthreads();
    const int4 a = own[0], b = own[1];
    row[0] = a.x;
    row[1] = a.y;
    row[2] = a.z;
    row[3] = a.w;
    row[4] = b.x;
    row[5] = b.y;
    row[6] = b.z;
    row[7] = b.w;
#pragma unroll
    for (int j = 1; j < kTilePer; ++j) row[j] = row[j] > row[j - 1] ? row[j] : row[j - 1];
    int32_t incl = row[kTilePer - 1];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t x = __shfl_up(incl, o, 64);
        if (lane_id() >= o) incl = x > incl ? x : incl;
    }
    if (lane_id() == kWave - 1) s_carry[tid / kWave] = incl;
    __syncthreads();
    int32_t run = __shfl_up(incl, 1, 64);
    if (lane_id() == 0) run = -1;
    run = u0 > run ? u0 : run;
#pragma unroll
    for (int w = 0; w < kTileThreads / kWave; ++w) run = w < tid / kWave && s_carry[w] > run ? s_carry[w] : run;
#pragma unroll
    for (int j = 0; j < kTilePer; ++j) row[j] = row[j] > run ? row[j] : run;
}

// The thread's kTilePer values of a slot array from slot i on; `past` beyond
// i1.  wide (the same for the whole workgroup): the tile is full and p
// 16-byte aligned.
__device__ __forceinline__ bool wide_tile(const void* p, int64_t i0, int64_t i1) {
    return i1 - i0 == kTile && (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}

__device__ __forceinline__ void tile_load(const int32_t* __restrict__ p, int64_t i, int64_t i1, bool wide, int32_t past,
                                          int32_t (&x)[kTilePer]) {
    if (wide) {
        const int4 a = reinterpret_cast<const int4*>(p + i)[0];
        const int4 b = reinterpret_cast<const int4*>(p + i)[1];
        x[0] = a.x;
        x[1] = a.y;
        x[2] = a.z;
        x[3] = a.w;
        x[4] = b.x;
        x[5] = b.y;
        x[6] = b.z;
        x[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < kTilePer; ++j) x[j] = i + j < i1 ? p[i + j] : past;
    }
}

}  // namespace
}  // namespace sclap
