// Cluster contraction on gfx950 (Section 3.1 contraction definition; Section
// 4.3 relabelling and quotient graph).
//
// Coarse ids are the ranks of the used labels (mark + exclusive scan).  The
// quotient graph is built row by row instead of by one global sort:
//   1. count, per fine node u, the slots u->v with C(u) != C(v), and add the
//      counts up per coarse row (one atomic per node: in the multilevel path
//      a cluster has at most U members, however many slots its rows hold);
//   2. scan the row counts into row offsets, give every node a block of its
//      row and scatter (C(v), w) of every such slot into its node's block
//      (at its rank; a row that spans slot tiles reserves each tile's part);
//   3. merge equal neighbours of each row, summing weights: rows of up to 64
//      entries in the registers of one wave (bitonic network over lanes), up
//      to 4096 in an LDS table of one workgroup, longer rows by chunks and then
//      by hash buckets;
//   4. scan the merged row lengths into the coarse offsets and copy;
//   5. for the canonical form (rows ascend by neighbour id, whatever order the
//      atomics of step 2 produced) order every row's distinct entries by an
//      LDS radix sort, rows of more than 8192 by one over (row, id) keys.
#include <climits>

#include "graph_ops.hpp"
#include "profile.hpp"
#include "tiles.hpp"

namespace sclap {

namespace {

constexpr int kWaveRow = 64;     // rows up to this length: one wave
constexpr int kBlockRow = 4096;  // up to this length: one workgroup, LDS table
constexpr int kRowClasses = 7;   // one wave; tables for up to 256, 512, .. 4096 entries; long

__global__ void mark_used_kernel(int32_t n, const int32_t* __restrict__ labels, int32_t* __restrict__ used) {
    const int32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v < n) used[labels[v]] = 1;
}

__global__ void map_kernel(int32_t n, const int32_t* __restrict__ labels, const int32_t* __restrict__ q,
                           const int32_t* __restrict__ vw, int32_t* __restrict__ C, int32_t* __restrict__ cvw) {
    const int32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    const int32_t cv = q[labels[v]];
    C[v] = cv;
    const int32_t c = vw ? vw[v] : 1;
    if (c) atomicAdd(&cvw[cv], c);
}

// probe_out[i] = number of used labels below probe[i] (probe[i] in [0, n]).
__global__ void probe_kernel(const int32_t* __restrict__ probe, int32_t nprobe, const int32_t* __restrict__ q,
                             int32_t n, const int32_t* __restrict__ total, int32_t* __restrict__ out) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < nprobe) out[i] = probe[i] < n ? q[probe[i]] : *total;
}

__device__ __forceinline__ int32_t block_sum_i32_256(int32_t v) {
    __shared__ int32_t sred[4];
    v = wave_sum(v);
    if (lane_id() == 0) sred[threadIdx.x >> 6] = v;
    __syncthreads();
    const int32_t t = sred[0] + sred[1] + sred[2] + sred[3];
    __syncthreads();
    return t;
}

// The inter-cluster slots before each slot of a tile, from one flag per slot
// (slot i0 + r * kTileThreads + thread in flag r): before[j] for slot j, and
// their number in before[kTile].  Rows lie one after the other in a tile, so a
// row's count, and a slot's rank within its row, are differences of two
// entries; counting wave by wave took an atomic per wave and row, whose return
// the writes of row_scatter waited for eight times in a row (128 M slots:
// 1.06 -> 0.60 ms, 2 TB/s; cross_count, bound by its gather, 1.00 -> 0.93).
__device__ __forceinline__ void tile_prefix(const bool (&flag)[kTilePer], int32_t* before) {
    constexpr int kGroups = kTile / 64;  // 64 consecutive slots each
    __shared__ int32_t s_group[kGroups];
    static_assert(kGroups <= 64, "one lane per group");
    const int lane = lane_id();
    const int wid = threadIdx.x / kWave;
    uint64_t m[kTilePer];
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        m[r] = __ballot(flag[r]);
        if (lane == 0) s_group[r * (kTileThreads / kWave) + wid] = __popcll(m[r]);
    }
    __syncthreads();
    const int32_t mine = lane < kGroups ? s_group[lane] : 0;
    int32_t incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        const int32_t base = __shfl(incl - mine, r * (kTileThreads / kWave) + wid, 64);
        before[r * kTileThreads + threadIdx.x] = base + __popcll(m[r] & ((1ULL << lane) - 1));
    }
    if (threadIdx.x == kWave - 1) before[kTile] = incl;
    __syncthreads();
}

// Step 1: inter-cluster slots per fine node, cross[u] (zero before: a row
// that lies in one tile is stored, the others' parts are added); keeps C(v) of
// every such slot for step 2 (-1 for the others), which then reads it in slot
// order instead of gathering it again.
__global__ void __launch_bounds__(kTileThreads) cross_count_kernel(const int64_t* __restrict__ xadj,
                                                                   const int32_t* __restrict__ adj, int32_t n,
                                                                   int64_t S, const int32_t* __restrict__ C,
                                                                   int32_t* __restrict__ cross,
                                                                   int32_t* __restrict__ cvs, const int32_t* __restrict__ trow) {
    __shared__ int32_t owner[kTile];
    __shared__ int32_t before[kTile + 1];
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int64_t i1 = i0 + kTile < S ? i0 + kTile : S;
    tile_owners(xadj, trow, static_cast<int64_t>(blockIdx.x), i0, i1, owner);
    // the gathers of all the thread's slots together
    int32_t u[kTilePer], cv[kTilePer], cu[kTilePer];
    bool e[kTilePer];
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        const int64_t i = i0 + r * kTileThreads + threadIdx.x;
        u[r] = i < i1 ? owner[i - i0] : -1;
        cv[r] = i < i1 ? adj[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        cv[r] = u[r] >= 0 ? C[cv[r]] : 0;
        cu[r] = u[r] >= 0 ? C[u[r]] : 0;
    }
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        e[r] = u[r] >= 0 && cu[r] != cv[r];
        if (u[r] >= 0) cvs[i0 + r * kTileThreads + threadIdx.x] = e[r] ? cv[r] : -1;
    }
    tile_prefix(e, before);
    for (int64_t v = trow[blockIdx.x] + static_cast<int64_t>(threadIdx.x); v <= trow[blockIdx.x + 1]; v += kTileThreads) {
        const int64_t b = xadj[v], end = xadj[v + 1];
        const int64_t lo = b > i0 ? b : i0, hi = end < i1 ? end : i1;
        if (lo >= hi) continue;
        const int32_t cnt = before[hi - i0] - before[lo - i0];
        if (lo == b && hi == end) cross[v] = cnt;
        else if (cnt) atomicAdd(&cross[v], cnt);
    }
}

// Per fine node: its coarse row grows by cross[u] ...
__global__ void row_count_kernel(int32_t n, const int32_t* __restrict__ C, const int32_t* __restrict__ cross,
                                 int32_t* __restrict__ rowcnt) {
    const int32_t u = blockIdx.x * 256 + threadIdx.x;
    if (u < n && cross[u]) atomicAdd(&rowcnt[C[u]], cross[u]);
}

// ... and, once rows are placed, each node reserves its block of the row.
__global__ void node_base_kernel(int32_t n, const int32_t* __restrict__ C, const int32_t* __restrict__ cross,
                                 const int64_t* __restrict__ rowoff, int32_t* __restrict__ fill,
                                 int64_t* __restrict__ nbase) {
    const int32_t u = blockIdx.x * 256 + threadIdx.x;
    if (u < n && cross[u]) nbase[u] = rowoff[C[u]] + atomicAdd(&fill[C[u]], cross[u]);
}

// Step 2: (C(v), w) of every inter-cluster slot into its node's block of the
// coarse row: at its rank, in rows that lie in one tile; the other rows (at most
// the tile's first and last) reserve the tile's part of their block.  All of a
// thread's reads are in flight together.  Unit weights (ew null) are not
// written: the merge knows them.
__global__ void __launch_bounds__(kTileThreads) row_scatter_kernel(const int64_t* __restrict__ xadj,
                                                                   const int32_t* __restrict__ cvs,
                                                                   const int32_t* __restrict__ ew, int64_t S,
                                                                   const int64_t* __restrict__ nbase,
                                                                   int32_t* __restrict__ nfill,
                                                                   int32_t* __restrict__ tk, int32_t* __restrict__ tw, const int32_t* __restrict__ trow) {
    __shared__ int32_t owner[kTile];
    __shared__ int32_t before[kTile + 1];
    __shared__ int32_t s_part[2];
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int64_t i1 = i0 + kTile < S ? i0 + kTile : S;
    tile_owners(xadj, trow, static_cast<int64_t>(blockIdx.x), i0, i1, owner);
    int32_t u[kTilePer], cv[kTilePer], wt[kTilePer];
    int64_t at[kTilePer], begin[kTilePer];
    bool e[kTilePer];
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        const int64_t i = i0 + r * kTileThreads + threadIdx.x;
        u[r] = i < i1 ? owner[i - i0] : -1;
        cv[r] = i < i1 ? cvs[i] : -1;
        wt[r] = i < i1 && ew ? ew[i] : 0;
        e[r] = cv[r] >= 0;
    }
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        at[r] = e[r] ? nbase[u[r]] : 0;
        begin[r] = e[r] ? xadj[u[r]] : 0;
    }
    tile_prefix(e, before);
    // the rows that reach beyond the tile, if any (one row may be both)
    const int32_t first = owner[0], last = owner[i1 - i0 - 1];
    const bool head = xadj[first] < i0, tail = xadj[last + 1] > i1;  // uniform
    if (threadIdx.x < 2) {
        const bool mine = threadIdx.x == 0 ? head : tail && !(head && first == last);
        const int32_t v = threadIdx.x == 0 ? first : last;
        int32_t base = 0;
        if (mine) {
            const int64_t b = xadj[v], end = xadj[v + 1];
            const int32_t cnt = before[(end < i1 ? end : i1) - i0] - before[b > i0 ? b - i0 : 0];
            if (cnt) base = atomicAdd(&nfill[v], cnt);
        }
        s_part[threadIdx.x] = base;
    }
    __syncthreads();
    const int32_t part0 = head ? s_part[0] : 0, part1 = s_part[1];
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        if (!e[r]) continue;
        const int32_t rank = before[r * kTileThreads + threadIdx.x] - before[begin[r] > i0 ? begin[r] - i0 : 0];
        at[r] += rank + (u[r] == first ? part0 : 0);
        if (u[r] == last && !(head && first == last)) at[r] += part1;
        tk[at[r]] = cv[r];
        if (ew) tw[at[r]] = wt[r];
    }
}

// Rows by length: 0 or 1 entries are final as they are; the others go to the
// list of their class: up to 64 entries (one wave), up to 256, 512, .. 4096 (one
// workgroup with a table of twice that) or long.
// (each workgroup takes kClassifyIters * 256 consecutive rows at a time and
// appends to each list with one atomic: the counters are few and hot)
constexpr int kClassifyIters = 16;

__global__ void __launch_bounds__(256) row_classify_kernel(int32_t nc, const int64_t* __restrict__ rowoff,
                                                           const int32_t* __restrict__ rowcnt,
                                                           int32_t* __restrict__ dcnt, int32_t* __restrict__ tw,
                                                           bool unit, int32_t* __restrict__ lists,
                                                           int32_t cap, uint32_t* __restrict__ counts) {
    for (int32_t base = blockIdx.x * (kClassifyIters * 256); base < nc; base += gridDim.x * (kClassifyIters * 256)) {
        uint32_t m[kRowClasses] = {};
        int32_t lens[kClassifyIters];
#pragma unroll
        for (int it = 0; it < kClassifyIters; ++it) {
            const int32_t r = base + it * 256 + static_cast<int32_t>(threadIdx.x);
            lens[it] = r < nc ? rowcnt[r] : -1;
        }
#pragma unroll
        for (int it = 0; it < kClassifyIters; ++it) {
            const int32_t r = base + it * 256 + static_cast<int32_t>(threadIdx.x);
            const int32_t len = lens[it];
            if (len < 0) continue;
            if (len <= 1) {
                dcnt[r] = len;
                if (unit && len == 1) tw[rowoff[r]] = 1;  // merged as it stands
                continue;
            }
#pragma unroll
            for (int c = 0; c < kRowClasses; ++c) {
                const int32_t lo = c == 0 ? 1 : (c == 1 ? kWaveRow : 128 << (c - 1));
                const int32_t hi = c == 0 ? kWaveRow : (c == kRowClasses - 1 ? INT_MAX : 128 << c);
                if (len > lo && len <= hi) m[c] |= 1u << it;
            }
        }
#pragma unroll
        for (int c = 0; c < kRowClasses; ++c) {
            uint32_t bits = m[c];
            if (!__syncthreads_or(bits != 0)) continue;
            uint32_t j = block_append_count(static_cast<uint32_t>(__popc(bits)), &counts[c]);
            while (bits) {
                const int it = __ffs(bits) - 1;
                bits &= bits - 1;
                lists[static_cast<int64_t>(c) * cap + j++] = base + it * 256 + static_cast<int32_t>(threadIdx.x);
            }
        }
    }
}

// Sorts (key, w) over the 64 lanes of a wave.
__device__ __forceinline__ void bitonic_wave(uint32_t& key, int32_t& w, int lane) {
    for (int k = 2; k <= 64; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const uint32_t ok = __shfl_xor(key, j, 64);
            const int32_t ow = __shfl_xor(w, j, 64);
            const bool up = (lane & k) == 0;
            const bool low = (lane & j) == 0;
            const bool take = low == up ? ok < key : ok > key;
            if (take) {
                key = ok;
                w = ow;
            }
        }
    }
}

// Merges the entries tk/tw[b, b + cnt), cnt <= kT / 2, in place in a table of kT
// LDS entries and returns the number of distinct ones in the last thread.  A
// thread's entries are all loaded before the table is needed, and it writes the
// ids that its own entries brought into the table (in no particular order)
// instead of searching the table for them (contraction of 128 M slots, chunks
// of long rows 0.65 -> 0.41 ms, rows of 2049..4096 entries 0.21 -> 0.10 ms).
template <int NT, int kT>
__device__ __forceinline__ int32_t merge_in_lds(int64_t b, int32_t cnt, int32_t* __restrict__ tk,
                                                int32_t* __restrict__ tw, bool unit, int32_t* keys, int32_t* sums) {
    constexpr int U = kT / 2 / NT;
    __shared__ int32_t s_w[NT / kWave];
    const int tid = threadIdx.x;
    int32_t x[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t j = tid + u * NT;
        x[u] = j < cnt ? tk[b + j] : -1;
        w[u] = j < cnt ? (unit ? 1 : tw[b + j]) : 0;
    }
    for (int j = 4 * tid; j < kT; j += 4 * NT) {
        *reinterpret_cast<int4*>(keys + j) = make_int4(-1, -1, -1, -1);
        *reinterpret_cast<int4*>(sums + j) = make_int4(0, 0, 0, 0);
    }
    __syncthreads();
    int32_t mine = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (x[u] < 0) continue;
        uint32_t h = slot_hash(static_cast<uint32_t>(x[u])) & (kT - 1);
        int32_t prev;
        while (true) {
            prev = atomicCAS(&keys[h], -1, x[u]);
            if (prev == -1 || prev == x[u]) break;
            h = (h + 1) & (kT - 1);
        }
        atomicAdd(&sums[h], w[u]);  // partial sums never exceed the final coarse weight
        w[u] = prev == -1 ? static_cast<int32_t>(h) : -1;
        if (prev == -1) ++mine;
        else x[u] = -1;
    }
    int32_t incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, 64);
        if (lane_id() >= o) incl += t;
    }
    if (lane_id() == kWave - 1) s_w[tid / kWave] = incl;
    __syncthreads();
    int32_t pos = incl - mine;
    for (int v = 0; v < tid / kWave; ++v) pos += s_w[v];
    const int32_t end = pos + mine;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (x[u] < 0) continue;
        tk[b + pos] = x[u];
        tw[b + pos] = sums[w[u]];
        ++pos;
    }
    return end;
}

// Rows of 2..64 entries: one wave per row sorts (C(v), w) over its lanes with a
// bitonic network and writes the merged row to the row's start.
__global__ void __launch_bounds__(256) wave_rows_kernel(const int32_t* __restrict__ list, uint32_t count,
                                                        const int64_t* __restrict__ rowoff,
                                                        const int32_t* __restrict__ rowcnt, int32_t* __restrict__ tk,
                                                        int32_t* __restrict__ tw, bool unit,
                                                        int32_t* __restrict__ dcnt) {
    const uint32_t wv = (blockIdx.x * 256 + threadIdx.x) >> 6;
    if (wv >= count) return;  // uniform per wave
    const int lane = lane_id();
    const int32_t row = list[wv];
    const int64_t b = rowoff[row];
    const int32_t len = rowcnt[row];
    uint32_t key = lane < len ? static_cast<uint32_t>(tk[b + lane]) : 0xFFFFFFFFu;
    int32_t w = lane < len ? (unit ? 1 : tw[b + lane]) : 0;
    bitonic_wave(key, w, lane);
    // merge equal neighbours: inclusive sums over the lanes, then per run
    const uint32_t prev = __shfl_up(key, 1, 64);
    const bool valid = lane < len;
    const bool head = valid && (lane == 0 || prev != key);
    int64_t incl = w;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    const uint64_t heads = __ballot(head);
    const uint64_t upto = (2ULL << lane) - 1;
    const uint64_t after = heads & ~upto;
    const int last = (after ? __ffsll(static_cast<long long>(after)) - 1 : len) - 1;  // last lane of this run
    const int64_t at_last = __shfl(incl, last < 0 ? 0 : last, 64);
    if (head) {
        const int pos = __popcll(heads & (upto >> 1));
        tk[b + pos] = static_cast<int32_t>(key);
        tw[b + pos] = static_cast<int32_t>(at_last - incl + w);
    }
    if (lane == 0) dcnt[row] = __popcll(heads);
}

// Orders rows of distinct entries by neighbour id: one workgroup of NW waves
// per row of up to NW * 512 entries, a stable least-significant-digit-first
// radix sort of (id, w) with 8-bit digits.  Elements live in registers (8 per
// thread, a wave holding consecutive ones) and meet in LDS once per digit: a
// wave ranks its elements by matching digits with ballots against counters of
// its own.  A bitonic network over the entries before they were merged took
// 4.0 ms on the rows of 65..4096 entries of a contracted R-MAT 2^22; merging
// first and ordering the distinct entries like this takes 1.0 ms.
template <int NW>
__global__ void __launch_bounds__(NW * 64) order_rows_kernel(const int32_t* __restrict__ list,
                                                             const int64_t* __restrict__ xadj,
                                                             int32_t* __restrict__ adj, int32_t* __restrict__ ew,
                                                             int bits) {
    constexpr int NT = NW * 64;
    constexpr int E = 8;
    constexpr int kD = 256;
    constexpr int kDT = NT < kD ? kD / NT : 1;  // digits per thread in the scan
    __shared__ uint64_t buf[NT * E];
    __shared__ uint32_t cnt[NW][kD];
    __shared__ uint32_t s_w[NW < 4 ? 1 : 4];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid >> 6;
    const int32_t row = list[blockIdx.x];
    const int64_t b = xadj[row];
    const int32_t len = static_cast<int32_t>(xadj[row + 1] - b);
    const int32_t rounds = (len + NT - 1) / NT;
    const int32_t first = w * rounds * 64 + lane;  // element r of this thread: first + 64 r
    uint64_t e[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int32_t i = first + 64 * r;
        e[r] = r < rounds && i < len ? (static_cast<uint64_t>(static_cast<uint32_t>(adj[b + i])) << 32) |
                                           static_cast<uint32_t>(ew[b + i])
                                     : 0;
    }
    const uint64_t lt = lanemask_lt();
    for (int shift = 0; shift < bits; shift += 8) {
#pragma unroll
        for (int q = 0; q < kD * NW / NT; ++q) cnt[w][lane + 64 * q] = 0;
        __syncthreads();
        uint32_t rank[E];
#pragma unroll
        for (int r = 0; r < E; ++r) {
            rank[r] = 0;
            if (r >= rounds) continue;  // uniform over the workgroup
            const bool valid = first + 64 * r < len;
            const uint32_t d = static_cast<uint32_t>(e[r] >> (32 + shift)) & (kD - 1);
            uint64_t match = __ballot(valid);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint64_t bal = __ballot((d >> q) & 1u);
                match &= ((d >> q) & 1u) ? bal : ~bal;
            }
            if (valid) rank[r] = cnt[w][d] + static_cast<uint32_t>(__popcll(match & lt));
            wave_sync();
            if (valid && (match & lt) == 0) cnt[w][d] += static_cast<uint32_t>(__popcll(match));
            wave_sync();
        }
        __syncthreads();
        // counts to first positions: thread t owns digits kDT * t ..
        uint32_t c[kDT][NW], tot[kDT], mine = 0;
        if (tid < kD / kDT) {
#pragma unroll
            for (int q = 0; q < kDT; ++q) {
                tot[q] = 0;
#pragma unroll
                for (int x = 0; x < NW; ++x) {
                    c[q][x] = cnt[x][kDT * tid + q];
                    tot[q] += c[q][x];
                }
                mine += tot[q];
            }
        }
        uint32_t incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        uint32_t run = incl - mine;
        if (NW >= 4) {
            if (lane == 63 && w < 4) s_w[w] = incl;
            __syncthreads();
            for (int x = 0; x < w && x < 4; ++x) run += s_w[x];
        }
        if (tid < kD / kDT) {
#pragma unroll
            for (int q = 0; q < kDT; ++q)
#pragma unroll
                for (int x = 0; x < NW; ++x) {
                    cnt[x][kDT * tid + q] = run;
                    run += c[q][x];
                }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; ++r) {
            if (r >= rounds || first + 64 * r >= len) continue;
            const uint32_t d = static_cast<uint32_t>(e[r] >> (32 + shift)) & (kD - 1);
            buf[cnt[w][d] + rank[r]] = e[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; ++r)
            if (r < rounds && first + 64 * r < len) e[r] = buf[first + 64 * r];
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int32_t i = first + 64 * r;
        if (r >= rounds || i >= len) continue;
        adj[b + i] = static_cast<int32_t>(e[r] >> 32);
        ew[b + i] = static_cast<int32_t>(e[r] & 0xFFFFFFFFULL);
    }
}

constexpr int kOrderMax = 8192;  // rows up to this length are ordered in LDS

// Rows to order, by length: one wave, up to 512, 2048 or 8192 entries, longer.
constexpr int kOrderClasses = 5;

__global__ void __launch_bounds__(256) order_classify_kernel(int32_t n, const int64_t* __restrict__ xadj,
                                                             int32_t* __restrict__ lists,
                                                             uint32_t* __restrict__ counts) {
    for (int32_t base = blockIdx.x * (kClassifyIters * 256); base < n; base += gridDim.x * (kClassifyIters * 256)) {
        uint32_t m[kOrderClasses] = {};
#pragma unroll
        for (int it = 0; it < kClassifyIters; ++it) {
            const int32_t r = base + it * 256 + static_cast<int32_t>(threadIdx.x);
            const int64_t len = r < n ? xadj[r + 1] - xadj[r] : 0;
            if (len > 1) {
                const int c = len <= 64 ? 0 : (len <= 512 ? 1 : (len <= 2048 ? 2 : (len <= kOrderMax ? 3 : 4)));
#pragma unroll
                for (int q = 0; q < kOrderClasses; ++q) m[q] |= q == c ? 1u << it : 0u;
            }
        }
#pragma unroll
        for (int c = 0; c < kOrderClasses; ++c) {
            uint32_t bits = m[c];
            if (!__syncthreads_or(bits != 0)) continue;
            uint32_t j = block_append_count(static_cast<uint32_t>(__popc(bits)), &counts[c]);
            while (bits) {
                const int it = __ffs(bits) - 1;
                bits &= bits - 1;
                lists[static_cast<int64_t>(c) * n + j++] = base + it * 256 + static_cast<int32_t>(threadIdx.x);
            }
        }
    }
}

// Rows of 2..64 distinct entries: one wave per row, bitonic network over the
// lanes.
__global__ void __launch_bounds__(256) order_wave_rows_kernel(const int32_t* __restrict__ list, uint32_t count,
                                                              const int64_t* __restrict__ xadj,
                                                              int32_t* __restrict__ adj, int32_t* __restrict__ ew) {
    const uint32_t wv = (blockIdx.x * 256 + threadIdx.x) >> 6;
    if (wv >= count) return;  // uniform per wave
    const int lane = lane_id();
    const int32_t row = list[wv];
    const int64_t b = xadj[row];
    const int32_t len = static_cast<int32_t>(xadj[row + 1] - b);
    uint32_t key = lane < len ? static_cast<uint32_t>(adj[b + lane]) : 0xFFFFFFFFu;
    int32_t w = lane < len ? ew[b + lane] : 0;
    bitonic_wave(key, w, lane);
    if (lane < len) {
        adj[b + lane] = static_cast<int32_t>(key);
        ew[b + lane] = w;
    }
}

// Longer rows: (row's place in the list << bn | id, w) over just those rows ...
__global__ void __launch_bounds__(256) long_keys_kernel(const int32_t* __restrict__ list, uint32_t l0,
                                                        const int64_t* __restrict__ loff,
                                                        const int64_t* __restrict__ xadj,
                                                        const int32_t* __restrict__ adj, const int32_t* __restrict__ ew,
                                                        int bn, uint64_t* __restrict__ keys,
                                                        uint32_t* __restrict__ vals) {
    const int32_t l = static_cast<int32_t>(l0 + blockIdx.y);
    const int64_t src = xadj[list[l]], dst = loff[l], len = loff[l + 1] - dst;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; j < len;
         j += static_cast<int64_t>(gridDim.x) * 256) {
        keys[dst + j] = (static_cast<uint64_t>(l) << bn) | static_cast<uint32_t>(adj[src + j]);
        vals[dst + j] = static_cast<uint32_t>(ew[src + j]);
    }
}

// ... and back in order.
__global__ void __launch_bounds__(256) long_write_kernel(const int32_t* __restrict__ list, uint32_t l0,
                                                         const int64_t* __restrict__ loff,
                                                         const int64_t* __restrict__ xadj,
                                                         const uint64_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ vals, int bn,
                                                         int32_t* __restrict__ adj, int32_t* __restrict__ ew) {
    const int32_t l = static_cast<int32_t>(l0 + blockIdx.y);
    const int64_t dst = xadj[list[l]], src = loff[l], len = loff[l + 1] - src;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; j < len;
         j += static_cast<int64_t>(gridDim.x) * 256) {
        adj[dst + j] = static_cast<int32_t>(keys[src + j] & ((1ULL << bn) - 1));
        ew[dst + j] = static_cast<int32_t>(vals[src + j]);
    }
}

__global__ void long_degrees_kernel(const int32_t* __restrict__ list, uint32_t nl, const int64_t* __restrict__ xadj,
                                    int32_t* __restrict__ lens) {
    const uint32_t l = blockIdx.x * 256 + threadIdx.x;
    if (l < nl) lens[l] = static_cast<int32_t>(xadj[list[l] + 1] - xadj[list[l]]);
}

// Rows longer than 4096 entries: chunks of each.
__global__ void long_lens_kernel(const int32_t* __restrict__ list, uint32_t nl, const int32_t* __restrict__ rowcnt,
                                 int32_t* __restrict__ nchunks, int32_t chunk) {
    const uint32_t l = blockIdx.x * 256 + threadIdx.x;
    if (l < nl) nchunks[l] = (rowcnt[list[l]] + chunk - 1) / chunk;
}

constexpr int kLongChunk = 8192;  // entries merged in LDS per workgroup before the sort
constexpr int kDedupThreads = 1024;

// Long-row chunks: chunk c of all long rows belongs to row list[crow[c]] and
// is that row's chunk number c - cfirst[crow[c]].
__global__ void long_chunks_kernel(uint32_t nl, const int64_t* __restrict__ cfirst, int32_t* __restrict__ crow) {
    const uint32_t l = blockIdx.x;
    if (l >= nl) return;
    for (int64_t c = cfirst[l] + threadIdx.x; c < cfirst[l + 1]; c += 256) crow[c] = static_cast<int32_t>(l);
}

// Merges equal neighbours inside one chunk in an LDS table and writes the
// chunk's distinct (C(v), summed w) back to the chunk's start.  Sums fit 32
// bits: a partial sum never exceeds the coarse edge's weight, and the edge
// weight total is checked to fit 31 bits.  Long rows of contracted hubs
// repeat their neighbours many times, so large chunks shrink what the
// bucket passes after this one move.
__global__ void __launch_bounds__(kDedupThreads) long_dedup_kernel(const int32_t* __restrict__ list,
                                                                   const int32_t* __restrict__ crow,
                                                                   const int64_t* __restrict__ cfirst,
                                                                   const int64_t* __restrict__ rowoff,
                                                                   const int32_t* __restrict__ rowcnt,
                                                                   int32_t* __restrict__ tk, int32_t* __restrict__ tw,
                                                                   bool unit, int32_t* __restrict__ ccnt) {
    constexpr int kT = 2 * kLongChunk;
    __shared__ __align__(16) int32_t keys[kT];
    __shared__ __align__(16) int32_t sums[kT];
    const int64_t c = blockIdx.x;
    const int32_t l = crow[c];
    const int32_t row = list[l];
    const int64_t j0 = (c - cfirst[l]) * kLongChunk;
    const int64_t len = rowcnt[row];
    const int32_t cnt = static_cast<int32_t>(j0 + kLongChunk < len ? kLongChunk : len - j0);
    const int32_t d = merge_in_lds<kDedupThreads, kT>(rowoff[row] + j0, cnt, tk, tw, unit, keys, sums);
    if (threadIdx.x == kDedupThreads - 1) ccnt[c] = d;
}

// loff[l] = coff[cfirst[l]]: first merged chunk entry of long row l
__global__ void long_offsets_kernel(uint32_t nl, const int64_t* __restrict__ cfirst, const int64_t* __restrict__ coff,
                                    int64_t* __restrict__ loff) {
    const uint32_t l = blockIdx.x * 256 + threadIdx.x;
    if (l <= nl) loff[l] = coff[cfirst[l]];
}

// Unsorted merge of rows of 65..4096 entries: one workgroup per row sums
// equal neighbours in an LDS table of kT >= 2 len slots and writes the
// distinct entries to the row's start, in the order of the slots that brought
// them into the table.  Rows are grouped by length so that short rows get small
// tables (less to clear, more workgroups per CU).
template <int kT>
__global__ void __launch_bounds__(256) block_hash_rows_kernel(const int32_t* __restrict__ list,
                                                              const int64_t* __restrict__ rowoff,
                                                              const int32_t* __restrict__ rowcnt,
                                                              int32_t* __restrict__ tk, int32_t* __restrict__ tw,
                                                              bool unit, int32_t* __restrict__ dcnt) {
    __shared__ __align__(16) int32_t keys[kT];
    __shared__ __align__(16) int32_t sums[kT];
    const int32_t row = list[blockIdx.x];
    const int32_t d = merge_in_lds<256, kT>(rowoff[row], rowcnt[row], tk, tw, unit, keys, sums);
    if (threadIdx.x == 255) dcnt[row] = d;
}

// Unsorted merge of long rows after the chunk merge, by buckets: the merged
// chunk entries of long row l are spread over P_l = ceil(m_l / kBucketMean)
// buckets by a hash of the neighbour id (so equal ids meet in one bucket),
// scattered bucket by bucket into a staging array, merged per bucket in an
// LDS table by one workgroup, and copied back into the row.  Every step
// streams the entries once; nothing probes a table in HBM.  A bucket whose
// distinct neighbours do not fit its LDS table raises a flag, and the caller
// then merges the long rows through per-row HBM tables instead.
constexpr int kBucketMean = 1024;   // merged entries per bucket on average (default)
constexpr int kBucketTable = 4096;  // LDS table slots of one bucket merge
constexpr int kBucketLds = 4096;    // rows with up to this many buckets count and reserve in LDS
constexpr int kBucketThreads = 1024;  // 8 entries of a chunk per thread, kept in registers between the passes

__device__ __forceinline__ uint32_t bucket_of(int32_t x, uint32_t P) {
    const uint32_t h = slot_hash(static_cast<uint32_t>(x) ^ 0x5BD1E995u);  // independent of the table slot
    return static_cast<uint32_t>((static_cast<uint64_t>(h) * P) >> 32);
}

__global__ void long_bucket_counts_kernel(uint32_t nl, const int64_t* __restrict__ loff, int32_t mean,
                                          const int32_t* __restrict__ list, const int64_t* __restrict__ cfirst,
                                          int32_t* __restrict__ dcnt, int32_t* __restrict__ nbk) {
    const uint32_t l = blockIdx.x * 256 + threadIdx.x;
    if (l >= nl) return;
    const int64_t m = loff[l + 1] - loff[l];
    if (cfirst[l + 1] - cfirst[l] == 1) {  // one chunk: its merge is the row's
        nbk[l] = 0;
        dcnt[list[l]] = static_cast<int32_t>(m);
        return;
    }
    // at most kBucketLds buckets: a row's buckets then count and reserve in
    // LDS; a bucket whose distinct neighbours overflow its table sends the
    // long rows to the HBM-table merge
    const int64_t q = m > mean ? (m + mean - 1) / mean : 1;
    nbk[l] = static_cast<int32_t>(q < kBucketLds ? q : kBucketLds);
}

// bucket q belongs to long row brow[q]
__global__ void long_bucket_rows_kernel(uint32_t nl, const int64_t* __restrict__ bfirst, int32_t* __restrict__ brow) {
    const uint32_t l = blockIdx.x;
    if (l >= nl) return;
    for (int64_t q = bfirst[l] + threadIdx.x; q < bfirst[l + 1]; q += 256) brow[q] = static_cast<int32_t>(l);
}

// Pass 1 (reserve = false): bucket sizes.  Pass 2 (reserve = true): every
// entry to its bucket's range of the staging arrays; each workgroup reserves
// its part of a bucket with one atomic per bucket it touches.  An entry is read
// once and keeps its rank in the bucket from the count to the write, and is
// staged as one 8-byte word, since the writes land on scattered lines (the
// three contractions of a 2^24-node partition: 6.3 -> 1.8 ms in pass 2).
template <bool kReserve>
__global__ void __launch_bounds__(kBucketThreads) long_bucket_scatter_kernel(
    const int32_t* __restrict__ list, const int32_t* __restrict__ crow, const int64_t* __restrict__ cfirst,
    const int32_t* __restrict__ ccnt, const int64_t* __restrict__ rowoff, const int64_t* __restrict__ bfirst,
    const int32_t* __restrict__ tk, const int32_t* __restrict__ tw, int32_t* __restrict__ bcount,
    const int64_t* __restrict__ boff, int32_t* __restrict__ bfill, int2* __restrict__ staged) {
    __shared__ int32_t lcnt[kBucketLds];
    __shared__ int32_t lbase[kReserve ? kBucketLds : 1];
    constexpr int U = kLongChunk / kBucketThreads;
    const int tid = threadIdx.x;
    const int64_t c = blockIdx.x;
    const int32_t l = crow[c];
    const int64_t src = rowoff[list[l]] + (c - cfirst[l]) * kLongChunk;
    const int32_t cnt = ccnt[c];
    const int64_t b0 = bfirst[l];
    const uint32_t P = static_cast<uint32_t>(bfirst[l + 1] - b0);
    if (P == 0) return;  // a one-chunk row, merged already
    int32_t x[U], w[U], rank[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t j = tid + u * kBucketThreads;
        x[u] = j < cnt ? tk[src + j] : -1;
        if (kReserve) w[u] = j < cnt ? tw[src + j] : 0;
    }
    for (uint32_t j = tid; j < P; j += kBucketThreads) lcnt[j] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) rank[u] = x[u] >= 0 ? atomicAdd(&lcnt[bucket_of(x[u], P)], 1) : 0;
    __syncthreads();
    for (uint32_t j = tid; j < P; j += kBucketThreads) {
        const int32_t k = lcnt[j];
        if (k == 0) continue;
        if (kReserve) lbase[j] = atomicAdd(&bfill[b0 + j], k);
        else atomicAdd(&bcount[b0 + j], k);
    }
    if (!kReserve) return;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (x[u] < 0) continue;
        const uint32_t q = bucket_of(x[u], P);
        staged[boff[b0 + q] + lbase[q] + rank[u]] = make_int2(x[u], w[u]);
    }
}

// One workgroup per bucket: equal neighbours summed in an LDS table, the
// distinct entries written back to the bucket's start, their number to qcnt.
__global__ void __launch_bounds__(256) long_bucket_merge_kernel(const int64_t* __restrict__ boff,
                                                                int2* __restrict__ staged, int32_t* __restrict__ qcnt,
                                                                uint32_t* __restrict__ overflow) {
    __shared__ int32_t keys[kBucketTable];
    __shared__ int32_t sums[kBucketTable];
    __shared__ int32_t s_w[4];
    __shared__ int32_t s_full;
    const int tid = threadIdx.x;
    const int64_t q = blockIdx.x;
    const int64_t b = boff[q];
    const int32_t len = static_cast<int32_t>(boff[q + 1] - b);
    for (int j = tid; j < kBucketTable; j += 256) {
        keys[j] = -1;
        sums[j] = 0;
    }
    if (tid == 0) s_full = 0;
    __syncthreads();
    constexpr int U = 4;
    bool full = false;
    for (int j0 = tid; j0 < len && !full; j0 += 256 * U) {
        int2 e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) e[u] = j0 + u * 256 < len ? staged[b + j0 + u * 256] : make_int2(-1, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (e[u].x < 0 || full) continue;
            uint32_t h = slot_hash(static_cast<uint32_t>(e[u].x)) & (kBucketTable - 1);
            int probes = 0;
            while (true) {
                const int32_t prev = atomicCAS(&keys[h], -1, e[u].x);
                if (prev == -1 || prev == e[u].x) break;
                h = (h + 1) & (kBucketTable - 1);
                if (++probes == kBucketTable) break;  // table full
            }
            full = probes == kBucketTable;
            if (!full) atomicAdd(&sums[h], e[u].y);  // partial sums never exceed the final coarse weight
        }
    }
    if (full) s_full = 1;
    __syncthreads();
    if (s_full) {
        if (tid == 0) atomicOr(overflow, 1u);
        return;
    }
    // exclusive prefix of the occupied slots, kPer consecutive slots per thread
    constexpr int kPer = kBucketTable / 256;
    int32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) mine += keys[tid * kPer + j] >= 0;
    int32_t incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t t = __shfl_up(incl, o, 64);
        if (lane_id() >= o) incl += t;
    }
    if (lane_id() == kWave - 1) s_w[tid / kWave] = incl;
    __syncthreads();
    int32_t pos = incl - mine;
    for (int w = 0; w < tid / kWave; ++w) pos += s_w[w];
    if (tid == 255) qcnt[q] = pos + mine;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int e = tid * kPer + j;
        if (keys[e] < 0) continue;
        staged[b + pos] = make_int2(keys[e], sums[e]);
        ++pos;
    }
}

__global__ void __launch_bounds__(256) long_bucket_write_kernel(const int32_t* __restrict__ list,
                                                                const int32_t* __restrict__ brow,
                                                                const int64_t* __restrict__ bfirst,
                                                                const int64_t* __restrict__ boff,
                                                                const int64_t* __restrict__ qoff,
                                                                const int32_t* __restrict__ qcnt,
                                                                const int64_t* __restrict__ rowoff,
                                                                const int2* __restrict__ staged,
                                                                int32_t* __restrict__ tk, int32_t* __restrict__ tw,
                                                                int32_t* __restrict__ dcnt) {
    const int64_t q = blockIdx.x;
    const int32_t l = brow[q];
    const int32_t row = list[l];
    const int64_t q0 = bfirst[l];
    const int64_t dst = rowoff[row] + (qoff[q] - qoff[q0]);
    const int64_t src = boff[q];
    const int32_t cnt = qcnt[q];
    for (int32_t j = threadIdx.x; j < cnt; j += 256) {
        const int2 e = staged[src + j];
        tk[dst + j] = e.x;
        tw[dst + j] = e.y;
    }
    if (q == q0 && threadIdx.x == 0) dcnt[row] = static_cast<int32_t>(qoff[bfirst[l + 1]] - qoff[q0]);
}

// Unsorted merge of long rows after the chunk merge: one open-addressing
// table in HBM per row (at least twice its merged entries, a power of two),
// filled with atomics, then compacted chunk by chunk.
constexpr int kTabChunk = 4096;

__global__ void long_table_sizes_kernel(uint32_t nl, const int64_t* __restrict__ loff, int64_t* __restrict__ tsz,
                                        int64_t* __restrict__ tch) {
    const uint32_t l = blockIdx.x * 256 + threadIdx.x;
    if (l >= nl) return;
    const int64_t want = 2 * (loff[l + 1] - loff[l]);
    int64_t t = kTabChunk;
    while (t < want) t <<= 1;
    tsz[l] = t;
    tch[l] = t / kTabChunk;
}

__global__ void __launch_bounds__(256) long_table_insert_kernel(const int32_t* __restrict__ list,
                                                                const int32_t* __restrict__ crow,
                                                                const int64_t* __restrict__ cfirst,
                                                                const int32_t* __restrict__ ccnt,
                                                                const int64_t* __restrict__ rowoff,
                                                                const int32_t* __restrict__ tk,
                                                                const int32_t* __restrict__ tw,
                                                                const int64_t* __restrict__ toff,
                                                                const int64_t* __restrict__ tsz,
                                                                int32_t* __restrict__ gk, int32_t* __restrict__ gv) {
    const int64_t c = blockIdx.x;  // one merged chunk per workgroup
    const int32_t l = crow[c];
    const int64_t src = rowoff[list[l]] + (c - cfirst[l]) * kLongChunk;
    int32_t* keys = gk + toff[l];
    int32_t* vals = gv + toff[l];
    const uint64_t mask = static_cast<uint64_t>(tsz[l]) - 1;
    for (int32_t j = threadIdx.x; j < ccnt[c]; j += 256) {
        const int32_t x = tk[src + j];
        uint64_t h = slot_hash(static_cast<uint32_t>(x)) & mask;
        while (true) {
            const int32_t prev = atomicCAS(&keys[h], -1, x);
            if (prev == -1 || prev == x) break;
            h = (h + 1) & mask;
        }
        atomicAdd(&vals[h], tw[src + j]);
    }
}

// table chunk q belongs to row tl[q]
__global__ void long_table_chunks_kernel(uint32_t nl, const int64_t* __restrict__ tcfirst, int32_t* __restrict__ tl) {
    const uint32_t l = blockIdx.x;
    if (l >= nl) return;
    for (int64_t q = tcfirst[l] + threadIdx.x; q < tcfirst[l + 1]; q += 256) tl[q] = static_cast<int32_t>(l);
}

__global__ void __launch_bounds__(256) long_table_count_kernel(const int32_t* __restrict__ tl,
                                                               const int64_t* __restrict__ tcfirst,
                                                               const int64_t* __restrict__ toff,
                                                               const int32_t* __restrict__ gk,
                                                               int32_t* __restrict__ qcnt) {
    const int64_t q = blockIdx.x;
    const int32_t l = tl[q];
    const int64_t base = toff[l] + (q - tcfirst[l]) * kTabChunk;
    int32_t c = 0;
    for (int j = threadIdx.x; j < kTabChunk; j += 256) c += gk[base + j] >= 0;
    c = block_sum_i32_256(c);
    if (threadIdx.x == 0) qcnt[q] = c;
}

__global__ void __launch_bounds__(256) long_table_write_kernel(const int32_t* __restrict__ list,
                                                               const int32_t* __restrict__ tl,
                                                               const int64_t* __restrict__ tcfirst,
                                                               const int64_t* __restrict__ toff,
                                                               const int64_t* __restrict__ qoff,
                                                               const int64_t* __restrict__ rowoff,
                                                               const int32_t* __restrict__ gk,
                                                               const int32_t* __restrict__ gv,
                                                               int32_t* __restrict__ tk, int32_t* __restrict__ tw,
                                                               int32_t* __restrict__ dcnt) {
    __shared__ int32_t s_cnt[256];
    const int64_t q = blockIdx.x;
    const int32_t l = tl[q];
    const int32_t row = list[l];
    const int64_t base = toff[l] + (q - tcfirst[l]) * kTabChunk;
    constexpr int kPer = kTabChunk / 256;
    const int tid = threadIdx.x;
    int32_t mine = 0;
    for (int j = 0; j < kPer; ++j) mine += gk[base + tid * kPer + j] >= 0;
    s_cnt[tid] = mine;
    __syncthreads();
    if (tid == 0) {
        int32_t run = 0;
        for (int t = 0; t < 256; ++t) {
            const int32_t x = s_cnt[t];
            s_cnt[t] = run;
            run += x;
        }
    }
    __syncthreads();
    int64_t pos = rowoff[row] + (qoff[q] - qoff[tcfirst[l]]) + s_cnt[tid];
    for (int j = 0; j < kPer; ++j) {
        const int64_t e = base + tid * kPer + j;
        if (gk[e] < 0) continue;
        tk[pos] = gk[e];
        tw[pos] = gv[e];
        ++pos;
    }
    if (q == tcfirst[l] && tid == 0) dcnt[row] = static_cast<int32_t>(qoff[tcfirst[l + 1]] - qoff[tcfirst[l]]);
}

// Step 4: the merged prefix of every row to its place in the coarse CSR.
__global__ void __launch_bounds__(kTileThreads) row_copy_kernel(const int64_t* __restrict__ rowoff, int32_t nc, int64_t m,
                                                                const int32_t* __restrict__ dcnt,
                                                                const int64_t* __restrict__ cxadj,
                                                                const int32_t* __restrict__ tk,
                                                                const int32_t* __restrict__ tw,
                                                                int32_t* __restrict__ cadj, int32_t* __restrict__ cew, const int32_t* __restrict__ trow) {
    __shared__ int32_t owner[kTile];
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int64_t i1 = i0 + kTile < m ? i0 + kTile : m;
    tile_owners(rowoff, trow, static_cast<int64_t>(blockIdx.x), i0, i1, owner);
    int64_t li[kTilePer], to[kTilePer];
    int32_t cnt[kTilePer];
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        const int64_t i = i0 + r * kTileThreads + threadIdx.x;
        const int32_t row = i < i1 ? owner[i - i0] : -1;
        li[r] = row >= 0 ? i - rowoff[row] : 0;
        cnt[r] = row >= 0 ? dcnt[row] : 0;
        to[r] = row >= 0 ? cxadj[row] : 0;
    }
    int32_t k[kTilePer], w[kTilePer];
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        const int64_t i = i0 + r * kTileThreads + threadIdx.x;
        k[r] = li[r] < cnt[r] ? tk[i] : 0;
        w[r] = li[r] < cnt[r] ? tw[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < kTilePer; ++r) {
        if (li[r] >= cnt[r]) continue;
        cadj[to[r] + li[r]] = k[r];
        cew[to[r] + li[r]] = w[r];
    }
}

// Long rows (unsorted) merged by buckets; false if a bucket's distinct
// neighbours overflowed its LDS table (tk/tw untouched then).
bool bucket_merge_long_rows(uint32_t nl, const int32_t* llist, int64_t nch, const int32_t* crow,
                            const int64_t* cfirst, const int32_t* ccnt, const int64_t* loff, int64_t ml,
                            const int64_t* rowoff, int32_t* tk, int32_t* tw, int32_t* dcnt, int32_t mean,
                            hipStream_t s) {
    ProfScope ps("contract_long_buckets", 40.0 * static_cast<double>(ml), s);
    DBuf<int32_t> nbk(nl, s);
    DBuf<int64_t> bfirst(static_cast<size_t>(nl) + 1, s);
    long_bucket_counts_kernel<<<grid_for(nl, 256), 256, 0, s>>>(nl, loff, mean, llist, cfirst, dcnt, nbk.get());
    LAUNCHCHK();
    exclusive_scan_i32_to_i64(nbk.get(), bfirst.get(), nl, bfirst.get() + nl, s);
    int64_t NB = 0;
    read_back(&NB, bfirst.get() + nl, sizeof(int64_t), s);
    if (NB == 0) return true;  // every long row was one chunk
    DBuf<int32_t> brow(NB, s), zeros(2 * NB + 1, s), qcnt(NB, s);  // bucket sizes, entries placed, overflow flag
    int32_t* const bcount = zeros.get();
    int32_t* const bfill = bcount + NB;
    uint32_t* const overflow = reinterpret_cast<uint32_t*>(bfill + NB);
    DBuf<int64_t> boff(static_cast<size_t>(NB) + 1, s), qoff(static_cast<size_t>(NB) + 1, s);
    DBuf<int2> staged(std::max<int64_t>(ml, 1), s);
    long_bucket_rows_kernel<<<nl, 256, 0, s>>>(nl, bfirst.get(), brow.get());
    LAUNCHCHK();
    fill_i32(zeros.get(), 0, 2 * NB + 1, s);
    long_bucket_scatter_kernel<false><<<static_cast<unsigned>(nch), kBucketThreads, 0, s>>>(
        llist, crow, cfirst, ccnt, rowoff, bfirst.get(), tk, tw, bcount, nullptr, nullptr, nullptr);
    LAUNCHCHK();
    exclusive_scan_i32_to_i64(bcount, boff.get(), NB, boff.get() + NB, s);
    long_bucket_scatter_kernel<true><<<static_cast<unsigned>(nch), kBucketThreads, 0, s>>>(
        llist, crow, cfirst, ccnt, rowoff, bfirst.get(), tk, tw, nullptr, boff.get(), bfill, staged.get());
    LAUNCHCHK();
    long_bucket_merge_kernel<<<static_cast<unsigned>(NB), 256, 0, s>>>(boff.get(), staged.get(), qcnt.get(), overflow);
    LAUNCHCHK();
    uint32_t over = 0;
    read_back(&over, overflow, sizeof(uint32_t), s);
    if (over) return false;
    exclusive_scan_i32_to_i64(qcnt.get(), qoff.get(), NB, qoff.get() + NB, s);
    long_bucket_write_kernel<<<static_cast<unsigned>(NB), 256, 0, s>>>(llist, brow.get(), bfirst.get(), boff.get(),
                                                                      qoff.get(), qcnt.get(), rowoff, staged.get(),
                                                                      tk, tw, dcnt);
    LAUNCHCHK();
    return true;
}

}  // namespace

// Merges every row r of the entries tk/tw[rowoff[r] .. rowoff[r] + rowcnt[r])
// in place (unit: every weight is 1, and tw is written but not read); dcnt[r]
// receives the number of distinct neighbours, written at the row's start in no
// particular order.
static void merge_rows(int32_t nc, int64_t m, const int64_t* rowoff, const int32_t* rowcnt, int32_t* tk, int32_t* tw,
                       bool unit, int32_t* dcnt, hipStream_t s, int32_t bucket_mean = 0) {
    DBuf<int32_t> lists(kRowClasses * static_cast<size_t>(nc), s);
    DBuf<uint32_t> counts(kRowClasses, s);
    uint32_t hc[kRowClasses] = {};
    auto list_of = [&](int c) { return lists.get() + static_cast<size_t>(c) * nc; };
    {
        ProfScope ps("contract_rows", 16.0 * static_cast<double>(m), s);
        fill_u32(counts.get(), 0, kRowClasses, s);
        row_classify_kernel<<<std::min(grid_for(nc, 256 * kClassifyIters), 1024u), 256, 0, s>>>(
            nc, rowoff, rowcnt, dcnt, tw, unit, lists.get(), nc, counts.get());
        LAUNCHCHK();
        read_back(hc, counts.get(), sizeof(hc), s);
        if (hc[5]) block_hash_rows_kernel<8192><<<hc[5], 256, 0, s>>>(list_of(5), rowoff, rowcnt, tk, tw, unit, dcnt);
        if (hc[4]) block_hash_rows_kernel<4096><<<hc[4], 256, 0, s>>>(list_of(4), rowoff, rowcnt, tk, tw, unit, dcnt);
        if (hc[3]) block_hash_rows_kernel<2048><<<hc[3], 256, 0, s>>>(list_of(3), rowoff, rowcnt, tk, tw, unit, dcnt);
        if (hc[2]) block_hash_rows_kernel<1024><<<hc[2], 256, 0, s>>>(list_of(2), rowoff, rowcnt, tk, tw, unit, dcnt);
        if (hc[1]) block_hash_rows_kernel<512><<<hc[1], 256, 0, s>>>(list_of(1), rowoff, rowcnt, tk, tw, unit, dcnt);
        if (hc[0])
            wave_rows_kernel<<<grid_for(static_cast<int64_t>(hc[0]) * 64, 256), 256, 0, s>>>(list_of(0), hc[0], rowoff,
                                                                                            rowcnt, tk, tw, unit, dcnt);
        LAUNCHCHK();
    }
    if (hc[kRowClasses - 1] > 0) {
        ProfScope ps("contract_long_rows", 0, s);
        const uint32_t nl = hc[kRowClasses - 1];
        const int32_t* llist = list_of(kRowClasses - 1);
        // chunks of the long rows, each merged in LDS first
        DBuf<int32_t> lens(nl, s);
        DBuf<int64_t> cfirst(static_cast<size_t>(nl) + 1, s);
        long_lens_kernel<<<grid_for(nl, 256), 256, 0, s>>>(llist, nl, rowcnt, lens.get(), kLongChunk);
        LAUNCHCHK();
        exclusive_scan_i32_to_i64(lens.get(), cfirst.get(), nl, cfirst.get() + nl, s);
        int64_t nch = 0;
        read_back(&nch, cfirst.get() + nl, sizeof(int64_t), s);
        DBuf<int32_t> crow(nch, s), ccnt(nch, s);
        DBuf<int64_t> coff(static_cast<size_t>(nch) + 1, s), loff(static_cast<size_t>(nl) + 1, s);
        {
            ProfScope ps_m("contract_long_merge", 0, s);
            long_chunks_kernel<<<nl, 256, 0, s>>>(nl, cfirst.get(), crow.get());
            LAUNCHCHK();
            long_dedup_kernel<<<static_cast<unsigned>(nch), kDedupThreads, 0, s>>>(llist, crow.get(), cfirst.get(),
                                                                                   rowoff, rowcnt, tk, tw, unit, ccnt.get());
            LAUNCHCHK();
        }
        exclusive_scan_i32_to_i64(ccnt.get(), coff.get(), nch, coff.get() + nch, s);
        int64_t ml = 0;
        read_back(&ml, coff.get() + nch, sizeof(int64_t), s);
        long_offsets_kernel<<<grid_for(static_cast<int64_t>(nl) + 1, 256), 256, 0, s>>>(nl, cfirst.get(), coff.get(),
                                                                                         loff.get());
        LAUNCHCHK();
        if (bucket_merge_long_rows(nl, llist, nch, crow.get(), cfirst.get(), ccnt.get(), loff.get(), ml,
                                              rowoff, tk, tw, dcnt, bucket_mean > 0 ? bucket_mean : kBucketMean, s))
            return;
        {  // a bucket overflowed: per-row tables in HBM
            DBuf<int64_t> tsz(nl, s), tch(nl, s), toff(static_cast<size_t>(nl) + 1, s),
                tcfirst(static_cast<size_t>(nl) + 1, s);
            long_table_sizes_kernel<<<grid_for(nl, 256), 256, 0, s>>>(nl, loff.get(), tsz.get(), tch.get());
            LAUNCHCHK();
            // offsets: [0, inclusive sums]
            fill_i64(toff.get(), 0, 1, s);
            fill_i64(tcfirst.get(), 0, 1, s);
            inclusive_scan_i64(tsz.get(), toff.get() + 1, nl, s);
            inclusive_scan_i64(tch.get(), tcfirst.get() + 1, nl, s);
            int64_t hts[2] = {0, 0};
            const ReadItem items[2] = {{&hts[0], toff.get() + nl, sizeof(int64_t)},
                                       {&hts[1], tcfirst.get() + nl, sizeof(int64_t)}};
            read_back(items, 2, s);
            const int64_t ttot = hts[0], nq = hts[1];
            DBuf<int32_t> gk(ttot, s), gv(ttot, s), tl(nq, s), qcnt(nq, s);
            DBuf<int64_t> qoff(static_cast<size_t>(nq) + 1, s), qt(1, s);
            fill_i32(gk.get(), -1, ttot, s);
            fill_i32(gv.get(), 0, ttot, s);
            {
                ProfScope ps_i("contract_long_insert", 0, s);
                long_table_insert_kernel<<<static_cast<unsigned>(nch), 256, 0, s>>>(
                    llist, crow.get(), cfirst.get(), ccnt.get(), rowoff, tk, tw, toff.get(), tsz.get(), gk.get(),
                    gv.get());
                LAUNCHCHK();
            }
            long_table_chunks_kernel<<<nl, 256, 0, s>>>(nl, tcfirst.get(), tl.get());
            LAUNCHCHK();
            long_table_count_kernel<<<static_cast<unsigned>(nq), 256, 0, s>>>(tl.get(), tcfirst.get(), toff.get(),
                                                                            gk.get(), qcnt.get());
            LAUNCHCHK();
            exclusive_scan_i32_to_i64(qcnt.get(), qoff.get(), nq, qt.get(), s);
            HIPCHK(hipMemcpyAsync(qoff.get() + nq, qt.get(), sizeof(int64_t), hipMemcpyDeviceToDevice, s));
            long_table_write_kernel<<<static_cast<unsigned>(nq), 256, 0, s>>>(llist, tl.get(), tcfirst.get(),
                                                                            toff.get(), qoff.get(), rowoff, gk.get(),
                                                                            gv.get(), tk, tw, dcnt);
            LAUNCHCHK();
        }
    }
}

// Orders every row of a CSR of distinct entries by neighbour id, in place.
static void order_rows(int32_t n, const int64_t* xadj, int32_t* adj, int32_t* ew, hipStream_t s) {
    if (n <= 0) return;
    const int bn = std::max(1, bits_for(static_cast<uint64_t>(n - 1)));
    DBuf<int32_t> lists(kOrderClasses * static_cast<size_t>(n), s);
    DBuf<uint32_t> counts(kOrderClasses, s);
    uint32_t hc[kOrderClasses] = {};
    auto list_of = [&](int c) { return lists.get() + static_cast<size_t>(c) * n; };
    fill_u32(counts.get(), 0, kOrderClasses, s);
    order_classify_kernel<<<std::min(grid_for(n, 256 * kClassifyIters), 1024u), 256, 0, s>>>(n, xadj, lists.get(),
                                                                                             counts.get());
    LAUNCHCHK();
    read_back(hc, counts.get(), sizeof(hc), s);
    if (hc[3]) order_rows_kernel<16><<<hc[3], 1024, 0, s>>>(list_of(3), xadj, adj, ew, bn);
    if (hc[2]) order_rows_kernel<4><<<hc[2], 256, 0, s>>>(list_of(2), xadj, adj, ew, bn);
    if (hc[1]) order_rows_kernel<1><<<hc[1], 64, 0, s>>>(list_of(1), xadj, adj, ew, bn);
    if (hc[0])
        order_wave_rows_kernel<<<grid_for(static_cast<int64_t>(hc[0]) * 64, 256), 256, 0, s>>>(list_of(0), hc[0], xadj,
                                                                                              adj, ew);
    LAUNCHCHK();
    const uint32_t nl = hc[4];
    if (nl == 0) return;
    ProfScope ps("contract_long_sort", 0, s);
    DBuf<int32_t> lens(nl, s);
    DBuf<int64_t> loff(static_cast<size_t>(nl) + 1, s);
    long_degrees_kernel<<<grid_for(nl, 256), 256, 0, s>>>(list_of(4), nl, xadj, lens.get());
    LAUNCHCHK();
    exclusive_scan_i32_to_i64(lens.get(), loff.get(), nl, loff.get() + nl, s);
    int64_t ml = 0;
    read_back(&ml, loff.get() + nl, sizeof(int64_t), s);
    DBuf<uint64_t> keys(ml, s), ktmp(ml, s);
    DBuf<uint32_t> vals(ml, s), vtmp(ml, s);
    // rows in groups that fit the grid's second dimension
    constexpr uint32_t kRows = 32768;
    for (uint32_t l0 = 0; l0 < nl; l0 += kRows) {
        const uint32_t cnt = std::min(kRows, nl - l0);
        long_keys_kernel<<<dim3(16, cnt), 256, 0, s>>>(list_of(4), l0, loff.get(), xadj, adj, ew, bn, keys.get(),
                                                       vals.get());
        LAUNCHCHK();
    }
    RadixScratch rs;
    radix_sort_pairs(keys.get(), vals.get(), ktmp.get(), vtmp.get(), ml, 0,
                     bn + std::max(1, bits_for(static_cast<uint64_t>(nl - 1))), rs, s);
    for (uint32_t l0 = 0; l0 < nl; l0 += kRows) {
        const uint32_t cnt = std::min(kRows, nl - l0);
        long_write_kernel<<<dim3(16, cnt), 256, 0, s>>>(list_of(4), l0, loff.get(), xadj, keys.get(), vals.get(), bn,
                                                        adj, ew);
        LAUNCHCHK();
    }
}

void contract(const DevGraph& g, const int32_t* labels, int32_t* C, OwnedDevGraph& coarse, hipStream_t s,
              const int32_t* probe, int32_t nprobe, int32_t* probe_out, bool sorted, int32_t bucket_mean) {
    const int32_t n = g.n;
    if (n == 0) {
        coarse.n = 0;
        coarse.S = 0;
        coarse.xadj.alloc(1, s);
        fill_i64(coarse.xadj.get(), 0, 1, s);
        if (nprobe > 0) fill_i32(probe_out, 0, nprobe, s);
        return;
    }
    // coarse ids: ranks of the used labels
    DBuf<int32_t> node_zeros(3 * static_cast<size_t>(n), s);  // ranks, inter-cluster slots, slots placed, per node
    int32_t* const q = node_zeros.get();
    int32_t* const cross = q + n;
    int32_t* const nfill = cross + n;
    DBuf<int32_t> total(1, s);
    fill_i32(q, 0, 3 * static_cast<int64_t>(n), s);
    mark_used_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, labels, q);
    LAUNCHCHK();
    exclusive_scan_i32(q, q, n, total.get(), s);
    if (nprobe > 0) {
        probe_kernel<<<grid_for(nprobe, 256), 256, 0, s>>>(probe, nprobe, q, n, total.get(), probe_out);
        LAUNCHCHK();
    }
    int32_t nc = 0;
    read_back(&nc, total.get(), sizeof(int32_t), s);
    coarse.n = nc;
    coarse.vw.alloc(nc, s);
    DBuf<int32_t> row_zeros(2 * static_cast<size_t>(nc), s);  // entries and entries placed, per coarse row
    int32_t* const rowcnt = row_zeros.get();
    int32_t* const fill = rowcnt + nc;
    fill_i32(coarse.vw.get(), 0, nc, s);
    fill_i32(rowcnt, 0, 2 * static_cast<int64_t>(nc), s);
    map_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, labels, q, g.vw, C, coarse.vw.get());
    LAUNCHCHK();
    coarse.xadj.alloc(static_cast<size_t>(nc) + 1, s);
    const int64_t ntiles = (g.S + kTile - 1) / kTile;

    // 1 + 2: inter-cluster slots bucketed by coarse source row
    DBuf<int64_t> rowoff(static_cast<size_t>(nc) + 1, s);
    int64_t m = 0;
    DBuf<int32_t> cvs(g.S > 0 ? g.S : 1, s);  // C(v) of every slot
    TileRows gtiles(g.xadj, n, g.S, s);
    if (g.S > 0) {
        ProfScope ps("contract_count", (8.0 + 8.0) * static_cast<double>(g.S) + 8.0 * n, s);
        cross_count_kernel<<<static_cast<unsigned>(ntiles), kTileThreads, 0, s>>>(g.xadj, g.adj, n, g.S, C,
                                                                                   cross, cvs.get(),
                                                                                   gtiles.trow.get());
        LAUNCHCHK();
        row_count_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, C, cross, rowcnt);
        LAUNCHCHK();
    }
    exclusive_scan_i32_to_i64(rowcnt, rowoff.get(), nc, rowoff.get() + nc, s);
    read_back(&m, rowoff.get() + nc, sizeof(int64_t), s);
    if (m == 0) {
        coarse.S = 0;
        coarse.adj.alloc(1, s);
        coarse.ew.alloc(1, s);
        fill_i64(coarse.xadj.get(), 0, static_cast<int64_t>(nc) + 1, s);
        HIPCHK(hipStreamSynchronize(s));
        return;
    }
    DBuf<int32_t> tk(m, s), tw(m, s);
    {
        ProfScope ps("contract_emit", (4.0 + (g.ew ? 4.0 : 0.0)) * static_cast<double>(g.S) + 8.0 * n + 8.0 * m, s);
        DBuf<int64_t> nbase(n, s);
        node_base_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, C, cross, rowoff.get(), fill, nbase.get());
        LAUNCHCHK();
        row_scatter_kernel<<<static_cast<unsigned>(ntiles), kTileThreads, 0, s>>>(
            g.xadj, cvs.get(), g.ew, g.S, nbase.get(), nfill, tk.get(), tw.get(), gtiles.trow.get());
        LAUNCHCHK();
    }
    cvs.release();

    // 3: merge every row
    DBuf<int32_t> dcnt(nc, s);
    merge_rows(nc, m, rowoff.get(), rowcnt, tk.get(), tw.get(), !g.ew, dcnt.get(), s, bucket_mean);

    // 4: coarse offsets and the merged rows
    ProfScope ps_copy("contract_copy", 16.0 * static_cast<double>(m), s);
    exclusive_scan_i32_to_i64(dcnt.get(), coarse.xadj.get(), nc, coarse.xadj.get() + nc, s);
    int64_t Sc = 0;
    read_back(&Sc, coarse.xadj.get() + nc, sizeof(int64_t), s);
    coarse.S = Sc;
    coarse.adj.alloc(std::max<int64_t>(Sc, 1), s);
    coarse.ew.alloc(std::max<int64_t>(Sc, 1), s);
    const int64_t mtiles = (m + kTile - 1) / kTile;
    TileRows ctiles(rowoff.get(), nc, m, s);
    row_copy_kernel<<<static_cast<unsigned>(mtiles), kTileThreads, 0, s>>>(rowoff.get(), nc, m, dcnt.get(),
                                                                           coarse.xadj.get(), tk.get(), tw.get(),
                                                                           coarse.adj.get(), coarse.ew.get(),
                                                                           ctiles.trow.get());
    LAUNCHCHK();
    // 5: and, for the canonical form, every row in order (of its distinct
    // entries, which are a third to a half of those merged above)
    if (sorted) order_rows(nc, coarse.xadj.get(), coarse.adj.get(), coarse.ew.get(), s);
    HIPCHK(hipStreamSynchronize(s));
}

void sort_rows(OwnedDevGraph& g, hipStream_t s) {
    if (g.n == 0 || g.S == 0) return;
    ProfScope ps("contract_sort_rows", 16.0 * static_cast<double>(g.S), s);
    order_rows(g.n, g.xadj.get(), g.adj.get(), g.ew.get(), s);
    HIPCHK(hipStreamSynchronize(s));
}

}  // namespace sclap
