// Size-constrained label propagation (SCLaP) kernels for gfx950.
//
// Follows Section 3.1 (Label Propagation with Size Constraints) of
// Meyerhenke, Sanders, Schulz (2014): a visited node moves to the eligible
// neighbouring label (cluster or block) of strongest connection, eligible
// meaning the label stays within the bound after the move; during refinement
// a node of an overloaded block moves to the best eligible block regardless
// of its own.  The paper's asynchronous visiting is realised as hash-coloured
// sub-rounds: every node of colour s is evaluated against the state at the
// start of sub-round s, then each target admits its candidates in
// (gain desc, node asc) order while it stays within the bound, then the moves
// are applied.  All arithmetic is integer, so the result does not depend on
// thread order.
//
// Node evaluation is bucketed by degree:
//   lane   one lane per node, neighbour labels kept in registers (deg <= 16;
//          deg <= 4 on small graphs)
//   group  16, 32 or 64 lanes per node, open-addressing table in LDS (deg <= 256)
//   block  one workgroup per node with an LDS table of 16, 64 or 80 KB
//          (deg <= 1024, 4096, 8192)
//   hub    the row is cut into 4096-slot chunks; each workgroup sums its
//          chunk in an LDS table and appends the chunk's distinct labels to
//          lists by label partition; one workgroup per partition then sums its
//          list in LDS, and the launch that counts the candidates picks the
//          best partition winner
// Large colours launch the buckets side by side on three streams; small ones
// run them in one launch, or two where rows need a table over 16 KB.  Large
// refinements count a long row's block sums once and keep them up to date
// (kept sums) instead of evaluating the row's slots in every round; after a
// sub-round that moved much they are counted afresh.
// The per-node connection table maps a neighbour label to the summed weight
// of the edges to it (Section 4.1 uses hashing with linear probing for this).
//
// Evaluation writes each node's result at the node's position in the
// sub-round's schedule, so no counter is shared.  Per-label sums use
// LDS-private histograms when the label space is small (refinement: k blocks).
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "lp.hpp"
#include "profile.hpp"
#include "sclap.h"

namespace sclap {

namespace {

// buckets: lane4, lane16, group16 (16 lanes per node), group32, wave,
// block (3 table sizes), hub
constexpr int kNB = 9;
constexpr int kHubBucket = kNB - 1;
constexpr int kLaneSmall = 4;
constexpr int kLaneMax = 16;
constexpr int kG16Max = 32;  // 16 lanes and a 64-entry table per node
constexpr int kG32Max = 64;  // 32 lanes and a 128-entry table per node
constexpr int kWaveTable = 512;
constexpr int kWaveMaxDeg = kWaveTable / 2;
// the workgroup bucket with the longest rows (up to kBlockMaxDeg slots): a
// 10240-entry table (80 KB, probed modulo its size) by default, which leaves
// room on the compute unit for a workgroup with a 64 KB table; the 16384-entry
// power-of-two table (128 KB) as a tuning choice
constexpr int kBlockTable = 10240;
constexpr int kBlockTablePow2 = 16384;
constexpr int kBlockMaxDeg = kBlockTablePow2 / 2;
constexpr int kBlock1Max = 1024;  // 256 threads, 16 KB table
constexpr int kBlock2Max = 4096;  // 1024 threads, 64 KB table (512 with dense sums)
constexpr int kHubTable = 8192;          // LDS table of a hub chunk workgroup (64 KB: two per CU)
constexpr int kHubChunk = kHubTable / 2; // slots per hub workgroup (table load <= 1/2)
constexpr int kHubDenseChunk = 8192;     // slots per hub workgroup with dense block arrays
constexpr int kSmallLabels = 4096;       // LDS-private histograms up to this many labels
constexpr int kCountInEval = 1 << 13;    // colours up to this size count candidates while they evaluate,
constexpr int kCountShortRows = 1 << 14;  // and up to this one where no row has more than 256 slots
constexpr int kMaxBlocks = 512;          // grid cap of the grid-stride candidate kernels
constexpr int kSmallSeg = 16384;         // large colours: segments up to this length have one selecting workgroup
constexpr int kSegChunk = 16384;         // entries per workgroup in the multi-workgroup selection
constexpr int kLargeBlocks = 256;        // grid of the multi-workgroup selection kernel
constexpr int kLargeThreads = 1024;      // and its workgroup size
constexpr int64_t kKeptMinSlots = 1 << 24;  // with fewer slots in long enough rows no sums are kept,
constexpr int64_t kKeptColourSlots = 1 << 22;  // nor with fewer of them per colour
constexpr int32_t kKeptPerSlot = 4;         // a row keeps its sums when it has at least dense_k / 4 slots
constexpr int kUpkeepLongBlocks = 512;      // grid of upkeep_long_kernel
constexpr int kFreshShare = 6;  // after a sub-round that moved more than this part of its slots no sums hold

struct Counters {
    unsigned long long segs;  // segments claimed (high word), entries reserved in them (low word)
    int32_t gmin;             // gain range of the entries
    int32_t gmax;
    uint32_t nlarge;    // segments longer than one workgroup selects from
    uint32_t nlchunks;  // kSegChunk-entry chunks of those segments
    uint32_t bad_color;
    uint32_t nlong;     // chunks of long rows whose node moved (upkeep of kept sums)
    unsigned long long moved;  // slots of the nodes that moved, about (where sums are kept)
};

// Which colours' kept sums hold (see eval_kept_kernel): the mask as the last
// sub-round left it, unless that sub-round moved too much for the upkeep to be
// worth it; then no sums hold until their colour's rows are counted afresh.
struct Fresh {
    const uint32_t* mask;  // bit per colour (null: no sums are kept, or every row is counted)
    const Counters* last;  // the last sub-round's counters
    unsigned long long limit;  // slots it may have moved
};

__device__ __forceinline__ uint32_t fresh_mask(const Fresh& F) { return F.last->moved > F.limit ? 0u : *F.mask; }

// One schedule entry: a node and where its row lies.  Laid out in schedule
// order, so that an evaluation reads 16 consecutive bytes per node instead of
// the node id and then two offsets somewhere in xadj (one dependent load less
// at the start of every evaluation).
struct __align__(16) Row {
    int64_t begin;
    int32_t deg;
    int32_t node;
};

struct EvalArgs {
    const int32_t* adj;
    int64_t S;  // slots of the graph (bound of the vector loads of short rows)
    const int32_t* ew;
    const int32_t* vw;
    const int32_t* label;
    // Narrow copies of label for the neighbour gathers when every label fits
    // 8 or 16 bits (refinement: blocks): a cache line then holds 4 or 2
    // times as many neighbours' labels.  Null when not kept.
    const uint8_t* label8;
    const uint16_t* label16;
    const int32_t* w;
    int64_t bound;
    uint64_t tp;  // H(seed, 2, level, phase, round)
    int32_t refine;
    // several graphs in one launch; gid == null: one graph, the scalars above
    const int32_t* gid;      // [n] graph of each node
    const uint64_t* g_tp;    // [G] tie prefix of each graph for this round
    const int64_t* g_bound;  // [G] bound of each graph's labels
    const int32_t* g_lbase;  // [G] first label of each graph
    // Quiet nodes: evaluated with no neighbouring label connected more strongly
    // than their own, not overloaded, and no neighbour has moved since.  Such a
    // node emits nothing while it stays quiet and its block is not overloaded
    // (its connections are unchanged), so it need not be evaluated again.
    uint8_t* quiet;     // [n] flags (null: not tracked); see quiet_mode()
    const uint32_t* rcnt;  // candidates of each round so far (device)
    int32_t round;         // this round
    int32_t quiet_n;       // nodes of the graph (the tracking threshold is 1/8 of them)
    int32_t dense_k;    // > 0: every node's labels are lbase + [0, dense_k) (refinement blocks)
    // the previous round's candidate count (null in the first round): after a
    // round without candidates the state is a fixed point and the evaluation
    // of the later rounds is skipped
    const uint32_t* gate;
    const Row* rows;  // schedule entries of this launch
    int32_t count;
    int32_t* ct;  // per entry: target label or -1
    int32_t* cg;  // per entry: gain
    // Candidate totals, counted as the results are stored (null: by a launch of
    // their own, which sums in LDS first); entry of label t: t << acc_shift
    unsigned long long* acc;
    int32_t acc_shift;
    int32_t* sums;  // kept block sums of the launch's rows, dense_k per entry (null: not kept)
    Fresh fresh;
    int32_t colour;  // of the launch's rows
};

__device__ __forceinline__ bool sums_hold(const EvalArgs& A) {
    return A.fresh.mask && ((fresh_mask(A.fresh) >> A.colour) & 1u);
}

// A round runs only while the previous one had candidates (gate: that
// round's candidate count, null for the first round).  Rounds are enqueued
// before the previous round's count is known (ahead of the host, or all of
// a level's rounds at once in a captured graph), so every kernel checks the
// gate: after a round without candidates the following ones do nothing.
__device__ __forceinline__ bool stopped(const uint32_t* gate) { return gate && *gate == 0; }

// Quiet-node tracking: marks are written from two rounds after the first
// round with at most n/8 candidates on, and used to skip nodes one round
// later (1: mark, 2: mark and skip, 0: off).  Derived from the per-round
// candidate counts on the device, so it needs no host decision per round.
__device__ __forceinline__ int quiet_mode(const uint8_t* quiet, const uint32_t* rcnt, int32_t round, int32_t n) {
    if (!quiet) return 0;
    for (int32_t q = 0; q + 2 <= round; ++q)
        if (static_cast<int64_t>(rcnt[q]) * 8 <= n) return q + 2 < round ? 2 : 1;
    return 0;
}

__device__ __forceinline__ int quiet_mode(const EvalArgs& A) { return quiet_mode(A.quiet, A.rcnt, A.round, A.quiet_n); }

// ------------------------------------------------------- selection helpers

__device__ __forceinline__ int32_t nbr_label(const EvalArgs& A, int32_t u) {
    if (A.label8) return A.label8[u];
    if (A.label16) return A.label16[u];
    return A.label[u];
}

// Per-node constants: the tie prefix and bound of the node's graph and the
// graph's first label (ties hash graph-local label ids).
struct Ctx {
    uint64_t tp;
    int64_t bound;
    int32_t lbase;
};

__device__ __forceinline__ Ctx ctx_of(const EvalArgs& A, int32_t v) {
    if (A.gid) {
        const int32_t g = A.gid[v];
        return Ctx{A.g_tp[g], A.g_bound[g], A.g_lbase[g]};
    }
    return Ctx{A.tp, A.bound, 0};
}

// Best eligible label seen so far under the total order
// (conn desc, tie(x) asc, x asc); tie(x) = mix(tp ^ x) is computed lazily,
// only when two labels have equal connection.
struct Best {
    int32_t conn;
    int32_t x;
    uint64_t tie;
    bool tv;
};

__device__ __forceinline__ void best_init(Best& b) {
    b.conn = -1;
    b.x = -1;
    b.tie = 0;
    b.tv = false;
}

__device__ __forceinline__ uint64_t tie_of(const Ctx& kx, int32_t x) {
    return mix64(kx.tp ^ static_cast<uint64_t>(static_cast<uint32_t>(x - kx.lbase)));
}

__device__ __forceinline__ void best_consider(Best& b, int32_t x, int32_t conn, const Ctx& kx) {
    if (b.x < 0 || conn > b.conn) {
        b.conn = conn;
        b.x = x;
        b.tv = false;
        return;
    }
    if (conn < b.conn) return;
    const uint64_t tx = tie_of(kx, x);
    if (!b.tv) {
        b.tie = tie_of(kx, b.x);
        b.tv = true;
    }
    if (tx < b.tie || (tx == b.tie && x < b.x)) {
        b.x = x;
        b.tie = tx;
    }
}

__device__ __forceinline__ uint64_t best_tie(const Best& b, const Ctx& kx) { return b.tv ? b.tie : tie_of(kx, b.x); }

// Reductions over aligned groups of G lanes of a wave (G a power of two <= 64).
template <int G>
__device__ __forceinline__ int32_t group_max(int32_t v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        const int32_t u = __shfl_xor(v, o, 64);
        v = u > v ? u : v;
    }
    return v;
}

template <int G>
__device__ __forceinline__ int32_t group_min(int32_t v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        const int32_t u = __shfl_xor(v, o, 64);
        v = u < v ? u : v;
    }
    return v;
}

template <int G>
__device__ __forceinline__ uint64_t group_min_u64(uint64_t v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) {
        const uint32_t lo = __shfl_xor(static_cast<uint32_t>(v), o, 64);
        const uint32_t hi = __shfl_xor(static_cast<uint32_t>(v >> 32), o, 64);
        const uint64_t u = (static_cast<uint64_t>(hi) << 32) | lo;
        v = u < v ? u : v;
    }
    return v;
}

template <int G>
__device__ __forceinline__ bool group_any(bool b) {
    const uint64_t m = __ballot(b);
    if (G == 64) return m != 0;
    const int base = lane_id() & ~(G - 1);
    return ((m >> base) & ((1ULL << G) - 1)) != 0;
}

// Group-wide argmax; every lane of the group gets the winning (x, conn) and
// its tie key.  Most nodes have no eligible label of positive gain after the
// first rounds, which one vote of the lanes tells.
template <int G>
__device__ __forceinline__ void group_argmax(const Best& b, const Ctx& kx, int32_t& out_x, int32_t& out_conn,
                                             uint64_t& out_tie) {
    out_x = -1;
    out_conn = -1;
    out_tie = ~0ULL;
    if (!group_any<G>(b.x >= 0)) return;
    const int32_t bc = b.x >= 0 ? b.conn : -1;
    const int32_t maxc = group_max<G>(bc);
    const bool top = b.x >= 0 && bc == maxc;
    const uint64_t tk = top ? best_tie(b, kx) : ~0ULL;
    out_tie = group_min_u64<G>(tk);
    const int32_t xx = (top && tk == out_tie) ? b.x : INT_MAX;
    out_x = group_min<G>(xx);
    out_conn = maxc;
}

// Combines one candidate per wave (written to LDS by each wave's lane 0).
__device__ __forceinline__ void combine_into(int32_t& bc, uint64_t& bt, int32_t& bx, int32_t c2, uint64_t t2,
                                             int32_t x2) {
    if (x2 < 0) return;
    if (bx < 0 || c2 > bc || (c2 == bc && (t2 < bt || (t2 == bt && x2 < bx)))) {
        bc = c2;
        bt = t2;
        bx = x2;
    }
}

__device__ __forceinline__ bool eligible(const EvalArgs& A, int32_t x, int32_t c, const Ctx& kx) {
    return static_cast<int64_t>(A.w[x]) + c <= kx.bound;
}

// Candidate total of a target: count in the high word, weight in the low one
// (a label's weight never exceeds c(V) <= 2^31 - 1, so no carry; the candidates
// of a heavy graph are counted without their weights, see Admission::heavy).
__device__ __forceinline__ unsigned long long acc_of(int32_t cnt, int32_t weight) {
    return (static_cast<unsigned long long>(static_cast<uint32_t>(cnt)) << 32) | static_cast<uint32_t>(weight);
}

// The eligible labels of a table (or of a lane's registers) are looked at in
// groups whose label weights are read together: one after the other, each
// read's latency (some 0.7 us) bounded the evaluation of small colours.
template <int U>
__device__ __forceinline__ void consider_group(const EvalArgs& A, const Ctx& kx, const int32_t* x, const int32_t* conn,
                                               int32_t c, int32_t own, bool over, Best& best, bool& blocked) {
    int32_t wx[U];
    bool need[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        blocked |= x[u] >= 0 && conn[u] > own;
        // a move needs a positive gain unless the own block is overloaded
        need[u] = x[u] >= 0 && (over || conn[u] > own) && (best.x < 0 || conn[u] >= best.conn);
        wx[u] = need[u] ? A.w[x[u]] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (need[u] && (best.x < 0 || conn[u] >= best.conn) && static_cast<int64_t>(wx[u]) + c <= kx.bound)
            best_consider(best, x[u], conn[u], kx);
}

// Decision for a node given its best eligible label (x, conn) and the
// connection to its own label: a move needs a positive gain, or an overloaded
// own block during refinement.  Returns the target or -1.
__device__ __forceinline__ int32_t store_decision(const EvalArgs& A, int32_t i, int32_t x, int32_t conn, int32_t own,
                                                  bool over) {
    int32_t t = -1, gain = 0;
    if (x >= 0) {
        gain = conn - own;
        if (over || gain > 0) t = x;
    }
    A.ct[i] = t;
    A.cg[i] = gain;
    return t;
}

// The same, and the candidate counted if the evaluation counts them.
__device__ __forceinline__ void store_result(const EvalArgs& A, int32_t i, int32_t x, int32_t conn, int32_t own,
                                             bool over, int32_t c) {
    const int32_t t = store_decision(A, i, x, conn, own, over);
    if (A.acc && t >= 0) atomicAdd(&A.acc[t << A.acc_shift], acc_of(1, c));
}

// Counts the candidates of a whole wave (t: -1 or the lane's target).  Nodes of
// few neighbours often want the same label (all the leaves of a star do), and
// adds to one address are served one every 12 ns, so a target that many lanes
// share gets one add: the first lane's target is looked at, and the next one's.
__device__ __forceinline__ void count_lanes(const EvalArgs& A, int32_t t, int32_t c) {
    constexpr int kMany = 8;
    uint64_t todo = __ballot(t >= 0);
#pragma unroll
    for (int tries = 0; tries < 2; ++tries) {
        if (__popcll(todo) < kMany) break;  // uniform
        const int first = __ffsll(static_cast<long long>(todo)) - 1;
        const int32_t t0 = __builtin_amdgcn_readlane(t, first);
        const uint64_t same = __ballot(t == t0);
        todo &= ~same;
        const int cnt = __popcll(same);
        if (cnt < kMany) continue;
        const int32_t weight = A.vw ? wave_sum(t == t0 ? c : 0) : cnt;
        if (lane_id() == first) atomicAdd(&A.acc[t0 << A.acc_shift], acc_of(cnt, weight));
        if (t == t0) t = -1;
    }
    if (t >= 0) atomicAdd(&A.acc[t << A.acc_shift], acc_of(1, c));
}

// True if v is quiet and may skip evaluation (its block is not overloaded).
__device__ __forceinline__ bool skip_quiet(const EvalArgs& A, int qm, int32_t v, const Ctx& kx) {
    if (qm < 2 || !A.quiet[v]) return false;
    return !A.refine || A.w[A.label[v]] <= kx.bound;
}

__device__ __forceinline__ uint32_t table_size_for(int32_t d, uint32_t lo, uint32_t hi) {
    uint32_t t = lo;
    while (t < 2u * static_cast<uint32_t>(d) && t < hi) t <<= 1;
    return t;
}

// Linear-probing insert of (x, wt) into a table of 2^k entries (key -1 =
// empty), in LDS or HBM.  The table always has a free entry for a new key.
// Returns the entry if x is new to the table, else -1.
__device__ __forceinline__ int32_t table_add(int32_t* keys, int32_t* vals, uint32_t mask, int32_t x, int32_t wt) {
    uint32_t h = slot_hash(static_cast<uint32_t>(x)) & mask;
    while (true) {
        const int32_t prev = atomicCAS(&keys[h], -1, x);
        if (prev == -1 || prev == x) {
            atomicAdd(&vals[h], wt);
            return prev == -1 ? static_cast<int32_t>(h) : -1;
        }
        h = (h + 1) & mask;
    }
}

// The same for a table of any size tsz: the first probe is a hash of x scaled
// to [0, tsz), and probing wraps at tsz.
__device__ __forceinline__ int32_t table_add_scaled(int32_t* keys, int32_t* vals, uint32_t tsz, uint32_t hash,
                                                    int32_t x, int32_t wt) {
    uint32_t h = static_cast<uint32_t>((static_cast<uint64_t>(hash) * tsz) >> 32);
    while (true) {
        const int32_t prev = atomicCAS(&keys[h], -1, x);
        if (prev == -1 || prev == x) {
            atomicAdd(&vals[h], wt);
            return prev == -1 ? static_cast<int32_t>(h) : -1;
        }
        h = h + 1 == tsz ? 0u : h + 1;
    }
}

__device__ __forceinline__ int32_t table_add_sized(int32_t* keys, int32_t* vals, uint32_t tsz, int32_t x, int32_t wt) {
    return table_add_scaled(keys, vals, tsz, slot_hash(static_cast<uint32_t>(x)), x, wt);
}

// Value of key x in such a table (0: absent; the table has a free entry or
// holds x).
template <bool kPow2>
__device__ __forceinline__ int32_t table_find(const int32_t* keys, const int32_t* vals, uint32_t tsz, int32_t x) {
    const uint32_t sh = slot_hash(static_cast<uint32_t>(x));
    uint32_t h = kPow2 ? sh & (tsz - 1) : static_cast<uint32_t>((static_cast<uint64_t>(sh) * tsz) >> 32);
    while (true) {
        const int32_t k = keys[h];
        if (k == x) return vals[h];
        if (k == -1) return 0;
        h = h + 1 == tsz ? 0u : h + 1;
    }
}

// Looks at entries first, first + STEP, ... of a table of tsz entries, U at a
// time, for the best eligible label other than a.
template <int STEP, int U>
__device__ __forceinline__ void scan_table(const EvalArgs& A, const Ctx& kx, const int32_t* keys, const int32_t* vals,
                                           uint32_t tsz, uint32_t first, int32_t a, int32_t c, int32_t own, bool over,
                                           Best& best, bool& blocked) {
    for (uint32_t j0 = first; j0 < tsz; j0 += STEP * U) {
        int32_t x[U], cn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t j = j0 + u * STEP;
            x[u] = j < tsz ? keys[j] : -1;
            cn[u] = j < tsz ? vals[j] : 0;
            if (x[u] == a) x[u] = -1;
        }
        consider_group<U>(A, kx, x, cn, c, own, over, best, blocked);
    }
}

// Empties a table of tsz entries (a multiple of 4) with 16-byte stores.
template <int NT>
__device__ __forceinline__ void table_clear(int32_t* keys, int32_t* vals, uint32_t tsz, int tid) {
    for (uint32_t j = 4 * tid; j < tsz; j += 4 * NT) {
        *reinterpret_cast<int4*>(keys + j) = make_int4(-1, -1, -1, -1);
        *reinterpret_cast<int4*>(vals + j) = make_int4(0, 0, 0, 0);
    }
}

// A thread's slots of a row of up to NT * U: the neighbours' labels, and for
// each the table entry if this slot brought the label into the table (else
// -1).  A table's distinct labels are then found through these entries: reading
// a table of two to four entries per slot from end to end took more
// instructions than filling it (with the vote in group_argmax: clustering of a
// weighted power-law graph, 2^22 nodes, 10 rounds, 20.8 -> 19.9 ms; partition
// of 2^24 nodes 228.4 -> 223.0 ms).
template <int U>
struct RowSlots {
    int32_t x[U];
    int32_t at[U];
};

// Adds the slots [b, b+d) of a row, d <= NT * U, to an empty table of tsz
// entries; all of the thread's gathers are in flight before it inserts.  kPow2:
// tsz is a power of two (masked probes), else any size (table_add_sized).
template <int NT, int U, bool kPow2 = true>
__device__ __forceinline__ void insert_slots(const EvalArgs& A, int64_t b, int32_t d, int32_t* keys, int32_t* vals,
                                             uint32_t tsz, int tid, RowSlots<U>& R) {
    int32_t wt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t j = tid + u * NT;
        R.x[u] = j < d ? A.adj[b + j] : 0;
        wt[u] = j < d ? (A.ew ? A.ew[b + j] : 1) : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) R.x[u] = tid + u * NT < d ? nbr_label(A, R.x[u]) : -1;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        R.at[u] = -1;
        if (R.x[u] < 0) continue;
        R.at[u] = kPow2 ? table_add(keys, vals, tsz - 1, R.x[u], wt[u])
                        : table_add_sized(keys, vals, tsz, R.x[u], wt[u]);
    }
}

// Looks at the labels that the thread's slots brought into the table for the
// best eligible one other than a.
template <int U>
__device__ __forceinline__ void consider_slots(const EvalArgs& A, const Ctx& kx, const RowSlots<U>& R,
                                               const int32_t* vals, int32_t a, int32_t c, int32_t own, bool over,
                                               Best& best, bool& blocked) {
    constexpr int V = U < 4 ? U : 4;
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += V) {
        int32_t x[V], cn[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int32_t at = R.at[u0 + u];
            x[u] = at >= 0 && R.x[u0 + u] != a ? R.x[u0 + u] : -1;
            cn[u] = x[u] >= 0 ? vals[at] : 0;
        }
        consider_group<V>(A, kx, x, cn, c, own, over, best, blocked);
    }
}

// ------------------------------------------------------------ lane bucket

// A short row's neighbour ids and weights, then the neighbours' labels.
// The row is read with 16-byte loads from the aligned address at or below
// its start when the aligned window lies inside the arrays (one lane per
// row: a wave's scalar loads each touch 64 rows, so fewer, wider loads
// spend less of the load unit's time); -1 and 0 past the row's end.
template <int MAXD>
__device__ __forceinline__ void lane_words(const int32_t* base, int64_t b, int d, int64_t S, int32_t* out, bool& vec) {
    constexpr int NQ = MAXD / 4 + 1;
    const int off = static_cast<int>((reinterpret_cast<uintptr_t>(base + b) & 15u) >> 2);
    const int64_t b0 = b - off;
    const int nq = (off + d + 3) >> 2;
    vec = b0 >= 0 && b0 + 4 * static_cast<int64_t>(nq) <= S;
    if (!vec) return;
    int32_t r[4 * NQ];
    const int4* q = reinterpret_cast<const int4*>(base + b0);
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        int4 w = make_int4(0, 0, 0, 0);
        if (k < nq) w = q[k];
        r[4 * k] = w.x;
        r[4 * k + 1] = w.y;
        r[4 * k + 2] = w.z;
        r[4 * k + 3] = w.w;
    }
#pragma unroll
    for (int j = 0; j < MAXD; ++j) {
        const int32_t x0 = r[j], x1 = r[j + 1], x2 = r[j + 2], x3 = r[j + 3];
        out[j] = off == 0 ? x0 : off == 1 ? x1 : off == 2 ? x2 : x3;
    }
}

template <int MAXD>
__device__ __forceinline__ void lane_row(const EvalArgs& A, int64_t b, int d, int32_t* lab, int32_t* wt) {
    bool vec;
    lane_words<MAXD>(A.adj, b, d, A.S, lab, vec);
    if (vec) {
        if (A.ew) {
            bool vec_w;
            lane_words<MAXD>(A.ew, b, d, A.S, wt, vec_w);
            if (!vec_w)
#pragma unroll
                for (int j = 0; j < MAXD; ++j) wt[j] = j < d ? A.ew[b + j] : 0;
        }
#pragma unroll
        for (int j = 0; j < MAXD; ++j) {
            lab[j] = j < d ? nbr_label(A, lab[j]) : -1;
            if (!A.ew) wt[j] = j < d ? 1 : 0;
            else if (j >= d) wt[j] = 0;
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < MAXD; ++j) {
        if (j < d) {
            lab[j] = nbr_label(A, A.adj[b + j]);
            wt[j] = A.ew ? A.ew[b + j] : 1;
        } else {
            lab[j] = -1;
            wt[j] = 0;
        }
    }
}

// The target of the node at entry i, or -1; c gets its weight.
template <int MAXD>
__device__ __forceinline__ int32_t eval_lane_node(const EvalArgs& A, int32_t i, int32_t& c) {
    const Row row = A.rows[i];
    if (stopped(A.gate)) return -1;
    const int qm = quiet_mode(A);
    const int32_t v = row.node;
    const Ctx kx = ctx_of(A, v);
    if (skip_quiet(A, qm, v, kx)) return store_decision(A, i, -1, 0, 0, false);
    const int d = row.deg;
    const int32_t a = A.label[v];
    c = A.vw ? A.vw[v] : 1;
    int32_t lab[MAXD], conn[MAXD];
    const bool over = A.refine && A.w[a] > kx.bound;
    lane_row<MAXD>(A, row.begin, d, lab, conn);
    int32_t own = 0;
#pragma unroll
    for (int j = 0; j < MAXD; ++j) own += (lab[j] == a) ? conn[j] : 0;
    // slot weights to label sums: each slot of the first occurrence of a label
    // collects the later ones, which drop out
#pragma unroll
    for (int j = 0; j < MAXD; ++j) {
        if (lab[j] == a) lab[j] = -1;
#pragma unroll
        for (int j2 = j + 1; j2 < MAXD; ++j2) {
            const bool same = lab[j] >= 0 && lab[j2] == lab[j];
            conn[j] += same ? conn[j2] : 0;
            lab[j2] = same ? -1 : lab[j2];
        }
    }
    Best best;
    best_init(best);
    bool blocked = false;  // some other neighbouring label is connected more strongly
    constexpr int U = MAXD < 8 ? MAXD : 8;
#pragma unroll
    for (int j = 0; j < MAXD; j += U) consider_group<U>(A, kx, lab + j, conn + j, c, own, over, best, blocked);
    if (qm) A.quiet[v] = (!over && !blocked) ? 1 : 0;
    return store_decision(A, i, best.x, best.conn, own, over);
}

template <int MAXD>
__device__ __forceinline__ void eval_lane_body(const EvalArgs& A, int32_t bid) {
    const int32_t i = bid * 256 + static_cast<int32_t>(threadIdx.x);
    int32_t c = 0;
    const int32_t t = i < A.count ? eval_lane_node<MAXD>(A, i, c) : -1;
    if (A.acc) count_lanes(A, t, c);
}

template <int MAXD>
__global__ void __launch_bounds__(256) eval_lane_kernel(EvalArgs A) {
    eval_lane_body<MAXD>(A, blockIdx.x);
}

// --------------------------------------------------- group and wave buckets

// G lanes per node (G = 16, 32 or 64: 256 / G nodes per workgroup), each
// group with an open-addressing table of T entries in LDS.
// LDS: 2 * (256 / G) * T int32 (the groups' key tables, then their sums).
template <int G, int T>  // rows of up to T / 2 slots
__device__ __forceinline__ void eval_group_body(const EvalArgs& A, int32_t bid, int32_t* lds) {
    constexpr int NG = 256 / G;
    const int grp = threadIdx.x / G;
    const int gl = threadIdx.x % G;
    const int node_i = bid * NG + grp;
    if (node_i >= A.count) return;  // uniform per group
    const Row row = A.rows[node_i];
    if (stopped(A.gate)) return;
    const int qm = quiet_mode(A);
    int32_t* keys = lds + grp * T;
    int32_t* vals = lds + (NG + grp) * T;
    const int32_t v = row.node;
    const Ctx kx = ctx_of(A, v);
    if (skip_quiet(A, qm, v, kx)) {
        if (gl == 0) store_result(A, node_i, -1, 0, 0, false, 0);
        return;
    }
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    const bool over = A.refine && A.w[a] > kx.bound;
    const uint32_t tsz = table_size_for(row.deg, T < 64 ? T : 64, T);
    table_clear<G>(keys, vals, tsz, gl);
    wave_sync();
    RowSlots<T / 2 / G> slots;
    insert_slots<G, T / 2 / G>(A, row.begin, row.deg, keys, vals, tsz, gl, slots);
    wave_sync();
    const int32_t own = table_find<true>(keys, vals, tsz, a);
    Best best;
    best_init(best);
    bool blocked = false;  // some other neighbouring label is connected more strongly
    consider_slots(A, kx, slots, vals, a, c, own, over, best, blocked);
    int32_t bx, bconn;
    uint64_t btie;
    group_argmax<G>(best, kx, bx, bconn, btie);
    const bool any_blocked = group_any<G>(blocked);
    if (gl == 0) {
        store_result(A, node_i, bx, bconn, own, over, c);
        if (qm) A.quiet[v] = (!over && !any_blocked) ? 1 : 0;
    }
}

template <int G, int T>
__global__ void __launch_bounds__(256) eval_group_kernel(EvalArgs A) {
    __shared__ __align__(16) int32_t lds[2 * (256 / G) * T];
    eval_group_body<G, T>(A, blockIdx.x, lds);
}

// ----------------------------------------------------------- block bucket

// LDS of the block bodies: per-wave winners (tie keys, labels, sums) then
// the body's table.
template <int NT>
struct BlockScratch {
    uint64_t tie[NT / 64];
    int32_t conn[NT / 64];
    int32_t x[NT / 64];
};

// Rows of up to NT * U slots.  LDS: BlockScratch<NT> then 2 * TABLE int32
// (keys, then sums).
template <int NT, int TABLE, int U>
__device__ __forceinline__ void eval_block_body(const EvalArgs& A, int32_t bid, unsigned char* lds) {
    BlockScratch<NT>& S = *reinterpret_cast<BlockScratch<NT>*>(lds);
    int32_t* keys = reinterpret_cast<int32_t*>(lds + sizeof(BlockScratch<NT>));
    int32_t* vals = keys + TABLE;
    int32_t* s_conn = S.conn;
    int32_t* s_x = S.x;
    uint64_t* s_tie = S.tie;
    const int tid = threadIdx.x;
    const int wid = tid >> 6;
    const int lane = lane_id();
    const Row row = A.rows[bid];
    if (stopped(A.gate)) return;  // uniform over the grid
    const int qm = quiet_mode(A);
    const int32_t v = row.node;
    const Ctx kx = ctx_of(A, v);
    if (skip_quiet(A, qm, v, kx)) {  // uniform over the workgroup
        if (tid == 0) store_result(A, bid, -1, 0, 0, false, 0);
        return;
    }
    const int32_t d = row.deg;
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    const bool over = A.refine && A.w[a] > kx.bound;
    constexpr bool kPow2 = (TABLE & (TABLE - 1)) == 0;
    const uint32_t tsz = kPow2 ? table_size_for(d, 512, TABLE) : static_cast<uint32_t>(TABLE);
    table_clear<NT>(keys, vals, tsz, tid);
    __syncthreads();
    RowSlots<U> slots;
    insert_slots<NT, U, kPow2>(A, row.begin, d, keys, vals, tsz, tid, slots);
    __syncthreads();
    const int32_t own = table_find<kPow2>(keys, vals, tsz, a);
    Best best;
    best_init(best);
    bool blocked = false;
    consider_slots(A, kx, slots, vals, a, c, own, over, best, blocked);
    int32_t bx, bconn;
    uint64_t btie;
    group_argmax<64>(best, kx, bx, bconn, btie);
    if (lane == 0) {
        s_conn[wid] = bconn;
        s_x[wid] = bx;
        s_tie[wid] = btie;
    }
    const int any_blocked = __syncthreads_or(blocked);
    if (tid == 0) {
        int32_t fc = -1, fx = -1;
        uint64_t ft = ~0ULL;
        for (int w = 0; w < NT / 64; ++w) combine_into(fc, ft, fx, s_conn[w], s_tie[w], s_x[w]);
        store_result(A, bid, fx, fc, own, over, c);
        if (qm) A.quiet[v] = (!over && !any_blocked) ? 1 : 0;
    }
}

template <int NT, int TABLE, int U>
__global__ void __launch_bounds__(NT) eval_block_kernel(EvalArgs A) {
    __shared__ __align__(16) unsigned char lds[sizeof(BlockScratch<NT>) + 2 * TABLE * sizeof(int32_t)];
    eval_block_body<NT, TABLE, U>(A, blockIdx.x, lds);
}

// ------------------------------------------------------------- hub bucket

struct HubArgs {
    const int32_t* hub_plog;     // [H] log2 of the hub's partition count
    const int32_t* hub_pbase;    // [H+1] first partition of each hub
    const int32_t* hub_cap;      // [H] entries per partition region
    const int32_t* chunk_hub;    // [nchunks]
    const int32_t* part_hub;     // [nparts]
    const int64_t* hub_rbase;    // [H] first region entry of the hub
    const int64_t* hub_obase;    // [H] first overflow entry of the hub
    const int64_t* hub_toff;     // [H] first entry of the hub's HBM table (two per slot)
    const int64_t* chunk_begin;  // [nchunks] first slot of the chunk
    int32_t* rcount;   // [nparts] entries reserved per partition    } zero before
    int32_t* ocount;   // [H] overflow entries                      } and after
    uint32_t* tfill;   // [H] entries of the HBM table given out    } every
    int32_t* hub_own;  // [H] connection to the own label           } sub-round
    int32_t* ekeys;    // partition regions (label, summed weight)
    int32_t* evals;
    int32_t* okeys;    // overflow of full regions
    int32_t* ovals;
    int32_t* gkeys;    // HBM tables
    int32_t* gvals;
    int32_t* w_conn;   // winners per partition
    uint64_t* w_tie;
    int32_t* w_x;
    int32_t part_limit;  // partitions with more entries are summed in HBM
    int32_t count;       // hubs of the colour (0: none); their entries are the colour's last
    int32_t* hub_sum;    // dense refinement: a row of dense_k sums per hub, else null
};

constexpr int kHubThreads = 1024;
constexpr int kPartThreads = 256;
constexpr int kPartTable = 4096;  // 32 KB LDS table of a partition workgroup (four per CU)
constexpr int kMaxPartLog = 11;   // at most 2048 partitions per hub

__device__ __forceinline__ uint32_t part_of(int32_t x, int32_t plog) {
    return plog == 0 ? 0u : (slot_hash(static_cast<uint32_t>(x)) >> (32 - plog));
}

// Sums one chunk of a hub row in an LDS table, then scatters the chunk's
// distinct (label, weight) entries into the hub's label partitions.
// LDS: 2 * kHubTable int32, then 2 << kMaxPartLog.
constexpr size_t kHubLds = (2 * kHubTable + (2 << kMaxPartLog)) * sizeof(int32_t);

__device__ __forceinline__ void hub_chunk_body(const EvalArgs& A, const HubArgs& H, int32_t bid, unsigned char* lds) {
    int32_t* keys = reinterpret_cast<int32_t*>(lds);
    int32_t* vals = keys + kHubTable;
    uint32_t* pcount = reinterpret_cast<uint32_t*>(vals + kHubTable);
    int32_t* pbase = vals + kHubTable + (1 << kMaxPartLog);
    constexpr int U = kHubChunk / kHubThreads;
    if (stopped(A.gate)) return;  // uniform over the grid
    const int tid = threadIdx.x;
    const int32_t h = H.chunk_hub[bid];
    const int64_t begin = H.chunk_begin[bid];
    const int64_t row_end = A.rows[h].begin + A.rows[h].deg;
    const int64_t end = begin + kHubChunk < row_end ? begin + kHubChunk : row_end;
    const uint32_t tsz = table_size_for(static_cast<int32_t>(end - begin), 1024, kHubTable);
    const int32_t plog = H.hub_plog[h];
    const int32_t P = 1 << plog;
    table_clear<kHubThreads>(keys, vals, tsz, tid);
    for (int32_t j = tid; j < P; j += kHubThreads) pcount[j] = 0;
    __syncthreads();
    RowSlots<U> slots;
    insert_slots<kHubThreads, U>(A, begin, static_cast<int32_t>(end - begin), keys, vals, tsz, tid, slots);
    uint32_t rank[U];  // of the label within its partition's list
#pragma unroll
    for (int u = 0; u < U; ++u)
        rank[u] = slots.at[u] >= 0 ? atomicAdd(&pcount[part_of(slots.x[u], plog)], 1u) : 0;
    __syncthreads();
    for (int32_t j = tid; j < P; j += kHubThreads) {
        const uint32_t c = pcount[j];
        pbase[j] = c ? atomicAdd(&H.rcount[H.hub_pbase[h] + j], static_cast<int32_t>(c)) : 0;
    }
    __syncthreads();
    const int32_t cap = H.hub_cap[h];
    const int64_t rb = H.hub_rbase[h];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (slots.at[u] < 0) continue;
        const int32_t x = slots.x[u], wt = vals[slots.at[u]];
        const uint32_t p = part_of(x, plog);
        const int32_t idx = pbase[p] + static_cast<int32_t>(rank[u]);
        if (idx < cap) {
            const int64_t at = rb + static_cast<int64_t>(p) * cap + idx;
            H.ekeys[at] = x;
            H.evals[at] = wt;
        } else {  // region full: the rest of the partition goes to the hub's overflow list
            const int64_t at = H.hub_obase[h] + atomicAdd(&H.ocount[h], 1);
            H.okeys[at] = x;
            H.ovals[at] = wt;
        }
    }
}

__global__ void __launch_bounds__(kHubThreads) hub_chunk_kernel(EvalArgs A, HubArgs H) {
    __shared__ __align__(16) unsigned char lds[kHubLds];
    hub_chunk_body(A, H, blockIdx.x, lds);
}

__device__ __forceinline__ int32_t block_sum_part(int32_t v, int32_t* s_red) {
    v = wave_sum(v);
    if (lane_id() == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    int32_t t = 0;
    for (int w = 0; w < kPartThreads / 64; ++w) t += s_red[w];
    __syncthreads();
    return t;
}

// Orders a workgroup's accesses to a table in device memory that no other
// workgroup touches: its waves share one L1 and one L2, so it is enough that
// every wave's stores and atomics have reached the L2.  A device-scope fence
// also writes back and invalidates the L2 (hub of 2^22 slots, 2048 partitions:
// 123 us per launch with two fences per wave, 85 us like this).
__device__ __forceinline__ void table_sync() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Best eligible label of a hub partition of more than part_limit entries.
// Partitions share no label, so the partition's workgroup sums it alone, in its
// own stretch of the hub's table in HBM (twice its entries; all partitions
// together have at most as many entries as the hub has slots).  One workgroup
// that summed every partition of such a hub in turn took 54 ms for a hub of
// 2^22 slots with distinct labels; side by side the partitions take 85 us.
__device__ void hub_part_in_hbm(const EvalArgs& A, const HubArgs& H, const Ctx& kx, int32_t h, int32_t p,
                                int64_t r0, int32_t in_region, int32_t ov, int32_t total, int32_t a, int32_t c,
                                Best& best) {
    __shared__ uint32_t s_first;
    const int tid = threadIdx.x;
    const uint32_t tsz = 2u * static_cast<uint32_t>(total);
    if (tid == 0) s_first = atomicAdd(&H.tfill[h], tsz);
    __syncthreads();
    int32_t* gk = H.gkeys + H.hub_toff[h] + s_first;
    int32_t* gv = H.gvals + H.hub_toff[h] + s_first;
    for (int64_t j = tid; j < tsz; j += kPartThreads) {
        __hip_atomic_store(&gk[j], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&gv[j], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    table_sync();
    // the partition's labels share the top plog bits of their hash
    const int32_t plog = H.hub_plog[h];
    auto add = [&](int32_t x, int32_t wt) {
        table_add_scaled(gk, gv, tsz, slot_hash(static_cast<uint32_t>(x)) << plog, x, wt);
    };
    for (int32_t j = tid; j < in_region; j += kPartThreads) add(H.ekeys[r0 + j], H.evals[r0 + j]);
    const int64_t ob = H.hub_obase[h];
    for (int32_t j = tid; j < ov; j += kPartThreads) {
        const int32_t x = H.okeys[ob + j];
        if (part_of(x, plog) == static_cast<uint32_t>(p)) add(x, H.ovals[ob + j]);
    }
    table_sync();
    for (int64_t j = tid; j < tsz; j += kPartThreads) {
        const int32_t x = __hip_atomic_load(&gk[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (x < 0) continue;
        const int32_t conn = __hip_atomic_load(&gv[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (x == a) {
            H.hub_own[h] = conn;
            continue;
        }
        if (best.x >= 0 && conn < best.conn) continue;
        if (!eligible(A, x, c, kx)) continue;
        best_consider(best, x, conn, kx);
    }
}

// One workgroup per label partition of a hub: sums the partition's entries
// in LDS (more than part_limit of them: in HBM) and writes the partition's best
// eligible label.
__global__ void __launch_bounds__(kPartThreads) hub_part_kernel(EvalArgs A, HubArgs H) {
    __shared__ __align__(16) int32_t keys[kPartTable];
    __shared__ __align__(16) int32_t vals[kPartTable];
    __shared__ int32_t s_red[kPartThreads / 64];
    __shared__ int32_t s_conn[kPartThreads / 64];
    __shared__ int32_t s_x[kPartThreads / 64];
    __shared__ uint64_t s_tie[kPartThreads / 64];
    if (stopped(A.gate)) return;  // uniform over the grid
    const int tid = threadIdx.x;
    const int32_t gp = blockIdx.x;
    const int32_t h = H.part_hub[gp];
    const int32_t p = gp - H.hub_pbase[h];
    const int32_t plog = H.hub_plog[h];
    const int32_t cap = H.hub_cap[h];
    const int32_t in_region = H.rcount[gp] < cap ? H.rcount[gp] : cap;
    const int32_t ov = H.ocount[h];
    const int64_t ob = H.hub_obase[h];
    int32_t mine = 0;
    for (int32_t j = tid; j < ov; j += kPartThreads) mine += part_of(H.okeys[ob + j], plog) == static_cast<uint32_t>(p);
    const int32_t total = in_region + (ov > 0 ? block_sum_part(mine, s_red) : 0);
    const int64_t r0 = H.hub_rbase[h] + static_cast<int64_t>(p) * cap;
    const int32_t v = A.rows[h].node;
    const Ctx kx = ctx_of(A, v);
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    // only the partition of a holds a; the others' best labels are compared
    // with its connection by hub_decide
    Best best;
    best_init(best);
    if (total > H.part_limit) {  // uniform over the workgroup
        hub_part_in_hbm(A, H, kx, h, p, r0, in_region, ov, total, a, c, best);
    } else {
        const uint32_t tsz = table_size_for(total, 256, kPartTable);
        const uint32_t mask = tsz - 1;
        table_clear<kPartThreads>(keys, vals, tsz, tid);
        __syncthreads();
        constexpr int U = kPartTable / 2 / kPartThreads;
        RowSlots<U> slots;
        {
            int32_t wt[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t j = tid + u * kPartThreads;
                slots.x[u] = j < in_region ? H.ekeys[r0 + j] : -1;
                wt[u] = j < in_region ? H.evals[r0 + j] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                slots.at[u] = slots.x[u] >= 0 ? table_add(keys, vals, mask, slots.x[u], wt[u]) : -1;
        }
        for (int32_t j = tid; j < ov; j += kPartThreads) {
            const int32_t x = H.okeys[ob + j];
            if (part_of(x, plog) == static_cast<uint32_t>(p)) table_add(keys, vals, mask, x, H.ovals[ob + j]);
        }
        __syncthreads();
        if (tid == 0 && part_of(a, plog) == static_cast<uint32_t>(p))
            H.hub_own[h] = table_find<true>(keys, vals, tsz, a);
        bool blocked = false;
        // labels that only the overflow list names are found in the table itself
        if (ov > 0) scan_table<kPartThreads, 4>(A, kx, keys, vals, tsz, tid, a, c, 0, true, best, blocked);
        else consider_slots(A, kx, slots, vals, a, c, 0, true, best, blocked);
    }
    int32_t bx, bconn;
    uint64_t btie;
    group_argmax<64>(best, kx, bx, bconn, btie);
    const int wid = tid >> 6;
    if (lane_id() == 0) {
        s_conn[wid] = bconn;
        s_x[wid] = bx;
        s_tie[wid] = btie;
    }
    __syncthreads();
    if (tid == 0) {
        int32_t fc = -1, fx = -1;
        uint64_t ft = ~0ULL;
        for (int w = 0; w < kPartThreads / 64; ++w) combine_into(fc, ft, fx, s_conn[w], s_tie[w], s_x[w]);
        H.w_conn[gp] = fc;
        H.w_tie[gp] = ft;
        H.w_x[gp] = fx;
    }
}

// Best of the threads' candidates for a workgroup of 256; thread 0 has it.
__device__ __forceinline__ void block_combine(int32_t& fc, uint64_t& ft, int32_t& fx) {
    __shared__ int32_t s_conn[4];
    __shared__ int32_t s_x[4];
    __shared__ uint64_t s_tie[4];
    const int32_t maxc = wave_max(fx >= 0 ? fc : -1);
    const bool top = fx >= 0 && fc == maxc;
    const uint64_t mt = wave_min_u64(top ? ft : ~0ULL);
    const int32_t bx = wave_min((top && ft == mt) ? fx : INT_MAX);
    if (lane_id() == 0) {
        s_conn[threadIdx.x >> 6] = maxc;
        s_x[threadIdx.x >> 6] = maxc >= 0 ? bx : -1;
        s_tie[threadIdx.x >> 6] = mt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        fc = -1;
        fx = -1;
        ft = ~0ULL;
        for (int w = 0; w < 4; ++w) combine_into(fc, ft, fx, s_conn[w], s_tie[w], s_x[w]);
    }
}

// Decision of hub h by one workgroup of 256, from the winners of its
// partitions; afterwards the hub's counters are zero again.
__device__ void hub_decide(const EvalArgs& A, const HubArgs& H, int32_t h) {
    const int tid = threadIdx.x;
    const int32_t v = A.rows[h].node;
    const Ctx kx = ctx_of(A, v);
    const int32_t a = A.label[v];
    const int32_t p0 = H.hub_pbase[h], p1 = H.hub_pbase[h + 1];
    int32_t fc = -1, fx = -1;
    uint64_t ft = ~0ULL;
    const int32_t own = H.hub_own[h];
    constexpr int U = 4;
    for (int32_t j = p0 + tid; j < p1; j += 256 * U) {
        int32_t cn[U], x[U];
        uint64_t ti[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = j + u * 256 < p1;
            cn[u] = in ? H.w_conn[j + u * 256] : -1;
            x[u] = in ? H.w_x[j + u * 256] : -1;
            ti[u] = in ? H.w_tie[j + u * 256] : ~0ULL;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) combine_into(fc, ft, fx, cn[u], ti[u], x[u]);
    }
    block_combine(fc, ft, fx);
    if (tid == 0) store_result(A, h, fx, fc, own, A.refine && A.w[a] > kx.bound, A.vw ? A.vw[v] : 1);
    __syncthreads();  // every thread has read the counters
    for (int32_t j = p0 + tid; j < p1; j += 256) H.rcount[j] = 0;
    if (tid == 0) {
        H.ocount[h] = 0;
        H.tfill[h] = 0;
        H.hub_own[h] = 0;
    }
}

// ------------------------------------------------ dense refinement buckets
//
// During refinement a node's labels are its graph's blocks, so connections
// are summed in a dense array of dense_k entries (one LDS atomic add per
// slot, no probing) instead of a hash table.

constexpr int kDenseMax = 256;

// Adds the slots [b, b+d) of a row to conn with LDS atomics (STRIDE lanes,
// U batches of loads in flight).
template <int STRIDE>
__device__ __forceinline__ void dense_slots(const EvalArgs& A, const Ctx& kx, int64_t b, int32_t d, int32_t* conn,
                                            int lane_in_set) {
    constexpr int U = 4;
    for (int32_t j0 = lane_in_set; j0 < d; j0 += STRIDE * U) {
        int32_t x[U], wt[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t j = j0 + u * STRIDE;
            x[u] = j < d ? A.adj[b + j] : -1;
            wt[u] = j < d ? (A.ew ? A.ew[b + j] : 1) : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = x[u] >= 0 ? nbr_label(A, x[u]) - kx.lbase : -1;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (x[u] >= 0) atomicAdd(&conn[x[u]], wt[u]);
    }
}

// Best eligible block of a node from its dense connections (lane j of the
// set scans entries j, j + STEP, ..., four at a time).
template <int STEP>
__device__ __forceinline__ void dense_best(const EvalArgs& A, const Ctx& kx, const int32_t* conn, int32_t a,
                                           int32_t c, int32_t own, bool over, int first, Best& best, bool& blocked) {
    constexpr int U = 4;
    const int32_t la = a - kx.lbase;
    for (int j0 = first; j0 < A.dense_k; j0 += STEP * U) {
        int32_t x[U], cn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = j0 + u * STEP;
            cn[u] = j < A.dense_k ? conn[j] : 0;
            // not a neighbouring block, or the own one
            x[u] = cn[u] == 0 || j == la ? -1 : j + kx.lbase;
        }
        consider_group<U>(A, kx, x, cn, c, own, over, best, blocked);
    }
}

// LDS: (256 / G) * kDenseMax int32 (each group's block sums).
template <int G>
__device__ __forceinline__ void eval_dense_group_body(const EvalArgs& A, int32_t bid, int32_t* lds) {
    constexpr int NG = 256 / G;
    const int grp = threadIdx.x / G;
    const int gl = threadIdx.x % G;
    const int node_i = bid * NG + grp;
    if (node_i >= A.count) return;  // uniform per group
    const Row row = A.rows[node_i];
    if (stopped(A.gate)) return;
    const int qm = quiet_mode(A);
    int32_t* conn = lds + grp * kDenseMax;
    const int32_t v = row.node;
    const Ctx kx = ctx_of(A, v);
    if (skip_quiet(A, qm, v, kx)) {
        if (gl == 0) store_result(A, node_i, -1, 0, 0, false, 0);
        return;
    }
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    const bool over = A.w[a] > kx.bound;
    for (int32_t j = gl; j < A.dense_k; j += G) conn[j] = 0;
    wave_sync();
    dense_slots<G>(A, kx, row.begin, row.deg, conn, gl);
    wave_sync();
    const int32_t own = conn[a - kx.lbase];
    if (A.sums)
        for (int32_t j = gl; j < A.dense_k; j += G) A.sums[static_cast<int64_t>(node_i) * A.dense_k + j] = conn[j];
    Best best;
    best_init(best);
    bool blocked = false;
    dense_best<G>(A, kx, conn, a, c, own, over, gl, best, blocked);
    int32_t bx, bconn;
    uint64_t btie;
    group_argmax<G>(best, kx, bx, bconn, btie);
    const bool any_blocked = group_any<G>(blocked);
    if (gl == 0) {
        store_result(A, node_i, bx, bconn, own, over, c);
        if (qm) A.quiet[v] = (!over && !any_blocked) ? 1 : 0;
    }
}

template <int G>
__global__ void __launch_bounds__(256) eval_dense_group_kernel(EvalArgs A) {
    __shared__ int32_t lds[(256 / G) * kDenseMax];
    eval_dense_group_body<G>(A, blockIdx.x, lds);
}

// LDS: BlockScratch<NT> then kDenseMax int32 (the node's block sums).
template <int NT>
__device__ __forceinline__ void eval_dense_block_body(const EvalArgs& A, int32_t bid, unsigned char* lds) {
    BlockScratch<NT>& S = *reinterpret_cast<BlockScratch<NT>*>(lds);
    int32_t* conn = reinterpret_cast<int32_t*>(lds + sizeof(BlockScratch<NT>));
    int32_t* s_conn = S.conn;
    int32_t* s_x = S.x;
    uint64_t* s_tie = S.tie;
    const int tid = threadIdx.x;
    const int wid = tid >> 6;
    const Row row = A.rows[bid];
    if (stopped(A.gate)) return;  // uniform over the grid
    const int qm = quiet_mode(A);
    const int32_t v = row.node;
    const Ctx kx = ctx_of(A, v);
    if (skip_quiet(A, qm, v, kx)) {  // uniform over the workgroup
        if (tid == 0) store_result(A, bid, -1, 0, 0, false, 0);
        return;
    }
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    const bool over = A.w[a] > kx.bound;
    for (int32_t j = tid; j < A.dense_k; j += NT) conn[j] = 0;
    __syncthreads();
    dense_slots<NT>(A, kx, row.begin, row.deg, conn, tid);
    __syncthreads();
    const int32_t own = conn[a - kx.lbase];
    if (A.sums)
        for (int32_t j = tid; j < A.dense_k; j += NT) A.sums[static_cast<int64_t>(bid) * A.dense_k + j] = conn[j];
    Best best;
    best_init(best);
    bool blocked = false;
    dense_best<NT>(A, kx, conn, a, c, own, over, tid, best, blocked);
    int32_t bx, bconn;
    uint64_t btie;
    group_argmax<64>(best, kx, bx, bconn, btie);
    if (lane_id() == 0) {
        s_conn[wid] = bconn;
        s_x[wid] = bx;
        s_tie[wid] = btie;
    }
    const int any_blocked = __syncthreads_or(blocked);
    if (tid == 0) {
        int32_t fc = -1, fx = -1;
        uint64_t ft = ~0ULL;
        for (int w = 0; w < NT / 64; ++w) combine_into(fc, ft, fx, s_conn[w], s_tie[w], s_x[w]);
        store_result(A, bid, fx, fc, own, over, c);
        if (qm) A.quiet[v] = (!over && !any_blocked) ? 1 : 0;
    }
}

template <int NT>
__global__ void __launch_bounds__(NT) eval_dense_block_kernel(EvalArgs A) {
    __shared__ __align__(16) unsigned char lds[sizeof(BlockScratch<NT>) + kDenseMax * sizeof(int32_t)];
    eval_dense_block_body<NT>(A, blockIdx.x, lds);
}

// Hubs: every chunk of a hub's row adds its dense sums to the hub's row of
// hub_sum (dense_k entries per hub) ...
template <int NT>
__device__ __forceinline__ void hub_dense_chunk_body(const EvalArgs& A, const HubArgs& H, int32_t bid, int32_t* conn) {
    if (stopped(A.gate)) return;  // uniform over the grid
    const int tid = threadIdx.x;
    const int32_t h = H.chunk_hub[bid];
    const Row row = A.rows[h];
    const Ctx kx = ctx_of(A, row.node);
    const int64_t begin = H.chunk_begin[bid];
    const int64_t row_end = row.begin + row.deg;
    const int64_t end = begin + kHubDenseChunk < row_end ? begin + kHubDenseChunk : row_end;
    for (int32_t j = tid; j < A.dense_k; j += NT) conn[j] = 0;
    __syncthreads();
    dense_slots<NT>(A, kx, begin, static_cast<int32_t>(end - begin), conn, tid);
    __syncthreads();
    for (int32_t j = tid; j < A.dense_k; j += NT)
        if (conn[j]) atomicAdd(&H.hub_sum[static_cast<int64_t>(h) * A.dense_k + j], conn[j]);
}

__global__ void __launch_bounds__(kHubThreads) hub_dense_chunk_kernel(EvalArgs A, HubArgs H) {
    __shared__ int32_t conn[kDenseMax];
    hub_dense_chunk_body<kHubThreads>(A, H, blockIdx.x, conn);
}

// ... then a workgroup of 256 decides and clears the hub's row.
__device__ void hub_dense_decide(const EvalArgs& A, const HubArgs& H, int32_t h) {
    const int tid = threadIdx.x;
    const int32_t v = A.rows[h].node;
    const Ctx kx = ctx_of(A, v);
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    int32_t* conn = H.hub_sum + static_cast<int64_t>(h) * A.dense_k;
    const int32_t own = conn[a - kx.lbase];
    const bool over = A.w[a] > kx.bound;
    Best best;
    best_init(best);
    bool blocked = false;
    dense_best<256>(A, kx, conn, a, c, own, over, tid, best, blocked);
    int32_t fc = best.conn, fx = best.x;
    uint64_t ft = best.x >= 0 ? best_tie(best, kx) : ~0ULL;
    block_combine(fc, ft, fx);
    if (tid == 0) store_result(A, h, fx, fc, own, over, c);
    __syncthreads();  // every thread has read the row
    for (int32_t j = tid; j < A.dense_k; j += 256) {
        if (A.sums) A.sums[static_cast<int64_t>(h) * A.dense_k + j] = conn[j];
        conn[j] = 0;
    }
}

// Kept sums: where a refinement starts from a good partition few nodes move
// (levels of a power-law graph of 2^22 nodes, 64 blocks: 0.1-2.5 % of a colour's
// slots belong to nodes that move in a sub-round; a partition a tenth of whose
// nodes were placed anew: 3-10 % in the first round), so the block sums of long
// rows stay in HBM.  The first round's evaluation writes them, the neighbours of
// every node that moves are corrected (upkeep), and later rounds read dense_k
// integers per row, hubs included, instead of gathering a label per slot.  The
// sums are the same integers a new count would give.  From a bad start up to all
// of a colour's slots move, and two atomics per slot, many on the same hubs' few
// words, cost far more than a new count (power-law graph of 2^22 nodes, 10 rounds
// from 2 random blocks 14.4 ms and 5.8 without sums, from a single pool 23.6 and
// 5.1; into one of 64 random blocks 29.3 and 12.2).  After a sub-round that moved
// over a sixth of its slots no correction is made, the sums hold no longer, and
// each colour's rows are counted afresh when their turn comes (Fresh): 6.0, 6.4
// and 8.2 ms.  A sixth, because a mesh of 2^22 nodes whose 64 random blocks move an
// eighth to a seventh of the slots in most of ten rounds is corrected in 14.0 ms
// and counted afresh in 15.3.  G lanes per row, each
// with its U sums loaded before anything else is known about the row: the
// kernel is a stream of 4 * dense_k bytes per row (2^24 nodes, 512 M slots, 64
// blocks, one colour: 180 k rows in 110 us beside the short rows, where the
// gathers of those rows took 700 us).
template <int G>
__global__ void __launch_bounds__(256) eval_kept_kernel(EvalArgs A) {
    constexpr int U = 4;  // G * U >= dense_k
    const int gl = threadIdx.x % G;
    const int32_t i = static_cast<int32_t>(blockIdx.x) * (256 / G) + static_cast<int32_t>(threadIdx.x) / G;
    if (i >= A.count) return;  // uniform per group
    const Row row = A.rows[i];
    if (stopped(A.gate) || !sums_hold(A)) return;
    const int32_t* conn = A.sums + static_cast<int64_t>(i) * A.dense_k;
    int32_t cn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) cn[u] = gl + u * G < A.dense_k ? conn[gl + u * G] : 0;
    const int qm = quiet_mode(A);
    const int32_t v = row.node;
    const Ctx kx = ctx_of(A, v);
    if (skip_quiet(A, qm, v, kx)) {
        if (gl == 0) store_result(A, i, -1, 0, 0, false, 0);
        return;
    }
    const int32_t a = A.label[v];
    const int32_t c = A.vw ? A.vw[v] : 1;
    const bool over = A.w[a] > kx.bound;
    const int32_t la = a - kx.lbase;
    int32_t own = 0;
    int32_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t at = __shfl(cn[u], la % G, G);
        if (la / G == u) own = at;
        x[u] = cn[u] == 0 || gl + u * G == la ? -1 : gl + u * G + kx.lbase;
    }
    Best best;
    best_init(best);
    bool blocked = false;
    consider_group<U>(A, kx, x, cn, c, own, over, best, blocked);
    int32_t bx, bconn;
    uint64_t btie;
    group_argmax<G>(best, kx, bx, bconn, btie);
    const bool any_blocked = group_any<G>(blocked);
    if (gl == 0) {
        store_result(A, i, bx, bconn, own, over, c);
        if (qm) A.quiet[v] = (!over && !any_blocked) ? 1 : 0;
    }
}

// ------------------------------------------------- small colours, fused

// The buckets of a small colour in one launch: consecutive workgroup ranges
// belong to the buckets, the longest rows first, and each workgroup runs its
// bucket's body on an LDS buffer sized for the largest.  Separate launches, one
// after the other on one stream, cost 2.3 us each before they do any work and
// leave most of the device idle.  Hash tables: rows of up to 1 024 slots (one
// lane, 16, 32 or 64 lanes, or one 256-thread workgroup per node).  Dense
// refinement: rows of any length, hub chunks among them, since the sums take
// only dense_k entries.
constexpr int kFusedHash = 6;    // buckets 0..5
constexpr int kFusedDense = 9;   // buckets 0..7 and the hub chunks

struct FusedBuckets {
    const Row* rows[kFusedDense];
    int32_t* sums[kFusedDense];
    int32_t* ct[kFusedDense];
    int32_t* cg[kFusedDense];
    int32_t count[kFusedDense];
    int32_t end[kFusedDense];  // workgroups up to and including the bucket's, from the last bucket down
};

constexpr size_t cmax(size_t a, size_t b) { return a > b ? a : b; }
constexpr size_t kFusedLds =
    cmax(cmax(2 * 16 * (2 * kG16Max) * sizeof(int32_t), 2 * 8 * (2 * kG32Max) * sizeof(int32_t)),
         cmax(cmax(2 * 4 * kWaveTable * sizeof(int32_t), sizeof(BlockScratch<256>) + 2 * (2 * kBlock1Max) * sizeof(int32_t)),
              cmax(16 * kDenseMax * sizeof(int32_t), sizeof(BlockScratch<256>) + kDenseMax * sizeof(int32_t))));

template <bool kDense>
__device__ __forceinline__ void eval_fused_body(EvalArgs& A, const FusedBuckets& F, const HubArgs& H, int32_t block,
                                                unsigned char* lds) {
    int b = (kDense ? kFusedDense : kFusedHash) - 1;
    int32_t first = 0;
    while (b > 0 && block >= F.end[b]) first = F.end[b--];
    const int32_t bid = block - first;
    A.rows = F.rows[b];
    A.count = F.count[b];
    A.ct = F.ct[b];
    A.cg = F.cg[b];
    A.sums = F.sums[b];
    int32_t* l32 = reinterpret_cast<int32_t*>(lds);
    switch (b) {  // uniform over the workgroup
        case 0:
            eval_lane_body<kLaneSmall>(A, bid);
            break;
        case 1:
            eval_lane_body<kLaneMax>(A, bid);
            break;
        case 2:
            if (kDense) eval_dense_group_body<16>(A, bid, l32);
            else eval_group_body<16, 2 * kG16Max>(A, bid, l32);
            break;
        case 3:
            if (kDense) eval_dense_group_body<32>(A, bid, l32);
            else eval_group_body<32, 2 * kG32Max>(A, bid, l32);
            break;
        case 4:
            if (kDense) eval_dense_group_body<64>(A, bid, l32);
            else eval_group_body<64, kWaveTable>(A, bid, l32);
            break;
        case kFusedDense - 1:
            if (kDense) hub_dense_chunk_body<256>(A, H, bid, l32);
            break;
        default:
            if (kDense) eval_dense_block_body<256>(A, bid, lds);
            else eval_block_body<256, 2 * kBlock1Max, kBlock1Max / 256>(A, bid, lds);
            break;
    }
}

template <bool kDense>
__global__ void __launch_bounds__(256) eval_fused_kernel(EvalArgs A, FusedBuckets F, HubArgs H) {
    __shared__ __align__(16) unsigned char lds[kFusedLds];
    eval_fused_body<kDense>(A, F, H, blockIdx.x, lds);
}

// The rows with kept sums counted afresh, where the sums hold no longer (after
// the first round seldom: the workgroups, few enough to come and go in a
// launch's time, take the places of the buckets in turn).
constexpr int kRecountBlocks = 2048;

__global__ void __launch_bounds__(256) eval_recount_kernel(EvalArgs A, FusedBuckets F, HubArgs H, int32_t blocks) {
    __shared__ __align__(16) unsigned char lds[kFusedLds];
    if (stopped(A.gate) || sums_hold(A)) return;  // uniform over the grid
    for (int32_t block = blockIdx.x; block < blocks; block += gridDim.x) {
        eval_fused_body<true>(A, F, H, block, lds);
        __syncthreads();  // the buffer is used again
    }
}

// The rows of a small colour that need a larger table, in one launch: hub
// chunks first, then the rows of up to 8 192 and of up to 4 096 slots.  80 KB
// of LDS: two workgroups per compute unit.
constexpr size_t kBigLds = kHubLds;
constexpr int kBigTable = static_cast<int>((kBigLds - sizeof(BlockScratch<kHubThreads>)) / (2 * sizeof(int32_t)));

__global__ void __launch_bounds__(kHubThreads) eval_big_kernel(EvalArgs A, FusedBuckets F, HubArgs H) {
    __shared__ __align__(16) unsigned char lds[kBigLds];
    const int32_t bid = blockIdx.x;
    if (bid < F.end[kHubBucket]) {
        A.rows = F.rows[kHubBucket];
        hub_chunk_body(A, H, bid, lds);
        return;
    }
    const int b = bid < F.end[7] ? 7 : 6;
    A.rows = F.rows[b];
    A.count = F.count[b];
    A.ct = F.ct[b];
    A.cg = F.cg[b];
    if (b == 7) eval_block_body<kHubThreads, kBigTable, kBlockMaxDeg / kHubThreads>(A, bid - F.end[kHubBucket], lds);
    else eval_block_body<kHubThreads, 2 * kBlock2Max, kBlock2Max / kHubThreads>(A, bid - F.end[7], lds);
}

// ------------------------------------------------- candidates and admission
//
// After the evaluation a sub-round needs three launches (more only when a
// target may have more candidates than one workgroup selects):
//   accumulate  per-target weight and count of the candidates
//   admit       candidates whose target takes all of its candidates are
//               admitted, the others are written into their target's segment
//   finish      moves the admitted ones; every segment finds its target's
//               boundary and moves the entries below it
// A launch that follows another on the same stream costs about 2.3 us on this
// GPU before it does any work, and an atomic on an address that other
// workgroups also add to costs 12 ns per add (4096 adds to one address:
// 50 us; spread over 4096 addresses: 2.4 us), so the chain is short, grids
// stay at a few hundred workgroups, and sums are combined in LDS first.

// Bound of a target label: one scalar, or per graph through the label's graph.
struct Bounds {
    int64_t bound;
    const int32_t* lgid;     // [nw] graph of each label, or null
    const int64_t* g_bound;  // [G]
};

__device__ __forceinline__ int64_t bound_of(const Bounds& B, int32_t t) {
    return B.lgid ? B.g_bound[B.lgid[t]] : B.bound;
}

// Slot of label t in a block-local open-addressing table of T entries (T at
// least twice the keys a block inserts).
template <int T>
__device__ __forceinline__ int32_t agg_insert(int32_t* keys, int32_t t) {
    uint32_t h = slot_hash(static_cast<uint32_t>(t)) & (T - 1);
    while (true) {
        const int32_t k = atomicCAS(&keys[h], -1, t);
        if (k == t || k == -1) return static_cast<int32_t>(h);
        h = (h + 1) & (T - 1);
    }
}

// Label spaces up to this size (blocks of a refinement): LDS sums are indexed
// by the label itself, every workgroup lays the segments out by itself, and the
// counters all workgroups add to stand one per 128-byte line (adds to one line
// are served one after the other, some 3 ns each).  Up to kSmallLabels in large
// colours, whose 512 workgroups would otherwise each add to most of the labels,
// 16 or 32 of them in a line, for every 2048 entries (mesh of 2^22 nodes, 1 500
// blocks: totals and admission 340 us a sub-round, 76 like this); not in a
// batch, where the entries of a workgroup have few targets.
constexpr int kDirectLabels = 1024;
constexpr int64_t kDirectColour = 1 << 18;  // colours above this size
constexpr int kAccShift = 4;    // acc[t << kAccShift] (8-byte entries)
constexpr int kFillShift = 5;   // seg_fill[t << kFillShift] (4-byte entries)

// Decides the hubs of the colour (workgroup h < H.count: hub h, from what the
// evaluation launches left), and counts the candidates:
// acc[t] += (1, c(v)) over the candidates of the sub-round, summed per block
// in LDS first so that a label many nodes aim at (a hub's cluster) costs one
// global atomic per block and chunk, not one per candidate.  Each block takes
// R * 256 consecutive entries at a time.
// kLabels: label spaces up to this size are summed directly, 0: through a table.
template <int kLabels, int R>
__global__ void __launch_bounds__(256) accumulate_kernel(EvalArgs E, HubArgs H, const int32_t* __restrict__ ct,
                                                         const int32_t* __restrict__ nodes, int32_t count,
                                                         unsigned long long* __restrict__ acc, int32_t nw,
                                                         bool heavy) {
    constexpr bool kDirect = kLabels > 0;
    if (stopped(E.gate)) return;  // uniform over the grid
    const int32_t* vw = E.vw;
    if (static_cast<int32_t>(blockIdx.x) < H.count) {
        const int32_t h = blockIdx.x;
        if (sums_hold(E)) {
            // decided from its sums, with the other rows that keep theirs
        } else if (H.hub_sum) {
            hub_dense_decide(E, H, h);
        } else {
            hub_decide(E, H, h);
        }
        if (threadIdx.x == 0 && E.ct[h] >= 0) {
            const int32_t t = E.ct[h];
            const int32_t c = heavy ? 0 : vw ? vw[E.rows[h].node] : 1;
            atomicAdd(&acc[kDirect ? t << kAccShift : t], acc_of(1, c));
        }
        return;
    }
    const int32_t bid = static_cast<int32_t>(blockIdx.x) - H.count;
    const int32_t nblocks = static_cast<int32_t>(gridDim.x) - H.count;
    constexpr int T = 512 * R;
    constexpr int kSlots = kDirect ? kLabels : T;
    __shared__ int32_t keys[kDirect ? 1 : T];
    __shared__ int32_t lsum[kSlots];
    __shared__ int32_t lcnt[kSlots];
    const int32_t nslots = kDirect ? nw : T;
    for (int j = threadIdx.x; j < nslots; j += 256) {
        if (!kDirect) keys[j] = -1;
        lsum[j] = 0;
        lcnt[j] = 0;
    }
    __syncthreads();
    for (int64_t base = static_cast<int64_t>(bid) * (R * 256); base < count;
         base += static_cast<int64_t>(nblocks) * (R * 256)) {
        // all of the thread's loads of the chunk first, then the LDS updates
        int32_t tr[R], cr[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t p = base + r * 256 + threadIdx.x;
            tr[r] = p < count ? ct[p] : -1;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t p = base + r * 256 + threadIdx.x;
            cr[r] = tr[r] >= 0 && !heavy ? (vw ? vw[nodes[p]] : 1) : 0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (tr[r] < 0) continue;
            const int32_t i = kDirect ? tr[r] : agg_insert<T>(keys, tr[r]);
            if (cr[r]) atomicAdd(&lsum[i], cr[r]);
            atomicAdd(&lcnt[i], 1);
        }
        if (!kDirect) {  // flush this chunk's labels
            __syncthreads();
            const bool more = base + static_cast<int64_t>(nblocks) * (R * 256) < count;  // uniform
            for (int j = threadIdx.x; j < T; j += 256) {
                const int32_t t = keys[j];
                if (t >= 0) {
                    atomicAdd(&acc[t], acc_of(lcnt[j], lsum[j]));
                    if (more) {
                        keys[j] = -1;
                        lsum[j] = 0;
                        lcnt[j] = 0;
                    }
                }
            }
            if (more) __syncthreads();
        }
    }
    if (kDirect) {
        __syncthreads();
        for (int j = threadIdx.x; j < nw; j += 256)
            if (lcnt[j]) atomicAdd(&acc[j << kAccShift], acc_of(lcnt[j], lsum[j]));
    }
}

// A target that cannot take all its candidates: `len` entries from `base` in
// the segment arrays, of which the longest prefix in key order whose weight
// stays within `room` moves.
struct Segment {
    int32_t t, base, len, room;
};

// An entry is stored as [gain][node] and ordered by the key
// (gmax - gain) << bits_v | node (gain descending, node ascending), which is
// formed when it is read: gmax, the largest gain in a segment, is known only
// once every entry has been written.
__device__ __forceinline__ uint64_t entry_of(int32_t gain, int32_t v) {
    return (static_cast<uint64_t>(static_cast<uint32_t>(gain)) << 32) | static_cast<uint32_t>(v);
}

__device__ __forceinline__ uint64_t key_of(uint64_t e, int32_t gmax, int bits_v) {
    return (static_cast<uint64_t>(static_cast<int64_t>(gmax) - static_cast<int32_t>(e >> 32)) << bits_v) |
           (e & 0xFFFFFFFFULL);
}

__device__ __forceinline__ int32_t node_of(uint64_t e) { return static_cast<int32_t>(e & 0xFFFFFFFFULL); }

// Multi-workgroup selection for segments longer than the single-workgroup
// limit: most-significant-digit-first with kLDigit-bit digits and per-segment
// histograms in HBM. A segment is registered when its target claims it: it
// takes the next large index l and a run of kSegChunk-entry chunks.
constexpr int kLDigit = 12;
constexpr int kLBins = 1 << kLDigit;

struct LargeSel {
    int32_t* target;    // [nlarge] target of each large segment
    int32_t* base;      // [nlarge] its first entry
    int32_t* len;       // [nlarge] its entries
    int32_t* chunk0;    // [nlarge] its first chunk
    int32_t* owner;     // [nlchunks] large segment of each chunk
    uint32_t* hist;     // [nlarge][kLBins] weight per digit (heavy graphs: 64 bits each)
    uint64_t* prefix;   // [nlarge] digits fixed so far, at the end the boundary key
    int32_t* room;      // [nlarge] weight still admissible below the prefix
    uint32_t* done;     // [nlarge] chunks finished with the current digit
};

__device__ __forceinline__ int32_t seg_chunks(int32_t len) { return (len + kSegChunk - 1) / kSegChunk; }

// Per-colour admission state shared by the kernels below.
struct Admission {
    const int32_t* ct;     // per entry of the colour: target or -1
    const int32_t* cg;     // per entry: gain
    const int32_t* nodes;  // per entry: node
    int32_t count;
    const int32_t* vw;
    int32_t* w;
    int32_t nw;
    unsigned long long* acc;
    // A heavy graph's candidates may weigh more than 32 bits hold: every target
    // selects, from their count alone, and the selection sums in 64 bits.
    bool heavy;
    Bounds B;
    uint8_t* ok;
    int32_t* seg_off;   // [nw] first entry of the target's segment, -1 none, -2 being claimed
    int32_t* seg_fill;  // per label: entries written
    Segment* seg;
    uint64_t* sent;  // segment entries and their weights
    int32_t* swt;
    LargeSel L;
    int32_t small_max;  // longer segments: multi-workgroup selection
    int32_t acc_shift;   // acc[t << acc_shift], seg_fill[t << fill_shift]: kAccShift
    int32_t fill_shift;  // and kFillShift where segments are laid out directly (no seg_off then), else 0
    int bits_v;
    int32_t* label;
    uint8_t* label8;
    uint16_t* label16;
    uint16_t* prev;      // [n] label that a node left in this sub-round, else kStayed (null: not needed)
    const int64_t* xadj;  // for the slots of the nodes that moved (where prev is kept)
    uint32_t* fresh;      // the mask of Fresh: this colour's sums hold from here on (null: none are kept)
    unsigned long long fresh_limit;  // of the last sub-round, whose counters are ctr_next
    int32_t colour;
    Counters* ctr;       // this sub-round's counters
    Counters* ctr_next;  // the next sub-round's: cleared here, no kernel reads them any more
    const uint32_t* gate;
    uint32_t* round_cnt;  // candidates of the round
    uint32_t* host_cnt;   // where the round's last sub-round reports them to the host (null: not the last)
};

// A segment's room: below its candidates' weight, or no more than a label may weigh.
__device__ __forceinline__ int32_t room32(int64_t room) {
    return static_cast<int32_t>(room < INT_MAX ? room : INT_MAX);
}

// Records segment sid and, when it is longer than small_max, gives it a large
// index.
__device__ __forceinline__ void record_segment(const Admission& A, uint32_t sid, const Segment& g) {
    A.seg[sid] = g;
    if (g.len <= A.small_max) return;
    const uint32_t l = atomicAdd(&A.ctr->nlarge, 1u);
    const int32_t nch = seg_chunks(g.len);
    const int32_t c0 = static_cast<int32_t>(atomicAdd(&A.ctr->nlchunks, static_cast<uint32_t>(nch)));
    A.L.target[l] = g.t;
    A.L.base[l] = g.base;
    A.L.len[l] = g.len;
    A.L.chunk0[l] = c0;
    A.L.prefix[l] = 0;
    A.L.room[l] = g.room;
    for (int32_t c = 0; c < nch; ++c) A.L.owner[c0 + c] = static_cast<int32_t>(l);
}

// Gives target t a segment of len entries and publishes seg_off[t] last.
__device__ __forceinline__ void claim_segment(const Admission& A, int32_t t, int32_t len, int32_t room) {
    const unsigned long long at = atomicAdd(&A.ctr->segs, acc_of(1, len));
    const int32_t base = static_cast<int32_t>(at & 0xFFFFFFFFULL);
    record_segment(A, static_cast<uint32_t>(at >> 32), Segment{t, base, len, room});
    __hip_atomic_store(&A.seg_off[t], base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroup's candidates and its segment entries' gain range into the
// counters.
__device__ __forceinline__ void note_gains(const Admission& A, int32_t found, int32_t gmin, int32_t gmax) {
    __shared__ int32_t s_min[4], s_max[4], s_cnt[4];
    gmin = wave_min(gmin);
    gmax = wave_max(gmax);
    found = wave_sum(found);
    if (lane_id() == 0) {
        s_min[threadIdx.x >> 6] = gmin;
        s_max[threadIdx.x >> 6] = gmax;
        s_cnt[threadIdx.x >> 6] = found;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int32_t a = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
        const int32_t b = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
        const int32_t n = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        if (a <= b) {
            atomicMin(&A.ctr->gmin, a);
            atomicMax(&A.ctr->gmax, b);
        }
        if (n) atomicAdd(A.round_cnt, static_cast<uint32_t>(n));
    }
}

// Admits every candidate whose target takes all its candidates and writes the
// others into their targets' segments.  The first block to meet such a target
// claims its segment; a block that meets it while the claim is being
// published waits for the offset.  That wait ends: a block makes all its
// claims of a chunk, which wait for nothing, before it reads any offset, and
// a claim is published by a wave that is already running.
template <int R>
__global__ void __launch_bounds__(256) admit_kernel(Admission A) {
    constexpr int T = 512 * R;
    __shared__ int32_t keys[T];
    __shared__ int32_t lcnt[T];
    __shared__ int32_t lbase[T];  // room of the target, then its first entry for this block
    __shared__ int32_t llen[T];
    if (stopped(A.gate)) return;  // uniform over the grid
    int32_t gmin = INT_MAX, gmax = INT_MIN;
    int32_t found = 0;
    for (int64_t base = static_cast<int64_t>(blockIdx.x) * (R * 256); base < A.count;
         base += static_cast<int64_t>(gridDim.x) * (R * 256)) {
        int32_t tr[R], gr[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t p = base + r * 256 + threadIdx.x;
            tr[r] = p < A.count ? A.ct[p] : -1;
            gr[r] = p < A.count ? A.cg[p] : 0;
        }
        unsigned long long ar[R];
        int32_t wr[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ar[r] = tr[r] >= 0 ? A.acc[tr[r]] : 0;
            wr[r] = tr[r] >= 0 ? A.w[tr[r]] : 0;
        }
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t p = base + r * 256 + threadIdx.x;
            bool slow = false;
            if (tr[r] >= 0) {
                const int64_t room = bound_of(A.B, tr[r]) - static_cast<int64_t>(wr[r]);
                slow = A.heavy || static_cast<int64_t>(ar[r] & 0xFFFFFFFFULL) > room;
                wr[r] = room32(room);
                ++found;
            }
            if (p < A.count) A.ok[p] = tr[r] >= 0 && !slow ? 1 : 0;
            if (!slow) tr[r] = -1;
            any |= slow;
        }
        if (!__syncthreads_or(any)) continue;  // also: the previous chunk's table is no longer in use
        for (int j = threadIdx.x; j < T; j += 256) {
            keys[j] = -1;
            lcnt[j] = 0;
        }
        __syncthreads();
        int32_t slot[R], rank[R], vr[R], cr[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t p = base + r * 256 + threadIdx.x;
            vr[r] = tr[r] >= 0 ? A.nodes[p] : 0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            slot[r] = tr[r] >= 0 ? agg_insert<T>(keys, tr[r]) : 0;
            rank[r] = tr[r] >= 0 ? atomicAdd(&lcnt[slot[r]], 1) : 0;
            if (tr[r] >= 0) {  // the same values from every candidate of the target
                lbase[slot[r]] = wr[r];
                llen[slot[r]] = static_cast<int32_t>(ar[r] >> 32);
            }
            cr[r] = tr[r] >= 0 ? (A.vw ? A.vw[vr[r]] : 1) : 0;
        }
        __syncthreads();
        for (int j = threadIdx.x; j < T; j += 256) {
            const int32_t t = keys[j];
            if (t >= 0 && atomicCAS(&A.seg_off[t], -1, -2) == -1) claim_segment(A, t, llen[j], lbase[j]);
        }
        __syncthreads();
        for (int j = threadIdx.x; j < T; j += 256) {
            const int32_t t = keys[j];
            if (t < 0) continue;
            int32_t o = __hip_atomic_load(&A.seg_off[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while (o < 0) {
                __builtin_amdgcn_s_sleep(1);
                o = __hip_atomic_load(&A.seg_off[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            lbase[j] = o + atomicAdd(&A.seg_fill[t], lcnt[j]);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (tr[r] < 0) continue;
            const int32_t at = lbase[slot[r]] + rank[r];
            A.sent[at] = entry_of(gr[r], vr[r]);
            A.swt[at] = cr[r];
            gmin = gr[r] < gmin ? gr[r] : gmin;
            gmax = gr[r] > gmax ? gr[r] : gmax;
        }
    }
    note_gains(A, found, gmin, gmax);
}

// The same for at most kLabels labels: the segments' layout follows from
// the candidate totals alone (a prefix sum over the labels), so every
// workgroup computes it, claims and waits are not needed, and each workgroup
// reserves its entries of a segment once, for a whole run of the colour.  With
// claims and a reservation per 2048 entries, 500 workgroups adding to the same
// 64 or 100 labels took 74-128 us a sub-round on R-MAT 2^21 and 2^24.
template <int kLabels>
__global__ void __launch_bounds__(256) admit_direct_kernel(Admission A) {
    constexpr int kPer = kLabels / 256;
    __shared__ int32_t lcnt[kLabels];
    __shared__ int32_t lbase[kLabels];  // first entry of the label's segment, -1: takes all its candidates
    __shared__ unsigned long long s_wave[4];
    if (stopped(A.gate)) return;  // uniform over the grid
    const int tid = threadIdx.x;
    // thread tid: labels kPer * tid ..
    unsigned long long mine = 0;  // segments (high word) and their entries
    Segment g[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int32_t t = kPer * tid + q;
        g[q] = Segment{t, 0, 0, 0};
        if (t >= A.nw) continue;
        const unsigned long long a = A.acc[t << kAccShift];
        if (a == 0) continue;
        const int64_t room = bound_of(A.B, t) - static_cast<int64_t>(A.w[t]);
        if (!A.heavy && static_cast<int64_t>(a & 0xFFFFFFFFULL) <= room) continue;
        g[q].len = static_cast<int32_t>(a >> 32);
        g[q].room = room32(room);
        mine += acc_of(1, g[q].len);
    }
    unsigned long long incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long u = shfl_up_u64(incl, o);
        if (lane_id() >= o) incl += u;
    }
    if (lane_id() == 63) s_wave[tid >> 6] = incl;
    __syncthreads();
    unsigned long long run = incl - mine, total = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        run += q < (tid >> 6) ? s_wave[q] : 0;
        total += s_wave[q];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        g[q].base = static_cast<int32_t>(run & 0xFFFFFFFFULL);
        lcnt[kPer * tid + q] = 0;
        lbase[kPer * tid + q] = g[q].len ? g[q].base : -1;
        if (g[q].len) {
            if (blockIdx.x == 0) record_segment(A, static_cast<uint32_t>(run >> 32), g[q]);
            run += acc_of(1, g[q].len);
        }
    }
    if (blockIdx.x == 0 && tid == 0) A.ctr->segs = total;
    __syncthreads();
    // this workgroup's run of the colour, U entries per thread at a time
    constexpr int U = 4;
    const int64_t per = ((A.count + gridDim.x - 1) / gridDim.x + 255) / 256 * 256;
    const int64_t p_begin = blockIdx.x * per + tid;
    const int64_t p_end = blockIdx.x * per + per < A.count ? blockIdx.x * per + per : A.count;
    bool any = false;
    int32_t found = 0;
    for (int64_t p0 = p_begin; p0 < p_end; p0 += 256 * U) {
        int32_t tr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) tr[u] = p0 + u * 256 < p_end ? A.ct[p0 + u * 256] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (p0 + u * 256 >= p_end) continue;
            const bool slow = tr[u] >= 0 && lbase[tr[u]] >= 0;
            A.ok[p0 + u * 256] = tr[u] >= 0 && !slow ? 1 : 0;
            if (slow) atomicAdd(&lcnt[tr[u]], 1);
            any |= slow;
            found += tr[u] >= 0;
        }
    }
    any = __syncthreads_or(any);
    for (int j = tid; any && j < A.nw; j += 256) {
        const int32_t c = lcnt[j];
        if (c) lbase[j] += atomicAdd(&A.seg_fill[j << kFillShift], c);
        lcnt[j] = 0;
    }
    __syncthreads();
    int32_t gmin = INT_MAX, gmax = INT_MIN;
    for (int64_t p0 = p_begin; any && p0 < p_end; p0 += 256 * U) {
        int32_t tr[U], gr[U], vr[U], cr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            tr[u] = p0 + u * 256 < p_end ? A.ct[p0 + u * 256] : -1;
            if (tr[u] >= 0 && lbase[tr[u]] < 0) tr[u] = -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            gr[u] = tr[u] >= 0 ? A.cg[p0 + u * 256] : 0;
            vr[u] = tr[u] >= 0 ? A.nodes[p0 + u * 256] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) cr[u] = tr[u] >= 0 ? (A.vw ? A.vw[vr[u]] : 1) : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (tr[u] < 0) continue;
            const int32_t at = lbase[tr[u]] + atomicAdd(&lcnt[tr[u]], 1);
            A.sent[at] = entry_of(gr[u], vr[u]);
            A.swt[at] = cr[u];
            gmin = gr[u] < gmin ? gr[u] : gmin;
            gmax = gr[u] > gmax ? gr[u] : gmax;
        }
    }
    note_gains(A, found, gmin, gmax);
}

__device__ __forceinline__ int bits_of(uint64_t x) { return x ? 64 - __clzll(static_cast<long long>(x)) : 0; }

// Bits of the sub-round's keys: the gain range, then the node id.
__device__ __forceinline__ int key_bits(const Counters* ctr, int bits_v) {
    return bits_of(static_cast<uint64_t>(static_cast<int64_t>(ctr->gmax) - ctr->gmin)) + bits_v;
}

// Sums of candidates' weights, and the histogram bins they are summed in: 32 bits
// (the weights sum to at most 2^31 - 1), for heavy graphs 64.
template <bool kHeavy>
struct Sums {
    using S = int32_t;
    using Bin = uint32_t;
};
template <>
struct Sums<true> {
    using S = int64_t;
    using Bin = unsigned long long;
};

// Boundary digit of a histogram held as kPerT consecutive digits per thread
// (hv): the first digit whose cumulative weight exceeds room (the last digit
// when none below it does); *s_d and *s_run (the weight of the digits before
// it) are set for the whole block.  S: the type of the weight sums (Sums).
template <int NT, int kPerT, typename S>
__device__ __forceinline__ void block_pick_digit(const S* hv, int32_t room, S* s_wave, int* s_d, int32_t* s_run) {
    const int j = threadIdx.x;
    const int lane = lane_id();
    S local = 0;
#pragma unroll
    for (int q = 0; q < kPerT; ++q) local += hv[q];
    S incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const S u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) s_wave[j >> 6] = incl;
    __syncthreads();
    S before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
        const S x = s_wave[q];
        before += q < (j >> 6) ? x : 0;
        total += x;
    }
    incl += before;
    const S excl = incl - local;
    // the digit where the admissible weight runs out (monotone: one thread),
    // else the last digit
    if (total <= room) {
        if (j == NT - 1) {
            *s_d = NT * kPerT - 1;
            *s_run = static_cast<int32_t>(incl - hv[kPerT - 1]);  // at most room, here and below
        }
    } else if (incl > room && excl <= room) {
        S run = excl;
        int d = kPerT * j + kPerT - 1;
        for (int q = 0; q < kPerT - 1; ++q) {
            if (run + hv[q] > room) {
                d = kPerT * j + q;
                break;
            }
            run += hv[q];
        }
        *s_d = d;
        *s_run = static_cast<int32_t>(run);
    }
    __syncthreads();
}

// One digit of the multi-workgroup selection per launch, most significant
// first: launch j of nlaunch handles digit passes - 1 - j.  Every block adds
// its chunk's weight histogram to the segment's histogram in HBM; the last
// block to finish a segment picks that segment's boundary digit (no block
// waits for another).  Keys rarely need more digits than the host launches;
// when they do, the last block of each segment in the final launch finishes
// the remaining digits alone, over the whole segment.  After the last digit
// L.prefix holds the segment's boundary key.
template <bool kHeavy>
__global__ void __launch_bounds__(kLargeThreads) large_pass_kernel(LargeSel L, int launch, int nlaunch, int bits_v,
                                                                   const uint64_t* __restrict__ sent,
                                                                   const int32_t* __restrict__ swt,
                                                                   const Counters* ctr) {
    constexpr int NT = kLargeThreads;
    constexpr int kPerT = kLBins / NT;
    constexpr int U = 4;
    using S = typename Sums<kHeavy>::S;
    using Bin = typename Sums<kHeavy>::Bin;
    __shared__ Bin h[kLBins];
    __shared__ S s_wave[NT / 64];
    __shared__ int s_last, s_d;
    __shared__ int32_t s_run;
    const int total_bits = key_bits(ctr, bits_v);
    const int32_t gmax = ctr->gmax;
    const int passes = total_bits > 0 ? (total_bits + kLDigit - 1) / kLDigit : 1;
    const int pass = passes - 1 - launch;
    const uint32_t nlarge = ctr->nlarge;
    if (pass < 0 || nlarge == 0) return;  // uniform over the grid
    const bool finish = launch == nlaunch - 1;
    const int shift = kLDigit * pass;
    const uint64_t above = shift + kLDigit >= 64 ? 0ULL : ~0ULL << (shift + kLDigit);  // digits already fixed
    const int32_t nch = static_cast<int32_t>(ctr->nlchunks);
    const int j = threadIdx.x;
    // adds the weights of entries [i0, i1) of a segment whose key matches
    // prefix on the digits above `sh` to the LDS histogram of digit `sh`
    auto accumulate = [&](int32_t base, int32_t i0, int32_t i1, uint64_t prefix, uint64_t ab, int sh) {
        for (int32_t i = i0 + j; i < i1; i += NT * U) {
            uint64_t k[U];
            int32_t wt[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t x = i + u * NT;
                k[u] = x < i1 ? sent[base + x] : 0;
                wt[u] = x < i1 ? swt[base + x] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t key = key_of(k[u], gmax, bits_v);
                if (wt[u] && (key & ab) == prefix)
                    atomicAdd(&h[(key >> sh) & (kLBins - 1)], static_cast<Bin>(wt[u]));
            }
        }
    };
    for (int32_t c = blockIdx.x; c < nch; c += gridDim.x) {
        const int32_t l = L.owner[c];
        const int32_t base = L.base[l];
        const int32_t len = L.len[l];
        const int32_t i0 = (c - L.chunk0[l]) * kSegChunk;
        const int32_t i1 = i0 + kSegChunk < len ? i0 + kSegChunk : len;
        const uint64_t prefix = L.prefix[l];
        Bin* hl = reinterpret_cast<Bin*>(L.hist) + static_cast<size_t>(l) * kLBins;
        for (int q = j; q < kLBins; q += NT) h[q] = 0;
        __syncthreads();
        accumulate(base, i0, i1, prefix, above, shift);
        __syncthreads();
        for (int q = j; q < kLBins; q += NT)
            if (h[q]) atomicAdd(&hl[q], h[q]);
        // the barrier orders every thread's adds before thread 0's release
        // fence, and thread 0's acquire fence before every thread's reads (a
        // device-scope fence writes back and invalidates the L2, so one
        // thread issues it, not every wave)
        __syncthreads();
        if (j == 0) {
            const uint32_t nchunks = static_cast<uint32_t>(seg_chunks(len));
            __threadfence();
            const bool last = atomicAdd(&L.done[l], 1u) == nchunks - 1;
            if (last) __threadfence();
            s_last = last;
        }
        __syncthreads();
        if (s_last) {  // block-uniform
            // thread j holds digits kPerT*j .. kPerT*j + kPerT-1
            S hv[kPerT];
#pragma unroll
            for (int q = 0; q < kPerT; ++q)
                hv[q] = static_cast<S>(
                    __hip_atomic_load(&hl[kPerT * j + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            int32_t room = L.room[l];
            block_pick_digit<NT, kPerT>(hv, room, s_wave, &s_d, &s_run);
#pragma unroll
            for (int q = 0; q < kPerT; ++q) hl[kPerT * j + q] = 0;
            uint64_t np = prefix | (static_cast<uint64_t>(s_d) << shift);
            room -= s_run;
            if (finish) {
                for (int q2 = pass - 1; q2 >= 0; --q2) {  // remaining digits, this block alone
                    const int sh = kLDigit * q2;
                    __syncthreads();
                    for (int q = j; q < kLBins; q += NT) h[q] = 0;
                    __syncthreads();
                    accumulate(base, 0, len, np, ~0ULL << (sh + kLDigit), sh);
                    __syncthreads();
#pragma unroll
                    for (int q = 0; q < kPerT; ++q) hv[q] = static_cast<S>(h[kPerT * j + q]);
                    block_pick_digit<NT, kPerT>(hv, room, s_wave, &s_d, &s_run);
                    np |= static_cast<uint64_t>(s_d) << sh;
                    room -= s_run;
                }
            }
            if (j == 0) {
                L.room[l] = room;
                L.prefix[l] = np;
                L.done[l] = 0;
            }
        }
        __syncthreads();
    }
}

// The per-sub-round counters back to their empty state.
__device__ __forceinline__ void clear_subround(Counters* ctr) {
    ctr->segs = 0;
    ctr->gmin = INT_MAX;
    ctr->gmax = INT_MIN;
    ctr->nlarge = 0;
    ctr->nlchunks = 0;
    ctr->nlong = 0;
    ctr->moved = 0;
}

// Moves node v (weight c) to label t.  The departure goes to delta (LDS, small
// label spaces) or to the label's weight; the caller books the arrivals.
template <bool kSmall>
__device__ __forceinline__ void depart_and_move(const Admission& A, int32_t v, int32_t a, int32_t t, int32_t c,
                                                int32_t* delta) {
    A.label[v] = t;
    if (A.prev) A.prev[v] = static_cast<uint16_t>(a);
    if (A.label8) A.label8[v] = static_cast<uint8_t>(t);
    if (A.label16) A.label16[v] = static_cast<uint16_t>(t);
    if (c) {
        if (kSmall) atomicSub(&delta[a], c);
        else atomicSub(&A.w[a], c);
    }
}

// Slots of a node that moved, where they are counted.  They only decide how the
// next sub-rounds come by the sums, so a thread looks one of its nodes up and
// takes the others it moves at the same time for as long: two more reads per
// moved node took 15 us of a launch that moves 120 000.
__device__ __forceinline__ int64_t moved_slots(const Admission& A, int32_t v) {
    return A.prev ? A.xadj[v + 1] - A.xadj[v] : 0;
}

// Adds the workgroup's moved slots up (nothing where they are not counted).
template <int NT>
__device__ __forceinline__ void note_moved(const Admission& A, int64_t moved) {
    if (!A.prev) return;  // uniform over the grid
    __shared__ int64_t s_moved[NT / 64];
    moved = wave_sum(moved);
    if (lane_id() == 0) s_moved[threadIdx.x >> 6] = moved;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < NT / 64; ++w) moved += s_moved[w];
    if (moved) atomicAdd(&A.ctr->moved, static_cast<unsigned long long>(moved));
}

template <bool kSmall>
__device__ __forceinline__ void arrive(const Admission& A, int32_t t, int32_t c, int32_t* delta) {
    if (!c) return;
    if (kSmall) atomicAdd(&delta[t], c);
    else atomicAdd(&A.w[t], c);
}

constexpr int kFinishThreads = 1024;
constexpr int kFinishMax = 65536;  // longest segment one workgroup of finish_kernel selects from
// workgroups for the segments and (at most) for the admitted candidates; in
// small label spaces every workgroup adds to the same few lines of weights, so
// fewer move, and no more select than there are labels, each with one segment
// at most (mesh of 2^22 nodes, 5 rounds, 300, 1 000 and 5 000 blocks with a
// segment each: 9.0, 11.0 and 15.2 ms with 32 to 96 selecting workgroups, 7.5,
// 8.0 and 12.3 like this; refinement of 2^21 nodes into 100 blocks 7.52 -> 7.34)
constexpr int kSegBlocks = 256;
constexpr int kMoveBlocks = 192;
constexpr int kSegBlocksSmall = 32;
constexpr int kMoveBlocksSmall = 64;

// Moves the admitted candidates, and selects and moves the admitted prefix of
// every segment of up to small_max entries: the entries whose inclusive
// weight prefix in key order stays within the target's room (node weights are
// >= 0, so those are exactly the ones below the first that does not fit).
// Up to 64 entries: one wave, every lane sums the entries not above its own.
// Longer ones: the workgroup finds the boundary key most significant digit
// first, 12 bits at a time, in an LDS histogram, and moves what is below it.
// Segments hold 2-50 entries in most sub-rounds and thousands in the first
// ones; one launch for all lengths replaced a scatter, a selection and an
// apply launch of about 5 us each.
template <bool kSmall, bool kHeavy>
__global__ void __launch_bounds__(kFinishThreads) finish_kernel(Admission A, uint32_t seg_blocks) {
    constexpr int NT = kFinishThreads;
    constexpr int kPerT = kLBins / NT;
    using S = typename Sums<kHeavy>::S;
    using Bin = typename Sums<kHeavy>::Bin;
    __shared__ Bin hist[kLBins];
    __shared__ int32_t delta[kSmall ? kSmallLabels : 1];
    __shared__ S s_wave[NT / 64];
    __shared__ int s_d;
    __shared__ int32_t s_run;
    const int tid = threadIdx.x;
    if (A.host_cnt && blockIdx.x == 0 && tid == 0) *A.host_cnt = *A.round_cnt;
    if (stopped(A.gate)) return;  // uniform over the grid: nothing was counted either
    const int lane = lane_id();
    if (blockIdx.x == 0 && tid == 0) {
        // before this sub-round's moves, which its counters tell the next one
        if (A.fresh) *A.fresh = fresh_mask(Fresh{A.fresh, A.ctr_next, A.fresh_limit}) | (1u << A.colour);
        clear_subround(A.ctr_next);
    }
    int64_t moved = 0;
    if (kSmall) {
        for (int j = tid; j < A.nw; j += NT) delta[j] = 0;
        __syncthreads();
    }
    // the first workgroups take the segments, the others the admitted
    // candidates: both are chains of dependent reads, which then overlap
    const bool takes_segs = blockIdx.x < seg_blocks;
    const uint32_t nseg = takes_segs ? static_cast<uint32_t>(A.ctr->segs >> 32) : 0;
    const int32_t gmax = A.ctr->gmax;
    // segments of up to 64 entries, one wave each (bookkeeping of the others)
    for (uint32_t sid = blockIdx.x * (NT / 64) + __builtin_amdgcn_readfirstlane(tid >> 6); sid < nseg;
         sid += seg_blocks * (NT / 64)) {
        const Segment sg = A.seg[sid];
        if (lane == 0) {
            if (A.seg_off) A.seg_off[sg.t] = -1;
            A.seg_fill[sg.t << A.fill_shift] = 0;
        }
        if (sg.len > 64 || sg.len > A.small_max) continue;
        const uint64_t e = lane < sg.len ? A.sent[sg.base + lane] : 0;
        const int32_t c = lane < sg.len ? A.swt[sg.base + lane] : 0;
        const int32_t v = node_of(e);
        const int32_t a = lane < sg.len ? A.label[v] : 0;
        const uint64_t k = key_of(e, gmax, A.bits_v);
        S incl = 0;
        for (int j = 0; j < sg.len; ++j) {
            const uint32_t klo = __builtin_amdgcn_readlane(static_cast<uint32_t>(k), j);
            const uint32_t khi = __builtin_amdgcn_readlane(static_cast<uint32_t>(k >> 32), j);
            const int32_t cj = static_cast<int32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(c), j));
            incl += ((static_cast<uint64_t>(khi) << 32) | klo) <= k ? cj : 0;
        }
        const bool in = lane < sg.len && incl <= sg.room;
        if (in) {
            moved += moved_slots(A, v);
            depart_and_move<kSmall>(A, v, a, sg.t, c, delta);
        }
        const int32_t sum = wave_sum(in ? c : 0);
        if (lane == 0) arrive<kSmall>(A, sg.t, sum, delta);
    }
    // longer ones, one workgroup each
    const int total_bits = key_bits(A.ctr, A.bits_v);
    const int passes = total_bits > 0 ? (total_bits + kLDigit - 1) / kLDigit : 1;
    for (uint32_t sid = blockIdx.x; sid < nseg; sid += seg_blocks) {
        const Segment sg = A.seg[sid];
        if (sg.len <= 64 || sg.len > A.small_max) continue;  // uniform over the workgroup
        // the first entry per thread stays in registers over the passes
        const uint64_t e0 = tid < sg.len ? A.sent[sg.base + tid] : 0;
        const int32_t c0 = tid < sg.len ? A.swt[sg.base + tid] : 0;
        const uint64_t k0 = key_of(e0, gmax, A.bits_v);
        uint64_t np = 0;
        int32_t room = sg.room;
        for (int pass = passes - 1; pass >= 0; --pass) {
            const int sh = kLDigit * pass;
            const uint64_t above = sh + kLDigit >= 64 ? 0ULL : ~0ULL << (sh + kLDigit);
            for (int q = tid; q < kLBins; q += NT) hist[q] = 0;
            __syncthreads();
            if (c0 && (k0 & above) == np) atomicAdd(&hist[(k0 >> sh) & (kLBins - 1)], static_cast<Bin>(c0));
            constexpr int U = 4;
            for (int32_t i = tid + NT; i < sg.len; i += NT * U) {
                uint64_t e[U];
                int32_t c[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t x = i + u * NT;
                    e[u] = x < sg.len ? A.sent[sg.base + x] : 0;
                    c[u] = x < sg.len ? A.swt[sg.base + x] : 0;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint64_t k = key_of(e[u], gmax, A.bits_v);
                    if (c[u] && (k & above) == np)
                        atomicAdd(&hist[(k >> sh) & (kLBins - 1)], static_cast<Bin>(c[u]));
                }
            }
            __syncthreads();
            S hv[kPerT];
#pragma unroll
            for (int q = 0; q < kPerT; ++q) hv[q] = static_cast<S>(hist[kPerT * tid + q]);
            block_pick_digit<NT, kPerT>(hv, room, s_wave, &s_d, &s_run);
            np |= static_cast<uint64_t>(s_d) << sh;
            room -= s_run;
            __syncthreads();  // s_d, s_run and hist are written again by the next pass
        }
        int32_t sum = 0, cnt = 0;
        int64_t slots = 0;
        for (int32_t i = tid; i < sg.len; i += NT) {
            const uint64_t e = i == tid ? e0 : A.sent[sg.base + i];
            if (key_of(e, gmax, A.bits_v) >= np) continue;
            const int32_t c = i == tid ? c0 : A.swt[sg.base + i];
            const int32_t v = node_of(e);
            const int32_t a = A.label[v];
            if (cnt++ == 0) slots = moved_slots(A, v);
            depart_and_move<kSmall>(A, v, a, sg.t, c, delta);
            sum += c;
        }
        moved += slots * cnt;
        sum = wave_sum(sum);
        if (lane == 0) arrive<kSmall>(A, sg.t, sum, delta);
    }
    // admitted candidates, U grid-stride positions per thread at a time: their
    // loads are issued together, level by level, before the updates
    constexpr int U = 4;
    const int64_t stride = static_cast<int64_t>(gridDim.x - seg_blocks) * NT;
    for (int64_t p0 = takes_segs ? A.count : static_cast<int64_t>(blockIdx.x - seg_blocks) * NT + tid; p0 < A.count;
         p0 += stride * U) {
        int32_t tq[U], vq[U], aq[U], cq[U];
        bool oq[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * stride;
            tq[u] = p < A.count ? A.ct[p] : -1;
            oq[u] = p < A.count && A.ok[p];
            vq[u] = p < A.count ? A.nodes[p] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            aq[u] = oq[u] ? A.label[vq[u]] : 0;
            cq[u] = oq[u] ? (A.vw ? A.vw[vq[u]] : 1) : 0;
        }
        int32_t cnt = 0, v1 = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v1 = oq[u] ? vq[u] : v1;
            cnt += oq[u];
        }
        const int64_t slots = cnt ? moved_slots(A, v1) : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (tq[u] < 0) continue;
            A.acc[tq[u] << A.acc_shift] = 0;
            if (!oq[u]) continue;
            depart_and_move<kSmall>(A, vq[u], aq[u], tq[u], cq[u], delta);
            arrive<kSmall>(A, tq[u], cq[u], delta);
        }
        moved += slots * cnt;
    }
    note_moved<NT>(A, moved);
    if (kSmall) {
        __syncthreads();
        for (int j = tid; j < A.nw; j += NT)
            if (delta[j]) atomicAdd(&A.w[j], delta[j]);
    }
}

// Moves the admitted prefix of the segments selected by large_pass_kernel.
template <bool kSmall>
__global__ void __launch_bounds__(256) large_move_kernel(Admission A) {
    __shared__ int32_t delta[kSmall ? kSmallLabels : 1];
    if (A.ctr->nlarge == 0) return;  // uniform over the grid
    if (kSmall) {
        for (int j = threadIdx.x; j < A.nw; j += 256) delta[j] = 0;
        __syncthreads();
    }
    const int32_t gmax = A.ctr->gmax;
    int64_t moved = 0;
    const int32_t nch = static_cast<int32_t>(A.ctr->nlchunks);
    constexpr int kParts = kSegChunk / 1024;  // a workgroup takes 1024 entries of a chunk at a time
    for (int32_t cp = blockIdx.x; cp < nch * kParts; cp += gridDim.x) {
        const int32_t c = cp / kParts;
        const int32_t l = A.L.owner[c];
        const int32_t base = A.L.base[l];
        const int32_t i0 = (c - A.L.chunk0[l]) * kSegChunk + (cp % kParts) * 1024;
        const int32_t i1 = min(i0 + 1024, A.L.len[l]);
        const uint64_t end = A.L.prefix[l];
        const int32_t t = A.L.target[l];
        int32_t sum = 0, cnt = 0;
        int64_t slots = 0;
        for (int32_t i = i0 + static_cast<int32_t>(threadIdx.x); i < i1; i += 256) {
            const uint64_t e = A.sent[base + i];
            if (key_of(e, gmax, A.bits_v) >= end) continue;
            const int32_t wt = A.swt[base + i];
            const int32_t v = node_of(e);
            const int32_t a = A.label[v];
            if (cnt++ == 0) slots = moved_slots(A, v);
            depart_and_move<kSmall>(A, v, a, t, wt, delta);
            sum += wt;
        }
        moved += slots * cnt;
        sum = wave_sum(sum);
        if (lane_id() == 0) arrive<kSmall>(A, t, sum, delta);
    }
    note_moved<256>(A, moved);
    if (kSmall) {
        __syncthreads();
        for (int j = threadIdx.x; j < A.nw; j += 256)
            if (delta[j]) atomicAdd(&A.w[j], delta[j]);
    }
}

// Admission state before the first sub-round: no candidates, no segments, no
// large segments in progress, no candidates counted in any round; and the
// narrow copy of the labels, if one is kept.
__global__ void __launch_bounds__(256) init_admission_kernel(unsigned long long* __restrict__ acc,
                                                             int64_t acc_n, int32_t* __restrict__ seg_off,
                                                             int64_t off_n, int32_t* __restrict__ seg_fill,
                                                             int64_t fill_n,
                                                             uint32_t* __restrict__ lhist, int64_t lhist_n,
                                                             uint32_t* __restrict__ ldone, int64_t ldone_n,
                                                             uint32_t* __restrict__ rcnt, int32_t rounds,
                                                             Counters* ctr, const int32_t* __restrict__ label,
                                                             int32_t n, uint8_t* __restrict__ label8,
                                                             uint16_t* __restrict__ label16) {
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t i = i0; i < acc_n; i += stride) acc[i] = 0;
    for (int64_t i = i0; i < off_n; i += stride) seg_off[i] = -1;
    for (int64_t i = i0; i < fill_n; i += stride) seg_fill[i] = 0;
    for (int64_t i = i0; i < lhist_n; i += stride) lhist[i] = 0;
    for (int64_t i = i0; i < ldone_n; i += stride) ldone[i] = 0;
    for (int64_t i = i0; i < rounds; i += stride) rcnt[i] = 0;
    if (label8)
        for (int64_t i = i0; i < n; i += stride) label8[i] = static_cast<uint8_t>(label[i]);
    if (label16)
        for (int64_t i = i0; i < n; i += stride) label16[i] = static_cast<uint16_t>(label[i]);
    if (i0 == 0) {
        clear_subround(ctr);
        clear_subround(ctr + 1);
    }
}

// After a sub-round: every neighbour of a node that moved is no longer quiet.
// A workgroup lays the rows of the movers among its 256 schedule entries end to
// end and takes a slot per thread: a wave that walked one mover's row after the
// other waited for two dependent reads per mover (64 graphs of a batch: 11.1 -> 8.2 us
// per launch, hubs among the movers).
__global__ void __launch_bounds__(256) unquiet_kernel(const int32_t* __restrict__ ct,
                                                      const int32_t* __restrict__ label,
                                                      const int32_t* __restrict__ nodes, int32_t count,
                                                      const int64_t* __restrict__ xadj,
                                                      const int32_t* __restrict__ adj, uint8_t* __restrict__ quiet,
                                                      const uint32_t* __restrict__ gate,
                                                      const uint32_t* __restrict__ rcnt, int32_t round, int32_t qn) {
    __shared__ int64_t s_pre[256], s_begin[256], s_wave[4];
    if (stopped(gate) || quiet_mode(quiet, rcnt, round, qn) == 0) return;  // uniform over the grid
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wid = tid >> 6;
    const int64_t p = static_cast<int64_t>(blockIdx.x) * 256 + tid;
    // a candidate that holds its target label now (its own differed before)
    const int32_t t = p < count ? ct[p] : -1;
    const int32_t v = t >= 0 ? nodes[p] : 0;
    const bool mover = t >= 0 && label[v] == t;
    if (!__syncthreads_or(mover)) return;
    const int64_t b = mover ? xadj[v] : 0;
    const int64_t d = mover ? xadj[v + 1] - b : 0;
    int64_t incl = d;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t x = static_cast<int64_t>(shfl_up_u64(static_cast<uint64_t>(incl), o));
        if (lane >= o) incl += x;
    }
    if (lane == 63) s_wave[wid] = incl;
    __syncthreads();
    int64_t before = incl - d, total = 0;
    for (int w = 0; w < 4; ++w) {
        if (w < wid) before += s_wave[w];
        total += s_wave[w];
    }
    s_pre[tid] = before;
    s_begin[tid] = b;
    __syncthreads();
    constexpr int U = 4;
    for (int64_t j0 = tid; j0 < total; j0 += 256 * U) {
        int32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = j0 + u * 256;
            int lo = 0;  // the last entry whose slots begin at or before this one
#pragma unroll
            for (int step = 128; step > 0; step >>= 1)
                if (s_pre[lo + step] <= at) lo += step;
            x[u] = at < total ? adj[s_begin[lo] + (at - s_pre[lo])] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (x[u] >= 0) quiet[x[u]] = 0;
    }
}

// ----------------------------------------------------- upkeep of kept sums

// After a sub-round, on the way to the next one's evaluation: the nodes that
// moved are found by their entries of prev (a stream of 2 bytes per node) and
// each of their slots corrects two sums of the neighbour at its end, if that
// keeps sums.  A workgroup lays the rows of its movers end to end and takes a
// slot per thread, since most movers have a handful; rows over kUpkeepLong
// slots become chunks for a second launch, so that no workgroup is left with
// a hub (20 M slots per colour, first later rounds: 49 + 23 -> 20 + 11 us).
// Two dependent reads and two atomics per slot; on random lines those ran at
// 18 G/s.

// Index of every scheduled node's kept sums with its colour above, -1 for short
// rows; the colours' kept rows follow each other.
constexpr int kKeptBits = 27;

struct KeptRanges {
    int32_t nsub;
    int32_t from[16], to[16];  // schedule positions of each colour's kept rows
    int32_t base[16];          // index of the first
    int32_t end[16];           // schedule position after the colour
};

__global__ void __launch_bounds__(256) kept_index_kernel(KeptRanges K, const int32_t* __restrict__ nodes, int32_t count,
                                                         int32_t* __restrict__ kidx) {
    const int32_t p = static_cast<int32_t>(blockIdx.x) * 256 + static_cast<int32_t>(threadIdx.x);
    if (p >= count) return;
    int sc = 0;
    while (sc < K.nsub - 1 && p >= K.end[sc]) ++sc;
    kidx[nodes[p]] = p >= K.from[sc] && p < K.to[sc] ? (sc << kKeptBits) | (K.base[sc] + (p - K.from[sc])) : -1;
}

constexpr uint32_t kStayed = 0xFFFF;
constexpr int kUpkeepPer = 8;           // nodes per thread: one 16-byte load of prev
constexpr int kUpkeepLong = 1024;       // longer rows are cut into chunks of this many slots

struct Upkeep {
    int32_t n;
    uint16_t* prev;
    const int32_t* label;
    const int64_t* xadj;
    const int32_t* adj;
    const int32_t* ew;
    const int32_t* gid;
    const int32_t* g_lbase;
    const int32_t* kidx;
    Fresh fresh;
    int32_t* sums;
    int32_t k;
    int4* chunks;  // node, old label, new label, chunk
    Counters* ctr;
    const uint32_t* gate;
};

// U slots of rows whose nodes moved from block `from` to `to` (slot -1: none).
template <int U>
__device__ __forceinline__ void upkeep_slots(const Upkeep& K, uint32_t fresh, const int64_t* slot, const int32_t* from,
                                             const int32_t* to) {
    int32_t v[U], wt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        v[u] = slot[u] >= 0 ? K.adj[slot[u]] : -1;
        wt[u] = slot[u] >= 0 && K.ew ? K.ew[slot[u]] : 1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = v[u] >= 0 ? K.kidx[v[u]] : -1;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        // rows whose sums do not hold are left alone: they may be being counted
        if (v[u] < 0 || !((fresh >> (v[u] >> kKeptBits)) & 1u)) continue;
        int32_t* conn = K.sums + static_cast<int64_t>(v[u] & ((1 << kKeptBits) - 1)) * K.k;
        atomicSub(&conn[from[u]], wt[u]);
        atomicAdd(&conn[to[u]], wt[u]);
    }
}

__global__ void __launch_bounds__(256) upkeep_kernel(Upkeep K) {
    constexpr int kNodes = 256 * kUpkeepPer;
    __shared__ int32_t s_node[kNodes];
    __shared__ uint16_t s_from[kNodes];
    __shared__ int64_t s_begin[256];
    __shared__ int32_t s_pre[256], s_f[256], s_t[256];
    __shared__ int32_t s_wave[4];
    if (stopped(K.gate)) return;  // uniform over the grid
    const uint32_t fresh = fresh_mask(K.fresh);
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wid = tid >> 6;
    const int64_t v0 = (static_cast<int64_t>(blockIdx.x) * 256 + tid) * kUpkeepPer;
    uint32_t pv[kUpkeepPer];
    if (v0 + kUpkeepPer <= K.n) {
        const uint4 q = *reinterpret_cast<const uint4*>(K.prev + v0);
        const uint32_t w4[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < kUpkeepPer; ++j) pv[j] = (w4[j / 2] >> (16 * (j & 1))) & 0xFFFFu;
    } else {
#pragma unroll
        for (int j = 0; j < kUpkeepPer; ++j) pv[j] = v0 + j < K.n ? K.prev[v0 + j] : kStayed;
    }
    int32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kUpkeepPer; ++j) mine += pv[j] != kStayed;
    if (fresh == 0) {  // uniform over the grid: nothing to correct, but the moves are dealt with
#pragma unroll
        for (int j = 0; j < kUpkeepPer; ++j)
            if (pv[j] != kStayed) K.prev[v0 + j] = static_cast<uint16_t>(kStayed);
        return;
    }
    if (__syncthreads_or(mine) == 0) return;
    // exclusive sum of v over the workgroup; *total gets the whole
    auto block_prefix = [&](int32_t v, int32_t* total) {
        int32_t inc = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t t = __shfl_up(inc, o, 64);
            if (lane >= o) inc += t;
        }
        __syncthreads();  // s_wave may still be read
        if (lane == 63) s_wave[wid] = inc;
        __syncthreads();
        int32_t before = 0, all = 0;
        for (int w = 0; w < 4; ++w) {
            if (w < wid) before += s_wave[w];
            all += s_wave[w];
        }
        *total = all;
        return before + inc - v;
    };
    int32_t m;
    int32_t at = block_prefix(mine, &m);
#pragma unroll
    for (int j = 0; j < kUpkeepPer; ++j) {
        if (pv[j] == kStayed) continue;
        s_node[at] = static_cast<int32_t>(v0 + j);
        s_from[at] = static_cast<uint16_t>(pv[j]);
        K.prev[v0 + j] = static_cast<uint16_t>(kStayed);
        ++at;
    }
    __syncthreads();
    // 256 movers at a time: their rows one after the other, a thread per slot
    for (int32_t m0 = 0; m0 < m; m0 += 256) {
        int32_t d = 0;
        if (m0 + tid < m) {
            const int32_t v = s_node[m0 + tid];
            const int64_t b = K.xadj[v], e = K.xadj[v + 1];
            const int32_t lb = K.gid ? K.g_lbase[K.gid[v]] : 0;
            const int32_t f = static_cast<int32_t>(s_from[m0 + tid]) - lb, t = K.label[v] - lb;
            if (e - b > kUpkeepLong) {
                const int32_t nch = static_cast<int32_t>((e - b + kUpkeepLong - 1) / kUpkeepLong);
                const uint32_t c0 = atomicAdd(&K.ctr->nlong, static_cast<uint32_t>(nch));
                for (int32_t q = 0; q < nch; ++q) K.chunks[c0 + q] = make_int4(v, f, t, q);
            } else {
                d = static_cast<int32_t>(e - b);
            }
            s_begin[tid] = b;
            s_f[tid] = f;
            s_t[tid] = t;
        }
        int32_t total;
        const int32_t pre = block_prefix(d, &total);
        s_pre[tid] = pre;
        __syncthreads();
        constexpr int U = 4;
        for (int32_t j0 = tid; j0 < total; j0 += 256 * U) {
            int64_t slot[U];
            int32_t f[U], t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t j = j0 + u * 256;
                int lo = 0;  // the last mover whose slots begin at or before j
#pragma unroll
                for (int step = 128; step > 0; step >>= 1)
                    if (s_pre[lo + step] <= j) lo += step;
                slot[u] = j < total ? s_begin[lo] + (j - s_pre[lo]) : -1;
                f[u] = s_f[lo];
                t[u] = s_t[lo];
            }
            upkeep_slots<U>(K, fresh, slot, f, t);
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) upkeep_long_kernel(Upkeep K) {
    if (stopped(K.gate)) return;
    const uint32_t fresh = fresh_mask(K.fresh);
    const uint32_t nch = K.ctr->nlong;
    for (uint32_t q = blockIdx.x; q < nch; q += gridDim.x) {
        const int4 c = K.chunks[q];
        const int64_t b = K.xadj[c.x] + static_cast<int64_t>(c.w) * kUpkeepLong;
        const int64_t e = min(b + kUpkeepLong, K.xadj[c.x + 1]);
        constexpr int U = 4;
        for (int64_t j0 = b + threadIdx.x; j0 < e; j0 += 256 * U) {
            int64_t slot[U];
            int32_t f[U], t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                slot[u] = j0 + u * 256 < e ? j0 + u * 256 : -1;
                f[u] = c.y;
                t[u] = c.z;
            }
            upkeep_slots<U>(K, fresh, slot, f, t);
        }
    }
}

// --------------------------------------------------------------- schedule

// Upper degree of each bucket but the hub bucket (non-decreasing).
struct Thresholds {
    int32_t t[kNB - 1];
};

// The schedule takes three launches: every wave counts the categories of its
// run of 64 * R consecutive nodes (classify), a prefix sum over (category, run)
// gives each run its places (place), and every wave ranks its nodes and writes
// their rows (scatter); ids ascend inside a category.  A general radix sort of
// (category, node) pairs, copies back, and a launch for the rows took eleven.

// Category of a node: colour * kNB + degree bucket; degree-0 nodes and nodes of
// inactive graphs never move and go to the extra category ncat.
struct Classes {
    int32_t n;
    const int64_t* xadj;
    const int32_t* color_override;
    uint64_t hc;
    const int32_t* gid;  // several graphs (null: one): the graph of each node, its hash, first node and state
    const uint64_t* g_hc;
    const int32_t* g_nbase;
    const uint8_t* g_active;
    int32_t nsub;
    Thresholds th;
};

constexpr int kMaxCat = 16 * kNB + 1;
constexpr int kSlotCopies = 8;  // arrays of slot totals the workgroups add to in turn

template <int R>
__global__ void __launch_bounds__(256) classify_kernel(Classes K, uint8_t* __restrict__ cat, int32_t nruns,
                                                       uint32_t* __restrict__ run_cnt,
                                                       unsigned long long* __restrict__ cat_slots, Counters* ctr) {
    __shared__ uint32_t hist[4][kMaxCat];
    __shared__ unsigned long long shist[kMaxCat];
    const int ncat = K.nsub * kNB;
    const int w = threadIdx.x >> 6;
    const int lane = lane_id();
    for (int j = threadIdx.x; j < 4 * kMaxCat; j += 256) hist[j / kMaxCat][j % kMaxCat] = 0;
    for (int j = threadIdx.x; j < kMaxCat; j += 256) shist[j] = 0;
    __syncthreads();
    const int32_t run = blockIdx.x * 4 + w;
#pragma unroll 4
    for (int r = 0; r < R; ++r) {
        const int64_t v64 = static_cast<int64_t>(run) * (64 * R) + r * 64 + lane;
        if (v64 >= K.n) continue;
        const int32_t v = static_cast<int32_t>(v64);
        const int64_t d = K.xadj[v + 1] - K.xadj[v];
        uint64_t hcv = K.hc;
        int32_t lv = v;  // graph-local id
        bool act = true;
        if (K.gid) {
            const int32_t g = K.gid[v];
            hcv = K.g_hc[g];
            lv = v - K.g_nbase[g];
            act = K.g_active[g] != 0;
        }
        int32_t col;
        if (K.color_override) {
            col = K.color_override[v];
            if (col < 0 || col >= K.nsub) {
                ctr->bad_color = 1;
                col = 0;
            }
        } else {
            col = static_cast<int32_t>(mix64(hcv ^ static_cast<uint64_t>(static_cast<uint32_t>(lv))) %
                                       static_cast<uint64_t>(K.nsub));
        }
        int32_t bucket = kHubBucket;
#pragma unroll
        for (int j = kHubBucket - 1; j >= 0; --j)
            if (d <= K.th.t[j]) bucket = j;
        const int32_t c = (d == 0 || !act) ? ncat : col * kNB + bucket;
        cat[v] = static_cast<uint8_t>(c);
        atomicAdd(&hist[w][c], 1u);
        if (d) atomicAdd(&shist[c], static_cast<unsigned long long>(d));
    }
    __syncthreads();
    for (int j = threadIdx.x; j < 4 * (ncat + 1); j += 256) {
        const int32_t q = blockIdx.x * 4 + (j & 3), c = j >> 2;
        if (q < nruns) run_cnt[static_cast<int64_t>(c) * nruns + q] = hist[j & 3][c];
    }
    unsigned long long* slots = cat_slots + (blockIdx.x % kSlotCopies) * kMaxCat;
    for (int j = threadIdx.x; j <= ncat; j += 256)
        if (shist[j]) atomicAdd(&slots[j], shist[j]);
}

// run_cnt[c][q] to the first place of run q in category c, one workgroup per
// category; cat_count[c] its nodes.
__global__ void __launch_bounds__(1024) place_kernel(int32_t nruns, uint32_t* __restrict__ run_cnt,
                                                     const uint32_t* __restrict__ counts_in,
                                                     uint32_t* __restrict__ cat_count) {
    __shared__ uint32_t s_w[16];
    const int tid = threadIdx.x;
    const int64_t c = blockIdx.x;
    auto block_sum = [&](uint32_t x) {
        x = wave_sum(x);
        if (lane_id() == 0) s_w[tid >> 6] = x;
        __syncthreads();
        uint32_t t = 0;
        for (int q = 0; q < 16; ++q) t += s_w[q];
        __syncthreads();
        return t;
    };
    uint32_t before = 0;
    for (int64_t j = tid; j < c * nruns; j += 1024) before += counts_in[j];
    uint32_t base = block_sum(before);
    const uint32_t first = base;
    for (int32_t q0 = 0; q0 < nruns; q0 += 1024) {
        const uint32_t x = q0 + tid < nruns ? counts_in[c * nruns + q0 + tid] : 0;
        uint32_t incl = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(incl, o, 64);
            if (lane_id() >= o) incl += u;
        }
        if (lane_id() == 63) s_w[tid >> 6] = incl;
        __syncthreads();
        uint32_t pre = 0, total = 0;
        for (int q = 0; q < 16; ++q) {
            pre += q < (tid >> 6) ? s_w[q] : 0;
            total += s_w[q];
        }
        __syncthreads();
        if (q0 + tid < nruns) run_cnt[c * nruns + q0 + tid] = base + pre + incl - x;
        base += total;
    }
    if (tid == 0) cat_count[c] = base - first;
}

// The rows of the schedule.  A row of 2^31 slots or more does not occur: its
// slots would be distinct neighbours or repeated edges whose weights sum past
// 2^31 - 1.  Nodes that never move have no row.
template <int R>
__global__ void __launch_bounds__(256) schedule_kernel(int32_t n, const int64_t* __restrict__ xadj,
                                                       const uint8_t* __restrict__ cat, int32_t ncat, int32_t nruns,
                                                       const uint32_t* __restrict__ place, Row* __restrict__ rows,
                                                       int32_t* __restrict__ nodes) {
    __shared__ uint32_t at[4][kMaxCat];
    const int w = threadIdx.x >> 6;
    const int lane = lane_id();
    const int32_t run = blockIdx.x * 4 + w;
    if (run >= nruns) return;  // whole waves; no workgroup barrier below
    for (int c = lane; c < ncat; c += 64) at[w][c] = place[static_cast<int64_t>(c) * nruns + run];
    wave_sync();
    const uint64_t lt = lanemask_lt();
#pragma unroll 2
    for (int r = 0; r < R; ++r) {
        const int64_t v64 = static_cast<int64_t>(run) * (64 * R) + r * 64 + lane;
        const bool in = v64 < n;
        const int32_t v = static_cast<int32_t>(in ? v64 : 0);
        const int32_t c = in ? cat[v] : ncat;
        const int64_t b = xadj[v];
        const int64_t e = xadj[v + 1];
        uint64_t match = __ballot(c < ncat);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint64_t bal = __ballot((c >> q) & 1);
            match &= ((c >> q) & 1) ? bal : ~bal;
        }
        uint32_t pos = 0;
        if (c < ncat) pos = at[w][c] + static_cast<uint32_t>(__popcll(match & lt));
        wave_sync();
        if (c < ncat && (match & lt) == 0) at[w][c] += static_cast<uint32_t>(__popcll(match));
        wave_sync();
        if (c < ncat) {
            rows[pos] = Row{b, static_cast<int32_t>(e - b), v};
            nodes[pos] = v;
        }
    }
}

// Every node its own cluster: labels[v] = v, w[v] = c(v).
__global__ void __launch_bounds__(256) singletons_kernel(int32_t n, const int32_t* __restrict__ vw,
                                                         int32_t* __restrict__ labels, int32_t* __restrict__ w) {
    const int32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    labels[v] = v;
    w[v] = vw ? vw[v] : 1;
}

// Per-graph hash prefixes H(seed_g, tag, level, phase[, round]).
__global__ void graph_prefix_kernel(int32_t G, const uint64_t* __restrict__ seed, uint64_t tag, uint64_t level,
                                    uint64_t phase, int64_t round, uint64_t* __restrict__ out) {
    const int32_t g = blockIdx.x * 256 + threadIdx.x;
    if (g >= G) return;
    uint64_t h = mix64(seed[g]);
    h = mix64(h ^ tag);
    h = mix64(h ^ level);
    h = mix64(h ^ phase);
    if (round >= 0) h = mix64(h ^ static_cast<uint64_t>(round));
    out[g] = h;
}

constexpr int kLWChunk = 2048;  // nodes per block and step of label_weights_kernel<false>

template <bool kSmall>
__global__ void __launch_bounds__(256) label_weights_kernel(int32_t n, const int32_t* __restrict__ label,
                                                            const int32_t* __restrict__ vw, int32_t* __restrict__ w,
                                                            int32_t nw) {
    __shared__ int32_t loc[kSmallLabels];
    if (kSmall) {
        for (int j = threadIdx.x; j < nw; j += 256) loc[j] = 0;
        __syncthreads();
        for (int32_t v = blockIdx.x * 256 + threadIdx.x; v < n; v += gridDim.x * 256) {
            const int32_t c = vw ? vw[v] : 1;
            if (c) atomicAdd(&loc[label[v]], c);
        }
        __syncthreads();
        for (int j = threadIdx.x; j < nw; j += 256)
            if (loc[j]) atomicAdd(&w[j], loc[j]);
        return;
    }
    // Large label spaces, kLWChunk consecutive nodes per block at a time: when
    // their labels span fewer than kSmallLabels ids (the blocks of the few
    // graphs a chunk of a batch covers, or a run of singleton clusters), they
    // are summed in LDS first, so a label many nodes share costs one global
    // atomic per chunk; otherwise every node adds to HBM directly.
    constexpr int R = kLWChunk / 256;
    __shared__ int32_t s_lo[4], s_hi[4];
    for (int64_t base = static_cast<int64_t>(blockIdx.x) * kLWChunk; base < n;
         base += static_cast<int64_t>(gridDim.x) * kLWChunk) {
        int32_t lab[R], cw[R];
        int32_t lo = INT_MAX, hi = INT_MIN;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t v = base + r * 256 + threadIdx.x;
            lab[r] = v < n ? label[v] : -1;
            cw[r] = v < n ? (vw ? vw[v] : 1) : 0;
            if (lab[r] >= 0) {
                lo = lab[r] < lo ? lab[r] : lo;
                hi = lab[r] > hi ? lab[r] : hi;
            }
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane_id() == 0) {
            s_lo[threadIdx.x >> 6] = lo;
            s_hi[threadIdx.x >> 6] = hi;
        }
        __syncthreads();
        lo = min(min(s_lo[0], s_lo[1]), min(s_lo[2], s_lo[3]));
        hi = max(max(s_hi[0], s_hi[1]), max(s_hi[2], s_hi[3]));
        const int64_t span = static_cast<int64_t>(hi) - lo + 1;
        if (span > 0 && span <= kSmallLabels) {
            for (int j = threadIdx.x; j < span; j += 256) loc[j] = 0;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (cw[r]) atomicAdd(&loc[lab[r] - lo], cw[r]);
            __syncthreads();
            for (int j = threadIdx.x; j < span; j += 256)
                if (loc[j]) atomicAdd(&w[lo + j], loc[j]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (cw[r]) atomicAdd(&w[lab[r]], cw[r]);
        }
        __syncthreads();  // s_lo, s_hi and loc are reused by the next chunk
    }
}

// Per-colour hub metadata built on the host after the schedule is known.
struct HubPlan {
    int32_t count = 0;
    int32_t nchunks = 0;
    int32_t nparts = 0;
    int64_t at[9] = {};  // first 8-byte word of each array in the plans' buffer
};

// Side streams for the independent evaluation launches of a sub-round
// (default priority, created once per thread).  fork() makes them wait for
// the work already on the caller's stream, join() makes the caller's stream
// wait for them.  The hub chain, usually the longest, stays on the caller's
// stream, so the join mostly waits on work that has already finished (a
// cross-stream wait on unfinished work costs the device some 20 us).
class EvalStreams {
  public:
    static constexpr int kN = 2;
    EvalStreams() {
        for (int i = 0; i < kN; ++i) {
            HIPCHK(hipStreamCreateWithFlags(&st_[i], hipStreamNonBlocking));
            HIPCHK(hipEventCreateWithFlags(&done_[i], hipEventDisableTiming));
        }
        HIPCHK(hipEventCreateWithFlags(&start_, hipEventDisableTiming));
    }
    EvalStreams(const EvalStreams&) = delete;
    EvalStreams& operator=(const EvalStreams&) = delete;
    void fork(hipStream_t s) {
        HIPCHK(hipEventRecord(start_, s));
        for (int i = 0; i < kN; ++i) HIPCHK(hipStreamWaitEvent(st_[i], start_, 0));
    }
    void join(hipStream_t s) {
        for (int i = 0; i < kN; ++i) {
            HIPCHK(hipEventRecord(done_[i], st_[i]));
            HIPCHK(hipStreamWaitEvent(s, done_[i], 0));
        }
    }
    // heavy buckets (large rows) apart from each other and from the hubs
    hipStream_t bucket(int bk) const {
        static const int kMap[kNB - 1] = {0, 0, 1, 1, 1, 0, 1, 0};
        return st_[kMap[bk]];
    }

  private:
    hipStream_t st_[kN];
    hipEvent_t done_[kN];
    hipEvent_t start_;
};

EvalStreams& eval_streams() {
    thread_local EvalStreams e;
    return e;
}

// Pinned host copies of the per-round candidate counts (grown as needed,
// kept for the thread's lifetime).
thread_local uint32_t* t_host_rc = nullptr;
thread_local int32_t t_host_rc_cap = 0;

uint32_t* host_round_counts(int32_t rounds) {
    if (rounds > t_host_rc_cap) {
        if (t_host_rc) HIPCHK(hipHostFree(t_host_rc));
        t_host_rc_cap = std::max(rounds, 64);
        HIPCHK(hipHostMalloc(reinterpret_cast<void**>(&t_host_rc), sizeof(uint32_t) * t_host_rc_cap,
                             hipHostMallocPortable | hipHostMallocCoherent));
    }
    return t_host_rc;
}

// Two events marking the end of consecutive rounds (per thread).
struct RoundEvents {
    hipEvent_t ev[2];
    RoundEvents() {
        for (hipEvent_t& e : ev) HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    }
};

RoundEvents& round_events() {
    thread_local RoundEvents r;
    return r;
}

// Records the work enqueued on the capture stream cs (and on streams joined
// to it) while it lives into a graph, when enabled; run() instantiates it,
// launches it on the caller's stream and waits.  The caller's stream may be
// the null stream, which cannot be captured itself.  If an error unwinds
// before run(), the capture is ended and discarded.
class GraphCapture {
  public:
    GraphCapture(hipStream_t cs, hipStream_t exec, bool on) : s_(cs), exec_(exec), on_(on) {
        if (on_) HIPCHK(hipStreamBeginCapture(s_, hipStreamCaptureModeThreadLocal));
    }
    GraphCapture(const GraphCapture&) = delete;
    GraphCapture& operator=(const GraphCapture&) = delete;
    void run() {
        if (!on_) return;
        on_ = false;
        hipGraph_t graph = nullptr;
        HIPCHK(hipStreamEndCapture(s_, &graph));
        hipGraphExec_t exec = nullptr;
        const hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(graph);
            HIPCHK(e);
        }
        const hipError_t l = hipGraphLaunch(exec, exec_);
        const hipError_t w = l == hipSuccess ? hipStreamSynchronize(exec_) : l;
        (void)hipGraphExecDestroy(exec);
        (void)hipGraphDestroy(graph);
        HIPCHK(w);
    }
    ~GraphCapture() {
        if (!on_) return;
        hipGraph_t graph = nullptr;
        if (hipStreamEndCapture(s_, &graph) == hipSuccess && graph) (void)hipGraphDestroy(graph);
    }

  private:
    hipStream_t s_;
    hipStream_t exec_;
    bool on_;
};

// The stream rounds are captured on (per thread, default priority).
hipStream_t capture_stream() {
    struct Holder {
        hipStream_t st;
        Holder() { HIPCHK(hipStreamCreateWithFlags(&st, hipStreamNonBlocking)); }
    };
    thread_local Holder h;
    return h.st;
}

unsigned capped_grid(int64_t items) {
    const int64_t g = (items + 255) / 256;
    return static_cast<unsigned>(g < 1 ? 1 : (g > kMaxBlocks ? kMaxBlocks : g));
}

}  // namespace

void singletons(const DevGraph& g, int32_t* labels, int32_t* w, hipStream_t s) {
    if (g.n <= 0) return;
    singletons_kernel<<<grid_for(g.n, 256), 256, 0, s>>>(g.n, g.vw, labels, w);
    LAUNCHCHK();
}

void label_weights(const DevGraph& g, const int32_t* label, int32_t* w, int32_t nw, hipStream_t s) {
    fill_i32(w, 0, nw, s);
    if (g.n > 0) {
        if (nw <= kSmallLabels)
            label_weights_kernel<true><<<capped_grid(g.n), 256, 0, s>>>(g.n, label, g.vw, w, nw);
        else
            label_weights_kernel<false><<<static_cast<unsigned>(std::min<int64_t>((g.n + kLWChunk - 1) / kLWChunk,
                                                                                  kMaxBlocks)),
                                          256, 0, s>>>(g.n, label, g.vw, w, nw);
        LAUNCHCHK();
    }
}

// One lane per node is the cheapest form, but the slowest one when there are
// too few nodes to fill the device: up to 2^17 nodes only rows of up to 4 slots
// take it (40 sub-rounds of clustering / of refinement, power-law graph of
// 2^14 nodes: 1.40 -> 1.14 / 1.64 -> 1.33 ms; of 2^20 nodes: 5.76 -> 5.92 /
// 4.96 -> 5.11 ms, so larger graphs keep 16).
int32_t default_lane_max(int32_t n) { return n <= (1 << 17) ? kLaneSmall : kLaneMax; }

LPResult run_lp(const DevGraph& g, int32_t phase, int32_t level, uint64_t seed, int32_t nsub, int32_t rounds,
                int64_t bound, int32_t* label, int32_t* w, int32_t nw, const int32_t* color_override,
                const LPTuning& tune, hipStream_t s, const MultiGraph* mg) {
    LPResult res;
    const int32_t n = g.n;
    if (n == 0 || rounds <= 0) return res;
    if (nsub < 1 || nsub > 16) fail(-1, "subrounds must be in 1..16");
    const bool small = nw <= kSmallLabels;
    static const bool trace = std::getenv("SCLAP_TRACE") != nullptr;  // per sub-round counts on stderr

    // --- schedule: nodes grouped by (colour, degree bucket), ascending ids
    const int32_t ncat = nsub * kNB;
    Thresholds th;
    {
        const int32_t lane = std::max(1, std::min(tune.lane_max > 0 ? tune.lane_max : default_lane_max(n), kLaneMax));
        const int32_t wave = std::max(lane, std::min(tune.wave_max, kWaveMaxDeg));
        const int32_t block = std::max(wave, std::min(tune.block_max, kBlockMaxDeg));
        th.t[0] = std::min(kLaneSmall, lane);
        th.t[1] = lane;
        th.t[2] = std::max(lane, std::min(kG16Max, wave));
        th.t[3] = std::max(th.t[2], std::min(kG32Max, wave));
        th.t[4] = wave;
        th.t[5] = std::min(block, std::max(wave, kBlock1Max));
        th.t[6] = std::min(block, std::max(th.t[5], kBlock2Max));
        th.t[7] = block;
    }
    // nodes per wave of the scheduling kernels: enough waves for a small graph,
    // few runs for a large one
    const int per_run = n <= (1 << 16) ? 1 : (n <= (1 << 20) ? 4 : 16);
    const int32_t nruns = static_cast<int32_t>((static_cast<int64_t>(n) + 64 * per_run - 1) / (64 * per_run));
    DBuf<uint8_t> cat(n, s);
    DBuf<uint32_t> run_cnt(static_cast<size_t>(ncat + 1) * nruns, s), place(static_cast<size_t>(ncat + 1) * nruns, s);
    DBuf<uint32_t> cat_count(ncat + 1, s);
    DBuf<int32_t> order(n, s);
    DBuf<Row> sched(n, s);
    // slot totals of the categories, then the two counter sets
    constexpr size_t kSlotWords = kSlotCopies * kMaxCat;
    DBuf<unsigned long long> cat_slots(kSlotWords + 2 * sizeof(Counters) / 8, s);
    Counters* const ctr = reinterpret_cast<Counters*>(cat_slots.get() + kSlotWords);
    fill_u32(reinterpret_cast<uint32_t*>(cat_slots.get()), 0, 2 * (kSlotWords + 2 * sizeof(Counters) / 8), s);
    const uint64_t hc = hash_prefix({seed, 1, static_cast<uint64_t>(static_cast<uint32_t>(level)),
                                     static_cast<uint64_t>(static_cast<uint32_t>(phase))});
    const uint64_t lvl64 = static_cast<uint64_t>(static_cast<uint32_t>(level));
    const uint64_t ph64 = static_cast<uint64_t>(static_cast<uint32_t>(phase));
    DBuf<uint64_t> g_hc, g_tp;
    if (mg) {
        g_hc.alloc(std::max(mg->G, 1), s);
        g_tp.alloc(std::max(mg->G, 1), s);
        graph_prefix_kernel<<<grid_for(mg->G, 256), 256, 0, s>>>(mg->G, mg->seed, 1, lvl64, ph64, -1, g_hc.get());
        LAUNCHCHK();
    }
    {
        ProfScope ps("lp_schedule", 0, s);
        const Classes K{n, g.xadj, color_override, hc, mg ? mg->gid : nullptr, g_hc.get(), mg ? mg->nbase : nullptr,
                        mg ? mg->active : nullptr, nsub, th};
        const unsigned gb = grid_for(nruns, 4);
        auto classify = per_run == 1 ? classify_kernel<1> : per_run == 4 ? classify_kernel<4> : classify_kernel<16>;
        classify<<<gb, 256, 0, s>>>(K, cat.get(), nruns, run_cnt.get(), cat_slots.get(), ctr);
        LAUNCHCHK();
        place_kernel<<<ncat + 1, 1024, 0, s>>>(nruns, place.get(), run_cnt.get(), cat_count.get());
        LAUNCHCHK();
        auto schedule = per_run == 1 ? schedule_kernel<1> : per_run == 4 ? schedule_kernel<4> : schedule_kernel<16>;
        schedule<<<gb, 256, 0, s>>>(n, g.xadj, cat.get(), ncat, nruns, place.get(), sched.get(), order.get());
        LAUNCHCHK();
    }
    std::vector<uint32_t> cnt(ncat + 1);
    std::vector<unsigned long long> cslots(kSlotWords);
    Counters hctr;
    {
        const ReadItem items[3] = {{cnt.data(), cat_count.get(), (ncat + 1) * sizeof(uint32_t)},
                                   {cslots.data(), cat_slots.get(), kSlotWords * sizeof(unsigned long long)},
                                   {&hctr, ctr, sizeof(Counters)}};
        read_back(items, 3, s);
    }
    for (size_t q = kMaxCat; q < kSlotWords; ++q) cslots[q % kMaxCat] += cslots[q];
    if (hctr.bad_color) fail(-1, "color_override value outside [0, subrounds)");
    std::vector<int64_t> off(ncat + 2, 0);
    for (int32_t j = 0; j <= ncat; ++j) off[j + 1] = off[j] + cnt[j];
    const int32_t* nodes = order.get();
    const Row* rows = sched.get();

    // --- hub plans per colour: the hubs' rows in one read, all plans in one copy
    std::vector<HubPlan> plans(nsub);
    int64_t max_region = 0, max_over = 0, max_table = 0, max_win = 0, max_hub_ints = 0;
    // refinement labels fit dense arrays when there are few enough blocks
    // (the same test sets EvalArgs::dense_k below); hub chunks are then longer
    const int32_t dense_labels = phase != kCluster ? (mg ? mg->max_labels : nw) : 0;
    const int64_t hub_chunk = dense_labels > 0 && dense_labels <= kDenseMax ? kHubDenseChunk : kHubChunk;
    std::vector<std::vector<Row>> hub_rows(nsub);
    std::vector<ReadItem> hub_reads;
    for (int32_t sc = 0; sc < nsub; ++sc) {
        const int32_t cat = sc * kNB + kHubBucket;
        hub_rows[sc].resize(cnt[cat]);
        if (cnt[cat]) hub_reads.push_back(ReadItem{hub_rows[sc].data(), rows + off[cat], cnt[cat] * sizeof(Row)});
    }
    DBuf<int64_t> plan_buf;
    if (!hub_reads.empty()) {
        read_back(hub_reads.data(), static_cast<int>(hub_reads.size()), s);
        std::vector<int64_t> all;  // the plans' arrays, each from a multiple of 8 bytes
        auto put = [&](const auto& vec) {
            const size_t at = all.size();
            const size_t bytes = vec.size() * sizeof(vec[0]);
            all.resize(at + (bytes + 7) / 8, 0);
            if (bytes) std::memcpy(all.data() + at, vec.data(), bytes);
            return static_cast<int64_t>(at);
        };
        for (int32_t sc = 0; sc < nsub; ++sc) {
            const std::vector<Row>& hr = hub_rows[sc];
            const int32_t H = static_cast<int32_t>(hr.size());
            HubPlan& P = plans[sc];
            P.count = H;
            if (H == 0) continue;
            std::vector<int32_t> plog(H), pbase(H + 1), cap(H), chub, phub;
            std::vector<int64_t> rbase(H), obase(H), toff(H), cbeg;
            int64_t rtot = 0, otot = 0, ttot = 0;
            int32_t np = 0;
            for (int32_t h = 0; h < H; ++h) {
                const int64_t hd = hr[h].deg;
                // at most 1024 entries per label partition on average (half the
                // LDS table's limit), at most 2048 partitions
                int32_t lg = 0;
                while (lg < kMaxPartLog && (static_cast<int64_t>(1024) << lg) < hd) ++lg;
                plog[h] = lg;
                const int64_t per = (hd + (1LL << lg) - 1) >> lg;
                cap[h] = static_cast<int32_t>(std::min<int64_t>(2 * per + 64, hd));
                if (tune.hub_region_cap > 0) cap[h] = std::min(cap[h], tune.hub_region_cap);
                pbase[h] = np;
                phub.insert(phub.end(), static_cast<size_t>(1) << lg, h);
                np += 1 << lg;
                rbase[h] = rtot;
                rtot += static_cast<int64_t>(cap[h]) << lg;
                obase[h] = otot;
                otot += hd;
                toff[h] = ttot;
                ttot += 2 * hd;
                for (int64_t sl = 0; sl < hd; sl += hub_chunk) {
                    chub.push_back(h);
                    cbeg.push_back(hr[h].begin + sl);
                }
            }
            pbase[H] = np;
            P.nchunks = static_cast<int32_t>(chub.size());
            P.nparts = np;
            P.at[0] = put(plog);
            P.at[1] = put(pbase);
            P.at[2] = put(cap);
            P.at[3] = put(chub);
            P.at[4] = put(phub);
            P.at[5] = put(rbase);
            P.at[6] = put(obase);
            P.at[7] = put(toff);
            P.at[8] = put(cbeg);
            max_region = std::max(max_region, rtot);
            max_over = std::max(max_over, otot);
            max_table = std::max(max_table, ttot);
            max_win = std::max(max_win, static_cast<int64_t>(np));
            max_hub_ints = std::max(max_hub_ints, static_cast<int64_t>(np) + 3 * static_cast<int64_t>(H));
        }
        plan_buf.alloc(all.size(), s);
        upload_once(plan_buf.get(), all.data(), all.size() * sizeof(int64_t), s);
    }
    DBuf<int32_t> ekeys, evals, okeys, ovals, gkeys, gvals, hub_ints, w_conn, w_x;
    DBuf<uint64_t> w_tie;
    if (max_win > 0) {
        ekeys.alloc(max_region, s);
        evals.alloc(max_region, s);
        okeys.alloc(max_over, s);
        ovals.alloc(max_over, s);
        gkeys.alloc(max_table, s);
        gvals.alloc(max_table, s);
        hub_ints.alloc(max_hub_ints, s);
        fill_i32(hub_ints.get(), 0, max_hub_ints, s);
        w_conn.alloc(max_win, s);
        w_x.alloc(max_win, s);
        w_tie.alloc(max_win, s);
    }

    // --- per-entry candidate buffers: at most the nodes of one colour
    int64_t max_color = 0;
    for (int32_t sc = 0; sc < nsub; ++sc) max_color = std::max(max_color, off[(sc + 1) * kNB] - off[sc * kNB]);
    const int64_t cap = std::max<int64_t>(max_color, 1);
    const bool direct = nw <= kDirectLabels || (nw <= kSmallLabels && cap > kDirectColour && !mg);
    const int64_t acc_n = static_cast<int64_t>(nw) << (direct ? kAccShift : 0);
    const int64_t fill_n = static_cast<int64_t>(nw) << (direct ? kFillShift : 0);
    DBuf<int32_t> ct(cap, s), cg(cap, s), seg_off(direct ? 0 : nw, s), seg_fill(fill_n, s), swt(cap, s);
    DBuf<unsigned long long> acc(acc_n, s);
    DBuf<Segment> seg(std::min<int64_t>(cap, nw), s);
    DBuf<uint8_t> ok(cap, s);
    DBuf<uint64_t> sent(cap, s);
    // segments longer than small_max are selected by several workgroups.  By
    // default a colour of up to kFinishMax nodes leaves every segment to one
    // workgroup and launches no further kernel (three to four launches of
    // 2 us each, against 20-80 us in the first sub-rounds, whose segments
    // alone are that long); larger colours split segments over kSmallSeg in a
    // launch per digit.  Up to 65 536 entries per workgroup and one launch for
    // the others, in colours of up to 2^18 nodes, gained nothing on a partition
    // of 2^20 nodes (28.25 and 27.21 ms, 28.35 and 27.30 like this) and 5 % on
    // a mesh of 741 000 (8.6 and 9.1 ms), and lost where the segments are that
    // long (8 hubs of 500 000 slots, refinement into 1 000 blocks: 2.09 ms, 1.47
    // like this).
    const int32_t small_max = tune.select_small_max > 0 ? std::min(tune.select_small_max, kFinishMax)
                              : cap <= kFinishMax       ? kFinishMax
                                                        : kSmallSeg;
    const bool use_large = cap > small_max;
    const int64_t max_large = use_large ? cap / small_max + 1 : 0;
    const int64_t max_lchunks = use_large ? cap / kSegChunk + max_large : 0;
    DBuf<int32_t> ltarget(max_large, s), lbase(max_large, s), llen(max_large, s), lchunk0(max_large, s);
    DBuf<int32_t> lowner(max_lchunks, s);
    const int64_t lhist_n = max_large * kLBins * (g.heavy ? 2 : 1);
    DBuf<uint32_t> lhist(lhist_n, s);
    DBuf<uint64_t> lprefix(max_large, s);
    DBuf<int32_t> lroom(max_large, s);
    DBuf<uint32_t> ldone(max_large, s);
    // launches of the multi-workgroup selection: enough digits for node ids
    // plus a 12-bit gain range; wider keys (node id bits plus at most 32 bits
    // of gain range) finish in the last launch
    const int max_launches = (bits_for(static_cast<uint64_t>(n - 1)) + 32 + kLDigit - 1) / kLDigit;
    const int sel_launches =
        tune.select_launches > 0
            ? std::min(tune.select_launches, max_launches)
            : std::min(max_launches, (bits_for(static_cast<uint64_t>(n - 1)) + 12 + kLDigit - 1) / kLDigit);
    DBuf<uint32_t> rcnt(std::max(rounds, 1), s);  // candidates per round, read back one round late (see stopped())
    DBuf<uint8_t> lab8;
    DBuf<uint16_t> lab16;
    if (nw <= 256) lab8.alloc(n, s);
    else if (nw <= 65536) lab16.alloc(n, s);
    const int64_t init_items = std::max({fill_n, lhist_n, nw <= 65536 ? static_cast<int64_t>(n) : 0});
    init_admission_kernel<<<std::min(grid_for(init_items, 256), 4096u), 256, 0, s>>>(
        acc.get(), acc_n, seg_off.get(), direct ? 0 : nw, seg_fill.get(), fill_n, lhist.get(), lhist_n, ldone.get(),
        max_large, rcnt.get(), rounds, ctr, label, n, lab8.get(), lab16.get());
    LAUNCHCHK();

    EvalArgs A;
    A.adj = g.adj;
    A.S = g.S;
    A.ew = g.ew;
    A.vw = g.vw;
    A.label = label;
    A.w = w;
    A.bound = bound;
    A.refine = phase != kCluster ? 1 : 0;  // the initial phase follows the refinement rules
    A.gid = mg ? mg->gid : nullptr;
    A.g_tp = g_tp.get();
    A.g_bound = mg ? mg->bound : nullptr;
    A.g_lbase = mg ? mg->lbase : nullptr;
    const Bounds BB{bound, mg ? mg->lgid : nullptr, mg ? mg->bound : nullptr};
    // refinement labels are blocks: dense connection arrays when few enough
    const int32_t dense_k = dense_labels;
    A.dense_k = dense_k > 0 && dense_k <= kDenseMax ? dense_k : 0;
    const bool dense = A.dense_k > 0;
    DBuf<int32_t> hub_sum;
    if (dense) {
        int64_t max_hubs = 1;
        for (const HubPlan& P : plans) max_hubs = std::max<int64_t>(max_hubs, P.count);
        hub_sum.alloc(max_hubs * A.dense_k, s);
        fill_i32(hub_sum.get(), 0, max_hubs * A.dense_k, s);
    }
    A.label8 = lab8.get();
    A.label16 = lab16.get();
    // quiet-node tracking starts once a round has few candidates (marking the
    // neighbours of every mover is then cheap) and skipping one round later;
    // the kernels derive the start from the per-round counts (quiet_mode)
    DBuf<uint8_t> quiet;
    // the default (0) leaves it off here; the batch driver turns it on
    const bool track_quiet = tune.skip_quiet > 0;
    if (track_quiet) {
        quiet.alloc(n, s);
        fill_u8(quiet.get(), 0, n, s);
    }
    A.quiet = quiet.get();
    A.quiet_n = n;
    bool long_rows = false;  // longer than the wave bucket's
    for (int32_t j = 0; j < ncat; ++j) long_rows |= j % kNB > 4 && cnt[j] > 0;
    // Kept sums (see eval_kept_kernel).  A row keeps its sums when reading them
    // is no more work than its slots: at least one slot per kKeptPerSlot blocks,
    // which also bounds the memory, by 16 bytes per slot of those rows.  The
    // upkeep finds a mover's neighbours in its row, so the graph must be known to
    // be symmetric.  Below kKeptMinSlots the two launches of the upkeep and the
    // separate launch for the kept rows cost more than the gathers (refinement of
    // a power-law graph, 10 rounds, 16 blocks: whole partition of 2^20 nodes, 31
    // M slots, 29.7 ms without, 28.7 ms with; levels of 2 to 16 M slots kept too:
    // 31.0 ms).  Nor with colours of under 2^22 slots, which evaluate all rows in
    // one launch and have nothing beside which the upkeep could run (refinement
    // of that graph, 16 colours of 2 M slots, 100 blocks: 12.1 ms with, 10.4
    // without; 4 colours 5.5 and 6.2).  Where the memory is not to be had, nothing
    // is kept.
    int32_t kept_bucket = 2;
    while (kept_bucket < kHubBucket && (th.t[kept_bucket - 1] + 1) * kKeptPerSlot < A.dense_k) ++kept_bucket;
    int64_t kept_slots = 0;
    for (int32_t j = 0; j < ncat; ++j)
        if (j % kNB >= kept_bucket) kept_slots += static_cast<int64_t>(cslots[j]);
    KeptRanges kr = {};
    kr.nsub = nsub;
    int32_t kept_rows = 0;
    for (int32_t sc = 0; sc < nsub; ++sc) {
        kr.from[sc] = static_cast<int32_t>(off[sc * kNB + kept_bucket]);
        kr.to[sc] = kr.end[sc] = static_cast<int32_t>(off[(sc + 1) * kNB]);
        kr.base[sc] = kept_rows;
        kept_rows += kr.to[sc] - kr.from[sc];
    }
    bool keep = dense && g.symmetric && rounds > 2 && kept_slots >= std::max(kKeptMinSlots, nsub * kKeptColourSlots) &&
                nw < static_cast<int32_t>(kStayed);
    // hub rows are kept whatever their length, which the options may set low
    if (static_cast<int64_t>(kept_rows) * A.dense_k > kKeptPerSlot * kept_slots || kept_rows >= 1 << kKeptBits) keep = false;
    DBuf<int32_t> sums, kidx;
    DBuf<uint16_t> prev;
    DBuf<int4> up_chunks;
    DBuf<uint32_t> fresh(1, s);
    if (keep) {
        try {
            sums.alloc(static_cast<size_t>(kept_rows) * A.dense_k, s);
            kidx.alloc(n, s);
            prev.alloc(static_cast<size_t>(n) + 8, s);
            up_chunks.alloc(static_cast<size_t>(g.S / (kUpkeepLong / 2) + 1), s);
        } catch (const Error& e) {
            if (e.status != SCLAP_ERR_NO_MEMORY) throw;
            keep = false;
            sums.release();
            kidx.release();
            prev.release();
        }
    }
    if (keep) {
        fill_u32(reinterpret_cast<uint32_t*>(prev.get()), 0xFFFFFFFFu, (static_cast<int64_t>(n) + 8) / 2, s);
        kept_index_kernel<<<grid_for(off[ncat], 256), 256, 0, s>>>(kr, nodes, static_cast<int32_t>(off[ncat]), kidx.get());
        LAUNCHCHK();
        fill_u32(fresh.get(), 0, 1, s);
    }
    A.sums = nullptr;
    A.fresh = Fresh{};
    A.colour = 0;

    // Algorithmic bytes of one evaluation launch, the figure of one round's
    // minimal traffic per unit: per evaluated node 24 (its row offsets, own
    // label, node weight and the weight of one label), per slot 12 (the
    // neighbour id, the edge weight and the neighbour's label), whether or
    // not the kernel reads weights that hold only ones or narrow labels.
    const double node_bytes = 24.0;
    const double slot_bytes = 12.0;
    auto eval_bytes = [&](int64_t nodes_in, unsigned long long slots_in) {
        return node_bytes * static_cast<double>(nodes_in) + slot_bytes * static_cast<double>(slots_in);
    };
    const int bits_v = bits_for(static_cast<uint64_t>(n - 1));
    EvalStreams& evs = eval_streams();

    A.rcnt = rcnt.get();
    uint32_t* hrc = host_round_counts(rounds);
    std::fill(hrc, hrc + rounds, 0u);
    int32_t last_sub = -1;  // the last colour with nodes
    for (int32_t sc = 0; sc < nsub; ++sc)
        if (off[(sc + 1) * kNB] > off[sc * kNB]) last_sub = sc;
    RoundEvents& rev = round_events();
    bool halted = false;
    // bookkeeping of a finished round q (read back from the device)
    auto finish_round = [&](int32_t q) {
        HIPCHK(hipEventSynchronize(rev.ev[q & 1]));
        const uint32_t round_cands = hrc[q];
        res.rounds_run = q + 1;
        res.moves += round_cands;
        if (round_cands == 0) halted = true;
    };
    // Captured execution (tuning option): all rounds of this call are
    // recorded into one HIP graph and launched at once, so the host neither
    // launches kernel by kernel nor waits between rounds; rounds after one
    // without candidates run as gated no-ops (the result is the same, see
    // stopped()).  Not the default: on this GPU the graph runs the same
    // kernels about 1.5 times slower than the host's pipelined launches.  Not
    // while per-launch timing events or the trace are on (events recorded in
    // a graph cannot be timed).
    const bool capture = !trace && !profiler().on && tune.capture > 0;
    // the rounds are enqueued on the capture stream and the graph runs on the
    // caller's stream; buffers above were allocated on the caller's stream
    const hipStream_t caller = s;
    if (capture) s = capture_stream();
    GraphCapture rounds_graph(s, caller, capture);

    Admission M;
    M.ct = ct.get();
    M.cg = cg.get();
    M.vw = g.vw;
    M.w = w;
    M.nw = nw;
    M.acc = acc.get();
    M.heavy = g.heavy;
    M.B = BB;
    M.ok = ok.get();
    M.seg_off = seg_off.get();
    M.seg_fill = seg_fill.get();
    M.seg = seg.get();
    M.sent = sent.get();
    M.swt = swt.get();
    M.L = LargeSel{ltarget.get(), lbase.get(), llen.get(),    lchunk0.get(), lowner.get(),
                   lhist.get(),   lprefix.get(), lroom.get(), ldone.get()};
    M.small_max = small_max;
    M.acc_shift = direct ? kAccShift : 0;
    M.fill_shift = direct ? kFillShift : 0;
    M.bits_v = bits_v;
    M.label = label;
    M.label8 = lab8.get();
    M.label16 = lab16.get();
    M.prev = keep ? prev.get() : nullptr;
    M.xadj = g.xadj;
    M.fresh = keep ? fresh.get() : nullptr;
    M.fresh_limit = 0;  // before the first sub-round nothing has moved
    Upkeep up = {};
    up.n = n;
    up.prev = prev.get();
    up.label = label;
    up.xadj = g.xadj;
    up.adj = g.adj;
    up.ew = g.ew;
    up.gid = A.gid;
    up.g_lbase = A.g_lbase;
    up.kidx = kidx.get();
    up.sums = sums.get();
    up.k = A.dense_k;
    up.chunks = up_chunks.get();
    bool upkeep_due = false;  // the last sub-round's moves have not reached the kept sums
    int32_t step = 0;  // sub-rounds enqueued: they use the two counter sets in turn

    for (int32_t r = 0; r < rounds && !halted; ++r) {
        const uint32_t* gate = r > 0 ? rcnt.get() + (r - 1) : nullptr;
        if (mg) {
            graph_prefix_kernel<<<grid_for(mg->G, 256), 256, 0, s>>>(mg->G, mg->seed, 2, lvl64, ph64, r, g_tp.get());
            LAUNCHCHK();
        }
        A.round = r;
        A.gate = gate;
        A.tp = hash_prefix({seed, 2, static_cast<uint64_t>(static_cast<uint32_t>(level)),
                            static_cast<uint64_t>(static_cast<uint32_t>(phase)),
                            static_cast<uint64_t>(static_cast<uint32_t>(r))});
        for (int32_t sc = 0; sc < nsub; ++sc) {
            const int32_t c0 = sc * kNB;
            const int64_t ccount = off[c0 + kNB] - off[c0];
            if (ccount == 0) continue;
            const int32_t* cnodes = nodes + off[c0];
            // evaluation: one result per schedule entry of this colour; the
            // buckets are independent and run side by side on the evaluation
            // streams (hubs on the caller's stream), joined before admission
            unsigned long long colour_slots = 0;
            for (int32_t bk = 0; bk < kNB; ++bk) colour_slots += cslots[c0 + bk];
            const bool side = colour_slots >= (1ULL << 22);  // small colours stay on one stream
            if (side) evs.fork(s);
            const Fresh now{fresh.get(), ctr + (~step & 1), M.fresh_limit};  // as the last sub-round left the sums
            // the previous sub-round's moves reach the kept sums while the
            // evaluation streams take the short rows, which need none
            if (upkeep_due) {
                up.fresh = now;
                ProfScope ps("lp_upkeep", 0, s);
                upkeep_kernel<<<grid_for(n, 256 * kUpkeepPer), 256, 0, s>>>(up);
                LAUNCHCHK();
                upkeep_long_kernel<<<kUpkeepLongBlocks, 256, 0, s>>>(up);
                LAUNCHCHK();
                upkeep_due = false;
            }
            // hubs first: their chain (chunks, partitions, decision) is the
            // longest, so its workgroups should be dispatched before the
            // other buckets fill the device
            const HubPlan& P = plans[sc];
            HubArgs H = {};
            const bool kept_eval = keep && r > 0;  // rows from kept_bucket on: from their kept sums, if those hold
            A.fresh = kept_eval ? now : Fresh{};
            A.colour = sc;
            if (P.count > 0) {
                const int32_t Hn = P.count;
                H.count = Hn;
                const int64_t* pb = plan_buf.get();
                auto i32 = [&](int q) { return reinterpret_cast<const int32_t*>(pb + P.at[q]); };
                H.hub_plog = i32(0);
                H.hub_pbase = i32(1);
                H.hub_cap = i32(2);
                H.chunk_hub = i32(3);
                H.part_hub = i32(4);
                H.hub_rbase = pb + P.at[5];
                H.hub_obase = pb + P.at[6];
                H.hub_toff = pb + P.at[7];
                H.chunk_begin = pb + P.at[8];
                H.rcount = hub_ints.get();
                H.ocount = H.rcount + P.nparts;
                H.tfill = reinterpret_cast<uint32_t*>(H.ocount + Hn);
                H.hub_own = H.ocount + 2 * Hn;
                H.ekeys = ekeys.get();
                H.evals = evals.get();
                H.okeys = okeys.get();
                H.ovals = ovals.get();
                H.gkeys = gkeys.get();
                H.gvals = gvals.get();
                H.w_conn = w_conn.get();
                H.w_tie = w_tie.get();
                H.w_x = w_x.get();
                H.part_limit = std::max(1, std::min(tune.hub_part_limit, kPartTable / 2));
                H.hub_sum = hub_sum.get();
            }
            FusedBuckets F;
            for (int32_t bk = 0; bk < kNB; ++bk) {
                F.rows[bk] = rows + off[c0 + bk];
                F.ct[bk] = ct.get() + (off[c0 + bk] - off[c0]);
                F.cg[bk] = cg.get() + (off[c0 + bk] - off[c0]);
                F.count[bk] = static_cast<int32_t>(off[c0 + bk + 1] - off[c0 + bk]);
                F.end[bk] = 0;
                F.sums[bk] = keep && bk >= kept_bucket
                                 ? sums.get() + (kr.base[sc] + off[c0 + bk] - kr.from[sc]) * A.dense_k
                                 : nullptr;
            }
            auto use_bucket = [&](int32_t bk) {
                A.rows = F.rows[bk];
                A.count = F.count[bk];
                A.ct = F.ct[bk];
                A.cg = F.cg[bk];
                A.sums = F.sums[bk];
            };
            // workgroups of buckets hi..lo, the longest rows first
            auto lay_out = [&](int32_t hi, int32_t lo, double* bytes) {
                static const int32_t kPerBlock[kNB] = {256, 256, 16, 8, 4, 1, 1, 1, 1};  // nodes per workgroup
                int32_t blocks = 0;
                *bytes = 0;
                for (int32_t bk = hi; bk >= lo; --bk) {
                    blocks += bk == kHubBucket ? P.nchunks : (F.count[bk] + kPerBlock[bk] - 1) / kPerBlock[bk];
                    F.end[bk] = blocks;
                    *bytes += eval_bytes(F.count[bk], cslots[c0 + bk]);
                }
                return blocks;
            };
            // a small colour: the buckets of small tables in one launch, the
            // others in a second one
            const bool fused = !side && tune.fuse >= 0;
            // A small colour without hubs counts its candidates as the results
            // are stored: one launch less.  Adds to one address are served one
            // every 12 ns, and the candidates of a colour may all want the same
            // label.  Rows of a few slots then add once per wave (count_lanes);
            // longer ones add one by one, so the colour has at most 2^13 nodes
            // (with 2^14: 10 rounds over 15 000 nodes per colour of a power-law
            // graph 1.87 ms, 1.61 like this; 6 hubs as every node's neighbours
            // 0.66 and 0.48), or 2^14 where no row is long, so that no label
            // draws many to begin with (partition of a mesh with 12 500 nodes
            // per colour 3.47 ms, 3.64 with 2^13).
            const bool count_in_eval =
                fused && H.count == 0 && ccount <= (long_rows ? kCountInEval : kCountShortRows) && nw >= 8 && !g.heavy;
            A.acc = count_in_eval ? acc.get() : nullptr;
            A.acc_shift = direct ? kAccShift : 0;
            const bool big = fused && !dense && tune.block_table != kBlockTablePow2;
            int32_t bk_from = 0;
            if (fused) {
                bk_from = dense ? kNB : kFusedHash;
                double bytes;
                const int32_t blocks = lay_out(kept_eval ? kept_bucket - 1 : bk_from - 1, 0, &bytes);
                if (blocks > 0) {
                    ProfScope ps(A.refine ? "lp_refine_fused" : "lp_eval_fused", bytes, s);
                    if (dense) eval_fused_kernel<true><<<blocks, 256, 0, s>>>(A, F, H);
                    else eval_fused_kernel<false><<<blocks, 256, 0, s>>>(A, F, H);
                    LAUNCHCHK();
                }
            }
            if (big) {
                double bytes;
                const int32_t blocks = lay_out(kHubBucket, kFusedHash, &bytes);
                bk_from = kNB;
                if (blocks > 0) {
                    ProfScope ps(A.refine ? "lp_refine_big" : "lp_eval_big", bytes, s);
                    eval_big_kernel<<<blocks, kHubThreads, 0, s>>>(A, F, H);
                    LAUNCHCHK();
                }
            }
            if (H.count > 0 && !(fused && dense) && !kept_eval) {
                use_bucket(kHubBucket);
                if (dense) {
                    ProfScope ps("lp_refine_hub_dense", eval_bytes(P.count, cslots[c0 + kHubBucket]), s);
                    hub_dense_chunk_kernel<<<P.nchunks, kHubThreads, 0, s>>>(A, H);
                    LAUNCHCHK();
                } else {
                    if (!big) {
                        ProfScope ps(A.refine ? "lp_refine_hub_chunk" : "lp_eval_hub_chunk",
                                     eval_bytes(P.count, cslots[c0 + kHubBucket]), s);
                        hub_chunk_kernel<<<P.nchunks, kHubThreads, 0, s>>>(A, H);
                        LAUNCHCHK();
                    }
                    ProfScope ps(A.refine ? "lp_refine_hub_part" : "lp_eval_hub_part", 0, s);
                    hub_part_kernel<<<P.nparts, kPartThreads, 0, s>>>(A, H);
                    LAUNCHCHK();
                }
            }
            if (kept_eval && kr.to[sc] > kr.from[sc]) {
                double bytes;
                const int32_t blocks = lay_out(kHubBucket, kept_bucket, &bytes);
                {
                    // beside the upkeep and the kept rows, which are the longer chain
                    const hipStream_t bs = side ? evs.bucket(2) : s;
                    ProfScope ps("lp_refine_recount", 0, bs);
                    eval_recount_kernel<<<std::min(blocks, kRecountBlocks), 256, 0, bs>>>(A, F, H, blocks);
                    LAUNCHCHK();
                }
                use_bucket(kept_bucket);
                A.count = kr.to[sc] - kr.from[sc];
                ProfScope ps("lp_refine_kept", 4.0 * A.dense_k * A.count, s);
                if (A.dense_k <= 32) eval_kept_kernel<8><<<grid_for(A.count, 32), 256, 0, s>>>(A);
                else if (A.dense_k <= 64) eval_kept_kernel<16><<<grid_for(A.count, 16), 256, 0, s>>>(A);
                else if (A.dense_k <= 128) eval_kept_kernel<32><<<grid_for(A.count, 8), 256, 0, s>>>(A);
                else eval_kept_kernel<64><<<grid_for(A.count, 4), 256, 0, s>>>(A);
                LAUNCHCHK();
            }
            const int32_t bk_to = kept_eval ? kept_bucket : kHubBucket;
            for (int32_t bk = bk_from; bk < bk_to; ++bk) {
                const hipStream_t bs = side ? evs.bucket(bk) : s;
                const int64_t count = F.count[bk];
                if (count == 0) continue;
                use_bucket(bk);
                static const char* const kNames[2][kHubBucket] = {
                    {"lp_eval_lane4", "lp_eval_lane16", "lp_eval_group16", "lp_eval_group32", "lp_eval_wave",
                     "lp_eval_block1k", "lp_eval_block4k", "lp_eval_block8k"},
                    {"lp_refine_lane4", "lp_refine_lane16", "lp_refine_group16", "lp_refine_group32",
                     "lp_refine_wave", "lp_refine_block1k", "lp_refine_block4k", "lp_refine_block8k"}};
                ProfScope ps(kNames[A.refine][bk], eval_bytes(count, cslots[c0 + bk]), bs);
                const unsigned nb = static_cast<unsigned>(count);
                if (bk == 0) {
                    eval_lane_kernel<kLaneSmall><<<grid_for(count, 256), 256, 0, bs>>>(A);
                } else if (bk == 1) {
                    eval_lane_kernel<kLaneMax><<<grid_for(count, 256), 256, 0, bs>>>(A);
                } else if (dense) {  // refinement blocks: dense connection arrays
                    if (bk == 2) eval_dense_group_kernel<16><<<grid_for(count, 16), 256, 0, bs>>>(A);
                    else if (bk == 3) eval_dense_group_kernel<32><<<grid_for(count, 8), 256, 0, bs>>>(A);
                    else if (bk == 4) eval_dense_group_kernel<64><<<grid_for(count, 4), 256, 0, bs>>>(A);
                    else if (bk == 5) eval_dense_block_kernel<256><<<nb, 256, 0, bs>>>(A);
                    else if (bk == 6) eval_dense_block_kernel<512><<<nb, 512, 0, bs>>>(A);
                    else eval_dense_block_kernel<1024><<<nb, 1024, 0, bs>>>(A);
                } else if (bk == 2) {
                    eval_group_kernel<16, 2 * kG16Max><<<grid_for(count, 16), 256, 0, bs>>>(A);
                } else if (bk == 3) {
                    eval_group_kernel<32, 2 * kG32Max><<<grid_for(count, 8), 256, 0, bs>>>(A);
                } else if (bk == 4) {
                    eval_group_kernel<64, kWaveTable><<<grid_for(count, 4), 256, 0, bs>>>(A);
                } else if (bk == 5) {
                    eval_block_kernel<256, 2 * kBlock1Max, kBlock1Max / 256><<<nb, 256, 0, bs>>>(A);
                } else if (bk == 6) {
                    eval_block_kernel<1024, 2 * kBlock2Max, kBlock2Max / 1024><<<nb, 1024, 0, bs>>>(A);
                } else {
                    if (tune.block_table == kBlockTablePow2)
                        eval_block_kernel<1024, kBlockTablePow2, kBlockMaxDeg / 1024><<<nb, 1024, 0, bs>>>(A);
                    else
                        eval_block_kernel<1024, kBlockTable, kBlockMaxDeg / 1024><<<nb, 1024, 0, bs>>>(A);
                }
                LAUNCHCHK();
            }
            if (side) evs.join(s);

            // Entries per thread of the accumulating and admitting kernels: one
            // up to 2^16 entries, so that a small colour still has a workgroup
            // per 256 entries; more above, so that at most some 500 workgroups
            // add to the same counters and each thread has several loads in
            // flight.
            M.nodes = cnodes;
            M.count = static_cast<int32_t>(ccount);
            M.ctr = ctr + (step & 1);
            M.ctr_next = ctr + (~step & 1);
            M.gate = gate;
            M.round_cnt = rcnt.get() + r;
            M.host_cnt = sc == last_sub ? hrc + r : nullptr;
            M.colour = sc;
            ++step;
            const int per = ccount <= (1 << 16) ? 1 : (ccount <= (1 << 18) ? 4 : 8);
            const unsigned gc = static_cast<unsigned>(std::min<int64_t>(grid_for(ccount, 256 * per), kMaxBlocks));
            // every directly summing workgroup adds to every label
            const unsigned ga = direct ? std::min(gc, std::max(64u, static_cast<unsigned>(kMaxBlocks * kDirectLabels / nw))) : gc;
            {
                ProfScope ps(A.refine ? "lp_refine_admit" : "lp_admit", 0, s);
                if (!count_in_eval) {
                    auto accum = direct && nw > kDirectLabels ? accumulate_kernel<kSmallLabels, 8>
                                 : direct ? (per == 1   ? accumulate_kernel<kDirectLabels, 1>
                                             : per == 4 ? accumulate_kernel<kDirectLabels, 4>
                                                        : accumulate_kernel<kDirectLabels, 8>)
                                          : (per == 1   ? accumulate_kernel<0, 1>
                                             : per == 4 ? accumulate_kernel<0, 4>
                                                        : accumulate_kernel<0, 8>);
                    use_bucket(kHubBucket);
                    accum<<<ga + H.count, 256, 0, s>>>(A, H, ct.get(), cnodes, M.count - H.count, acc.get(), nw, g.heavy);
                    LAUNCHCHK();
                }
                auto admit = direct ? (nw > kDirectLabels ? admit_direct_kernel<kSmallLabels> : admit_direct_kernel<kDirectLabels>)
                             : per == 1 ? admit_kernel<1>
                             : per == 4 ? admit_kernel<4>
                                        : admit_kernel<8>;
                admit<<<std::min(gc, direct ? 256u : gc), 256, 0, s>>>(M);
                LAUNCHCHK();
            }
            if (trace) {
                uint32_t cands = 0;
                const ReadItem items[2] = {{&hctr, M.ctr, sizeof(Counters)},
                                           {&cands, rcnt.get() + r, sizeof(uint32_t)}};
                read_back(items, 2, s);
                const uint32_t slow = static_cast<uint32_t>(hctr.segs);
                fprintf(stderr, "[sclap] %s L%d r%d s%d n=%lld round cand=%u slow=%u targets=%u gain=[%d,%d] hubs=%d\n",
                        phase != kCluster ? "refine" : "cluster", level, r, sc, static_cast<long long>(ccount),
                        cands, slow, static_cast<uint32_t>(hctr.segs >> 32), slow ? hctr.gmin : 0,
                        slow ? hctr.gmax : 0, plans[sc].count);
            }
            {
                ProfScope ps("lp_apply", 0, s);
                const unsigned gseg = small ? std::max(kSegBlocksSmall, std::min(nw, kSegBlocks)) : kSegBlocks;
                const unsigned gmov = static_cast<unsigned>(std::min<int64_t>(
                    grid_for(ccount, kFinishThreads), small ? kMoveBlocksSmall : kMoveBlocks));
                auto finish = small ? (g.heavy ? finish_kernel<true, true> : finish_kernel<true, false>)
                                    : (g.heavy ? finish_kernel<false, true> : finish_kernel<false, false>);
                finish<<<gseg + gmov, kFinishThreads, 0, s>>>(M, gseg);
                LAUNCHCHK();
            }
            // a target has at most ccount candidates: no longer segment
            // unless the colour has more than the single-workgroup limit
            if (ccount > small_max) {
                ProfScope ps(A.refine ? "lp_refine_admit_select" : "lp_admit_select", 0, s);
                for (int launch = 0; launch < sel_launches; ++launch) {
                    auto pass = g.heavy ? large_pass_kernel<true> : large_pass_kernel<false>;
                    pass<<<kLargeBlocks, kLargeThreads, 0, s>>>(M.L, launch, sel_launches, bits_v, sent.get(),
                                                                swt.get(), M.ctr);
                    LAUNCHCHK();
                }
                if (small) large_move_kernel<true><<<kMaxBlocks, 256, 0, s>>>(M);
                else large_move_kernel<false><<<kMaxBlocks, 256, 0, s>>>(M);
                LAUNCHCHK();
            }
            if (keep) {
                M.fresh_limit = colour_slots / kFreshShare;
                up.ctr = M.ctr;
                up.gate = gate;
                upkeep_due = true;
            }
            if (A.quiet) {
                ProfScope ps("lp_unquiet", 0, s);
                unquiet_kernel<<<grid_for(ccount, 256), 256, 0, s>>>(ct.get(), label, cnodes,
                                                                      static_cast<int32_t>(ccount), g.xadj, g.adj,
                                                                      A.quiet, gate, rcnt.get(), r, n);
                LAUNCHCHK();
            }
        }
        // a round without candidates moved nothing (the first candidate of
        // every target is always admitted) and ends the run; its count, which
        // the last finish kernel wrote to host memory, is read while the next
        // round runs
        if (!capture) {
            HIPCHK(hipEventRecord(rev.ev[r & 1], s));
            if (r > 0) finish_round(r - 1);
        }
    }
    s = caller;
    if (capture) {
        rounds_graph.run();  // launches the graph on the caller's stream and waits for it
        for (int32_t q = 0; q < rounds && !halted; ++q) {
            res.rounds_run = q + 1;
            res.moves += hrc[q];
            if (hrc[q] == 0) halted = true;
        }
    } else if (!halted && rounds > 0) {
        finish_round(rounds - 1);
    }
    res.visits = static_cast<int64_t>(res.rounds_run) * g.S;
    HIPCHK(hipStreamSynchronize(s));
    if (profiler().on) profiler().collect();
    return res;
}

}  // namespace sclap
