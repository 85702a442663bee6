// Shared declarations between the host library and the HIP kernels of the
// biclique counter.  Device-side structures hold plain pointers into HBM.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bcdev {

typedef unsigned __int128 u128;

// One counting job: (graph side pair, p, q, root range) -> one result slot.
// "A" is the anchor side (L is drawn from it), "B" the other side.  Both CSRs
// are relabelled by rank, so orientation "w ranked after u" is "w > u".
struct Job {
    const uint64_t *ptrA;   // nA + 1
    const uint32_t *adjA;   // N(u) as sorted B ids
    const uint32_t *rposA;  // per edge u - v of adjA: position of u within N(v)
    const uint64_t *ptrB;   // nB + 1
    const uint32_t *adjB;   // N(v) as sorted A ids
    const u128 *binom;      // binom[n] = C(n, qA) for n in [0, binom_n)
    uint32_t nA, nB;
    uint32_t root_lo, root_hi;  // roots counted: ranks in [root_lo, root_hi)
    uint32_t pA, qA;
    uint32_t binom_n;       // table length (max degree of A + 1)
    uint32_t n_ovf;         // smallest n with C(n, qA) >= 2^128 (binom_n if none)
    uint32_t slot;          // result slot
    uint32_t n_u64;         // largest n with C(n, qA) < 2^64
    uint64_t deadline;      // device real-time clock tick after which the job gives up (0 = none)
    uint32_t n_u58;         // largest n with C(n, qA) < 2^58 (64 such values add up in 64 bits)
    uint32_t n_u28;         // largest n with C(n, qA) < 2^28 (16 such values add up in 32 bits)
    // hierarchical truncated bitmap of side A's rows (Section V-A): the row of
    // x is the 32-bit words htb_idx/htb_val[htb_off[x] .. htb_off[x+1]), word
    // i holding B ids 32i .. 32i+31 (bit j = id 32i + j); NULL when unused
    const uint64_t *htb_off;
    const uint32_t *htb_idx;
    const uint32_t *htb_val;
    // per-vertex counts of side A (two 64-bit words per vertex, by rank): the
    // bicliques each vertex is an L member of; NULL when not asked for (only
    // the global-set path fills them)
    uint64_t *pv;
    // the leaf tables of searches with 1 .. kColFixed vertices of side B fixed:
    // C(n, qA - 1), C(n, qA - 2), .., and where they pass the limits above
    struct {
        const u128 *binom;
        uint32_t n_ovf, n_u64, n_u58, n_u28;
    } less[3];
};

// One root of the global-set path (set intersections over the graph's own
// adjacency: HTB words or sorted id lists), in schedule order.
struct SetRoot {
    uint64_t id_off;        // its candidate ids: ids[id_off .. id_off + k)
    uint64_t task_begin;    // global index of its first task
    uint32_t job;
    uint32_t root;
    uint32_t k;
    uint32_t n_tasks;       // k - (pA - 2)
};

enum : uint32_t { SETS_HTB = 1, SETS_SORTED = 2 };

struct Slot;

struct SetParams {
    const Job *jobs;
    const SetRoot *roots;
    uint32_t n_roots;
    uint32_t task_chunk;
    uint64_t n_tasks;
    const uint32_t *ids;    // candidate ids of every root
    uint32_t mode;          // SETS_HTB or SETS_SORTED
    uint32_t instrument;
    uint32_t pure_dfs;      // nonzero: siblings one at a time, the lanes sharing each intersection
    uint32_t pad;
    uint64_t *slab;         // per-wave scratch
    uint64_t slab_words;
    unsigned long long *queue;
    Slot *slots;
};

// One root that owns enumeration tasks, in schedule (cost) order.
struct ActiveRoot {
    uint64_t pool_off;      // first word of its candidate rows in the pool
    uint64_t task_begin;    // global index of its first task
    uint32_t job;
    uint32_t root;          // anchor-side vertex (rank)
    uint32_t k;             // number of candidates (rows)
    uint32_t n_tasks;       // candidates that start a task, k - (pA - 2), times shares
    uint32_t shares;        // tasks each of these is shared out to, by its child rows (p_A >= 5; else 1)
    uint32_t pad;
};

// One root of the column search, in schedule order: its candidate rows
// transposed (one bitmap over the candidates per neighbour of the root), and
// either one unit that counts the whole root or one unit per neighbour.
struct ColRoot {
    uint64_t col_off;       // word w of column c is cols[col_off + w * du + c]
    uint64_t pool_off;      // its candidate rows in the pool
    uint64_t unit_begin;    // global index of its first unit
    uint32_t job;
    uint32_t k, du, wk;     // candidates, neighbours (columns), words per column
    uint32_t n_units;       // 1 (whole root) or du - (qA - 1): columns du - 1, du - 2, ...
    uint32_t whole;
};

// Result slot: exact 128-bit count as two 64-bit limbs plus status flags.
struct Slot {
    unsigned long long lo, hi;
    unsigned int flags;     // FLAG_* bits
    unsigned int pad;
    unsigned long long pair_ops, filter_ops;
    unsigned long long cyc_setup, cyc_compact, cyc_pair, cyc_filter;   // instrumented shader-clock sums
    unsigned long long pairs, pair_slots;   // instrumented: leaf pairs, and lane-slots spent on them
    unsigned long long cyc_pack;            // instrumented: compaction cycles of tasks that bit-pack S2
    unsigned long long pad3;
};

enum : unsigned {
    FLAG_OVERFLOW = 1u,     // count does not fit in 128 bits
    FLAG_CAPACITY = 2u,     // a scratch bound computed on the host was exceeded
    FLAG_MISMATCH = 4u,     // candidate count differs between the two wedge passes
    FLAG_TIMEOUT = 8u,      // the job's deadline passed before it finished
    FLAG_POOL = 16u,        // the row pool was too small for some root (rows built again)
};

constexpr int kWaveSize = 64;
constexpr int kWavesPerBlock = 4;
constexpr uint32_t kTripleRows = 96;   // nodes up to this many rows finish their last three levels at once
constexpr int kBlockThreads = kWaveSize * kWavesPerBlock;
constexpr uint32_t kColMax = 128;      // widest column search, in columns: lanes hold pairs,
constexpr uint32_t kColTripleMax = 64; // triples,
constexpr uint32_t kColQuadMax = 40;   // tuples of four,
constexpr uint32_t kColQuintMax = 28;  // or of five
constexpr uint32_t kColWords = 40;     // longest column searched, in 64-bit words
constexpr uint32_t kColBuf = 960;      // LDS words for a wave's columns
constexpr uint32_t kColMinQ = 2, kColMaxQ = 6;   // columns chosen
constexpr uint32_t kColMinP = 2, kColMaxP = 5;   // rows chosen
constexpr uint32_t kColRootWords = 64;     // longest column of a root searched unit by unit
constexpr uint32_t kColRootPlanes = 16;    // and its widest row, in 64-bit words
constexpr uint32_t kColFixed = 3;          // most columns fixed in a unit
constexpr uint32_t kColLessLen = 64 * kColRootPlanes + 1;   // entries of a unit's leaf table, if so many
constexpr uint32_t kNoJ = 0xffffffffu;     // no restriction to one child
constexpr uint32_t kOneChild = 0x40000000u;   // step of a child loop that ends after one
constexpr uint32_t kMaxShares = 64;        // most tasks a candidate's search is shared out to
constexpr int kSortCap = 4096;          // candidates sorted in LDS up to this many
constexpr int kRbWaves = 8;             // waves per large block of the fused per-root kernel
constexpr uint32_t kRbBigPerCu = 2;     // large blocks of it on a CU
constexpr int kRbWideWaves = 16;        // waves per wide block, one on a CU
constexpr uint32_t kRbWideDegree = 32768;   // widest root of a job from which on the large roots take wide blocks
static_assert(kRbWideDegree <= 65536, "large blocks count in 16 bits");
constexpr uint32_t kRbManyWedges = 32768;   // wedges a root has on average for which small blocks are not tried
constexpr uint32_t kRbSmallPerCu = 5;   // small blocks (four waves)
constexpr uint32_t kQueues = 16;        // counters of a task queue,
constexpr uint32_t kQueueStride = 16;   // this many 64-bit words apart
constexpr uint32_t kQueueWords = kQueues * kQueueStride;
constexpr uint32_t kSlotFlag = 0x80000000u;

constexpr uint32_t kShapeDegree = 32;   // neighbours past which a root's fill and spread are taken
constexpr float kSpreadUnit = 4096.0f;

// What the candidate pass finds of one root.
struct RootOut {
    uint64_t off;           // first word of its rows in the pool (~0: no rows)
    uint32_t k;             // candidates
    // of roots of more than kShapeDegree neighbours, from k_root_build (else 0):
    uint16_t fill;          // share of the rows' bits that are set, times 65535
    uint16_t spread;        // variance of the rows' bit counts over their mean squared, times kSpreadUnit, at most 65535
};

// Row storage of the candidate pass: each block reserves kRowChunk pool words at
// a time and hands them out, rows longer than an eighth of that are reserved by
// themselves.  So less than an eighth of a used-up chunk is left over, and a pool
// of row_pool_words(w, n) words serves n blocks whatever roots of w words in all
// they meet, in any order.
constexpr uint32_t kRowChunk = 4096;
__host__ __device__ constexpr uint64_t row_pool_words(uint64_t w, uint64_t n_blocks) { return w + w / 7 + n_blocks * kRowChunk + 1; }
struct RowChunk {
    unsigned long long at, end;
};
// The offset of need words of a pool of cap, ~0 if there is no room.  chunk:
// words reserved at once; reserve(n): the pool's head before it advanced by n.
template <typename F>
__host__ __device__ __forceinline__ unsigned long long take_rows(RowChunk &c, uint64_t need, uint64_t chunk, uint64_t cap, F reserve)
{
    if (8 * need > chunk) {
        const unsigned long long o = reserve(need);
        return o + need <= cap ? o : ~0ull;
    }
    if (c.end - c.at < need) {
        const unsigned long long o = reserve(chunk);
        if (o + chunk > cap) {
            c.at = c.end = 0;
            return o + need <= cap ? o : ~0ull;
        }
        c.at = o;
        c.end = o + chunk;
    }
    c.at += need;
    return c.at - need;
}

struct RootScratch {
    uint32_t *cnt;          // per block: nA_max counters, all zero between roots
    uint32_t *touched;      // per block: nA_max touched ids
    uint32_t *cand;         // per block: nA_max candidate ids (when k > kSortCap)
    uint64_t stride;        // elements per block in each array
};

struct RootParams {
    const Job *jobs;
    const uint64_t *job_root_prefix;   // first item of each job
    uint32_t n_jobs;
    uint32_t run, period;              // a job's items: `run` ranks out of every `period` (run 0: all)
    uint64_t total_roots;
    RootScratch sc;                    // of the large blocks
    uint64_t *pool;                    // candidate rows
    uint64_t pool_cap;                 // words
    uint64_t chunk;                    // pool words a block reserves at once (0: what each root needs)
    unsigned long long *pool_head;
    unsigned long long *queue;         // items of the first launch
    unsigned long long *queue_big;     // of the second
    unsigned long long *n_retry;       // roots left to the large blocks
    uint32_t *retry;                   // their items
    const uint32_t *list;              // items of the launch (null: all)
    const unsigned long long *n_list;
    RootOut *out;
    Slot *slots;
};

struct ColParams {
    const Job *jobs;
    const ColRoot *roots;
    uint32_t n_roots;
    uint32_t n_whole;       // roots [0, n_whole) are one unit each, taken one by one
    uint32_t unit_chunk;    // consecutive units of the other roots taken per queue pop
    uint32_t instrument;
    uint32_t timed;         // some job has a deadline
    uint64_t n_units;       // units of roots [n_whole, n_roots), or room in `units`
    const uint64_t *pool;   // candidate rows
    uint64_t *cols;         // candidate columns (k_transpose writes, k_columns reads)
    unsigned long long *queue;
    uint64_t *slab;         // per-wave columns that exceed the LDS (NULL: none may)
    // listed units are {root, col_pack of the fixed columns}
    const uint2 *units;     // the units of a later run (NULL: those of the roots)
    const unsigned long long *n_listed;   // and their number
    uint2 *split;           // units split by a further column (NULL: none are)
    unsigned long long *n_split;
    uint64_t split_cap;     // room in split
    uint4 *left;            // units that the row search takes: the same, and one child row or kNoJ
    unsigned long long *n_left;
    uint64_t left_cap;      // room in left: every unit fits, and a heavy one's children if they do
    uint64_t left_room;     // its entries: the long units lie from the end down,
    unsigned long long *n_long;   // this many
    uint32_t deep;          // a deep run may take them
    Slot *slots;
};

struct EnumParams {
    const Job *jobs;
    const ActiveRoot *roots;
    uint32_t n_roots;
    uint32_t task_chunk;    // consecutive tasks taken per queue pop (>= 1)
    uint64_t n_tasks;
    // the column search's roots and the units that it left to the row search
    // (the instances with COLS): task t is left[t * left_step], t < *n_left
    const ColRoot *col_roots;
    const uint4 *left;
    const unsigned long long *n_left;
    int32_t left_step;      // 1, or -1 for the long units (from the list's end down)
    const uint64_t *cols;
    const uint64_t *pool;
    uint64_t *slab;         // per-wave global scratch
    uint64_t slab_words;    // words per wave
    uint32_t lds_words;     // per-wave LDS words actually used (<= compiled cap)
    uint32_t instrument;
    uint32_t triple;        // nonzero: small nodes three levels above the leaves take the triple sweep
    uint32_t split_rows;    // level-2 blocks with more rows are split into queued subtasks
    uint32_t split_cap;     // subtask ring entries (0 = no splitting)
    uint4 *ring;            // subtask ring, split_cap entries, all zero at launch
    unsigned long long *sub_head;   // [0] subtask entries claimed, [2] split heap words taken (zero at launch)
    unsigned long long *sub_tail;   // subtask entries reserved (zero at launch)
    uint64_t *split_heap;   // level-2 blocks of split tasks
    uint64_t split_heap_words;
    unsigned long long *wave_clock; // instrumented: per wavefront {first task start, end} device clock ticks
    unsigned long long *queue;   // task counter: tasks popped in the low 40 bits; with splitting on,
                                 // wavefronts still running a popped chunk in the bits above
    Slot *slots;
};

// Launchers (defined in bc_kernels.hip).  All run on `stream` and return the
// launch status.
hipError_t launch_fill_u32(uint32_t *p, uint64_t n, uint32_t v, hipStream_t stream);
hipError_t launch_fill_slots(Slot *slots, uint32_t n, hipStream_t stream);
hipError_t launch_degree_sum(const Job *jobs, const uint32_t *job_ids, uint32_t n_jobs,
                             Slot *slots, hipStream_t stream);
hipError_t launch_cand_count(const Job *jobs, const uint64_t *job_root_prefix, uint32_t n_jobs,
                             uint64_t total_roots, RootScratch scratch, uint32_t n_blocks,
                             unsigned long long *queue, RootOut *out, Slot *slots, hipStream_t stream);
// LDS of the largest block of launch_root_build.
uint32_t root_build_lds();
// Candidate counts and rows in one kernel; rows go to pool[out[r].off ..]
// (bump-allocated from *pool_head, capacity pool_cap words).  n_small blocks of
// four waves take every root and list those too large for them in retry; then
// n_big large or wide blocks take these (n_small 0: all).  Large blocks: no root
// of kRbWideDegree neighbours or more.
hipError_t launch_root_build(const RootParams &prm, uint32_t n_small, uint32_t n_big, bool wide, bool per_vertex,
                             hipStream_t stream);
hipError_t launch_rows_build(const Job *jobs, const ActiveRoot *roots, uint32_t n_roots,
                             uint64_t *pool, RootScratch scratch, uint32_t n_blocks,
                             unsigned long long *queue, Slot *slots, hipStream_t stream);
hipError_t launch_enumerate(const EnumParams &prm, uint32_t n_blocks, hipStream_t stream);
// The column search: k_transpose writes the columns of n_roots roots, k_columns
// counts their units and lists those that the row search has to take.
hipError_t launch_columns(const ColParams &prm, uint32_t n_blocks, hipStream_t stream);
// The long units that k_columns left: to the row search's list, or searched by
// columns after all.
hipError_t launch_columns_long(const ColParams &prm, uint32_t n_blocks, hipStream_t stream);
// The row search over the units listed by k_columns.
hipError_t launch_enumerate_left(const EnumParams &prm, uint32_t n_blocks, hipStream_t stream);
// Candidate ids of the global-set roots: for root r, the w > u sharing >= qA
// neighbours with u, in no particular order, written to ids[roots[r].id_off ..].
hipError_t launch_cand_ids(const Job *jobs, const SetRoot *roots, uint32_t n_roots, uint32_t *ids,
                           RootScratch scratch, uint32_t n_blocks, unsigned long long *queue, Slot *slots,
                           hipStream_t stream);
hipError_t launch_enumerate_sets(const SetParams &prm, uint32_t n_blocks, hipStream_t stream);

uint32_t max_lds_words_per_wave();

// The columns fixed in a unit, the last of its subsets first: ten bits each,
// all ones for none.
constexpr uint32_t kColNone = 1023;
constexpr uint32_t kColRootMax = kColNone;   // most neighbours of a root searched unit by unit: columns 0 .. kColNone - 1
static_assert(kColRootMax <= kColNone && kColRootMax <= 64 * kColRootPlanes, "a column's number is never kColNone");
__host__ __device__ constexpr uint32_t col_pack(uint32_t x, uint32_t y, uint32_t z) { return x | (y << 10) | (z << 20); }
__host__ __device__ constexpr uint32_t col_fixed(uint32_t pack, uint32_t i) { return (pack >> (10 * i)) & kColNone; }
// Whether a root of du neighbours and wk words of candidates can be searched unit by unit.
__host__ __device__ constexpr bool col_root_fits(uint32_t du, uint32_t wk) { return du <= kColRootMax && wk <= kColRootWords; }

// The column search chooses q of s columns of nw words.  It searches
// col_words words of them, kept col_stride words apart (two words more, so
// that the lanes' reads of different columns fall on different LDS banks, 20
// banks apart at eight words, and an even number for 16-byte reads), in LDS or,
// past kColBuf words, in the wave's slab (16 words and more only).
// col_loops of the q columns run through loops, each of which keeps one more
// AND in registers (hence fewer for long columns); the lanes hold tuples of
// the rest.
__host__ __device__ constexpr uint32_t col_stride(uint32_t nc) { return nc + 2; }
__host__ __device__ constexpr uint32_t col_words(uint32_t nw, uint32_t s)
{
    const uint32_t nc = nw <= 8 ? (nw + 1) & ~1u : nw <= 12 ? 12u : nw <= 16 ? 16u : nw <= 24 ? 24u : 40u;
    return nc < 16 && s * col_stride(nc) > kColBuf ? 16u : nc;
}
__host__ __device__ constexpr uint32_t col_loops(uint32_t q, uint32_t nc, uint32_t s)
{
    const uint32_t want = s > kColTripleMax ? (q > 2 ? q - 2 : 1) : q <= 4 ? 1 : q - 3;
    const uint32_t most = nc <= 8 ? 3 : nc <= 16 ? 2 : 1;
    return want < most ? want : most;
}
constexpr uint64_t kColSlabWords = (uint64_t)kColMax * (kColWords + 2);   // per wave

// Whether it can: q columns, room, tuple tables.
__host__ __device__ constexpr bool col_fits(uint32_t s, uint32_t nw, uint32_t q, bool slab)
{
    if (q < kColMinQ || q > kColMaxQ || s > kColMax || nw > kColWords) return false;
    const uint32_t nc = col_words(nw, s), R = q - col_loops(q, nc, s);
    return s <= (R <= 2 ? kColMax : R == 3 ? kColTripleMax : R == 4 ? kColQuadMax : kColQuintMax) &&
           (slab || s * col_stride(nc) <= kColBuf);
}

__host__ __device__ constexpr uint64_t choose(uint64_t n, uint32_t k)
{
    if (n < k) return 0;
    uint64_t c = 1;
    for (uint32_t i = 0; i < k; ++i) c = c * (n - i) / (i + 1);
    return c;
}

// Steps of the search with D loops: lane tuples, steps of the innermost loop
// and of the loops around it.  The lanes take the tuples of R = q - D columns
// that leave D behind them, 64 a round in colexicographic order (so that the
// tuples with a last column below x are the first choose(x, R)), and a round's
// loops start behind its first tuple's last column.
struct ColCost {
    uint32_t tuples, leaf, outer;
};
struct ColCosts {
    ColCost at[kColMaxQ - kColMinQ + 1][3][kColMax + 1];
    __host__ __device__ constexpr const ColCost &of(uint32_t q, uint32_t D, uint32_t s) const
    {
        return at[q - kColMinQ][D - 1][s];
    }
};
constexpr ColCosts make_col_costs()
{
    ColCosts t{};
    for (uint32_t q = kColMinQ; q <= kColMaxQ; ++q)
        for (uint32_t D = 1; D <= 3 && D < q; ++D)
            for (uint32_t s = q; s <= kColMax; ++s) {
                const uint32_t R = q - D;
                uint64_t leaf = 0, outer = 0, base = 0;
                for (uint32_t last = R - 1; last + D < s; ++last) {
                    const uint64_t n = s - 1 - last, end = choose(last + 1, R);
                    const uint64_t rounds = base < end ? (end - base + kWaveSize - 1) / kWaveSize : 0;
                    base += rounds * kWaveSize;
                    leaf += rounds * choose(n, D);
                    for (uint32_t d = 1; d < D; ++d) outer += rounds * choose(n, d);
                }
                ColCost &c = t.at[q - kColMinQ][D - 1][s];
                c.tuples = (uint32_t)choose(s - D, R);   // below 2^32 wherever col_fits
                c.leaf = leaf < 0xffffffffu ? (uint32_t)leaf : 0xffffffffu;
                c.outer = outer < 0xffffffffu ? (uint32_t)outer : 0xffffffffu;
            }
    return t;
}

// Estimated wave instructions of the search with tuples of R columns of nc words.
__host__ __device__ constexpr uint64_t col_estimate(const ColCost &c, uint64_t nc, uint32_t R)
{
    return c.leaf * (4 * nc + 8) + c.outer * (6 * nc + 8) + (c.tuples + 63) / 64 * (2 * R * nc + 40) + 100;
}

// Estimated wave instructions of the row search over m rows choosing p: one
// 16 x 16 product of pair sizes with its table reads costs about as much as
// 30 VALU instructions; below the pairs of the last list its nodes' own work
// dominates (measured at p = 4: six times the products).
__host__ __device__ constexpr uint64_t row_estimate(uint64_t m, uint32_t p)
{
    return p <= 1 ? m / 4 + 40 : p == 2 ? m * m / 17 + 60 : p == 3 ? m * m * m / 42 + 100
         : p == 4 ? m * m * m * m / 43 + 100 : m * m * m * m * m / 100 + 100;
}

// Reads the device real-time clock (s_memrealtime) into *out (device memory).
hipError_t launch_read_clock(uint64_t *out, hipStream_t stream);

}  // namespace bcdev
