// mce_internal.h -- types shared by the device kernels and the host runtime of
// libmce.so.  Not part of the public ABI (include/mce.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mce {

constexpr uint32_t kMaxN = 16384;
// Per-wavefront clique buffer in LDS: each buffered clique is the list of the
// non-empty 16-bit halves of its input-id bitset, one word per half
// (half index << 16 | bits), in increasing order; at most 64 cliques.
constexpr uint32_t kCliqueSlots = 512;
// Per-wavefront LDS histogram; larger clique sizes go straight to HBM.
constexpr uint32_t kHistLds = 64;
// Words at the head of a queue record: graph index; of a root unit, its pieces
// (16 bits, 0: one) and the number of this piece.
constexpr uint32_t kRecHeader = 2;
// Per-workgroup LDS: a header and a LIFO of units shared by its wavefronts.
constexpr uint32_t kWgHdrWords = 16;
constexpr uint32_t kLocalSlots = 8;
// LDS words of a wavefront before its frames: histogram (kHistLds u64), the
// clique buffer (kCliqueSlots words), 64 words that absorb the stores of lanes
// with nothing to store, a 32-word context block and a 128-word save area for
// the search loop's lane registers.  Then come the stack window, the slot of
// the current frame and some slack (lds_frame_words).
constexpr uint32_t kWaveFixedWords = kHistLds * 2 + kCliqueSlots + 64 + 32 + 128;

// Wavefront-lane layout of the search: one 32-bit word per lane and chunk.
// A graph with w32 + 1 <= 64 row words (n <= 2016) uses one chunk, larger ones
// two (the +1 is the input-id word of a row, read while w32 < 128), then four
// (n <= 8160) and eight (n <= kMaxN).
constexpr uint32_t kOneChunkMaxW32 = 63;
inline uint32_t search_chunks(uint32_t max_w32)
{
    return max_w32 <= kOneChunkMaxW32 ? 1u : max_w32 <= 127u ? 2u : max_w32 <= 255u ? 4u : 8u;
}

// Wavefronts per search workgroup at most: four for the wide layouts, whose
// registers per lane would not fit four wavefronts per SIMD.
constexpr uint32_t max_search_wpb(uint32_t chunks) { return chunks >= 4u ? 4u : 16u; }

// Lane search (search_kernel with LANE): a node whose P u X has at most
// kLaneMaxM vertices, and with R at most kLaneMaxS, is searched by all 64
// lanes on bitsets of its own vertices (two to four 32-bit words a lane).
// Its LDS area, after the wavefront's frames: the lanes' stacks
// (kLaneStackWords: frames of 2 N words a lane; at first the node's P, X, L and
// R are there), the rows of the node's subgraph (128 x 4 words), the vertices'
// ranks by input id and the node's candidates (128 bytes each), the input ids
// by rank (128 words), R's ranks (4 words) and what a bundle says of its node (4).
constexpr uint32_t kLaneMaxM = 121, kLaneMaxS = 128;
constexpr uint32_t kLaneStackWords = 1536;
constexpr uint32_t kLaneAreaWords = kLaneStackWords + 512 + 32 + 32 + 64 + 8;
// Lanes on their way to another workgroup, a record in HBM (rows of 64 words):
// each lane's state word, the tables of the lane area (4 rows), the rows of the
// subgraph (at most 8), L and R (2 N), the stacks.
constexpr uint32_t kBundleTables = 1, kBundleAdj = 5, kBundleWords = 64 * (5 + 8 + 8) + kLaneStackWords;
// A lane's frames below its LDS stack (kLaneStackWords / (128 N) frames) go
// to the wavefront's part of a buffer in HBM: levels of this many words.
constexpr uint32_t kLaneLevelWords = 64 * 2 * 4;
// Such levels a wavefront has at first, and at most (one a vertex of P).
constexpr uint32_t kLaneLevelsFirst = 16, kLaneLevelsFull = 124;

// Pieces of each of a batch graph's `units` root units that wants `chop` of
// them: every piece after a unit's first takes one of the pool's `limit` spare
// slots, of which the graphs before it asked for `asked` (granted or not).
// In 64 bits: the sum of what 2^32 graphs can ask for does not wrap, so all
// that is granted together fits in `limit`.
__host__ __device__ inline uint32_t pieces_granted(uint64_t asked, uint32_t units, uint32_t chop, uint32_t limit)
{
    return asked + (uint64_t)units * (chop - 1u) <= limit ? chop : 1u;
}

// What a lane search has counted since it last added to the wavefront's 64-bit
// totals.  A call ends with its node's tree, which has no bound (a Moon-Moser
// graph of 84 vertices is one node with 3^28 cliques below it), so the counts
// are added whenever they are due at a look, and a look comes after at most
// kLaneLookMax steps of 64 children.  (Held in 64 bits to the end of the call
// they cost batches of graphs 1% by their registers.)
constexpr uint32_t kLaneLookMax = 1u << 20;
struct LaneTotals {
    uint32_t children = 0, nodes = 0, cliques = 0;
    // one child of every busy lane: so many, and so many of them nodes
    __host__ __device__ void step(uint32_t c, uint32_t n)
    {
        children += c;
        nodes += n;
    }
    // (nodes and cliques are children too)
    __host__ __device__ bool due() const { return children >= 1u << 31; }
    template <class T> __host__ __device__ void add_to(T& t)
    {
        t.count += cliques;
        t.nodes += nodes;
        t.children += children;
        children = nodes = cliques = 0;
    }
};
static_assert((1ull << 31) + 2ull * 64 * kLaneLookMax < 1ull << 32, "LaneTotals");

// LDS stack frame (P, X, L and the row of the frame's next candidate,
// interleaved per lane, 16 bytes a lane): words per frame, and the slack after
// the last frame that absorbs the accesses of lanes past the row.  With one
// chunk a frame spans lanes 0..max_w32, so that the row's input-id word (lane
// w32) is kept.
inline uint32_t lds_frame_words(uint32_t max_w32)
{
    return search_chunks(max_w32) == 1 ? 4u * (max_w32 + 1u) : 256u * search_chunks(max_w32);
}
inline uint32_t lds_slack_words(uint32_t max_w32)
{
    return search_chunks(max_w32) == 1 ? 4u * (63u - max_w32) : 0u;
}
// Spill frame in HBM: (P, X, L, child id) per lane, 16 bytes a lane, all lanes.
inline uint32_t spill_frame_words(uint32_t max_w32) { return 256u * search_chunks(max_w32); }

// Stacks of a search in HBM: chunks of the spill pool (for levels of a
// wavefront's loop below its LDS window), levels a chunk holds, and levels of
// the lanes' stacks a wavefront has.
struct StackPlan {
    uint32_t levels, chunks, lane_levels;
};
// What searches of a handle were found to need beyond the first plan (each set
// by its own error bit: what one stack needs says nothing about the other).
struct StackNeeds {
    uint32_t chunks = 0;     // spill chunks (kErrSpill: one for every wavefront)
    bool deep = false;       // chunks of the full stack depth (kErrDepth)
    bool lanes_deep = false; // all the lanes' levels (kErrLaneDepth)
    bool operator==(const StackNeeds& o) const
    {
        return chunks == o.chunks && deep == o.deep && lanes_deep == o.lanes_deep;
    }
};
// Levels a spill chunk holds at first: enough for every search of these
// workloads.  With lanes the LDS window is of few levels (the lanes' stacks have
// most of the LDS) and any wavefront may need a chunk: each has one, of fewer
// levels.  Else 64 wavefronts have one on first use.
constexpr uint32_t kSpillLevelsFirst = 64, kLaneSpillLevelsFirst = 32, kSpillChunksFirst = 64;
// Chunks of the full depth with lanes: as many as fit in this, or 64 (n = 1000:
// 268; one for each of 3072 wavefronts would be 3 GB, and few searches have
// more than a few deep wavefronts).
constexpr uint64_t kDeepSpillBytes = 256ull << 20;
// full_levels: the stack's levels below the LDS window; frame_bytes: of one.
inline StackPlan plan_stacks(bool lanes, uint32_t waves, uint32_t full_levels, uint64_t frame_bytes, const StackNeeds& need)
{
    StackPlan p;
    p.levels = full_levels ? full_levels : 1u;
    const uint32_t first = lanes ? kLaneSpillLevelsFirst : kSpillLevelsFirst;
    uint64_t chunks = kSpillChunksFirst;
    if (need.deep) {
        if (lanes && kDeepSpillBytes / (frame_bytes * p.levels) > chunks) chunks = kDeepSpillBytes / (frame_bytes * p.levels);
    } else {
        if (p.levels > first) p.levels = first;
        if (lanes) chunks = waves;
    }
    if (chunks < need.chunks) chunks = need.chunks;
    p.chunks = (uint32_t)(chunks < waves ? chunks : waves);
    p.lane_levels = !lanes ? 0u : need.lanes_deep ? kLaneLevelsFull : kLaneLevelsFirst;
    return p;
}

// Cuts a plan to an area of fixed size, both stacks one after the other in it:
// with lanes every wavefront has a chunk, of fewer levels at first (down to
// kFixedSpillLevels) rather than fewer wavefronts; without, as many chunks as
// fit, and no more wavefronts than those once each needs one.  Returns the
// wavefronts that can run, at most `waves` (0: not one).
constexpr uint32_t kFixedSpillLevels = 4;
inline uint32_t fit_stacks(bool lanes, uint64_t area, uint32_t waves, uint64_t frame_bytes, const StackNeeds& need,
                           StackPlan* p)
{
    const uint64_t lane_bytes = 4ull * kLaneLevelWords * p->lane_levels;
    uint64_t w = waves;
    if (!lanes) {
        const uint64_t fit = area / (frame_bytes * p->levels);
        if (need.chunks != 0 && w > fit) w = fit;
        const uint64_t chunks = p->chunks < w ? p->chunks : w;
        p->chunks = (uint32_t)(chunks < fit ? chunks : fit);
        return p->chunks ? (uint32_t)w : 0u;
    }
    uint64_t least = p->levels;
    if (!need.deep && least > kFixedSpillLevels) least = kFixedSpillLevels;
    const uint64_t fit = area / (lane_bytes + frame_bytes * least);
    if (w > fit) w = fit;
    if (w == 0) return 0;
    const uint64_t levels = (area / w - lane_bytes) / frame_bytes;
    if (p->levels > levels) p->levels = (uint32_t)levels;
    p->chunks = (uint32_t)w;
    return (uint32_t)w;
}

// One graph of a handle, in device memory.
struct GraphDesc {
    uint32_t n;        // vertices
    uint32_t w32;      // 32-bit words of a bitset, ceil(n/32)
    uint32_t rw64;     // uint64 words of an input row, ceil(n/64)
    uint32_t rstride;  // uint32 words between renumbered rows: w32 + 1 (the last word of a
                       // row holds the vertex's input id)
    uint64_t in_off;   // first uint64 word of the input rows
    uint64_t adj_off;  // first uint32 word of the renumbered rows (row stride rstride)
    uint64_t ord_off;  // first entry of order[] (position -> input id)
    uint64_t hist_off; // first entry of the graph's histogram (n + 1 entries)
    // Local graphs (the root children of a sparse graph of more than 4096
    // vertices, each solved on the subgraph its neighbourhood induces): the
    // ids of a local graph are local ranks, reported through idmap; an
    // ordinary graph has idmap_off = kNoMap.
    uint64_t idmap_off; // first entry of the id map (local id -> input id), or kNoMap
    uint32_t res;       // the DevResult (and histogram) the graph's totals go to
    uint32_t pad;
};
// For a local graph, rw64 holds the root child's position in the whole graph
// and in_off the first word of its node's P and X bitsets (w32 words each,
// local positions) followed by the root child's own local id, in lpx.
constexpr uint64_t kNoMap = ~0ull;
// Vertices of a local graph at most (one-chunk layout: w32 + 1 <= 64).
constexpr uint32_t kLocalMaxN = 2016;
static_assert(sizeof(GraphDesc) == 64, "GraphDesc layout");

// Per-graph totals, accumulated with device atomics.
struct DevResult {
    unsigned long long count, nodes, children, dead_ends, hash_xor, hash_sum;
    unsigned long long root_branches;
    unsigned int omega, status;
    unsigned int unit_base, unit_count; // queue slots of the graph's root units
    unsigned int unit_chop, pad;        // pieces of each root unit
};

// Control block of one search launch.  Words written by many workgroups sit
// on cache lines of their own.
struct QueueCtl {
    unsigned int pool_next, pad_h[31]; // next root unit to hand out
    unsigned int pool_size; // root units written by the root kernels
    unsigned int chop;      // pieces each of a single graph's is handed out in (0: one)
    unsigned long long extra; // pool slots asked for by pieces of a batch's graphs, refused ones too
    unsigned int pad_t[28];
    unsigned int work, pad_w[31];      // root units not handed out + units in transit
                                       // + workgroups holding work; the search ends at 0
    unsigned int error, pad_e[31];
    unsigned long long donations, units;
    unsigned long long spill_next;           // next free chunk of the spill pool
    unsigned long long spill_levels_written; // stack levels stored in HBM
    unsigned long long checks, flushes;      // suspensions of the search loop, by reason
    unsigned long long busy_ticks, run_ticks; // wall-clock ticks on units / from start to exit, all wavefronts
    unsigned long long ramp_ticks, tail_ticks; // before the first unit / after the last one
    // enumerate output cursors, a cache line each: every flush of a clique
    // buffer adds to both, and with lanes most flushes are of a few cliques (the
    // end of a small node).  On one line enumerate of G(2016, 0.15) took 4.87 ms,
    // on two 2.51 (2.87 before the lanes), G(600, 0.2) 0.46 and 0.32 (0.49).
    unsigned long long pad_v[16];
    unsigned long long vcursor, pad_o[15];
    unsigned long long ocursor, pad_x[15];
};

// Mailbox of one search workgroup in HBM.  A workgroup out of work asks one
// other workgroup at a time: it writes its id + 1 into that workgroup's req
// word (compare-and-swap from 0), and the asked workgroup answers in the
// asker's state word: a unit (copied to the asker's record slot first) or a
// refusal.  The hint word says how many of the workgroup's wavefronts were
// busy when it last looked (0 when it holds no work), so that askers can
// prefer busy workgroups.  Each word has a cache line of its own.
struct Mailbox {
    unsigned int req, pad_r[31];   // asking workgroup + 1, 0: none
    unsigned int state, pad_s[31]; // answer to this workgroup's own question
    unsigned int hint, pad_b[31];  // busy wavefronts (a hint, written by the owner only)
};
constexpr unsigned int kMailNone = 0u, kMailUnit = 1u, kMailRefused = 2u, kMailBundle = 3u;

// Exit record of one search wavefront: its totals of the graph it worked on
// last (not yet added to that graph's result slot) and its counters.  The
// exit-fold kernel that runs after the search adds the records up, so that the
// wavefronts, which leave within microseconds of each other, issue no atomics
// on the same few words at once.
constexpr unsigned int kNoSlot = 0xffffffffu;
struct WaveExit {
    unsigned int res, omega; // result slot (kNoSlot: the wavefront held no graph), largest clique
    unsigned long long hist_off; // where hist adds into SearchParams.hist
    unsigned long long count, nodes, children, hash_xor, hash_sum;
    unsigned long long units, donations, spills, checks, flushes; // QueueCtl counters
    unsigned long long busy, run, ramp, tail;                     // wall-clock ticks (QueueCtl *_ticks)
    unsigned long long hist[kHistLds];
};
static_assert(sizeof(WaveExit) == 8 * (16 + kHistLds), "WaveExit layout");

// QueueCtl.error bits
constexpr unsigned int kErrSpill = 1u; // spill pool exhausted: rerun with a larger pool
constexpr unsigned int kErrDepth = 2u; // stack deeper than a spill chunk: rerun with chunks of full depth
constexpr unsigned int kErrLaneDepth = 64u; // a lane's stack deeper than its levels in HBM: rerun with all of them
constexpr unsigned int kErrWatchdog = 4u; // the search ran past its deadline
constexpr unsigned int kErrCancel = 16u;  // the host asked the search to stop (SearchParams.cancel)
constexpr unsigned int kErrClique = 8u;   // a clique with more non-empty 16-bit id groups than the
                                          // clique buffer's slots (only possible for n > 8192)
constexpr unsigned int kErrPool = 32u;    // root units past the pool's end (none is written there): a fault
                                          // in the host's or the root kernels' arithmetic

struct SearchParams {
    const GraphDesc* graphs;
    const uint32_t* adj;
    const uint32_t* order;
    DevResult* results;
    unsigned long long* hist;
    QueueCtl* ctl;
    uint32_t* rec;            // root units, cap * rec_words
    Mailbox* mail;            // one per workgroup
    uint32_t* mail_rec;       // one record slot per workgroup, rec_words each
    uint32_t* spill;          // per wavefront: spill_levels * slot_words
    uint32_t* verts;          // enumerate output (device) or nullptr
    unsigned long long* offs;
    unsigned long long verts_cap, offs_cap;
    uint32_t num_wg;          // search workgroups
    uint32_t rec_words;       // kRecHeader + 4 * w32cap
    uint32_t w32cap;          // bitset stride in LDS slots and records
    uint32_t slot_words;      // LDS frame stride (lds_frame_words)
    uint32_t spill_words;     // spill frame stride (spill_frame_words)
    uint32_t lds_depth;       // stack levels in LDS
    uint32_t spill_levels;    // stack levels in one spill chunk
    uint32_t spill_chunks;    // chunks in the spill pool
    uint32_t wave_lds_words;  // LDS words per wavefront
    uint32_t split_threshold;
    uint32_t check_interval;
    uint32_t enumerate;
    uint64_t watchdog_ticks;  // wall-clock ticks a wavefront may run (0 = no limit)
    uint32_t refresh_children; // children a workgroup processes between two looks at its mailbox
    uint32_t poll_iters;       // idle iterations between two looks at the end-of-search counter
    uint32_t* wave_state;     // per wavefront: kWave* phase (for deadline reports), or null
    WaveExit* exits;          // per wavefront (blockIdx.x * waves per workgroup + wavefront)
    uint32_t pivot_rule;      // kPivot*
    uint32_t pad0;
    // host-written word in coherent pinned host memory, or null: non-zero asks
    // the search to stop (a served job cancelled while it runs)
    const uint32_t* cancel;
    const uint32_t* idmap;    // id maps of local graphs (GraphDesc.idmap_off), or null
    // lane search: off (0) or on; nodes with fewer candidates than lane_min
    // stay with the wavefront's loop; lane_levels levels a wavefront in lspill
    uint32_t lane_on, lane_min, lane_levels;
    uint32_t chop_max; // pieces of root units at most, of a batch beyond the first of each unit (0: whole units)
    uint32_t pool_cap; // records in rec
    uint32_t pad1;
    uint32_t* lspill;
    uint32_t* mail_bundle; // one record of lanes per workgroup, kBundleWords each
};
// Pivot rules (SearchParams.pivot_rule, MCE_OPT_PIVOT).
constexpr uint32_t kPivotGreedy = 0, kPivotTomita = 1, kPivotTX = 2;

// Phases recorded in SearchParams.wave_state.
constexpr uint32_t kWaveIdle = 1, kWaveFetch = 2, kWaveBusy = 3, kWaveExited = 4;

// Dynamic LDS of one search workgroup.
inline uint32_t search_lds_bytes(uint32_t wave_lds_words, uint32_t rec_words, uint32_t waves)
{
    return 4u * (kWgHdrWords + kLocalSlots * rec_words + wave_lds_words * waves);
}

// Rows whose degrees stand for a graph's mean degree: every degree_stride(n)th.
constexpr uint32_t kDegreeRows = 16;
__host__ __device__ inline uint32_t degree_stride(uint32_t n) { return n > kDegreeRows ? (n + kDegreeRows - 1u) / kDegreeRows : 1u; }
__host__ __device__ inline uint32_t degree_rows(uint32_t n) { return (n + degree_stride(n) - 1u) / degree_stride(n); }
// Whether the search of a graph gains by lanes.  Not where most neighbourhoods
// are too large for them (121 vertices) and have so few edges that the next
// nodes are too small to be worth their set-up: the loop then has most of the
// work, and without the lanes' stacks more wavefronts.  Kept counts with lanes
// and without, us: G(1600, 0.06) 222, 219; 0.08 316, 270; 0.1 396, 360; 0.12
// 468, 528; G(2016, 0.08) 429, 353; 0.1 540, 524; 0.12 734, 858; G(1200, 0.08)
// 229, 216; 0.12 346, 352; G(1000, 0.08) 169, 196; 0.1 233, 230; G(800, 0.15)
// 268, 337.
constexpr float kLaneDegree = 96.f;
constexpr float kLaneDensity = 0.11f;
inline bool lanes_pay(float n, float degree) { return degree < kLaneDegree || degree > kLaneDensity * n; }
// Mean degree of a single graph of one word a lane, or of those of a batch that
// are large enough for the rule above, with their mean size, if they are half of
// the batch.
struct DegreeSample {
    uint64_t sum = 0, rows = 0, verts = 0, graphs = 0;
    static bool wanted(uint32_t n, uint32_t num_graphs)
    {
        return n != 0 && n <= 32u * kOneChunkMaxW32 && (num_graphs == 1 || kLaneDensity * (float)n > kLaneDegree);
    }
    void add(uint32_t n)
    {
        rows += degree_rows(n);
        verts += n;
        graphs++;
    }
    float degree() const { return rows ? (float)sum / (float)rows : 0.f; }
    bool lanes(uint32_t num_graphs) const
    {
        return graphs == 0 || 2 * graphs < num_graphs || lanes_pay((float)verts / (float)graphs, degree());
    }
};

// Host-side launchers (kernels.hip).
// flag: [0] gets 1 if the graph is not simple, [1] the sum of the sampled
// degrees if `sample`.
hipError_t launch_validate(const uint64_t* rows, uint32_t n, uint32_t rw, unsigned int* flag, bool sample,
                           hipStream_t s);
// max_words: the largest n * rw64 of the graphs (their input rows' words).
// nbr: for graphs whose rows do not fit in LDS, room for cap 16-bit entries
// a vertex (indexed like order), cap = order_list_cap(max_n, max_words), used
// for neighbour lists during the ordering, and done: a word a graph; nullptr
// (or cap 0): none.
uint32_t order_list_cap(uint32_t max_n, uint64_t max_words);
// Whether a handle of num_graphs graphs, `large` of them of more than
// kListMinN vertices, is ordered on lists where they can be: in a batch of
// graphs that are mostly smaller, the passes over all of them cost more than
// the lists save (prepare of 20,000 graphs of 17 vertices and one of 1500: 6.3
// ms on the device with lists, 1.1 without, 1.25 before there were lists here).
constexpr uint32_t kListMinN = 1024;
inline bool order_on_lists(uint32_t num_graphs, uint32_t large, uint32_t max_n)
{
    return num_graphs == 1u || max_n > 4096u || 8ull * large >= num_graphs;
}
hipError_t launch_order(const GraphDesc* graphs, uint32_t num_graphs, uint32_t max_n, uint64_t max_words,
                        const uint64_t* rows_in, uint32_t* order, uint16_t* nbr, uint32_t cap, uint32_t* done,
                        hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, uint32_t count, uint32_t value, hipStream_t s);
hipError_t launch_relabel(const GraphDesc* graphs, uint32_t num_graphs, uint32_t max_n,
                          const uint64_t* rows_in, const uint32_t* order, uint32_t* adj,
                          hipStream_t s);
// Zeroes the results, histogram, mailboxes and control block of a solve, and
// writes sp to params_out when that is not null.
hipError_t launch_reset(const SearchParams& sp, uint32_t num_graphs, uint64_t hist_total,
                        uint32_t workgroups, SearchParams* params_out, hipStream_t s);
hipError_t launch_root(const SearchParams& sp, uint32_t num_graphs, uint32_t max_w32,
                       uint64_t first, uint64_t last, uint32_t max_units, hipStream_t s);
hipError_t launch_subproblem(const SearchParams& sp, uint32_t max_w32, const uint32_t* bits, hipStream_t s);
// Local graphs of the root children of graph gparent (a single graph):
// per position, its degree with bit 31 set when it is a root child; then the
// local graphs themselves (rows, orders, id maps, the P and X bitsets of the
// root child's node at lpx + in_off); then, per solve, the root children with
// branch index in [first, last) as units (or leaves counted at once).
hipError_t launch_local_plan(const GraphDesc* gparent, const uint32_t* adj, uint32_t n, uint32_t* out, hipStream_t s);
hipError_t launch_local_build(const GraphDesc* gparent, const uint32_t* adj, const uint32_t* order, uint32_t n,
                              const GraphDesc* lgraphs, uint32_t count, uint32_t* ladj, uint32_t* lord,
                              uint32_t* lidmap, uint32_t* lpx, hipStream_t s);
hipError_t launch_local_units(const SearchParams& sp, const uint32_t* lpx, uint32_t count, uint32_t max_w32,
                              uint64_t first, uint64_t last, hipStream_t s);
hipError_t launch_search(const SearchParams& sp, const SearchParams* d_sp, uint32_t max_w32, uint32_t blocks,
                         uint32_t waves_per_block, hipStream_t s);
// Adds the exit records of the last search launch's `waves` wavefronts into
// the result slots, the histogram and the control block's counters.
hipError_t launch_exit_fold(const SearchParams& sp, uint32_t waves, hipStream_t s);
hipError_t search_occupancy(uint32_t max_w32, uint32_t rule, bool lanes, uint32_t waves_per_block, uint32_t lds_bytes,
                            int* blocks_per_cu);

} // namespace mce
