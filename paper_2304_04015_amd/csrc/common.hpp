// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "simrank.h"

namespace srk {

// ------------------------------------------------------------------ errors
void set_error(const std::string &msg);
void clear_error();
int fail(int code, const std::string &msg);

#define SRK_HIP(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return ::srk::fail(SIMRANK_EDEVICE, std::string(#expr) + ": " +                \
                                                    hipGetErrorString(e_));                \
    } while (0)

// --------------------------------------------------------------- constants
constexpr uint32_t NIL = 0xffffffffu;   // no successor / no segment
constexpr int MAX_CAP = 255;            // walk cap limit (lengths fit a byte)
constexpr int MAX_STITCH_CAP = 64;      // stitched walks: long walks span 64 steps
constexpr int64_t MAX_R = 1 << 24;
constexpr int64_t MAX_STRAT_N = (1 << 24) - 1;  // weighted sums stay below 2^64

// Query kinds (one meet-kernel instance each).
enum Kind : int32_t { K_PLAIN = 0, K_STITCHED = 1, K_STRAT = 2, N_KINDS = 3 };


// Meet-kernel tiling of the compacted source walks (see query.hip), per kind.
// The more walks of one node a block holds, the more of their early steps
// share rows in the CU's L1; LDS bounds the tile.  Measured per query:
//  - plain (medium graph, in the Infinity Cache): 1024-thread blocks, tiles of
//    up to 8192 walks / 24576 positions (148 KB of LDS, one block per CU):
//    50.5 ms, against 58.9 ms with 512 threads and 1024 / 4096;
//  - stratified (medium graph; its LDS also holds classes, shuffle keys and a
//    queue of prepared pairs): 1024 threads, 6144 / 20480: 99.6 ms, against
//    114.1 ms with 512 threads and 1024 / 4096;
//  - stitched: the plain kind's block and positions per tile (its private
//    heads are plain walks), with room in LDS for the waves' tail queues
//    (16 waves x 128 x 8 bytes): tiles of up to 6144 walks / 24576 positions.
#ifndef SRK_TILE_J
#define SRK_TILE_J 8192
#endif
#ifndef SRK_TILE_NODES
#define SRK_TILE_NODES 24576
#endif
#ifndef SRK_MEET_BLOCK
#define SRK_MEET_BLOCK 1024
#endif
#ifndef SRK_STITCH_TILE_J
#define SRK_STITCH_TILE_J 6144
#endif
#ifndef SRK_STITCH_TILE_NODES
#define SRK_STITCH_TILE_NODES 24576
#endif
#ifndef SRK_STITCH_MEET_BLOCK
#define SRK_STITCH_MEET_BLOCK 1024
#endif
#ifndef SRK_STRAT_TILE_J
#define SRK_STRAT_TILE_J 6144
#endif
#ifndef SRK_STRAT_TILE_NODES
#define SRK_STRAT_TILE_NODES 20480
#endif
#ifndef SRK_STRAT_MEET_BLOCK
#define SRK_STRAT_MEET_BLOCK 1024
#endif
constexpr int MEET_VB = 256;                // nodes v per work unit, at most
constexpr int MIN_TILE_J = 2048;            // smallest tile a query may be given (buffers are
                                            // sized for it: max_tiles_for)
__host__ __device__ constexpr int tile_j_of(int kind) {
    return kind == K_PLAIN ? SRK_TILE_J : kind == K_STITCHED ? SRK_STITCH_TILE_J : SRK_STRAT_TILE_J;
}
__host__ __device__ constexpr int tile_nodes_of(int kind) {   // < 2^16
    return kind == K_PLAIN ? SRK_TILE_NODES
           : kind == K_STITCHED ? SRK_STITCH_TILE_NODES : SRK_STRAT_TILE_NODES;
}
__host__ __device__ constexpr int meet_block_of(int kind) {
    return kind == K_PLAIN ? SRK_MEET_BLOCK
           : kind == K_STITCHED ? SRK_STITCH_MEET_BLOCK : SRK_STRAT_MEET_BLOCK;
}

// Rows of a packed graph's hubs that a kind's meet kernel has LDS for, beside
// its tile and a served request's preparation.  A graph with more hubs has the
// tiles of plain and stitched queries cut to HUB_TILE_NODES positions, to make
// room for HUB_ROWS.
__host__ __device__ constexpr int hub_rows_of(int kind) {
    return kind == K_PLAIN ? 1216 : kind == K_STITCHED ? 704 : 1472;
}
constexpr int HUB_TILE_NODES = 12288, HUB_ROWS = 6848;

// ------------------------------------------------------------ device graph
// Gather layout of the reversed graph.  Every node v owns the edge slots
// [o(v), o(v) + max(deg(v), 1)) of E; E[o(v) + k] describes the k-th
// in-neighbour u of v by (o(u), deg(u)), so one 8-byte gather moves a walk and
// already yields the row of the node it lands on.  o() is strictly increasing,
// so it identifies nodes; nodes without in-neighbours own one unused slot.
struct Index;

// Hubs a graph may have and still be packed (E4).
constexpr uint32_t HUB_CAP = HUB_ROWS;

struct Graph {
    int device = 0;
    int32_t n = 0;
    int64_t m = 0;
    int64_t m_slots = 0;          // sum over v of max(deg(v), 1)
    int32_t n_active = 0;         // nodes with deg >= 1
    int32_t max_deg = 0;
    uint2 *nodes = nullptr;       // [n]     (o(v), deg(v))
    uint2 *E = nullptr;           // [m_slots]
    uint32_t *E4 = nullptr;       // [m_slots] E packed for the meet kernels (graph.hip), or NULL
    uint2 *hubs = nullptr;        // [n_hubs] rows of the nodes whose degree E4 cannot hold
    int32_t obits = 0;            // bits of o() in an E4 entry; 0: there is no E4
    int32_t n_hubs = 0;
    uint32_t *node_of = nullptr;  // [m_slots] node id owning slot o (valid at o(v))
    int32_t *active = nullptr;    // [n_active] nodes with deg >= 1, ascending
    uint32_t *dbar = nullptr;     // [n] rows of the CSR that list v (v's in-degree in the
                                  //     reversed graph), counted at ingest
    hipStream_t stream = nullptr; // stream of the synchronous calls
    Index *index = nullptr;
    uint64_t index_gen = 0;       // counts replacements of the index (plans check it)
    int32_t tuned_vb = 0;         // nodes per meet work unit chosen by simrank_tune (0: default)
    int32_t tuned_tile_j[N_KINDS] = {0, 0, 0};   // source walks per LDS tile, per kind (0: default)
    int64_t bytes = 0;
};

// Stitched-walk index (see index.hip).
struct Index {
    int32_t seg_log2 = 3;
    int32_t seg_len = 8;          // 2^k
    int32_t width = 8;            // long-walk width in segments: 64 / 2^k
    int32_t levels = 3;           // doubling rounds: log2(width)
    double kappa = 1.0;
    double c = 0.6;               // decay of the segments' walks
    uint32_t T = 0;               // their continue threshold
    uint64_t seed = 0;
    int64_t segments = 0;
    int64_t *pool_off = nullptr;  // [n+1]
    uint32_t *seg = nullptr;      // [segments][seg_len] o() of positions 1..len, NIL after
    uint8_t *seg_lens = nullptr;  // [segments]
    uint32_t *succ = nullptr;     // [segments] successor slot or NIL
    uint32_t *chain = nullptr;    // [segments][width] slots of the long walk from sigma
    int64_t bytes = 0;
    double build_ms = 0;
    double segments_ms = 0, doubling_ms = 0;   // parts of build_ms
    uint64_t build_moves = 0;
};

// Read-only view of a graph's stitched index, as the kernels see it.
struct IndexView {
    const uint32_t *node_of;
    const int64_t *pool_off;
    const uint32_t *seg;
    const uint8_t *seg_lens;
    const uint32_t *chain;
    int32_t seg_len, width;
};

// Length-stratified estimator: the first slot of each length class and
// Lemma 5's per-class ratio Z_l / Zhat_l (computed on the host).
struct StratTab {
    uint32_t ccum[MAX_CAP + 2];   // ccum[l] = Zhat_0 + ... + Zhat_{l-1}; ccum[phi+1] = N
    double a[MAX_CAP + 1];
};

struct StratParams {
    double z = 0;                 // Algorithm 2's normaliser
    int32_t N = 0;                // walks per node, sum of Zhat_l
    int32_t phi = 0;              // walk length cap
    int32_t sb = 0;               // shuffle grid [0, sa) x [0, 2^sb), sa 2^sb >= N
    int32_t sa = 1;
};

// One query as the device kernels see it (one entry per query of a launch).
struct QueryDesc {
    const uint2 *nodes;
    const uint2 *E;
    const uint32_t *E4;    // the packed rows of the graph, if obits > 0
    const uint2 *hubs;
    int32_t obits, n_hubs;
    const int32_t *active;
    IndexView ix;
    uint32_t *sw;          // [R][L] source walk positions 1..L (o values)
    uint8_t *slen;         // [R rounded up to 256] lengths of a group member's source walks;
                           // a lone query's tiles' first units
    uint32_t *jj;          // [R] walk index of compact entry k
    uint32_t *joff;        // [R + 1] start of entry k in swc
    uint32_t *swc;         // [R * L] packed positions
    uint32_t *tiles;       // [max tiles + 1]
    uint32_t *meta;        // [8]: R1, packed positions, tiles, entries of the largest tile
    uint32_t *cnt;         // [n] meet counts (caller's; plain and stitched)
    double *out;           // [n] estimate or NULL
    uint32_t k0, k1;       // Philox key of the query's walks
    uint32_t T;            // continue threshold
    int32_t n, n_active, s, R, L;
    int32_t vb;            // nodes per work unit at most (<= MEET_VB); 0: sized on the device
    uint32_t cost;         // of a pair, for the sizes of units (pair_cost)
    int32_t kind;          // Kind
    int32_t items;         // items a wave takes at once, at most (item_chunk)
    int32_t tile_j;        // source walks per LDS tile, MIN_TILE_J .. tile_j_of(kind)
    int32_t tile_nodes;    // and their positions: tile_nodes_of(kind), or HUB_TILE_NODES
    // stratified only (R = N walks per node, L = phi)
    const StratTab *tab;
    uint8_t *scls;         // [R] length class of walk (s, j)
    unsigned long long *wsum;  // [n] weighted meet sums, 2^40 = weight 1 (caller's)
    double *out_n;         // [n] estimate normalised by the N pairs, or NULL
    double z;
    int32_t sa, sb;        // shuffle grid
};

// Rows that a meet kernel gathers (graph.hip): the 8 bytes of E, or those packed
// in 4; HUBS: packed, with the small tiles of a graph with many hubs; MIXED: as
// each query's graph has it.
enum Rows : int { ROWS_E, ROWS_PACKED, ROWS_HUBS, ROWS_MIXED };
// What a query can use.  E is better where all of it is within an XCD's L2
// (packed rows only add their decoding; n = 20,000, R = 38,005: 2,677 us with E,
// 2,717 packed), packed rows are beyond it (n = 2^18, R = 9,502: 11,681 and
// 9,455; stratified, N = 16,508: 20.2 and 18.1 ms).
constexpr int WANTS_E = 1, WANTS_PACKED = 2, WANTS_HUBS = 4, HAS_NONE = 8;
inline int rows_wish(const Graph &g, const QueryDesc &d) {
    if (g.obits == 0) return HAS_NONE;
    if (g.n_hubs > hub_rows_of(d.kind)) return d.tile_nodes == HUB_TILE_NODES ? WANTS_HUBS : HAS_NONE;
    return 8 * g.m_slots <= (int64_t)4 << 20 ? WANTS_E : WANTS_PACKED;
}
// Rows of a launch for queries of these wishes.  A kernel that asks its graph
// at each gather takes 2 to 4% longer, so it is left for queries of which only
// some can have packed rows.
inline Rows rows_of(int wishes) {
    return wishes == WANTS_HUBS                    ? ROWS_HUBS
           : !(wishes & WANTS_PACKED)              ? ROWS_E
           : !(wishes & (WANTS_HUBS | HAS_NONE))   ? ROWS_PACKED
                                                   : ROWS_MIXED;
}
// Positions of a tile of source walks.  The small tiles of a graph with many
// hubs are up to twice as many: they are taken where even units of one node
// could be numbered.
inline int32_t tile_nodes_for(const Graph &g, int kind, int32_t R, int32_t L) {
    const int64_t tiles = 2 + R / MIN_TILE_J + (int64_t)R * L / (HUB_TILE_NODES - L);
    return kind != K_STRAT && g.obits > 0 && g.n_hubs > hub_rows_of(kind) &&
                   tiles * g.n_active < (int64_t)1 << 31
               ? HUB_TILE_NODES : tile_nodes_of(kind);
}

// Settles the tiles of a launch's queries of one kind (`units` of them nominally)
// and returns their wishes.  Small tiles are for launches that read packed rows
// with them.  A graph with many hubs beside others is gathered from E, where they
// cost time (a query at n = 2^20, R = 9,502, 6,256 hubs, with one at n = 5,000: 50.4
// ms with 12,288 positions a tile, 49.6 with 24,576; with one at n = 150,000: 60.4 and
// 59.4); and they make the units up to twice as many.
inline int settle_tiles(const Graph *const *g, QueryDesc *const *d, size_t nq, int64_t units) {
    int wishes = 0;
    for (size_t i = 0; i < nq; ++i) wishes |= rows_wish(*g[i], *d[i]);
    if (!(wishes & WANTS_HUBS) || (rows_of(wishes) == ROWS_HUBS && units < (int64_t)1 << 30)) return wishes;
    wishes = 0;
    for (size_t i = 0; i < nq; ++i) {
        d[i]->tile_nodes = tile_nodes_of(d[i]->kind);
        wishes |= rows_wish(*g[i], *d[i]);
    }
    return wishes;
}

// A set of queries whose descriptors are already in device memory.
struct QuerySet {
    const QueryDesc *desc;        // device [nq]
    int32_t nq = 0;
    int32_t max_R = 0, max_n = 0;
    int64_t units_bound[N_KINDS] = {0, 0, 0};   // work units of each kind's queries, at most
    int rows[N_KINDS] = {0, 0, 0};              // rows_wish of each kind's queries
    uint32_t *units = nullptr;    // device [units_words(nq)]: unit offsets per kind, then cursors
    unsigned long long *counters = nullptr;  // device [CTR_WORDS]
    const struct GroupSet *groups = nullptr;  // grouped plain queries, if any
};

// Words of a query set's unit table: N_KINDS lists of nq + 1 offsets, then
// one cursor per kind.
inline size_t units_words(int32_t nq) { return (size_t)N_KINDS * ((size_t)nq + 1) + N_KINDS; }

// ------------------------------------------------------------ query groups
// In a batch, queries of one kind on one graph with the same walk key and walk
// parameters (c and cap; the stratified estimator's z and cap) have the same
// walk (v, j) from every node v: a group of up to GROUP_MAX such queries
// follows each walk once and tests it against every
// member's walk j of its own source (group.hip).  A member keeps its own
// descriptor (source walks, counts or weighted sums, estimate) with kind
// K_GROUPED, K_GROUPED_STITCHED or K_GROUPED_STRAT, which no per-kind unit list
// takes.
constexpr int GROUP_MAX = 32;
constexpr int32_t K_GROUPED = N_KINDS, K_GROUPED_STITCHED = N_KINDS + 1, K_GROUPED_STRAT = N_KINDS + 2;
// Groups of more than 8 stratified queries keep their 64-bit weighted sums for
// at most this many nodes per work unit (64 KB of LDS at 256 nodes; their tile
// is the smaller for it).
#ifndef SRK_GROUP_STRAT32_VB
#define SRK_GROUP_STRAT32_VB 256
#endif
constexpr int GROUP_STRAT32_VB = SRK_GROUP_STRAT32_VB;
// Kinds whose walks are the stratified estimator's (weighted sums, not counts).
__host__ __device__ inline bool strat_kind(int32_t kind) { return kind == K_STRAT || kind == K_GROUPED_STRAT; }

struct GroupDesc {
    const uint2 *nodes;
    const uint2 *E;
    const uint32_t *E4;
    const uint2 *hubs;
    int32_t obits, n_hubs;
    const int32_t *active;
    int32_t n_active, vb, n_chunks;
    int32_t G, L, Rmax;
    int32_t gw;                          // words of member lengths per entry: ceil(G / 4)
    int32_t wk;                          // walks: 0 plain, 1 stitched (index tails), 2 stratified
    IndexView ix;
    // stratified: the class table, N = R of every member, the shuffle grid
    const StratTab *tab;
    int32_t sa, sb;
    uint32_t k0, k1, T;
    int32_t s[GROUP_MAX];                // members' sources
    int32_t R[GROUP_MAX];
    const uint32_t *sw[GROUP_MAX];       // members' source walks [R][L]
    const uint8_t *slen[GROUP_MAX];      // and their lengths [R]
    uint32_t *cnt[GROUP_MAX];            // members' meet counts [n] (plain, stitched)
    unsigned long long *wsum[GROUP_MAX]; // members' weighted sums [n] (stratified)
    const uint8_t *scls[GROUP_MAX];      // classes of the members' walks [R] (stratified)
    // Compacted walks: entry e is a walk index jj[e] for which at least one
    // member's walk has a step; from pos[joff[e]], one block per step t of its
    // longest member walk: a word with bit q set for each member q whose walk
    // j has a position at step t, then those positions' marks (the low halves
    // of their o()) in member order, 0xffff up to a multiple of four words.
    // Member q's length is byte q of the entry's gw words glen[e gw ...].
    uint32_t *jj;                        // [Rmax]
    uint32_t *joff;                      // [Rmax + 1]
    uint32_t *glen;                      // [Rmax][gw]
    uint32_t *pos;                       // [group_pos_words]
    uint32_t *tiles;                     // [group_max_tiles + 1]
    uint32_t *meta;                      // [8]: entries, positions, tiles
};

// Kernel instance of a group: plain walks with up to 8 members (0) or more
// (1), stitched walks with up to 8 (2) or more (3), stratified walks with up
// to 8 (4) or more (5).
constexpr int GROUP_LISTS = 6;
__host__ __device__ inline int group_list(int32_t G, int32_t wk) { return 2 * wk + (G > 8 ? 1 : 0); }

// Rows of hubs that an instance has LDS for, and the rows a group can use: as a
// lone query (rows_wish).  A launch whose groups cannot all be packed reads E.
__host__ __device__ constexpr int group_hub_rows(int list) { return list == 5 ? 256 : 1536; }
inline int group_rows_wish(const Graph &g, int list) {
    if (g.obits == 0 || g.n_hubs > group_hub_rows(list)) return HAS_NONE;
    return 8 * g.m_slots <= (int64_t)4 << 20 ? WANTS_E : WANTS_PACKED;
}

struct GroupSet {
    const GroupDesc *desc = nullptr;     // device [ng]
    int32_t ng = 0;
    int32_t max_R = 0;                   // largest Rmax
    int64_t units_bound[GROUP_LISTS] = {};       // work units per kernel instance (group_list)
    int rows[GROUP_LISTS] = {};                  // group_rows_wish of its groups
    uint32_t *units = nullptr;           // device [group_units_words(ng)]
};
// Unit offsets of a group set: one list of ng + 1 offsets per instance, then
// one cursor per list.
inline size_t group_units_words(int32_t ng) { return GROUP_LISTS * ((size_t)ng + 1) + GROUP_LISTS; }

// Words of a group's compacted walks, at most: every member position, and one
// member word and up to three words of padding per step of each entry.
inline int64_t group_pos_words(int64_t Rmax, int64_t sum_RL, int32_t L) { return sum_RL + 4 * Rmax * L; }
// Tiles of a group's compacted walks, at most.
int32_t group_max_tiles(int64_t Rmax, int64_t sum_RL, int32_t L, int32_t G, int32_t wk);
// Nodes per work unit of a group of G members with walks wk on a graph with
// n_active nodes that have in-edges (the lone queries' tuning does not apply).
int32_t group_unit_nodes(int32_t n_active, int32_t G, int32_t wk);
// Fills a group's descriptor (all but its compaction buffers jj .. meta) from
// the descriptors of its G members (kinds K_GROUPED, K_GROUPED_STITCHED or
// K_GROUPED_STRAT, buffers attached).
void describe_group(const QueryDesc *const *members, int32_t G, GroupDesc *gd);
// Device bytes of a group's compaction buffers and their carving from `base`
// (256-byte aligned pieces); returns the bytes taken.
size_t group_buffers(GroupDesc *gd, int64_t sum_RL, char *base);
// Enqueues a query set's groups: compaction, unit offsets, the group meet
// kernel (after the members' source walks, before their estimates).
int launch_groups(const GroupSet &gs, unsigned long long *counters, hipStream_t st);

// ------------------------------------------------------------ serving ring
// The server's in-flight requests (server.hip) sit in a ring of entries that
// persistent meet kernels take work units from.  An entry has a claim word per
// kind, which holds everything a block needs to decide whether it may take units:
//   claim[kind] = seq << 32 | CLAIM_ZERO + units not yet claimed,
// so availability and age come from one atomic read, never from fields that a
// reuse of the entry may be rewriting.  An entry is published by the last kernel
// of its request's preparation: the other fields first, then its kind's word with
// all n_units units unclaimed (release).  A block that sees a word above
// CLAIM_ZERO takes up to a run of units by an atomic subtraction (acquire), and
// has those that the word it returns says were left: of that request, or of a
// later one of the kind if the entry has been published again since; none if it
// is CLAIM_ZERO or below, to which blocks that came too late move it (by a run
// each, far less than CLAIM_ZERO).  It then reads n_units, which stays until its
// units are finished (the first unit it took is n_units minus those left).  An
// entry published again as another kind leaves this kind's word exhausted.  The
// block that finishes the entry's last unit writes the estimate and then the
// entry's flag in host memory (the request's seq).
// seq is nonzero and below 2^30.
constexpr uint32_t CLAIM_ZERO = 1u << 20;
constexpr int RING_MAX = 64;
constexpr uint32_t RING_SEQ_LIMIT = 1u << 30;
struct RingCtl {
    unsigned long long claim[N_KINDS];   // see above; 0 = never published
    uint32_t n_units;           // tiles x node chunks of the request
    uint32_t done;              // units finished
};
struct StreamRing {
    QueryDesc *desc;                 // device [RING_MAX]
    RingCtl *ctl;                    // device [RING_MAX]
    unsigned long long *counters;    // device [RING_MAX][8]: work counters per entry
    uint32_t *flags;                 // pinned host [RING_MAX], written by the device
    int32_t entries;                 // entries in use, <= RING_MAX
};
// Serving (query.hip): enqueue on `st` the preparation of ring entry `slot`
// for the request described by d (its buffers attached): descriptor, init,
// source walks, publication (tiles and units).  Launch a persistent meet kernel of
// `kind` that takes units from every published entry of that kind and exits
// when none is left.  Bytes of device memory a request needs for its buffers.
int enqueue_ring_request(const QueryDesc &d, const StreamRing &ring, int32_t slot, uint32_t seq,
                         hipStream_t st);
int launch_ring_meet(Rows rows, int kind, const StreamRing &ring, hipStream_t st);
size_t request_bytes(const simrank_params &p, int mode, int32_t n);
// Carves a request's buffers (request_bytes of them) from base into d.
void carve_request(const simrank_params &p, int mode, int32_t n, char *base, QueryDesc *d);

// Per-query scratch.
struct Workspace {
    const Graph *g = nullptr;
    int32_t max_R = 0, max_L = 0;
    uint32_t *sw = nullptr;        // [max_R][max_L] source walk positions 1..L (o values)
    uint8_t *slen = nullptr;       // [max_R]
    uint32_t *jj = nullptr;        // [max_R] walk index of compact entry k
    uint32_t *joff = nullptr;      // [max_R + 1] start of entry k in swc
    uint32_t *swc = nullptr;       // [max_R * max_L] compact positions
    uint32_t *tiles = nullptr;     // [max tiles + 1] first compact entry of each tile
    uint32_t *meta = nullptr;      // [8]: R1, total nodes, n_tiles, ...
    unsigned long long *counters = nullptr;  // [CTR_WORDS] stats
    bool own_counters = false;
    QueryDesc *desc = nullptr;     // device [1]
    uint32_t *units = nullptr;     // device [units_words(1)]
    uint8_t *scls = nullptr;       // [max_R] stratified: class of walk (s, j)
    StratTab *tab = nullptr;       // device table of the last stratified query
    int32_t max_tiles = 0;
    hipEvent_t ev1 = nullptr;      // behind the query
    hipStream_t last_stream = nullptr;
    simrank_params last_params{};
    int32_t last_n = 0;
    bool pending = false;
};

enum Counter : int {
    C_MOVES = 0, C_DRAWS = 1, C_MEETS = 2, C_TAIL = 3, C_PAIRS = 4, C_SRC_MOVES = 5,
    C_UNITS = 6, C_SPARE = 7
};

// Work counters of a query set: the 8 totals, then CTR_SETS sets of 8 that the
// blocks add to (block b to set b mod CTR_SETS); k_estimate, the last kernel
// of every launch sequence, folds the sets into the totals.  One set for all
// blocks made the end of every meet launch a queue: atomics of all XCDs on one
// line complete about 16 ns apart, and a full grid's (256 blocks x 16 waves x
// 5 counters) took 330 us.  Measured per query (R = 1,521): 382 us before and 162 after at
// n = 5,003, 980 and 686 at n = 40,000.
constexpr int CTR_SETS = 64;
constexpr int CTR_SUMS = 8 * (1 + CTR_SETS);
// Behind them, device times of a lone query (ticks of the constant 100 MHz clock):
// start of its first kernel, end of the kernel before the meet kernel, start of
// the one behind it, end of the last one's block of the highest number.  (The
// latest of all its blocks' ends comes 1 us later, 22.7 and 24.0 us at n = 500, 577.1 and
// 577.8 at n = 2^22, and finding it took each query 0.3 us.)  HIP events there
// were packets of their own between the kernels and held each of them up by 3 to
// 6 us.  A query at n = 5,003 took 95 us with them and 84 without.
enum Stamp : int { STAMP_BEGIN = CTR_SUMS, STAMP_MEET = CTR_SUMS + 1, STAMP_MET = CTR_SUMS + 2,
                   STAMP_END = CTR_SUMS + 3 };
constexpr int CTR_WORDS = CTR_SUMS + 8;

// ----------------------------------------------------------------- helpers
int device_alloc(void **p, size_t bytes, int64_t *acct);
void device_free(void *p);

// Device-wide scans (scan.hip).  Exclusive sum of `in` (n values) into `out`
// (n values); returns the total in *total_dev (device scalar).  Temp storage
// is allocated and released by the call.
int scan_exclusive_u32_to_i64(const uint32_t *in, int64_t n, int64_t *out, int64_t *total_dev,
                              hipStream_t st);
int scan_exclusive_i64(const int64_t *in, int64_t n, int64_t *out, int64_t *total_dev,
                       hipStream_t st);
// Inclusive running maximum of u32 values, in place.
int scan_inclusive_max_u32(uint32_t *data, int64_t n, hipStream_t st);

// Queries (query.hip).
int query_params(const simrank_query *q, int32_t n, simrank_params *out, int *mode);
// Stratified estimator: z, N, phi, shuffle width and (if tab) the class table.
int strat_params(const simrank_query *q, int32_t n, StratParams *sp, StratTab *tab);
int32_t max_tiles_for(int32_t R, int32_t L);
// What a pair of stitched walks costs on average, 1 at least: the steps of its
// tail behind a head of `head` steps, in the 1.5 steps of a plain pair at c = 0.6.
uint32_t pair_cost(double c, int32_t L, int32_t head);
// Nodes per unit that the unit counts of a query are bounded with; a graph that
// was not tuned has its units sized on the device (lay_units, query.hip).
int32_t default_unit_nodes(const Graph *g);
// Work units of a query with nominal nodes per unit, which the launch limits
// are stated in; lay_units makes at most one per tile and 2^14 a launch more.
int64_t units_bound_of(const Graph *g, int32_t R, int32_t L);
IndexView index_view(const Graph *g);
// Fills everything but the buffers (sw .. out) of a descriptor.
void describe_query(const Graph *g, const simrank_query *q, const simrank_params &p, int mode,
                    QueryDesc *d);
// Enqueues init, source walks, tiles and units, meet and estimate for
// every query of the set.  one (may be NULL): the descriptor of a set of one
// query, not yet in device memory.
int launch_query_set(const QuerySet &qs, hipStream_t st, const QueryDesc *one = nullptr);
// Waits for the workspace's last query; its device time and its meet kernel's,
// in ms (each pointer may be NULL).
int query_times(const Workspace *ws, double *ms, double *meet_ms);
int enqueue_query(const Graph *g, const simrank_query *q, const simrank_params &p, int mode,
                  Workspace *ws, double *out_dev, uint32_t *counts_dev, hipStream_t st);
int enqueue_stratified(const Graph *g, const simrank_query *q, Workspace *ws, double *out_dev,
                       double *out_n_dev, unsigned long long *wsum_dev, hipStream_t st);
// counters: device [CTR_WORDS] of the caller's, or NULL for the workspace's own.
int workspace_init(const Graph *g, int32_t max_R, int32_t max_L, Workspace *ws,
                   unsigned long long *counters = nullptr);
void workspace_release(Workspace *ws);

// Index (index.hip).
void index_free(Index *ix);

inline unsigned grid_for(int64_t n, int block) {
    int64_t b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > 0x7fffffff) b = 0x7fffffff;
    return (unsigned)b;
}

uint32_t continue_threshold(double c);

}  // namespace srk

// The opaque handles of the C ABI are the internal objects.
struct simrank_graph : srk::Graph {};
struct simrank_workspace : srk::Workspace {};
