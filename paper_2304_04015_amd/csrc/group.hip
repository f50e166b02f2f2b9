// Query groups: queries of one batch (or of the server's waiting requests)
// that share a graph, a kind of walks, a walk key and the walks' parameters.
//
// The estimator of Section 3 pairs walk j of the source s with walk j of every
// node v.  The walk (v, j) draws its steps from counters (v, j, t, 0) under the
// query's key, so queries that share the key, the decay and the cap have the
// same walk (v, j) for every v and differ only in their source walks.  A group
// follows each walk (v, j) once and, at every step, compares its position with
// the same step of walk j of each member's source; a member drops out of the
// pair once it has met (counted once, as for a lone query) or its source walk
// has no further step.  The pair ends when the walk stops, reaches a node
// without in-neighbours, or no member is left.  Each member's counts are
// therefore exactly those of its lone run; the walks from the nodes are paid
// for once per group instead of once per query.  The same holds for stitched
// walks (their tails come from the shared index, entered by a draw keyed
// (v, j)) and for the stratified estimator's walks (walk j of v is the walk in
// slot pi_v(j), a function of v and the key; a meet adds Lemma 5's weight of
// the two walks' classes).
#include <algorithm>

#include "common.hpp"
#include "device_common.hpp"

namespace srk {
namespace {

// Tile shapes of the group meet kernel (walks and member positions per tile)
// for groups of up to 8 members and of up to 32; stratified walks keep 64-bit
// weighted sums in LDS, which take room from the tile (and, beyond 8 members,
// from the nodes per work unit).
#ifndef SRK_GROUP_TILE_J
#define SRK_GROUP_TILE_J 1280
#endif
#ifndef SRK_GROUP_TILE_NODES
#define SRK_GROUP_TILE_NODES 32768
#endif
#ifndef SRK_GROUP32_TILE_J
#define SRK_GROUP32_TILE_J 512
#endif
#ifndef SRK_GROUP32_TILE_NODES
#define SRK_GROUP32_TILE_NODES 28672
#endif
#ifndef SRK_GROUP32_STRAT_TILE_NODES
#define SRK_GROUP32_STRAT_TILE_NODES 20480
#endif
#ifndef SRK_GROUP_STRAT_TILE_J
#define SRK_GROUP_STRAT_TILE_J 1024
#endif
#ifndef SRK_GROUP_STRAT_TILE_NODES
#define SRK_GROUP_STRAT_TILE_NODES 24576
#endif
#ifndef SRK_GROUP_SLOTS
#define SRK_GROUP_SLOTS 2
#endif
constexpr int GROUP_BLOCK = 1024;
// GW: the instance's member capacity in words of four (2: up to 8 members, 8:
// up to 32; it sizes the per-member LDS counters and picks the tile shape);
// WK: walks (0 plain, 1 stitched, 2 stratified).
__host__ __device__ constexpr int group_tile_j(int GW, int WK) {
    return GW > 2 ? SRK_GROUP32_TILE_J : WK == 2 ? SRK_GROUP_STRAT_TILE_J : SRK_GROUP_TILE_J;
}
__host__ __device__ constexpr int group_tile_nodes(int GW, int WK) {   // < 2^16
    return GW > 2 ? (WK == 2 ? SRK_GROUP32_STRAT_TILE_NODES : SRK_GROUP32_TILE_NODES)
                  : WK == 2 ? SRK_GROUP_STRAT_TILE_NODES : SRK_GROUP_TILE_NODES;
}
// Nodes per work unit whose sums a stratified instance keeps in LDS.
__host__ __device__ constexpr int group_strat_vb(int GW) { return GW > 2 ? GROUP_STRAT32_VB : MEET_VB; }
// Words of an entry's block for a step with c member positions: the members'
// word and the positions' marks (half a word each), in whole 16-byte pieces.
__host__ __device__ constexpr uint32_t block_words(uint32_t c) { return ((c + 1u) / 2u + 4u) & ~3u; }
// A position's mark: the low half of its o().
__device__ __forceinline__ uint32_t mark_of(uint32_t o) { return o & 0xffffu; }
// a tile holds at least one entry of the longest form (L blocks of G positions)
static_assert(group_tile_nodes(2, 0) < 65536 && group_tile_nodes(2, 0) > 12 * MAX_CAP, "tile shape");
static_assert(group_tile_nodes(8, 0) < 65536 && group_tile_nodes(8, 0) > 36 * MAX_CAP, "tile shape");
static_assert(group_tile_nodes(2, 2) < 65536 && group_tile_nodes(2, 2) > 12 * MAX_CAP, "tile shape");
static_assert(group_tile_nodes(8, 2) < 65536 && group_tile_nodes(8, 2) > 36 * MAX_CAP, "tile shape");
static_assert(group_tile_nodes(2, 0) % 4 == 0 && group_tile_nodes(8, 0) % 4 == 0 &&
              group_tile_nodes(2, 2) % 4 == 0 && group_tile_nodes(8, 2) % 4 == 0, "16-byte pieces");
static_assert(GROUP_MAX == 32, "length words");

// The kernel instance (its GW) for groups of G members.
__host__ __device__ inline int group_gw(int32_t G) { return G <= 8 ? 2 : 8; }

// Length of member q in an entry's length words (byte q).
__device__ __forceinline__ uint32_t byte_of(uint32_t w, int q) { return (w >> (8 * (q & 3))) & 0xffu; }

// ------------------------------------------------------------ compaction
// Keeps the walk indices j for which at least one member's walk j has a step
// and packs the members' positions of walk j step by step: for each step t up
// to the longest member walk, the word of members with a position at t, then
// the marks of their positions at t in member order, 0xffff up to a multiple of
// four words (the meet kernel reads 16-byte pieces).  grid (x over blocks of PACK_J walk
// indices, y = group); a half wave packs an entry, one member per lane, and a
// block takes the room of its entries with one atomic on meta[0..1], so entries
// are in no order of j.  One block per group, a thread per walk index copying
// word by word, took 3.2 ms of the 66 ms of 32 queries on a graph of n = 2^18
// (R = 9,502); this takes 0.05, and cutting the tiles 0.03.
constexpr int PACK_J = 32;
__global__ __launch_bounds__(256) void k_group_pack(const GroupDesc *__restrict__ gd) {
    __shared__ uint32_t s_words[PACK_J], s_first[PACK_J + 1], s_base[2];
    const GroupDesc &d = gd[blockIdx.y];
    const int32_t j00 = (int32_t)blockIdx.x * PACK_J;
    if (j00 >= d.Rmax) return;
    const int32_t L = d.L, G = d.G, gw = d.gw;
    const int lane = threadIdx.x & 63, q = lane & 31, half = threadIdx.x >> 5;   // 8 half waves
    const bool member = q < G;
    const uint32_t hshift = (uint32_t)(lane & 32);
    const uint8_t *slen = member ? d.slen[q] : nullptr;
    const uint32_t *sw = member ? d.sw[q] : nullptr;
    const int32_t Rq = member ? d.R[q] : 0;
    uint32_t len[PACK_J / 8];
#pragma unroll
    for (int i = 0; i < PACK_J / 8; ++i) {
        const int32_t jl = i * 8 + half, j = j00 + jl;
        len[i] = j < Rq ? (uint32_t)slen[j] : 0u;
        uint32_t mx = len[i];
        for (int dd = 16; dd > 0; dd >>= 1) mx = max(mx, __shfl_xor(mx, dd, 32));
        uint32_t words = 0;
        for (uint32_t t = 0; __ballot(t < mx) != 0ull; ++t) {
            const uint32_t am = (uint32_t)(__ballot(t < len[i]) >> hshift);
            if (t < mx) words += block_words((uint32_t)__popc(am));
        }
        if (q == 0) s_words[jl] = words;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t w = threadIdx.x < PACK_J ? s_words[threadIdx.x] : 0u;
        const uint64_t has = __ballot(w > 0u);
        uint32_t inc = w;
        for (int dd = 1; dd < PACK_J; dd <<= 1) {
            const uint32_t y = __shfl_up(inc, dd, 64);
            if (lane >= dd) inc += y;
        }
        if (threadIdx.x < PACK_J) s_first[threadIdx.x] = inc - w;
        if (threadIdx.x == PACK_J - 1) {
            unsigned long long at = 0;
            if (has) at = atomicAdd((unsigned long long *)d.meta,
                                    ((unsigned long long)inc << 32) | (uint32_t)__popcll(has));
            s_base[0] = (uint32_t)at;
            s_base[1] = (uint32_t)(at >> 32);
        }
        if (threadIdx.x < PACK_J) s_words[threadIdx.x] = w ? lane_rank(has) : NIL;   // rank of the entry
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PACK_J / 8; ++i) {
        const int32_t jl = i * 8 + half, j = j00 + jl;
        const uint32_t rank = s_words[jl];
        const bool on = rank != NIL;
        const uint32_t k = s_base[0] + rank;
        uint32_t off = s_base[1] + s_first[jl];
        if (on && q == 0) {
            d.jj[k] = (uint32_t)j;
            d.joff[k] = off;
        }
        const uint32_t l1 = __shfl_down(len[i], 1, 32), l2 = __shfl_down(len[i], 2, 32),
                       l3 = __shfl_down(len[i], 3, 32);
        if (on && (q & 3) == 0 && (q >> 2) < gw)
            d.glen[(size_t)k * gw + (q >> 2)] = len[i] | (l1 << 8) | (l2 << 16) | (l3 << 24);
        uint32_t mx = on ? len[i] : 0u;
        for (int dd = 16; dd > 0; dd >>= 1) mx = max(mx, __shfl_xor(mx, dd, 32));
        const uint32_t *row = sw + (size_t)j * L;
        uint32_t next = len[i] > 0u ? row[0] : NIL;
        for (uint32_t t = 0; __ballot(t < mx) != 0ull; ++t) {
            const uint32_t here = next;
            next = t + 1 < len[i] ? row[t + 1] : NIL;   // the next step's load is on its way
            const uint32_t am = (uint32_t)(__ballot(t < len[i]) >> hshift);
            const uint32_t c = (uint32_t)__popc(am), bw = block_words(c);
            if (t < mx) {
                if (q == 0) d.pos[off] = am;
                uint16_t *marks = reinterpret_cast<uint16_t *>(d.pos + off + 1u);
                if (t < len[i]) marks[__popc(am & ((1u << q) - 1u))] = (uint16_t)mark_of(here);
                if ((uint32_t)q < 2u * (bw - 1u) - c) marks[c + (uint32_t)q] = 0xffffu;
                off += bw;
            }
        }
    }
}

// Tiles of one group per block: cuts the entries into tiles of at most TJ
// entries and TN words, each the longest run from the previous one's end
// (cut_tiles).  (TJ, TN) is the shape of the kernel instance that runs the
// group.
__global__ __launch_bounds__(64) void k_group_tiles(const GroupDesc *__restrict__ gd) {
    const GroupDesc &d = gd[blockIdx.x];
    const uint32_t TJ = (uint32_t)group_tile_j(group_gw(d.G), d.wk);
    const uint32_t TN = (uint32_t)group_tile_nodes(group_gw(d.G), d.wk);
    const uint32_t E1 = d.meta[0], total = d.meta[1];
    if (threadIdx.x == 0) d.joff[E1] = total;
    __threadfence_block();
    const uint32_t n_tiles = cut_tiles(d.joff, E1, TJ, TN, d.tiles, (int)threadIdx.x);
    if (threadIdx.x == 0) {
        d.tiles[n_tiles] = E1;
        d.meta[2] = n_tiles;
    }
}

// The groups' counters of packed entries start at zero.
__global__ void k_group_clear(const GroupDesc *__restrict__ gd) {
    if (threadIdx.x < 8) gd[blockIdx.x].meta[threadIdx.x] = 0u;
}

// Work-unit offsets of the groups (one block), one list per kernel instance
// (group_list: the walks, up to 8 members or more): ng + 1
// offsets each, then one cursor each.
__global__ __launch_bounds__(1024) void k_group_units(const GroupDesc *__restrict__ gd, int32_t ng,
                                                      uint32_t *__restrict__ units) {
    const int32_t per = (ng + (int32_t)blockDim.x - 1) / (int32_t)blockDim.x;
    const int32_t g0 = min(ng, (int32_t)threadIdx.x * per), g1 = min(ng, g0 + per);
    for (int list = 0; list < GROUP_LISTS; ++list) {
        uint32_t sum = 0;
        for (int32_t g = g0; g < g1; ++g)
            if (group_list(gd[g].G, gd[g].wk) == list) sum += gd[g].meta[2] * (uint32_t)gd[g].n_chunks;
        uint32_t total;
        uint32_t run = block_excl_sum(sum, &total);
        uint32_t *u = units + list * (ng + 1);
        for (int32_t g = g0; g < g1; ++g) {
            u[g] = run;
            if (group_list(gd[g].G, gd[g].wk) == list) run += gd[g].meta[2] * (uint32_t)gd[g].n_chunks;
        }
        if (threadIdx.x == 0) {
            u[ng] = total;
            units[GROUP_LISTS * (ng + 1) + list] = 0u;
        }
    }
}

// ------------------------------------------------------------ meet kernel
// The single-query meet kernel's scheme with a group in place of a query:
// persistent blocks take units (group, tile of its compacted walks, chunk of
// vb nodes with in-edges) from a device cursor, stage the tile's positions in
// LDS, and hand the pairs (v, entry) of a unit, v-major, to the waves in chunks
// of 64.  A lane keeps NS pairs in flight; a pair carries the LDS offset of
// its entry's block for the next step and the mask of members still tested.
// A step reads the positions of the members present at that step, then
// compares.  Counts go to 16-bit LDS counters per (member, node) (a unit
// holds at most TJ < 2^16 walks), flushed to the members' counts once per
// unit.  WK = 1 (stitched): the walk's first 2^k
// steps are its own draws, the rest is read from the segment index, one load
// per iteration, as in the single-query kernel.  WK = 2 (stratified): walk j
// of v is the fixed-length walk of slot pi_v(j) (the shuffle and the class
// search are done when the pair starts), it takes no stop draws, and a meet of
// member q adds Lemma 5's weight of the classes of walk j of s_q and of v to a
// 64-bit LDS sum per (member, node).

template <int GW>
struct GSlot {
    uint32_t left;     // steps left (16 bits): of the entry's longest member walk, or of walk
                       // (v, j) if that is shorter | node index << 16 | those at its start << 24
    uint32_t live;     // members still tested (bit q)
    uint32_t b;        // LDS offset of the entry's block for the next step
    uint32_t o, d;     // current node: slot offset in E and in-degree
    WalkDraws rng;
    uint32_t t;        // stitched: steps taken
    uint32_t ph;       // stitched: 0 head; 1 node id, 2 pool offsets, 3 segment length,
                       // 4 tail step; 5 chain, 6 next segment's length
    uint32_t tsig, tm, tu, tseg, tsl;   // stitched tail: entry slot, chain index, position,
                                        // segment, its length
    uint32_t cj;       // stratified: class of walk (v, j) | j << 8
};

// Compares the pair's position at step t with the members' positions at step t,
// for the lanes in `act`.  The entry's block for step t is the word of members
// with a position at t, then the marks of those positions in member order; the
// slot's offset b moves on to the next step's block (every step is compared
// once, in order).  Meets are rare on large graphs: the common step reads the
// block in 16-byte pieces and only asks whether any mark is the pair's (a meet, or
// one in 65,536 positions that differs in the other half).  Up to GROUP_FEW_HITS
// lanes with such a mark are taken in turn, and the whole wave compares the
// members' positions themselves, one per lane, in their walks' tables.  Beyond it
// each lane finds the places of its marks in the block and compares those
// members' positions: in turn, the wave waited for a load per lane, and groups on
// small graphs, where meets are frequent, took (8 members, R = 2,000) 671 us at n =
// 1,000, now 292, at n = 100 730 and 340, on a star of 1,000 nodes 1,635 and 615.
// Returns the members still tested that meet at this step.  Called by all lanes
// of a wave.
// The kernel is bound by these reads of LDS: with whole positions in the blocks
// 32 queries at n = 40,000, R = 1,521, took 1,812 us, with marks 1,314; at n = 2^18,
// R = 9,502: 50.1 ms and 47.9, bound by the gathers as well.
constexpr int GROUP_FEW_HITS = 4;
template <int GW, int WK>
__device__ __forceinline__ uint32_t group_compare(GSlot<GW> &w, bool act, const uint32_t *s_nodes,
                                                  const GroupDesc &d, int lane) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    auto as2 = [](uint32_t x) { return __builtin_bit_cast(u16x2, x); };
    bool hit = false;
    uint32_t am = 0;
    if (act) {
        const uint32_t mine = mark_of(w.o) | (w.o << 16);
        const uint4 *blk = reinterpret_cast<const uint4 *>(s_nodes + w.b);
        const uint4 h = blk[0];
        am = h.x;
        const uint32_t pieces = block_words((uint32_t)__popc(am)) >> 2;
        // the least difference of a mark, per half word
        u16x2 least = __builtin_elementwise_min(as2(h.y ^ mine), as2(h.z ^ mine));
        least = __builtin_elementwise_min(least, as2(h.w ^ mine));
        for (uint32_t i = 1; i < pieces; ++i) {
            const uint4 p = blk[i];
            least = __builtin_elementwise_min(least, __builtin_elementwise_min(as2(p.x ^ mine), as2(p.y ^ mine)));
            least = __builtin_elementwise_min(least, __builtin_elementwise_min(as2(p.z ^ mine), as2(p.w ^ mine)));
        }
        hit = least.x == 0 || least.y == 0;
        w.b += 4u * pieces;
    }
    uint32_t met = 0;
    if (const uint64_t hits = __ballot(hit)) {
        if (__popcll(hits) > GROUP_FEW_HITS) {
            if (hit) {
                // the places of the marks that are the pair's, then those members' positions
                const uint32_t mine = mark_of(w.o) | (w.o << 16);
                const uint32_t c = (uint32_t)__popc(am), words = block_words(c);
                const uint32_t *blk = s_nodes + w.b - words;
                uint32_t at = 0;
                for (uint32_t i = 0; 2u * i < c; ++i) {
                    const uint32_t x = blk[1u + i] ^ mine;
                    at |= ((x & 0xffffu) == 0u ? 1u : 0u) << (2u * i);
                    at |= (x >> 16 == 0u ? 2u : 0u) << (2u * i);
                }
                at &= c < 32u ? (1u << c) - 1u : 0xffffffffu;
                const uint32_t step = (w.left >> 24) - (w.left & 0xffffu);   // 1, 2, ..
                const uint32_t j = WK == 2 ? w.cj >> 8 : w.rng.j;
                for (; at; at &= at - 1u) {
                    // the member of place p is bit p of those set in am
                    uint32_t p = (uint32_t)__builtin_ctz(at), q = 0, rest = am;
#pragma unroll
                    for (uint32_t half = 16u; half > 0u; half >>= 1) {
                        const uint32_t low = (uint32_t)__popc(rest & ((1u << half) - 1u));
                        if (p >= low) {
                            p -= low;
                            q += half;
                            rest >>= half;
                        }
                    }
                    if (d.sw[q][(size_t)j * (size_t)d.L + step - 1u] == w.o) met |= 1u << q;
                }
            }
        } else {
            for (uint64_t hm = hits; hm != 0ull; hm &= hm - 1ull) {
                const int from = __builtin_ctzll(hm);
                const uint32_t fam = __builtin_amdgcn_readlane(am, from), fo = __builtin_amdgcn_readlane(w.o, from),
                               fleft = __builtin_amdgcn_readlane(w.left, from),
                               fj = WK == 2 ? (uint32_t)__builtin_amdgcn_readlane(w.cj, from) >> 8
                                            : (uint32_t)__builtin_amdgcn_readlane(w.rng.j, from);
                const uint32_t step = (fleft >> 24) - (fleft & 0xffffu);   // 1, 2, ..
                bool same = false;
                if (lane < 32 && ((fam >> lane) & 1u))
                    same = d.sw[lane][(size_t)fj * (size_t)d.L + step - 1u] == fo;
                const uint32_t who = (uint32_t)__ballot(same);
                if (lane == from) met = who;
            }
        }
    }
    return met & w.live;
}

template <int NS, int GW, int WK, bool PACKED>
__global__ __launch_bounds__(GROUP_BLOCK) void k_meet_group(const GroupDesc *__restrict__ gd, int32_t ng,
                                                            const uint32_t *__restrict__ ustart,
                                                            uint32_t *__restrict__ cursor,
                                                            unsigned long long *__restrict__ counters) {
    constexpr bool STITCHED = WK == 1, STRAT = WK == 2;
    constexpr int TJ = group_tile_j(GW, WK), TN = group_tile_nodes(GW, WK), GM = 4 * GW;
    constexpr int HL = group_hub_rows(2 * WK + (GW > 2 ? 1 : 0));
    __shared__ uint2 s_hub[PACKED ? HL : 1];   // rows of a packed graph's hubs
    __shared__ __attribute__((aligned(16))) uint32_t s_nodes[TN];
    __shared__ uint32_t s_jl[TJ];   // walk index of the entry (below 2^24) | longest member walk << 24
    __shared__ uint16_t s_off[TJ];
    __shared__ uint32_t s_cnt[STRAT ? 1 : GM / 2 * MEET_VB];   // members 2i, 2i+1 in the low, high half
    // stratified: weighted sums per (member, node), the nodes' shuffle keys,
    // the class starts
    constexpr int VBW = group_strat_vb(GW);
    __shared__ unsigned long long s_w[STRAT ? GM * VBW : 1];
    __shared__ uint4 s_fk[STRAT ? MEET_VB : 1];
    __shared__ uint32_t s_ccum[STRAT ? MAX_CAP + 2 : 1];
    __shared__ uint32_t s_vid[MEET_VB];
    __shared__ uint2 s_vrow[MEET_VB];
    __shared__ uint32_t s_srcm[MEET_VB];   // members whose source is the node
    __shared__ uint32_t s_unit, s_item;

    const int lane = threadIdx.x & 63;
    const uint32_t n_units = ustart[ng];
    uint32_t cur_g = 0xffffffffu, cur_tile = 0xffffffffu;
    uint32_t K = 0;
    Work work;

    for (;;) {
        if (threadIdx.x == 0) s_unit = atomicAdd(cursor, 1u);
        __syncthreads();
        const uint32_t unit = s_unit;
        if (unit >= n_units) break;
        int32_t lo = 0, hi = ng;
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (ustart[mid] <= unit) lo = mid; else hi = mid;
        }
        const int32_t gi = lo;
        const GroupDesc &d = gd[gi];
        const int32_t n_chunks = (int32_t)uni((uint32_t)d.n_chunks);
        const int32_t vb = (int32_t)uni((uint32_t)d.vb);
        const int32_t G = (int32_t)uni((uint32_t)d.G);
        const int32_t gw = (int32_t)uni((uint32_t)d.gw);
        const uint32_t local = unit - ustart[gi];
        const uint32_t tile = local / (uint32_t)n_chunks;
        const uint32_t chunk = local - tile * (uint32_t)n_chunks;
        const PhiloxKey key{uni(d.k0), uni(d.k1)};
        const uint32_t T = uni(d.T);
        const Gather rows = gather_of<HL>(d);
        const uint32_t gmask = G >= 32 ? 0xffffffffu : (1u << G) - 1u;
        const uint32_t NN = uni((uint32_t)d.Rmax), sa = uni((uint32_t)d.sa), sb = uni((uint32_t)d.sb);
        const int32_t phi = (int32_t)uni((uint32_t)d.L);
        if ((uint32_t)gi != cur_g || tile != cur_tile) {
            const uint32_t k0 = uni(d.tiles[tile]), k1 = uni(d.tiles[tile + 1]);
            const uint32_t nb = d.joff[k0], ne = d.joff[k1];
            K = k1 - k0;
            for (uint32_t i = threadIdx.x; i < K; i += blockDim.x) {
                s_off[i] = (uint16_t)(d.joff[k0 + i] - nb);
                uint32_t mx = 0;
                for (int32_t wd = 0; wd < gw; ++wd) {
                    const uint32_t lw = d.glen[(size_t)(k0 + i) * gw + wd];
                    mx = max(mx, max(max(byte_of(lw, 0), byte_of(lw, 1)), max(byte_of(lw, 2), byte_of(lw, 3))));
                }
                s_jl[i] = d.jj[k0 + i] | (mx << 24);
            }
            for (uint32_t i = threadIdx.x; i < ne - nb; i += blockDim.x) s_nodes[i] = d.pos[nb + i];
            if (STRAT)
                for (uint32_t i = threadIdx.x; i < (uint32_t)phi + 2; i += blockDim.x)
                    s_ccum[i] = d.tab->ccum[i];
            if (PACKED)
                for (uint32_t i = threadIdx.x; i < (uint32_t)d.n_hubs; i += blockDim.x) s_hub[i] = d.hubs[i];
            cur_g = (uint32_t)gi;
            cur_tile = tile;
        }
        const int32_t vbase = (int32_t)chunk * vb;
        const uint32_t nv = uni((uint32_t)min(vb, d.n_active - vbase));
        if (STRAT)
            for (uint32_t i = threadIdx.x; i < GM * VBW; i += blockDim.x) s_w[i] = 0ull;
        else
            for (uint32_t i = threadIdx.x; i < GM / 2 * MEET_VB; i += blockDim.x) s_cnt[i] = 0u;
        for (uint32_t i = threadIdx.x; i < nv; i += blockDim.x) {
            const uint32_t id = (uint32_t)d.active[vbase + (int32_t)i];
            s_vid[i] = id;
            s_vrow[i] = d.nodes[id];
            uint32_t m = 0;
            for (int32_t q = 0; q < G; ++q) m |= (uint32_t)((uint32_t)d.s[q] == id) << q;
            s_srcm[i] = m;
            if (STRAT) s_fk[i] = philox4x32_10(id, 0u, 0u, DOM_SHUFFLE, key);
        }
        if (threadIdx.x == 0) s_item = 0u;
        __syncthreads();

        // item i = vl * K + k for node vl < nv and entry k < K
        // (K and nv are the same in all lanes; said so, the refill's bookkeeping
        // stays in scalar registers)
        const uint32_t Ku = uni(K), total = nv * Ku;
        uint32_t ci = 0, ce = 0, cvl = 0, ck = 0;
        bool drained = false;
        // node cvl: its row, draw constants, the members tested (all but those
        // whose source it is; a member whose walk j is empty never reads a
        // position) and, stratified, its shuffle key
        uint32_t vo = 0, vd = 0, wa = 0, wb = 0, wcc = 0, vlive = 0;
        uint4 vfk = make_uint4(0u, 0u, 0u, 0u);
        uint32_t at_vl = NIL;
        auto enter_node = [&]() {
            at_vl = cvl;
            const uint2 row = s_vrow[cvl];
            vo = uni(row.x);
            vd = uni(row.y);
            const WalkDraws w = walk_draws_begin(uni(s_vid[cvl]), 0u, key, STRAT ? DOM_STRAT : DOM_WALK);
            wa = uni(w.a);
            wb = uni(w.b);
            wcc = uni(w.cc);
            vlive = gmask & ~uni(s_srcm[cvl]);
            if (STRAT) {
                const uint4 k = s_fk[cvl];
                vfk = make_uint4(uni(k.x), uni(k.y), uni(k.z), uni(k.w));
            }
        };
        // the wave's slots, and which lanes' have a pair
        GSlot<GW> sl[NS];
        uint64_t busy[NS];
#pragma unroll
        for (int qq = 0; qq < NS; ++qq) {
            sl[qq] = GSlot<GW>{};
            busy[qq] = 0ull;
        }

        for (;;) {
            // ---- refill idle slots; a pair with no member to test (each
            // member's source is v), or a stratified walk of class 0, is skipped
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) {
                uint64_t need = ~busy[qq];
                while (need != 0ull) {
                    if (ci == ce) {
                        if (drained) break;
                        uint32_t x = 0;
                        if (lane == 0) x = atomicAdd(&s_item, ITEM_CHUNK);
                        x = uni(x);
                        if (x >= total) {
                            drained = true;
                            break;
                        }
                        ci = x;
                        ce = min(x + ITEM_CHUNK, total);
                        cvl = uni(x / Ku);
                        ck = x - cvl * Ku;
                        if (cvl != at_vl) enter_node();
                    }
                    uint32_t take = min(ce - ci, Ku - ck);
                    if (vlive != 0u) {
                        take = min(take, (uint32_t)__popcll(need));
                        const uint32_t rank = lane_rank(need);
                        uint64_t mine = need & __ballot(rank < take);
                        const uint32_t k = min(ck + rank, Ku - 1u);
                        const uint32_t jl = s_jl[k], off = s_off[k];
                        uint32_t j = jl & 0xffffffu, left = jl >> 24, cv = 0;
                        if (STRAT) {
                            uint32_t r = 0;
                            if (in_mask(mine)) {
                                r = shuffle_slot(j, NN, sa, sb, vfk);
                                cv = slot_class(r, s_ccum, phi);
                            }
                            mine &= __ballot(cv > 0u);
                            left = min(left, cv);
                            cv |= j << 8;
                            j = r;
                        }
                        GSlot<GW> &w = sl[qq];
                        const bool me = in_mask(mine);
                        w.left = me ? left | (cvl << 16) | (left << 24) : w.left;
                        w.live = me ? vlive : w.live;
                        w.b = me ? off : w.b;
                        w.o = me ? vo : w.o;
                        w.d = me ? vd : w.d;
                        w.rng.j = me ? j : w.rng.j;
                        w.rng.a = me ? wa : w.rng.a;
                        w.rng.b = me ? wb : w.rng.b;
                        w.rng.cc = me ? wcc : w.rng.cc;
                        w.rng.mt = me ? 0ull : w.rng.mt;
                        if (STITCHED) {
                            w.t = me ? 0u : w.t;
                            w.ph = me ? 0u : w.ph;
                        }
                        if (STRAT) w.cj = me ? cv : w.cj;
                        work.pairs += (uint32_t)__popcll(mine);
                        busy[qq] |= mine;
                        need &= ~mine;
                    }
                    ci += take;
                    ck += take;
                    if (ck == Ku) {
                        ck = 0;
                        ++cvl;
                        if (ci < ce) enter_node();
                    }
                }
            }
            uint64_t any = 0ull;
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) any |= busy[qq];
            if (any == 0ull) {
                if (drained) break;
                continue;
            }

            // ---- head steps: draws, then one load per slot (a head step's
            // gather or the load its stitched tail phase needs), then compares
            uint64_t go[NS];
            uint32_t at[NS];
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) {
                const uint64_t head = STITCHED ? busy[qq] & __ballot(sl[qq].ph == 0u) : busy[qq];
                uint2 x = make_uint2(0u, 0u);
                if (!STITCHED || in_mask(head)) x = walk_draw_next(sl[qq].rng, key);
                work.draws += (uint32_t)__popcll(head);
                go[qq] = STRAT ? head : head & __ballot(x.x < T);
                if (STITCHED) busy[qq] &= ~(head & ~go[qq]);
                at[qq] = sl[qq].o + pick32(x.y, sl[qq].d);
            }
            uint2 e[NS];
            uint32_t tv[NS];
            int64_t tb[NS], te[NS];
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) {
                if (in_mask(go[qq])) {
                    if (PACKED) e[qq].x = rows.E4[at[qq]];
                    else e[qq] = load_edge(rows.E, at[qq]);
                }
                if (STITCHED && in_mask(busy[qq] & ~go[qq])) {
                    const GSlot<GW> &w = sl[qq];
                    switch (w.ph) {
                    case 1: tv[qq] = d.ix.node_of[w.o]; break;
                    case 2: tb[qq] = d.ix.pool_off[w.tsig]; te[qq] = d.ix.pool_off[w.tsig + 1]; break;
                    case 3:
                    case 6: tv[qq] = d.ix.seg_lens[w.tseg]; break;
                    case 4: tv[qq] = d.ix.seg[(size_t)w.tseg * d.ix.seg_len + w.tu]; break;
                    default: tv[qq] = d.ix.chain[(size_t)w.tsig * d.ix.width + w.tm + 1]; break;
                    }
                }
            }
            // ---- one compare per slot that reached a new position (a head
            // step's node, or a stitched tail step read from the index), then
            // the end tests of its phase; the other tail phases only advance
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) {
                GSlot<GW> &w = sl[qq];
                const bool head = in_mask(go[qq]);
                const bool tail_step = STITCHED && in_mask(busy[qq] & ~go[qq]) && w.ph == 4u;
                work.moves += (uint32_t)__popcll(go[qq]);
                if (head) {
                    const uint2 to = PACKED ? unpack_row(e[qq].x, rows.obits, s_hub) : e[qq];
                    w.o = to.x;
                    w.d = to.y;
                } else if (tail_step) {
                    ++work.tail;
                    w.o = tv[qq];
                    ++w.tu;
                }
                if (head || tail_step) {
                    --w.left;
                    if (STITCHED) ++w.t;
                }
                const uint32_t met = group_compare<GW, WK>(w, head || tail_step, s_nodes, d, lane);
                if (const uint64_t mm = __ballot(met != 0u)) {
                    uint32_t n_met = 0;
                    for (uint64_t m = mm; m; m &= m - 1ull)
                        n_met += (uint32_t)__popc(__builtin_amdgcn_readlane(met, __builtin_ctzll(m)));
                    work.meets += n_met;
                    if (met) {
                        const uint32_t vl = (w.left >> 16) & 0xffu;
                        w.live &= ~met;
                        for (uint32_t m = met; m; m &= m - 1u) {
                            const uint32_t q = (uint32_t)__builtin_ctz(m);
                            if (STRAT)
                                atomicAdd(&s_w[q * VBW + vl],
                                          strat_weight(d.tab->a, d.scls[q][w.cj >> 8], w.cj & 0xffu));
                            else
                                atomicAdd(&s_cnt[(q >> 1) * MEET_VB + vl], 1u << (16 * (q & 1u)));
                        }
                    }
                }
                // the pair ends with its last member walk (or, stratified, the
                // class of walk (v, j)), when every member tested has met, or
                // at a node without in-neighbours
                bool more = head && w.live != 0u && w.d != 0u && (w.left & 0xffffu) != 0u;
                if constexpr (!STITCHED) {
                    busy[qq] = __ballot(more);
                    continue;
                }
                if (more && w.t == (uint32_t)d.ix.seg_len)
                    w.ph = 1;   // the head made all its moves: enter a pool slot of this node
                if (in_mask(busy[qq] & ~go[qq])) {
                more = true;
                switch (w.ph) {
                case 1:   // the end node's id
                    w.tsig = tv[qq];
                    w.ph = 2;
                    break;
                case 2: { // its pool: slot picked by draw (v, j, 0, DOM_ENTRY)
                    const uint4 x = philox4x32_10(s_vid[(w.left >> 16) & 0xffu], w.rng.j, 0u, DOM_ENTRY, key);
                    w.tsig = (uint32_t)(tb[qq] + (int64_t)pick64(x.x, (uint64_t)(te[qq] - tb[qq])));
                    w.tseg = w.tsig;
                    w.tm = 0;
                    w.ph = 3;
                    break;
                }
                case 3:
                case 6:   // a segment's length
                    w.tsl = tv[qq];
                    w.tu = 0;
                    w.ph = 4;
                    if (w.tsl == 0u) more = false;
                    break;
                case 4:   // after a tail step
                    if (w.live == 0u || (w.left & 0xffffu) == 0u) {
                        more = false;
                    } else if (w.tu == w.tsl) {
                        if (w.tsl < (uint32_t)d.ix.seg_len || w.tm + 1 >= (uint32_t)d.ix.width)
                            more = false;
                        else
                            w.ph = 5;
                    }
                    break;
                default:  // the chain's next segment
                    ++w.tm;
                    w.tseg = tv[qq];
                    if (w.tseg == NIL) more = false;
                    else w.ph = 6;
                    break;
                }
                }
                busy[qq] = __ballot(more);
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < (uint32_t)G * nv; i += blockDim.x) {
            const uint32_t q = i / nv, vi = i - q * nv;
            if (STRAT) {
                const unsigned long long c = s_w[q * VBW + vi];
                if (c) atomicAdd(&d.wsum[q][s_vid[vi]], c);
            } else {
                const uint32_t c = (s_cnt[(q >> 1) * MEET_VB + vi] >> (16 * (q & 1u))) & 0xffffu;
                if (c) atomicAdd(&d.cnt[q][s_vid[vi]], c);
            }
        }
    }

    add_work(ctr_set(counters), work);
}

#ifndef SRK_GROUP_SLOTS_STITCHED
#define SRK_GROUP_SLOTS_STITCHED 2
#endif

template <int NS, int GW, int WK>
int group_grid_blocks() {
    static const int blocks = [] {
        int dev = 0, cus = 0, per = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_meet_group<NS, GW, WK, false>,
                                                           GROUP_BLOCK, 0);
        if (cus <= 0) cus = 256;
        if (per <= 0) per = 1;
        return cus * per;
    }();
    return blocks;
}

template <int NS, int GW, int WK>
void launch_group_list(const GroupSet &gs, int list, unsigned long long *counters, hipStream_t st) {
    if (gs.units_bound[list] <= 0) return;
    const int blocks = (int)std::min<int64_t>(gs.units_bound[list], group_grid_blocks<NS, GW, WK>());
    const auto kernel = rows_of(gs.rows[list]) == ROWS_PACKED ? k_meet_group<NS, GW, WK, true>
                                                              : k_meet_group<NS, GW, WK, false>;
    kernel<<<blocks, GROUP_BLOCK, 0, st>>>(
        gs.desc, gs.ng, gs.units + (size_t)list * (gs.ng + 1),
        gs.units + GROUP_LISTS * ((size_t)gs.ng + 1) + list, counters);
}

}  // namespace

int32_t group_max_tiles(int64_t Rmax, int64_t sum_RL, int32_t L, int32_t G, int32_t wk) {
    const int GW = group_gw(G);
    // (stated with whole positions in the blocks, of which there are never fewer words)
    const int64_t NW = group_tile_nodes(GW, wk) - (int64_t)((G + 4) & ~3) * L;
    return (int32_t)(2 + Rmax / group_tile_j(GW, wk) + group_pos_words(Rmax, sum_RL, L) / NW);
}

// A unit's pairs are (its vb nodes) x (the tile's entries); each unit has
// fixed work (the claim, three barriers, staging its nodes, flushing its
// counters, the wait for its longest pair).  A group's tile holds few entries
// (every entry carries all members' positions), so small units pay that work
// over few pairs: on the n = 2^22 graph a 32-member group took 855 ms with 256
// nodes per unit, 894 with 128, 971 with 64 and 1121 with 32 (stitched: 994 /
// 1049 / 1161 / 1366).  Groups therefore take the largest unit that still
// leaves 64 chunks of nodes, whatever the lone queries were tuned to.
int32_t group_unit_nodes(int32_t n_active, int32_t G, int32_t wk) {
    int32_t vb = MEET_VB;
    while (vb > 32 && (n_active + vb - 1) / vb < 64) vb >>= 1;
    if (wk == 2 && G > 8) vb = std::min(vb, GROUP_STRAT32_VB);   // the LDS sums' node limit
    return vb;
}

void describe_group(const QueryDesc *const *members, int32_t G, GroupDesc *gd) {
    const QueryDesc &d0 = *members[0];
    *gd = GroupDesc{};
    gd->nodes = d0.nodes;
    gd->E = d0.E;
    gd->E4 = d0.E4;
    gd->hubs = d0.hubs;
    gd->obits = d0.obits;
    gd->n_hubs = d0.n_hubs;
    gd->active = d0.active;
    gd->n_active = d0.n_active;
    gd->G = G;
    gd->gw = (G + 3) / 4;
    gd->wk = d0.kind == K_GROUPED_STITCHED ? 1 : d0.kind == K_GROUPED_STRAT ? 2 : 0;
    gd->vb = group_unit_nodes(d0.n_active, G, gd->wk);
    gd->n_chunks = (gd->n_active + gd->vb - 1) / gd->vb;
    gd->ix = d0.ix;
    gd->tab = d0.tab;
    gd->sa = d0.sa;
    gd->sb = d0.sb;
    gd->L = d0.L;
    gd->k0 = d0.k0;
    gd->k1 = d0.k1;
    gd->T = d0.T;
    for (int32_t q = 0; q < G; ++q) {
        const QueryDesc &dq = *members[q];
        gd->s[q] = dq.s;
        gd->R[q] = dq.R;
        gd->sw[q] = dq.sw;
        gd->slen[q] = dq.slen;
        gd->cnt[q] = dq.cnt;
        gd->wsum[q] = dq.wsum;
        gd->scls[q] = dq.scls;
        gd->Rmax = std::max(gd->Rmax, dq.R);
    }
}

size_t group_buffers(GroupDesc *gd, int64_t sum_RL, char *base) {
    size_t at = 0;
    auto take = [&](size_t b) {
        char *r = base ? base + at : nullptr;
        at += (b + 255) & ~(size_t)255;
        return r;
    };
    const int32_t mt = group_max_tiles(gd->Rmax, sum_RL, gd->L, gd->G, gd->wk);
    gd->jj = (uint32_t *)take(4 * (size_t)gd->Rmax);
    gd->joff = (uint32_t *)take(4 * ((size_t)gd->Rmax + 1));
    gd->glen = (uint32_t *)take(4 * (size_t)gd->Rmax * (size_t)gd->gw);
    gd->pos = (uint32_t *)take(4 * (size_t)group_pos_words(gd->Rmax, sum_RL, gd->L));
    gd->tiles = (uint32_t *)take(4 * ((size_t)mt + 1));
    gd->meta = (uint32_t *)take(32);
    return at;
}

static_assert(GROUP_LISTS == 6, "one launch below per group kernel instance");

int launch_groups(const GroupSet &gs, unsigned long long *counters, hipStream_t st) {
    if (gs.ng <= 0) return SIMRANK_OK;
    k_group_clear<<<gs.ng, 64, 0, st>>>(gs.desc);
    k_group_pack<<<dim3((unsigned)((gs.max_R + PACK_J - 1) / PACK_J), (unsigned)gs.ng), 256, 0, st>>>(gs.desc);
    k_group_tiles<<<gs.ng, 64, 0, st>>>(gs.desc);
    k_group_units<<<1, 1024, 0, st>>>(gs.desc, gs.ng, gs.units);
    launch_group_list<SRK_GROUP_SLOTS, 2, 0>(gs, 0, counters, st);
    launch_group_list<SRK_GROUP_SLOTS, 8, 0>(gs, 1, counters, st);
    launch_group_list<SRK_GROUP_SLOTS_STITCHED, 2, 1>(gs, 2, counters, st);
    launch_group_list<SRK_GROUP_SLOTS_STITCHED, 8, 1>(gs, 3, counters, st);
    launch_group_list<SRK_GROUP_SLOTS, 2, 2>(gs, 4, counters, st);
    launch_group_list<SRK_GROUP_SLOTS, 8, 2>(gs, 5, counters, st);
    SRK_HIP(hipGetLastError());
    return SIMRANK_OK;
}

}  // namespace srk
