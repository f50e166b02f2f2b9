// Single-source query: source walks, packed and cut into LDS tiles, the
// fused walk + meet + count kernel, and the estimate.
//
// Method (Section 2.2; Lemma 2; Section 3.2 pairing): walk j of the source s
// is paired with walk j of every node v, j < R; the pair meets if the two
// walks are on the same node at the same step; s_hat(s, v) = meets / R.
//
// The meet kernel generates walk (v, j) only as far as it can still meet walk
// (s, j): it stops at the first meeting step (a pair counts once, Section 4.4),
// when walk (v, j) stops, and when walk (s, j) has no later position.  This
// reads exactly the positions the meet test compares, so the counts equal
// those of full walks, while a pair costs about sum_t c^t = c / (1 - c) moves.
#include <math.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "common.hpp"
#include "device_common.hpp"
#include "philox.hpp"

namespace srk {
namespace {

// ------------------------------------------------------------ small kernels

// Clears a query's counts or sums and its meta words; x over nodes.
__device__ __forceinline__ void clear_query(const QueryDesc &d) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < 8) d.meta[threadIdx.x] = 0u;
    if (strat_kind(d.kind)) {
        for (int64_t v = i; v < d.n; v += (int64_t)gridDim.x * blockDim.x) d.wsum[v] = 0ull;
    } else {
        for (int64_t v = i; v < d.n; v += (int64_t)gridDim.x * blockDim.x) d.cnt[v] = 0u;
    }
}

// grid (x over nodes, y = query); clears `words` words of counters
__global__ void k_init(const QueryDesc *__restrict__ qd, unsigned long long *__restrict__ counters,
                       int32_t words) {
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int32_t w = threadIdx.x; w < words; w += blockDim.x) counters[w] = 0ull;
    clear_query(qd[blockIdx.y]);
}

// A stratified query's class table, which comes with the launch.
__global__ void k_put_tab(StratTab *dst, StratTab t) {
    for (int i = threadIdx.x; i < MAX_CAP + 2; i += blockDim.x) dst->ccum[i] = t.ccum[i];
    for (int i = threadIdx.x; i < MAX_CAP + 1; i += blockDim.x) dst->a[i] = t.a[i];
}

// The same for one query whose descriptor comes with the launch and is put in
// device memory for the kernels behind it; grid (x over nodes).
__global__ void k_init_one(QueryDesc *__restrict__ dst, QueryDesc d,
                           unsigned long long *__restrict__ counters, int32_t words) {
    if (blockIdx.x == 0) {
        for (int32_t w = threadIdx.x; w < words; w += blockDim.x) counters[w] = 0ull;
        if (threadIdx.x == 0) {
            *dst = d;
            if (words == CTR_SUMS) counters[STAMP_BEGIN] = wall_clock64();
        }
    }
    clear_query(d);
}

// s_hat(s, v) = cnt[v] / R; the pair (s, s) meets at step 0 for every j.
// Stratified (Algorithm 2): s~(s, v) = wsum[v] 2^-40 / z, and the variant
// normalised by the N pairs, s~(s, v) N / z; both are 1 at v = s.
__device__ __forceinline__ void estimate_one(const QueryDesc &d, int64_t v) {
    if (strat_kind(d.kind)) {
        const double x = (double)d.wsum[v] * 9.094947017729282379150390625e-13;   // 2^-40
        const double e = x / d.z;
        if (d.out) d.out[v] = (v == d.s) ? 1.0 : e;
        if (d.out_n) d.out_n[v] = (v == d.s) ? 1.0 : e * ((double)d.R / d.z);
        return;
    }
    if (v == d.s) d.cnt[v] = (uint32_t)d.R;
    if (d.out) d.out[v] = (v == d.s) ? 1.0 : (double)d.cnt[v] / (double)d.R;
}

// grid (x over nodes, y = query); the last kernel of a launch sequence, it also
// folds the sets of work counters into the totals.
__global__ void k_estimate(const QueryDesc *__restrict__ qd, unsigned long long *__restrict__ counters) {
    const unsigned long long begun = wall_clock64();
    const QueryDesc &d = qd[blockIdx.y];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 8) {
        unsigned long long sum = 0;
        for (int i = 1; i <= CTR_SETS; ++i) sum += counters[8 * i + threadIdx.x];
        counters[threadIdx.x] = sum;
        if (threadIdx.x == 0) counters[STAMP_MET] = begun;
    }
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < d.n;
         v += (int64_t)gridDim.x * blockDim.x)
        estimate_one(d, v);
    if (blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1 && threadIdx.x == 0)
        counters[STAMP_END] = wall_clock64();
}

// ------------------------------------------------------------ source walks
// Walk (s, j) for j < R: positions 1..len as o() values.  Stratified: walk j
// of s is the fixed-length walk generated in slot pi_s(j); its class goes to
// scls[j].  grid (x over j, y = query); sets: the counters are a query set's
// (CTR_SETS sets), else a ring entry's 8.
//
// A group member's walks go to its padded table (sw, slen), from which its
// group packs them.  A lone query's are packed here: the block keeps its walks'
// first WALK_LDS positions in LDS, drops the walks of length 0 (they can only
// meet at step 0, i.e. only the source itself), and takes room for the others'
// entries and positions with one atomic on meta[0..1]; so entries are in no
// order of j, and entry k + 1 starts where entry k ends.  Packing from the
// padded table by one block, a thread copying its walks word by word, took 13
// us at R = 1,521 and 60 at R = 9,502.  All kernels of a query but the meet
// kernel, before and now: 44 and 31 us at R = 1,521, 95 and 40 at R = 9,502,
// 305 and 45 at R = 38,005.
//
// A served request's walks run beside a persistent meet kernel, which leaves
// its compute unit a few KB of LDS: KEEP false keeps the positions in the
// padded table instead, from which each thread copies its own.
constexpr int WALK_LDS = 32;
template <bool KEEP>
__device__ __forceinline__ void source_walks(const QueryDesc &d, unsigned long long *counters,
                                             bool sets) {
    constexpr int HELD = KEEP ? WALK_LDS : 0;
    __shared__ uint32_t s_pos[KEEP ? WALK_LDS : 1][KEEP ? 256 : 1];
    __shared__ uint32_t s_at[2];
    const int32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if ((int32_t)(blockIdx.x * blockDim.x) >= d.R) return;
    const bool grouped = d.kind >= K_GROUPED;
    uint32_t *row = d.sw + (size_t)j * d.L;
    auto put = [&](int32_t t, uint32_t o) {   // position t + 1
        if (!grouped && t < HELD) s_pos[t][threadIdx.x] = o;
        else row[t] = o;
    };
    int32_t len = 0;
    if (j < d.R) {
        const PhiloxKey key{uni(d.k0), uni(d.k1)};
        const GlobalPtr<uint64_t> E = gp_uni((const uint64_t *)d.E);
        uint2 cur = d.nodes[d.s];
        // the draw of the next step is made while the step's gather is on its way
        if (strat_kind(d.kind)) {
            const uint4 fk = philox4x32_10((uint32_t)d.s, 0u, 0u, DOM_SHUFFLE, key);
            const uint32_t r = shuffle_slot((uint32_t)j, (uint32_t)d.R, (uint32_t)d.sa, (uint32_t)d.sb, fk);
            const uint32_t cls = slot_class(r, d.tab->ccum, d.L);
            WalkDraws w = walk_draws_begin((uint32_t)d.s, r, key, DOM_STRAT);
            uint2 x = walk_draw_next(w, key);
            for (int32_t t = 1; t <= (int32_t)cls; ++t) {
                if (cur.y == 0) break;
                const uint2 to = load_edge(E, cur.x + pick32(x.y, cur.y));
                x = walk_draw_next(w, key);
                cur = to;
                put(t - 1, cur.x);
                len = t;
            }
            d.scls[j] = (uint8_t)cls;
        } else {
            const bool stitched = d.kind == K_STITCHED || d.kind == K_GROUPED_STITCHED;
            const int32_t head = stitched ? min(d.ix.seg_len, d.L) : d.L;
            const uint32_t T = d.T;
            WalkDraws w = walk_draws_begin((uint32_t)d.s, (uint32_t)j, key);
            uint2 x = walk_draw_next(w, key);
            for (int32_t t = 1; t <= head; ++t) {
                if (x.x >= T || cur.y == 0) break;
                const uint2 to = load_edge(E, cur.x + pick32(x.y, cur.y));
                x = walk_draw_next(w, key);
                cur = to;
                put(t - 1, cur.x);
                len = t;
            }
            if (stitched && len == d.ix.seg_len && len < d.L) {
                const uint32_t y = d.ix.node_of[cur.x];
                const uint32_t sigma = entry_slot(d.ix, key, (uint32_t)d.s, (uint32_t)j, y);
                for (int32_t mm = 0; mm < d.ix.width && len < d.L; ++mm) {
                    const uint32_t sg = d.ix.chain[(size_t)sigma * d.ix.width + mm];
                    if (sg == NIL) break;
                    const int32_t sl = d.ix.seg_lens[sg];
                    for (int32_t u = 0; u < sl && len < d.L; ++u) {
                        put(len, d.ix.seg[(size_t)sg * d.ix.seg_len + u]);
                        ++len;
                    }
                    if (sl < d.ix.seg_len) break;
                }
            }
        }
        if (grouped) d.slen[j] = (uint8_t)len;
    }
    uint32_t entries, words;
    const uint32_t ek = block_excl_sum<uint32_t>(len > 0 ? 1u : 0u, &entries);
    const uint32_t eo = block_excl_sum<uint32_t>((uint32_t)len, &words);
    if (threadIdx.x == 0) {
        if (words) atomicAdd(&(sets ? ctr_set(counters) : counters)[C_SRC_MOVES], (unsigned long long)words);
        if (!grouped && entries) {
            const unsigned long long at =
                atomicAdd((unsigned long long *)d.meta, ((unsigned long long)words << 32) | entries);
            s_at[0] = (uint32_t)at;
            s_at[1] = (uint32_t)(at >> 32);
        }
    }
    if (grouped) return;
    __syncthreads();
    if (len == 0) return;
    const uint32_t k = s_at[0] + ek, off = s_at[1] + eo;
    d.jj[k] = (uint32_t)j;
    d.joff[k] = off;
    uint32_t *dst = d.swc + off;
    for (int32_t t = 0; t < min(len, HELD); ++t) dst[t] = s_pos[t][threadIdx.x];
    for (int32_t t = HELD; t < len; ++t) dst[t] = row[t];
}

template <bool KEEP>
__global__ __launch_bounds__(256) void k_source_walks(const QueryDesc *__restrict__ qd,
                                                      unsigned long long *__restrict__ counters,
                                                      bool sets) {
    source_walks<KEEP>(qd[blockIdx.y], counters, sets);
}

// The same for one query, its descriptor a kernel argument.
__global__ __launch_bounds__(256) void k_source_walks_one(QueryDesc d,
                                                          unsigned long long *__restrict__ counters) {
    source_walks<true>(d, counters, true);
}

// ------------------------------------------------------------ tiles
// First entries of a query's tiles.  HUB_TILE_NODES' tiles can be more than the
// buffer was sized for (max_tiles_for) where the positions may fill several:
// they lie where the source walks' padded table was, which the packing before
// was the last to read.
__device__ __forceinline__ uint32_t *tiles_of(const QueryDesc &d) {
    return d.tile_nodes == HUB_TILE_NODES && (uint64_t)d.R * (uint64_t)d.L > (uint64_t)HUB_TILE_NODES
               ? d.sw : d.tiles;
}

// Cuts the packed entries of a query into tiles that fit the meet kernel's LDS:
// with the kind's shape (TJ walks, TN positions), each tile is the longest run
// of walks from the previous one's end that holds at most TJ walks and TN
// positions (cut_tiles).  Called by all lanes of one wave.
__device__ void make_tiles(const QueryDesc &d, int lane) {
    const uint32_t R1 = d.meta[0], total = d.meta[1];
    const uint32_t TJ = (uint32_t)d.tile_j, TN = (uint32_t)d.tile_nodes;
    if (lane == 0) d.joff[R1] = total;
    uint32_t n_tiles, km = R1;
    if (R1 <= TJ && total <= TN) {
        n_tiles = R1 > 0u ? 1u : 0u;
        if (lane == 0 && R1 > 0u) tiles_of(d)[0] = 0u;
    } else {
        __threadfence_block();   // joff[R1] is read below
        n_tiles = cut_tiles(d.joff, R1, TJ, TN, tiles_of(d), lane);
        __threadfence_block();
        km = 0;
        for (uint32_t t = (uint32_t)lane; t < n_tiles; t += 64)
            km = max(km, (t + 1 < n_tiles ? tiles_of(d)[t + 1] : R1) - tiles_of(d)[t]);
        for (int dd = 32; dd > 0; dd >>= 1) km = max(km, __shfl_xor(km, dd, 64));
    }
    if (lane == 0) {
        tiles_of(d)[n_tiles] = R1;
        d.meta[2] = n_tiles;
        d.meta[3] = km;
    }
    __threadfence_block();
}

// ------------------------------------------------------------ work units
//
// A unit is a tile of a query's source walks and a run of its nodes with
// in-edges; a persistent block takes one at a time.  A unit costs a block 10
// to 25 us beside its pairs (claim, staging, the wait for its longest pair),
// and the grid waits for the block that ends last.  Unless the graph was
// tuned, the units of a launch therefore all hold about the same work, such
// that every block of the grid takes a whole number of rounds of them: one
// round per 2^27 pairs (about 0.5 ms), 16 at most, more only where MEET_VB nodes
// a unit ask for it.  A pair of stitched walks counts as several where its tail
// is long (pair_cost; up to 32 rounds then): tails are of very different lengths,
// and long units of them end far apart (c = 0.95, R = 2,000, segments of 1 and 4
// steps: counted as one and as several, n = 20,000: 8.64 and 6.80 ms, 6.09 and
// 5.55; n = 2^18: 154.4 and 153.4, 105.2 and 104.0).  Plain and
// stratified pairs count as one at any c: at c = 0.95 and 255 steps several rounds
// instead of one take 3.07 and 4.08 ms, one 2.85 and 3.67.  Meet kernel, with units of a fixed
// number of nodes by graph size (256 from 2^19 nodes with in-edges, 128, 64,
// 32 below) and with this rule: n = 500, R = 2,000: 96 and 32 us; n = 5,003,
// R = 1,521: 98 and 61; R = 9,502: 404 and 264; n = 40,000, R = 1,521: 386 and
// 303; R = 9,502: 1,738 and 1,680; n = 150,001, R = 9,502: 6,108 and 6,061;
// n = 2^18: 11.56 and 11.65 ms; n = 2^20: 50.3 ms both.
constexpr int UNIT_ROUNDS_LOG2_WORK = 27, UNIT_MAX_ROUNDS = 16, UNIT_MAX_ROUNDS_TAILS = 32;

// First unit of each tile and, behind them, the number of units: kept where a
// group member has its source walks' lengths.
// They and one word more fit there: 4 (3 + R / 2048 + R L / (12288 - L))
// bytes are fewer than R rounded up to 256, for every R and L up to MAX_CAP.
__device__ __forceinline__ uint32_t *tunits_of(const QueryDesc &d) {
    return reinterpret_cast<uint32_t *>(d.slen);
}

// Work of nodes x walks pairs of query d (below 2^62: 2^31 nodes, 2^24 walks, a
// cost of 43).
__device__ __forceinline__ uint64_t work_of(const QueryDesc &d, uint32_t nodes, uint32_t walks) {
    return (uint64_t)nodes * walks * d.cost;
}

// Rounds of units that a launch of `work` on `grid` blocks is cut into, its
// dearest pair costing `cost` and its largest full unit holding `most` of the
// work (MEET_VB nodes of its largest tile).
__device__ __forceinline__ uint64_t unit_rounds(uint64_t work, uint32_t cost, uint64_t most, uint32_t grid) {
    const uint64_t limit = cost > 1 ? UNIT_MAX_ROUNDS_TAILS : UNIT_MAX_ROUNDS;
    const uint64_t by_work = (work + ((1ull << UNIT_ROUNDS_LOG2_WORK) - 1)) >> UNIT_ROUNDS_LOG2_WORK;
    const uint64_t rounds = by_work < 1 ? 1 : by_work > limit ? limit : by_work;
    const uint64_t full = (most < 1 ? 1 : most) * grid;   // a round of full units
    const uint64_t least = (work + full - 1) / full;
    return rounds < least ? least : rounds;
}

__device__ __forceinline__ uint64_t work_each(uint64_t work, uint64_t units) {
    const uint64_t per = units ? (work + units - 1) / units : work;
    return per < 1 ? 1 : per;
}

// Work per unit of the queries of a kind in qd[0 .. nq).  A tile of few walks
// reaches MEET_VB nodes a unit below the common work, so it has more units than
// its share; the other tiles then take that many fewer.  Called by all lanes of
// one wave; results uniform.
__device__ uint64_t unit_work(const QueryDesc *qd, int32_t nq, int32_t kind, uint64_t work,
                              uint32_t cost, uint64_t most, uint32_t grid, int lane) {
    uint64_t units = unit_rounds(work, cost, most, grid) * grid;
    uint64_t per = work_each(work, units);
    for (int it = 0; it < 3; ++it) {
        unsigned long long small_work = 0, small_units = 0;
        for (int32_t q = 0; q < nq; ++q) {
            if (qd[q].kind != kind) continue;
            const uint32_t n = (uint32_t)qd[q].n_active, nt = qd[q].meta[2];
            const uint64_t least = (n + MEET_VB - 1) / MEET_VB;
            for (uint32_t t = (uint32_t)lane; t < nt; t += 64) {
                const uint64_t p = work_of(qd[q], n, tiles_of(qd[q])[t + 1] - tiles_of(qd[q])[t]);
                if (p < least * per) {
                    small_work += p;
                    small_units += least;
                }
            }
        }
        for (int dd = 32; dd > 0; dd >>= 1) {
            small_work += __shfl_xor(small_work, dd, 64);
            small_units += __shfl_xor(small_units, dd, 64);
        }
        if (small_units == 0ull || small_work >= work) break;
        while (units < small_units + grid / 2) units += grid;   // room for the others
        per = work_each(work - small_work, units - small_units);
    }
    return per;
}

// Lays the units of query d, of work `per` each where the graph is not tuned:
// writes the first unit of each tile and returns their number.  Called by all
// lanes of one wave.
__device__ uint32_t lay_units(const QueryDesc &d, uint64_t per, int lane) {
    const uint32_t nt = d.meta[2], n = (uint32_t)d.n_active;
    const uint32_t vb = d.vb > 0 ? (uint32_t)d.vb : (uint32_t)MEET_VB;
    uint32_t first = 0;
    for (uint32_t t0 = 0; t0 < nt; t0 += 64) {
        const uint32_t t = t0 + (uint32_t)lane;
        uint32_t c = 0;
        if (t < nt) {
            c = (n + vb - 1) / vb;
            if (d.vb <= 0 && n) {
                const uint64_t want = work_of(d, n, tiles_of(d)[t + 1] - tiles_of(d)[t]) / per;
                c = max(c, (uint32_t)min(want, (uint64_t)n));
            }
        }
        uint32_t inc = c;
        for (int dd = 1; dd < 64; dd <<= 1) {
            const uint32_t y = __shfl_up(inc, dd, 64);
            if (lane >= dd) inc += y;
        }
        if (t < nt) tunits_of(d)[t] = first + inc - c;
        first += __shfl(inc, 63, 64);
    }
    if (lane == 0) tunits_of(d)[nt] = first;
    return first;
}

// Tiles of one query per block, for sets of more than TILES_IN_UNITS queries.
constexpr int32_t TILES_IN_UNITS = 16;
__global__ __launch_bounds__(64) void k_tiles(const QueryDesc *__restrict__ qd) {
    const QueryDesc &d = qd[blockIdx.x];
    if (d.kind < N_KINDS) make_tiles(d, (int)threadIdx.x);
}

// Tiles (where there are few queries) and units of the queries (one block),
// then one list of nq + 1 offsets per kind (a query of another kind has
// no units in a list) and one cursor per kind.  grid: blocks of each kind's
// meet launch.
__global__ __launch_bounds__(1024) void k_unit_offsets(const QueryDesc *__restrict__ qd, int32_t nq,
                                                       uint32_t *units, uint3 grid,
                                                       unsigned long long *counters) {
    __shared__ unsigned long long s_work[N_KINDS], s_most[N_KINDS], s_per[N_KINDS];
    __shared__ uint32_t s_cost[N_KINDS];
    if (threadIdx.x < N_KINDS) {
        s_work[threadIdx.x] = s_most[threadIdx.x] = 0ull;
        s_cost[threadIdx.x] = 0u;
    }
    for (int32_t q = threadIdx.x >> 6; nq <= TILES_IN_UNITS && q < nq; q += (int32_t)(blockDim.x >> 6))
        if (qd[q].kind < N_KINDS) make_tiles(qd[q], (int)(threadIdx.x & 63));
    __syncthreads();
    for (int32_t q = threadIdx.x; q < nq; q += blockDim.x) {
        const int32_t kind = qd[q].kind;
        if (kind >= N_KINDS) continue;
        atomicAdd(&s_work[kind], (unsigned long long)work_of(qd[q], (uint32_t)qd[q].n_active, qd[q].meta[0]));
        atomicMax(&s_cost[kind], qd[q].cost);
        atomicMax(&s_most[kind], (unsigned long long)work_of(qd[q], MEET_VB, qd[q].meta[3]));
    }
    __syncthreads();
    if (threadIdx.x < 64 * N_KINDS) {
        // (many queries in one launch have units of all sizes: their common
        // work is not refined)
        const int kind = (int)(threadIdx.x >> 6);
        const uint64_t p = unit_work(qd, nq <= 16 ? nq : 0, kind, s_work[kind], s_cost[kind],
                                     s_most[kind], kind == 0 ? grid.x : kind == 1 ? grid.y : grid.z,
                                     (int)(threadIdx.x & 63));
        if ((threadIdx.x & 63) == 0) s_per[kind] = p;
    }
    __syncthreads();
    for (int32_t q = threadIdx.x >> 6; q < nq; q += (int32_t)(blockDim.x >> 6)) {
        const int32_t kind = qd[q].kind;
        uint32_t total = 0;
        if (kind < N_KINDS) total = lay_units(qd[q], s_per[kind], (int)(threadIdx.x & 63));
        if ((threadIdx.x & 63) < N_KINDS)
            units[(threadIdx.x & 63) * (nq + 1) + q] = (int32_t)(threadIdx.x & 63) == kind ? total : 0u;
    }
    __threadfence_block();
    __syncthreads();
    const int32_t per = (nq + blockDim.x - 1) / blockDim.x;
    const int32_t q0 = min(nq, (int32_t)threadIdx.x * per), q1 = min(nq, q0 + per);
    for (int list = 0; list < N_KINDS; ++list) {
        uint32_t *u = units + list * (nq + 1);
        uint32_t sum = 0;
        for (int32_t q = q0; q < q1; ++q) sum += u[q];
        uint32_t total;
        uint32_t run = block_excl_sum(sum, &total);
        for (int32_t q = q0; q < q1; ++q) {
            const uint32_t x = u[q];
            u[q] = run;
            run += x;
        }
        if (threadIdx.x == 0) {
            u[nq] = total;
            // (a meet launch's blocks take one unit each, then those from here)
            units[N_KINDS * (nq + 1) + list] = list == 0 ? grid.x : list == 1 ? grid.y : grid.z;
        }
    }
    if (threadIdx.x == 0) counters[STAMP_MEET] = wall_clock64();
}

// The same for a set of one query, its descriptor a kernel argument, by one
// wave.  Most queries of up to some 7,000 walks have one tile: their units
// follow from the two words that the source walks left.  (8 us before and 4
// now at R = 1,521: a chain of dependent reads.)
__global__ __launch_bounds__(64) void k_units_one(QueryDesc d, uint32_t *__restrict__ units,
                                                  uint3 grid, unsigned long long *counters) {
    const int lane = (int)threadIdx.x;
    const uint32_t blocks = d.kind == 0 ? grid.x : d.kind == 1 ? grid.y : grid.z;
    const uint32_t R1 = uni(d.meta[0]), total = uni(d.meta[1]), n = (uint32_t)d.n_active;
    uint32_t n_units = 0;
    if (R1 <= (uint32_t)d.tile_j && total <= (uint32_t)d.tile_nodes) {
        const uint32_t nt = R1 > 0u ? 1u : 0u;
        if (nt && n) {
            const uint32_t most = d.vb > 0 ? (uint32_t)d.vb : (uint32_t)MEET_VB;
            n_units = (n + most - 1) / most;
            if (d.vb <= 0) {
                // (rounds enough for full units: no tile is smaller than the others)
                const uint64_t work = work_of(d, n, R1);
                const uint64_t per = work_each(work, unit_rounds(work, d.cost, work_of(d, MEET_VB, R1), blocks) * blocks);
                n_units = max(n_units, (uint32_t)min(work / per, (uint64_t)n));
            }
        }
        if (lane == 0) {
            d.joff[R1] = total;
            tiles_of(d)[0] = 0u;
            tiles_of(d)[nt] = R1;
            d.meta[2] = nt;
            d.meta[3] = R1;
            tunits_of(d)[0] = 0u;
            tunits_of(d)[nt] = n_units;
        }
    } else {
        make_tiles(d, lane);
        n_units = lay_units(d, unit_work(&d, 1, d.kind, work_of(d, n, R1), d.cost, work_of(d, MEET_VB, d.meta[3]),
                                         blocks, lane), lane);
    }
    if (lane < N_KINDS) {
        units[lane * 2] = 0u;
        units[lane * 2 + 1] = lane == d.kind ? n_units : 0u;
        units[N_KINDS * 2 + lane] = lane == 0 ? grid.x : lane == 1 ? grid.y : grid.z;
    }
    if (lane == 0) counters[STAMP_MEET] = wall_clock64();
}

// ------------------------------------------------------------ meet kernel
//
// Persistent blocks take work units from a device cursor.  A unit is (query,
// tile of its source walks, run of its nodes with in-edges); the units
// of all queries of a launch form one list, so queries on graphs of any size
// share the launch and its tail.  A block stages its tile (walk ids, packed
// positions) in LDS once and keeps it while consecutive units share it, and
// stages the chunk's nodes (id, row) per unit.
//
// Inside a unit the pairs (v, k), v-major, are handed out from one block-wide
// cursor in chunks of 64 to 256 (items_for) to the waves, so all waves of a block
// work on the same few nodes v at a time: the rows a walk reads at its first two steps
// (v's own row and those of its in-neighbours) are then shared by the whole
// block and stay in the CU's L1.  Each lane runs NS independent pairs (slots)
// so that NS gathers per lane are in flight at once; a slot whose pair ended
// (stop, meet, or end of walk (s, j)) is refilled before the next step.
// A step: one Philox draw, a multiply-high neighbour pick, one gather of a row (4
// bytes where the graph's are packed, else 8 of E), one LDS compare.  Meets go to an LDS counter per node, flushed to the
// global counts once per unit.
//
// KIND selects the walks: K_PLAIN (sqrt(c)-walks), K_STITCHED (private head,
// then a tail read from the segment index) or K_STRAT (the stratified
// estimator's fixed-length walks: walk j of v has the class of slot pi_v(j),
// takes no stop draw, and a meet adds Lemma 5's weight of the two classes).
//
// Stitched walks run their private heads (the first 2^k steps, the plain
// walk's own draws) exactly as plain walks do.  A pair whose head made all its
// moves with both walks alive and apart is not continued on its slot: it goes
// to the wave's tail queue in LDS (unit-local node, tile entry, position) and
// the slot takes a new pair.  Whenever the queue holds a wave's worth of
// pairs, and once more when the unit's pairs are done, the wave follows 64
// queued tails at once through the index (the end node's pool slot drawn with
// (v, j, 0, 2), then the chain of segments), comparing with the tile in LDS.
// Heads thus keep the plain kernel's shape and rate, and the rarer tails do
// not hold slots of their own.

// Serving (STREAM): wave 0 of a block claims the next units from the ring:
// among published entries of the kernel's kind with unclaimed units, the
// oldest (smallest seq), all read from the entries' claim words alone; the
// claim (an acquire) counts down up to RING_RUN consecutive units (consecutive
// runs of nodes of one tile) from whatever the word holds when it arrives: a
// later request of the kind, or no units at all, in which case the word stays
// below CLAIM_ZERO and the block looks again.  (With a compare-and-swap, which
// fails whenever another block's came first, the grid's 256 blocks claimed one
// after another, 2 us each: one request, n = 5,000, R = 9,502, took 917 us, now
// 501; eight, every other at R = 1,521: 5,053 and 1,524.)
// The block fences only when it moves to a request it has not worked on
// (below), so its caches keep the graph's rows from unit to unit.
// *o_slot = RING_MAX when no entry has units left.
constexpr uint32_t RING_RUN = 4;
template <int KIND>
__device__ void ring_claim(const StreamRing &ring, int lane, uint32_t *o_slot, uint32_t *o_unit,
                           uint32_t *o_count, uint32_t *o_seq) {
    for (;;) {
        unsigned long long key = ~0ull, c = 0ull;
        if (lane < ring.entries) {
            c = __hip_atomic_load(&ring.ctl[lane].claim[KIND], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t)c > CLAIM_ZERO) key = ((c >> 32) << 32) | (uint32_t)lane;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(key, off, 64);
            key = o < key ? o : key;
        }
        if (key == ~0ull) {
            if (lane == 0) *o_slot = RING_MAX;
            return;
        }
        const int best = (int)(uint32_t)key;
        // runs shorten towards a request's end, so that its last units spread
        // over the blocks
        const uint32_t seen = (uint32_t)__shfl(c, best, 64) - CLAIM_ZERO;
        const uint32_t take = min(RING_RUN, max(1u, seen / (2u * gridDim.x)));
        bool won = false;
        if (lane == 0) {
            const unsigned long long old = __hip_atomic_fetch_add(
                &ring.ctl[best].claim[KIND], -(unsigned long long)take, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
            won = (uint32_t)old > CLAIM_ZERO;
            if (won) {
                const uint32_t left = (uint32_t)old - CLAIM_ZERO;
                const uint32_t nu = __hip_atomic_load(&ring.ctl[best].n_units, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
                *o_slot = (uint32_t)best;
                *o_unit = nu - left;
                *o_count = min(take, left);
                *o_seq = (uint32_t)(old >> 32);
            }
        }
        if (__shfl((int)won, 0, 64)) return;
    }
}

// Serving: a block reports `units` finished units of ring entry `slot`
// (request `tag`) and the work it did on them (the lanes' counters, which it
// then clears); the block whose report completes the entry writes the
// request's estimate and then its flag in host memory.  Block-wide.
__device__ void ring_report(const StreamRing &ring, const QueryDesc &d, uint32_t slot,
                            uint32_t tag, uint32_t units, Work &work, uint32_t *s_last) {
    // The entry's size is read before the report, while these units keep the entry
    // from being finished: behind it, another block may finish the entry and the
    // host publish it again, and the new request's size would be compared.  It is
    // read coherently: a plain load could return the size of an earlier request in
    // this entry from a cache and miss the last unit.
    uint32_t nu = 0;
    if (threadIdx.x == 0)
        nu = __hip_atomic_load(&ring.ctl[slot].n_units, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    add_work(ring.counters + (size_t)slot * 8, work);
    work = Work{};
    // every wave's counts are at the coherence point (atomics, waited for)
    // before one thread releases them with the block's report
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        const uint32_t old = atomicAdd(&ring.ctl[slot].done, units);
        *s_last = (old + units == nu) ? 1u : 0u;
    }
    __syncthreads();
    if (*s_last) {
        __threadfence();
        for (int64_t v = threadIdx.x; v < d.n; v += blockDim.x) estimate_one(d, v);
        __threadfence_system();
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(&ring.flags[slot], tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __syncthreads();
}

constexpr uint32_t DESC_WORDS = sizeof(QueryDesc) / 4;
static_assert(sizeof(QueryDesc) % 4 == 0, "whole words");
__device__ __forceinline__ const QueryDesc &desc_in(const uint32_t *words) {
    return *reinterpret_cast<const QueryDesc *>(words);
}
// A word of memory that another kernel may have written while this one runs.
__device__ __forceinline__ uint32_t coherent(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// At most 112 registers, which the attribute counts in pairs: 4 waves leave a
// SIMD 64 of its 512, and a wave of a served request's preparation fits beside.
template <int KIND, int NS, bool STREAM, int ROWS>
__global__ __launch_bounds__(meet_block_of(KIND)) __attribute__((amdgpu_num_vgpr(56)))
void k_meet(const QueryDesc *__restrict__ qd, int32_t nq,
            const uint32_t *__restrict__ ustart,
            uint32_t *__restrict__ cursor,
            unsigned long long *__restrict__ counters,
            StreamRing ring) {
    constexpr bool STITCHED = KIND == K_STITCHED;
    constexpr bool STRAT = KIND == K_STRAT;
    constexpr int TJ = tile_j_of(KIND), TN = ROWS == ROWS_HUBS ? HUB_TILE_NODES : tile_nodes_of(KIND);
    constexpr int HL = ROWS == ROWS_HUBS ? HUB_ROWS : hub_rows_of(KIND);
    __shared__ uint2 s_hub[ROWS == ROWS_E ? 1 : HL];   // rows of a packed graph's hubs
    __shared__ uint32_t s_nodes[TN];
    // the tile's entries: walk index j (below 2^24) | number of positions << 24,
    // and their LDS offset
    static_assert(MAX_R <= 1 << 24 && MAX_CAP < 256, "packed entries");
    __shared__ uint32_t s_jl[TJ];
    __shared__ uint16_t s_off[TJ];
    __shared__ uint32_t s_cnt[STRAT ? 1 : MEET_VB];
    __shared__ uint32_t s_vid[MEET_VB];
    __shared__ uint2 s_vrow[MEET_VB];
    __shared__ uint32_t s_unit, s_item, s_slot, s_seq, s_last, s_run, s_srcvl;
    // stratified: classes of the tile's source walks, class starts and the class
    // of each run of slots' first, the shuffle keys of the unit's nodes, weighted
    // sums
    __shared__ uint8_t s_cls[STRAT ? TJ : 1];
    __shared__ uint32_t s_ccum[STRAT ? MAX_CAP + 2 : 1];
    __shared__ uint4 s_fk[STRAT ? MEET_VB : 1];
    __shared__ uint8_t s_run_cls[STRAT ? CLASS_RUNS : 1];
    __shared__ unsigned long long s_w[STRAT ? MEET_VB : 1];
    // 64 prepared pairs per wave: (LDS offset | class of walk (s, j) << 16,
    // slot << 8 | class), LDS index of the last position
    __shared__ uint2 s_q[STRAT ? meet_block_of(KIND) : 1];
    __shared__ uint16_t s_qend[STRAT ? meet_block_of(KIND) : 1];
    // stitched: per-wave ring of pairs waiting for their tails, (vl << 16 | k, o)
    __shared__ uint2 s_tq[STITCHED ? (meet_block_of(KIND) / 64) * TAIL_Q : 1];

    // serving: the descriptor of the request worked on
    __shared__ __attribute__((aligned(16))) uint32_t s_desc[STREAM ? DESC_WORDS : 1];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t n_units = STREAM ? 0u : ustart[nq];
    uint32_t tq_head = 0, tq_tail = 0;   // stitched: the wave's tail ring (wave-uniform)
    // serving: the request whose finished units this block has not reported yet
    uint32_t acc_slot = 0, acc_tag = 0, acc_units = 0;
    uint32_t run_next = 0, run_left = 0;   // serving: claimed units not yet taken
    uint32_t next_unit = blockIdx.x;       // thread 0: taken while the unit before ran
    uint32_t cur_q = 0xffffffffu, cur_tile = 0xffffffffu;
    uint32_t K = 0;
    Work work;

    for (;;) {
        uint32_t unit = 0, tag_s = 0;
        if constexpr (STREAM) {
            if (run_left == 0u) {
                if (threadIdx.x < 64) ring_claim<KIND>(ring, lane, &s_slot, &s_unit, &s_run, &s_seq);
                __syncthreads();
                run_next = s_unit;
                run_left = s_slot < (uint32_t)RING_MAX ? s_run : 0u;
            }
            const uint32_t nslot = s_slot, nseq = s_seq;
            unit = run_next++;
            if (run_left) --run_left;
            // the block reports the units it finished of a request, and their
            // work, once: when it moves on to another request or runs out
            if (acc_units && (nslot >= (uint32_t)RING_MAX || nseq != acc_tag)) {
                ring_report(ring, desc_in(s_desc), acc_slot, acc_tag, acc_units, work, &s_last);
                acc_units = 0;
            }
            if (nslot >= (uint32_t)RING_MAX) break;
            tag_s = nseq;
            // a request this block has not worked on: see its descriptor and
            // buffers as its publication left them.  One wave's acquire
            // empties the CU's vector caches for all (its claim, an acquire
            // before a barrier, has done so too); a fence by each of a grid's
            // 4,096 waves, here and at the report, took half a millisecond a
            // request.  No fence empties the scalar cache, and ring entries and
            // pool memory are used again: the descriptor is read coherently
            // into LDS, and so are the other words at addresses that all lanes
            // share (coherent).
            if (tag_s != cur_q) {
                if (threadIdx.x < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                const uint32_t *from = reinterpret_cast<const uint32_t *>(&qd[nslot]);
                for (uint32_t i = threadIdx.x; i < DESC_WORDS; i += blockDim.x) s_desc[i] = coherent(from + i);
                __syncthreads();
            }
        } else {
            if (threadIdx.x == 0) s_unit = next_unit;
            __syncthreads();
            unit = s_unit;
            if (unit >= n_units) break;
            if (threadIdx.x == 0) next_unit = atomicAdd(cursor, 1u);
        }
        int32_t lo = 0;
        if constexpr (STREAM) {
            lo = (int32_t)s_slot;
        } else {
            // query of the unit: the last q with ustart[q] <= unit
            int32_t hi = nq;
            while (hi - lo > 1) {
                const int32_t mid = (lo + hi) >> 1;
                if (ustart[mid] <= unit) lo = mid; else hi = mid;
            }
        }
        const int32_t q = lo;
        const uint32_t local = STREAM ? unit : unit - ustart[q];
        const uint32_t tag = STREAM ? tag_s : (uint32_t)q;
        const QueryDesc &d = STREAM ? desc_in(s_desc) : qd[q];
        auto word = [](const uint32_t *p) { return STREAM ? coherent(p) : *p; };
        // tile of the unit: the last one that starts at or before it (a tile
        // of a query with units has at least one)
        uint32_t tile = 0, tile_hi = uni(word(d.meta + 2));
        while (tile_hi - tile > 1) {
            const uint32_t mid = (tile + tile_hi) >> 1;
            if (uni(word(tunits_of(d) + mid)) <= local) tile = mid; else tile_hi = mid;
        }
        const uint32_t unit0 = uni(word(tunits_of(d) + tile));
        const uint32_t chunks = uni(word(tunits_of(d) + tile + 1)) - unit0, chunk = local - unit0;
        const PhiloxKey key{uni(d.k0), uni(d.k1)};
        const uint32_t T = uni(d.T);
        const Gather rows = gather_of<HL>(d);
        const bool packed = ROWS == ROWS_PACKED || ROWS == ROWS_HUBS || (ROWS == ROWS_MIXED && rows.obits > 0u);
        const int32_t src = (int32_t)uni((uint32_t)d.s);
        const uint32_t NN = uni((uint32_t)d.R), sa = uni((uint32_t)d.sa), sb = uni((uint32_t)d.sb);
        const int32_t phi = (int32_t)uni((uint32_t)d.L);
        const uint32_t head_len = STITCHED ? uni((uint32_t)d.ix.seg_len) : 0u;
        const uint32_t run_log2 = STRAT ? class_run_log2(NN) : 0u;
        if (tag != cur_q || tile != cur_tile) {
            const uint32_t k0 = uni(word(tiles_of(d) + tile)), k1 = uni(word(tiles_of(d) + tile + 1));
            const uint32_t nb = uni(word(d.joff + k0)), ne = uni(word(d.joff + k1));
            K = k1 - k0;
            for (uint32_t i = threadIdx.x; i < K; i += blockDim.x) {
                const uint32_t jw = d.jj[k0 + i], at = d.joff[k0 + i];
                s_jl[i] = jw | ((d.joff[k0 + i + 1] - at) << 24);
                s_off[i] = (uint16_t)(at - nb);
                if (STRAT) s_cls[i] = d.scls[jw];
            }
            for (uint32_t i = threadIdx.x; i < ne - nb; i += blockDim.x) s_nodes[i] = d.swc[nb + i];
            if (STRAT) {
                for (uint32_t i = threadIdx.x; i < (uint32_t)phi + 2; i += blockDim.x)
                    s_ccum[i] = d.tab->ccum[i];
                for (uint32_t i = threadIdx.x; i <= (NN - 1u) >> run_log2; i += blockDim.x)
                    s_run_cls[i] = (uint8_t)slot_class(i << run_log2, d.tab->ccum, phi);
            }
            if (packed)
                for (uint32_t i = threadIdx.x; i < (uint32_t)d.n_hubs; i += blockDim.x) s_hub[i] = d.hubs[i];
            cur_q = tag;
            cur_tile = tile;
        }
        // the tile's units split the nodes evenly
        const uint32_t na = uni((uint32_t)d.n_active), nq0 = na / chunks, nrem = na - nq0 * chunks;
        const int32_t vbase = (int32_t)(chunk * nq0 + min(chunk, nrem));
        const uint32_t nv = nq0 + (chunk < nrem ? 1u : 0u);
        if (threadIdx.x == 0) {
            s_item = 0u;
            s_srcvl = NIL;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < MEET_VB; i += blockDim.x) {
            if (STRAT) s_w[i] = 0ull; else s_cnt[i] = 0u;
            if (i < nv) {
                const uint32_t id = (uint32_t)d.active[vbase + (int32_t)i];
                s_vid[i] = id;
                s_vrow[i] = d.nodes[id];
                if ((int32_t)id == src) s_srcvl = i;
                if (STRAT) s_fk[i] = philox4x32_10(id, 0u, 0u, DOM_SHUFFLE, key);
            }
        }
        __syncthreads();

        // Pairs of the unit: item i = vl * K + k for node vl < nv and walk k < K.
        // (K and nv are the same in all lanes; said so, the refill's bookkeeping
        // stays in scalar registers)
        // (stratified: an item is 64 walks of a node)
        const uint32_t Ku = uni(K), node_chunks = (Ku + 63u) >> 6;
        const uint32_t total = nv * (STRAT ? node_chunks : Ku);
        // wave-uniform chunk of items [ci, ce) and the (node, walk) of item ci
        uint32_t ci = 0, ce = 0, cvl = 0, ck = 0;
        uint32_t vo = 0, vd = 0, va = 0, vb = 0, vcc = 0;   // node cvl's row and draw constants
        const uint32_t srcvl = uni(s_srcvl), chunk_items =
            STRAT ? item_chunk(64u * total, uni((uint32_t)d.items)) >> 6 : item_chunk(total, uni((uint32_t)d.items));
        uint4 vfk = make_uint4(0u, 0u, 0u, 0u);             // stratified: and its shuffle key
        uint32_t at_vl = NIL;   // the node those are of
        auto enter_node = [&]() {
            at_vl = cvl;
            const uint2 row = s_vrow[cvl];
            vo = uni(row.x);
            vd = uni(row.y);
            const WalkDraws w = walk_draws_begin(uni(s_vid[cvl]), 0u, key, STRAT ? DOM_STRAT : DOM_WALK);
            va = uni(w.a);
            vb = uni(w.b);
            vcc = uni(w.cc);
            if (STRAT) {
                const uint4 k = s_fk[cvl];
                vfk = make_uint4(uni(k.x), uni(k.y), uni(k.z), uni(k.w));
            }
        };
        bool drained = false;
        uint32_t qh = 0, qn = 0;   // stratified: the wave's queue of prepared pairs [qh, qn)

        // The wave's slots, and which lanes' have a pair.  (Lane masks, and fills
        // that select: with a flag per lane and assignments under it the
        // compiler copied every slot's and the node's registers at each fill)
        Slot sl[NS];
        uint64_t busy[NS];
#pragma unroll
        for (int qq = 0; qq < NS; ++qq) {
            sl[qq] = Slot{};
            busy[qq] = 0ull;
        }

        // Stitched: follow the tails of the first `c` queued pairs (one per
        // lane) through the index; meets go to the unit's LDS counters.
        auto drain_tails = [&](uint32_t c) {
            bool met = false;
            if (lane < (int)c) {
                const uint2 r = s_tq[wave * TAIL_Q + ((tq_head + (uint32_t)lane) & (TAIL_Q - 1))];
                const uint32_t vl = r.x >> 16, k = r.x & 0xffffu;
                const uint32_t base = s_off[k], jl = s_jl[k], len = jl >> 24;
                const uint32_t seg_len = (uint32_t)d.ix.seg_len, width = (uint32_t)d.ix.width;
                const uint32_t y = d.ix.node_of[r.y];
                const int64_t pb = d.ix.pool_off[y];
                const int64_t pe = d.ix.pool_off[y + 1];
                const uint4 x = philox4x32_10(s_vid[vl], jl & 0xffffffu, 0u, DOM_ENTRY, key);
                const uint32_t sigma = (uint32_t)(pb + (int64_t)pick64(x.x, (uint64_t)(pe - pb)));
                const uint32_t *crow = d.ix.chain + (size_t)sigma * width;
                uint32_t t = seg_len;
                bool done = false;
                for (uint32_t mm = 0; mm < width && !done; ++mm) {
                    const uint32_t sg = crow[mm];
                    if (sg == NIL) break;
                    const uint32_t sln = d.ix.seg_lens[sg];
                    const uint32_t *srow = d.ix.seg + (size_t)sg * seg_len;
                    for (uint32_t u = 0; u < sln; ++u) {
                        ++t;
                        ++work.tail;
                        if (srow[u] == s_nodes[base + t - 1]) {
                            atomicAdd(&s_cnt[vl], 1u);
                            done = met = true;
                            break;
                        }
                        if (t == len) {
                            done = true;
                            break;
                        }
                    }
                    if (sln < seg_len) break;
                }
            }
            tq_head += c;
            work.meets += (uint32_t)__popcll(__ballot(met));
        };

        // The masked lanes' slot starts a pair of node cvl.
        auto start = [&](Slot &w, uint64_t mine, uint32_t at, uint32_t end, uint32_t j, uint32_t aux) {
            const bool me = in_mask(mine);
            w.at = me ? at : w.at;
            w.end = me ? end : w.end;
            w.o = me ? vo : w.o;
            w.d = me ? vd : w.d;
            w.rng.j = me ? j : w.rng.j;
            w.rng.a = me ? va : w.rng.a;
            w.rng.b = me ? vb : w.rng.b;
            w.rng.cc = me ? vcc : w.rng.cc;
            w.rng.mt = me ? 0ull : w.rng.mt;
            if (STRAT || STITCHED) w.aux = me ? aux : w.aux;
            work.pairs += (uint32_t)__popcll(mine);
        };

        for (;;) {
            // ---- refill idle slots from the block's cursor; a lane whose item
            // has nothing to walk (the source's own pair, or a stratified walk
            // of length 0) takes the next item
            if constexpr (STRAT) {
                // A pair's shuffle and class cost some eighty instructions: they
                // are done for 64 walks of one node at once by all lanes of the
                // wave, and the pairs with steps to walk wait in the wave's
                // queue in LDS until slots free up.  All that need not be done
                // by the third of the lanes that fill a slot is done there.
#pragma unroll
                for (int qq = 0; qq < NS; ++qq) {
                    uint64_t need = ~busy[qq];
                    while (need != 0ull) {
                        if (qh == qn) {
                            if (ci == ce) {
                                if (drained) break;
                                uint32_t x = 0;
                                if (lane == 0) x = atomicAdd(&s_item, chunk_items);
                                x = uni(x);
                                if (x >= total) {
                                    drained = true;
                                    break;
                                }
                                ci = x;
                                ce = min(x + chunk_items, total);
                                cvl = uni(x / node_chunks);
                                ck = x - cvl * node_chunks;
                            } else if (ck == node_chunks) {
                                ck = 0;
                                ++cvl;
                            }
                            if (cvl != at_vl) enter_node();
                            const uint32_t k = 64u * ck + (uint32_t)lane;
                            ++ci;
                            ++ck;
                            bool ok = k < Ku && cvl != srcvl;   // (the source's own pairs are not walked)
                            uint32_t r = 0, cv = 0, jl = 0;
                            if (ok) {
                                jl = s_jl[k];
                                r = shuffle_slot(jl & 0xffffffu, NN, sa, sb, vfk);
                                cv = s_run_cls[r >> run_log2];
                                while (s_ccum[cv + 1u] <= r) ++cv;   // (ends: ccum[phi + 1] = N > r)
                                ok = cv > 0u;
                            }
                            const uint64_t m = __ballot(ok);
                            if (ok) {
                                const uint32_t at = wave * 64 + lane_rank(m), off = s_off[k];
                                s_q[at] = make_uint2(off | ((uint32_t)s_cls[k] << 16), (r << 8) | cv);
                                s_qend[at] = (uint16_t)(off + min(jl >> 24, cv) - 1u);
                            }
                            qn = (uint32_t)__popcll(m);
                            qh = 0;
                            continue;
                        }
                        const uint32_t take = min(qn - qh, (uint32_t)__popcll(need));
                        const uint32_t rank = lane_rank(need);
                        const uint64_t mine = need & __ballot(rank < take);
                        const uint32_t from = wave * 64 + ((qh + rank) & 63u);
                        const uint2 e = s_q[from];
                        start(sl[qq], mine, e.x, s_qend[from] | (cvl << 16), e.y >> 8, e.y & 0xffu);
                        busy[qq] |= mine;
                        need &= ~mine;
                        qh += take;
                    }
                }
            } else {
#pragma unroll
                for (int qq = 0; qq < NS; ++qq) {
                    uint64_t need = ~busy[qq];
                    while (need != 0ull) {
                        if (ci == ce) {
                            if (drained) break;
                            uint32_t x = 0;
                            if (lane == 0) x = atomicAdd(&s_item, chunk_items);
                            x = uni(x);
                            if (x >= total) {
                                drained = true;
                                break;
                            }
                            ci = x;
                            ce = min(x + chunk_items, total);
                            cvl = uni(x / Ku);
                            ck = x - cvl * Ku;
                            if (cvl != at_vl) enter_node();
                        }
                        // the chunk's items of one node: its row and the draws'
                        // constants are uniform (per lane, with the constants
                        // formed anew for each pair and 64 items a chunk:
                        // n = 40,000, R = 9,502: 1,688 us against 1,501)
                        uint32_t take = min(ce - ci, Ku - ck);
                        if (cvl != srcvl) {   // (the source's own pairs are not walked)
                            take = min(take, (uint32_t)__popcll(need));
                            const uint32_t rank = lane_rank(need);
                            const uint64_t mine = need & __ballot(rank < take);
                            const uint32_t k = min(ck + rank, Ku - 1u);
                            const uint32_t jl = s_jl[k], off = s_off[k];
                            uint32_t end = off + (jl >> 24) + ((cvl << 16) - 1u);
                            if (STITCHED && jl >> 24 > head_len)
                                end = (off + head_len + ((cvl << 16) - 1u)) | HEAD_ONLY;
                            start(sl[qq], mine, off, end, jl & 0xffffffu, k);
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
            }
            uint64_t any = 0ull;
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) any |= busy[qq];
            // A refill round can hand out only pairs with nothing to walk: a
            // wave leaves only once the block's cursor is drained.
            if (any == 0ull) {
                if (drained && qh == qn) {
                    if constexpr (STITCHED) {
                        while (tq_tail != tq_head) drain_tails(min(64u, tq_tail - tq_head));
                    }
                    break;
                }
                continue;
            }

            // ---- head steps: draws, then all gathers, then the compares
            uint64_t go[NS];
            uint32_t from[NS];
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) {
                const uint2 x = walk_draw_next(sl[qq].rng, key);
                work.draws += (uint32_t)__popcll(busy[qq]);
                go[qq] = STRAT ? busy[qq] : busy[qq] & __ballot(x.x < T);
                from[qq] = sl[qq].o + pick32(x.y, sl[qq].d);
            }
            uint2 e[NS];
            if (packed) {
#pragma unroll
                for (int qq = 0; qq < NS; ++qq)
                    if (in_mask(go[qq])) e[qq].x = rows.E4[from[qq]];
            } else {
#pragma unroll
                for (int qq = 0; qq < NS; ++qq)
                    if (in_mask(go[qq])) e[qq] = load_edge(rows.E, from[qq]);
            }
            uint64_t tails[NS];
#pragma unroll
            for (int qq = 0; qq < NS; ++qq) {
                work.moves += (uint32_t)__popcll(go[qq]);
                Slot &w = sl[qq];
                bool met = false, more = false, tail = false;
                if (in_mask(go[qq])) {
                    const uint2 to = packed ? unpack_row(e[qq].x, rows.obits, s_hub) : e[qq];
                    w.o = to.x;
                    w.d = to.y;
                    met = w.o == s_nodes[w.at & 0xffffu];
                    const bool last = (uint16_t)w.at == (uint16_t)w.end;
                    more = !met && !last && w.d != 0u;
                    // stitched: a head that made all its moves queues its tail
                    if (STITCHED) tail = !met && last && w.d != 0u && w.end >= HEAD_ONLY;
                    ++w.at;
                }
                busy[qq] = __ballot(more);
                tails[qq] = STITCHED ? __ballot(tail) : 0ull;
                if (const uint64_t m = __ballot(met)) {
                    work.meets += (uint32_t)__popcll(m);
                    const uint32_t vl = (w.end >> 16) & 0xffu;
                    if (met) {
                        if (STRAT) atomicAdd(&s_w[vl], strat_weight(d.tab->a, w.at >> 16, w.aux));
                        else atomicAdd(&s_cnt[vl], 1u);
                    }
                }
            }
            if constexpr (STITCHED) {
                // queue the pairs whose heads ended open, then follow queued
                // tails while a wave's worth is waiting
#pragma unroll
                for (int qq = 0; qq < NS; ++qq) {
                    if (tails[qq] == 0ull) continue;
                    if (in_mask(tails[qq]))
                        s_tq[wave * TAIL_Q + ((tq_tail + lane_rank(tails[qq])) & (TAIL_Q - 1))] =
                            make_uint2((sl[qq].end & 0xff0000u) | sl[qq].aux, sl[qq].o);
                    tq_tail += (uint32_t)__popcll(tails[qq]);
                    if (tq_tail - tq_head >= 64u) drain_tails(64u);
                }
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < nv; i += blockDim.x) {
            if (STRAT) {
                const unsigned long long c = s_w[i];
                if (c) atomicAdd(&d.wsum[s_vid[i]], c);
            } else {
                const uint32_t c = s_cnt[i];
                if (c) atomicAdd(&d.cnt[s_vid[i]], c);
            }
        }
        if constexpr (STREAM) {
            ++acc_units;
            acc_slot = (uint32_t)q;
            acc_tag = tag;
        }
    }
    if constexpr (STREAM) return;

    add_work(ctr_set(counters), work);
}

// ------------------------------------------------------ walk materialisation

struct WalkArgs {
    const uint2 *nodes;
    const uint2 *E;
    IndexView ix;
    const int32_t *vs;
    const uint32_t *js;
    int64_t count;
    int32_t *paths;   // [count][L+1]
    int32_t *lens;
    PhiloxKey key;
    uint32_t T;
    int32_t L;
};

template <bool STITCHED>
__global__ __launch_bounds__(256) void k_walks(WalkArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.count) return;
    int32_t *row = a.paths + (size_t)i * (a.L + 1);
    const uint32_t v = (uint32_t)a.vs[i], j = a.js[i];
    row[0] = (int32_t)v;
    uint2 cur = a.nodes[v];
    const int32_t head = STITCHED ? min(a.ix.seg_len, a.L) : a.L;
    int32_t len = 0;
    for (int32_t t = 1; t <= head; ++t) {
        const uint4 x = philox4x32_10(v, j, (uint32_t)t, DOM_WALK, a.key);
        if (x.x >= a.T || cur.y == 0) break;
        cur = a.E[cur.x + pick32(x.y, cur.y)];
        row[t] = (int32_t)a.ix.node_of[cur.x];
        len = t;
    }
    if (STITCHED && len == a.ix.seg_len && len < a.L) {
        const uint32_t sigma = entry_slot(a.ix, a.key, v, j, (uint32_t)row[len]);
        for (int32_t mm = 0; mm < a.ix.width && len < a.L; ++mm) {
            const uint32_t sg = a.ix.chain[(size_t)sigma * a.ix.width + mm];
            if (sg == NIL) break;
            const int32_t sl = a.ix.seg_lens[sg];
            for (int32_t u = 0; u < sl && len < a.L; ++u) {
                ++len;
                row[len] = (int32_t)a.ix.node_of[a.ix.seg[(size_t)sg * a.ix.seg_len + u]];
            }
            if (sl < a.ix.seg_len) break;
        }
    }
    for (int32_t t = len + 1; t <= a.L; ++t) row[t] = -1;
    a.lens[i] = len;
}

// Stratified: walk j of v after the shuffle (the fixed-length walk of slot
// pi_v(j)); paths hold node ids, row[0] = v.
struct StratWalkArgs {
    const uint2 *nodes;
    const uint2 *E;
    const uint32_t *node_of;
    const StratTab *tab;
    const int32_t *vs;
    const uint32_t *js;
    int64_t count;
    int32_t *paths;   // [count][phi+1] or NULL
    int32_t *lens;    // or NULL
    uint32_t *slots;  // or NULL
    int32_t *classes; // or NULL
    PhiloxKey key;
    uint32_t N, sa, sb;
    int32_t phi;
};

__global__ __launch_bounds__(256) void k_walks_strat(StratWalkArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.count) return;
    const uint32_t v = (uint32_t)a.vs[i], j = a.js[i];
    const uint4 fk = philox4x32_10(v, 0u, 0u, DOM_SHUFFLE, a.key);
    const uint32_t r = shuffle_slot(j, a.N, a.sa, a.sb, fk);
    const uint32_t cls = slot_class(r, a.tab->ccum, a.phi);
    if (a.slots) a.slots[i] = r;
    if (a.classes) a.classes[i] = (int32_t)cls;
    if (!a.paths) return;
    int32_t *row = a.paths + (size_t)i * (a.phi + 1);
    row[0] = (int32_t)v;
    uint2 cur = a.nodes[v];
    int32_t len = 0;
    for (int32_t t = 1; t <= (int32_t)cls; ++t) {
        if (cur.y == 0) break;
        const uint4 x = philox4x32_10(v, r, (uint32_t)t, DOM_STRAT, a.key);
        cur = a.E[cur.x + pick32(x.y, cur.y)];
        row[t] = (int32_t)a.node_of[cur.x];
        len = t;
    }
    for (int32_t t = len + 1; t <= a.phi; ++t) row[t] = -1;
    a.lens[i] = len;
}

#ifndef SRK_MEET_SLOTS
#define SRK_MEET_SLOTS 2
#endif
#ifndef SRK_MEET_SLOTS_STITCHED
#define SRK_MEET_SLOTS_STITCHED 2
#endif

#ifndef SRK_MEET_SLOTS_STRAT
#define SRK_MEET_SLOTS_STRAT 2
#endif
// Stratified queries that gather packed rows wait for their gathers: a third
// pair per lane (with 2 and 3: n = 40,000, N = 16,508: 2,499 and 2,429 us; n =
// 2^18: 18.1 and 17.4 ms).  Those that gather E, from the L2 or with many hubs,
// have the more idle slots at a unit's end instead (n = 2,003: 55 and 62 us; n =
// 2^20: 17.3 and 17.5 ms).
#ifndef SRK_MEET_SLOTS_STRAT_PACKED
#define SRK_MEET_SLOTS_STRAT_PACKED 3
#endif

// Resident blocks of a meet-kernel instance on the whole device (computed
// once per process; a function-local static is initialised thread-safely).
template <int KIND, int NS, bool STREAM>
int meet_grid_blocks() {
    static const int blocks = [] {
        int dev = 0, cus = 0, per = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per, k_meet<KIND, NS, STREAM, ROWS_E>, meet_block_of(KIND), 0);
        if (cus <= 0) cus = 256;
        if (per <= 0) per = 1;
        return cus * per;
    }();
    return blocks;
}

template <int KIND, int NS>
void launch_meet(const QuerySet &qs, hipStream_t st) {
    const int blocks = meet_grid_blocks<KIND, NS, false>();
    const uint32_t *ustart = qs.units + (size_t)KIND * (qs.nq + 1);
    uint32_t *cursor = qs.units + (size_t)N_KINDS * (qs.nq + 1) + KIND;
    constexpr int NP = KIND == K_STRAT ? SRK_MEET_SLOTS_STRAT_PACKED : NS;
    const Rows rows = rows_of(qs.rows[KIND]);
    auto kernel = rows == ROWS_E        ? k_meet<KIND, NS, false, ROWS_E>
                  : rows == ROWS_PACKED ? k_meet<KIND, NP, false, ROWS_PACKED>
                                        : k_meet<KIND, NS, false, ROWS_MIXED>;
    if constexpr (KIND != K_STRAT)
        if (rows == ROWS_HUBS) kernel = k_meet<KIND, NS, false, ROWS_HUBS>;
    kernel<<<blocks, meet_block_of(KIND), 0, st>>>(qs.desc, qs.nq, ustart, cursor, qs.counters, StreamRing{});
}

template <int KIND, int NS>
void launch_meet_ring(Rows rows, const StreamRing &ring, hipStream_t st) {
    // (a server's requests are on one graph)
    auto kernel = rows == ROWS_E ? k_meet<KIND, NS, true, ROWS_E> : k_meet<KIND, NS, true, ROWS_PACKED>;
    if constexpr (KIND != K_STRAT)
        if (rows == ROWS_HUBS) kernel = k_meet<KIND, NS, true, ROWS_HUBS>;
    kernel<<<meet_grid_blocks<KIND, NS, true>(), meet_block_of(KIND), 0, st>>>(
        ring.desc, ring.entries, nullptr, nullptr, ring.counters, ring);
}

// Publication of a ring entry, the last kernel of its request's preparation:
// its units (for meet launches of `grid` blocks) and their count, then its
// claim word.  A request with nothing to walk is finished here:
// estimate, then its flag.  One block.
__global__ __launch_bounds__(256) void k_publish(StreamRing ring, int32_t slot, uint32_t seq,
                                                 uint32_t grid) {
    const QueryDesc &d = ring.desc[slot];
    __shared__ uint32_t s_nu;
    if (threadIdx.x < 64) {
        make_tiles(d, (int)threadIdx.x);
        const uint32_t nu = lay_units(
            d, unit_work(&d, 1, d.kind, work_of(d, (uint32_t)d.n_active, d.meta[0]), d.cost,
                         work_of(d, MEET_VB, d.meta[3]), grid, (int)threadIdx.x), (int)threadIdx.x);
        if (threadIdx.x == 0) s_nu = nu;
    }
    __syncthreads();
    const uint32_t nu = s_nu;
    if (nu > 0u) {
        if (threadIdx.x == 0) {
            RingCtl &c = ring.ctl[slot];
            c.n_units = nu;
            c.done = 0u;
            __threadfence();
            __hip_atomic_store(&c.claim[d.kind], ((unsigned long long)seq << 32) | (CLAIM_ZERO + nu),
                               __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    for (int64_t v = threadIdx.x; v < d.n; v += blockDim.x) estimate_one(d, v);
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&ring.flags[slot], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

IndexView index_view(const Graph *g) {
    IndexView v{};
    v.node_of = g->node_of;
    if (g->index) {
        v.pool_off = g->index->pool_off;
        v.seg = g->index->seg;
        v.seg_lens = g->index->seg_lens;
        v.chain = g->index->chain;
        v.seg_len = g->index->seg_len;
        v.width = g->index->width;
    }
    return v;
}

// Tiles of R walks of cap L, at most, for any kind and any tile a query may be
// given (the smallest shape).
int32_t max_tiles_for(int32_t R, int32_t L) {
    const int64_t TJ =
        std::min({MIN_TILE_J, tile_j_of(K_PLAIN), tile_j_of(K_STITCHED), tile_j_of(K_STRAT)});
    const int64_t NW =
        std::min({tile_nodes_of(K_PLAIN), tile_nodes_of(K_STITCHED), tile_nodes_of(K_STRAT)}) - L;
    return (int32_t)(2 + R / TJ + ((int64_t)R * L) / NW);
}

// Nodes per work unit that unit counts are bounded with (the tuner's choice, if
// any; else a nominal one by graph size).
int32_t default_unit_nodes(const Graph *g) {
    if (g->tuned_vb > 0) return g->tuned_vb;
    if (g->n_active >= (1 << 19)) return 256;
    if (g->n_active >= (1 << 17)) return 128;
    if (g->n_active >= (1 << 15)) return 64;
    return 32;
}

int64_t units_bound_of(const Graph *g, int32_t R, int32_t L) {
    const int64_t vb = default_unit_nodes(g);
    return (int64_t)max_tiles_for(R, L) * ((g->n_active + vb - 1) / vb);
}

// Items that a wave takes at once, at most.  The fewer, the closer together the
// block's pairs are and the more rows they share in the L1; the more, the fewer
// refills are cut short by a chunk's end.  Meet kernel with 64 / 128 / 256 / 512
// items: n = 20,000 (2.5 MB of E), R = 38,005: 2,978 / 2,701 / 2,575 / 2,549 us;
// n = 40,000 (5 MB), R = 9,502: 1,636 / 1,512 / 1,456 / 1,445; n = 150,001
// (19 MB): 6,144 / 6,013 / 6,063 / 6,238; n = 2^18 (33 MB): 11.60 / 11.70 /
// 11.92 / 12.40 ms; n = 2^20 (133 MB): 51.96 / 52.26 / 53.13 / 55.06.
static int32_t items_for(const Graph *g) {
    const int64_t e = 8 * g->m_slots;
    return e <= (int64_t)8 << 20 ? 256 : e <= (int64_t)24 << 20 ? 128 : 64;
}

uint32_t pair_cost(double c, int32_t L, int32_t head) {
    const double tail = pow(c, (double)head) * std::min(c / (1.0 - c), (double)std::max(L - head, 0));
    return (uint32_t)std::max(1.0, floor(tail / 1.5 + 0.5));
}

void describe_query(const Graph *g, const simrank_query *q, const simrank_params &p, int mode,
                    QueryDesc *d) {
    *d = QueryDesc{};
    d->nodes = g->nodes;
    d->E = g->E;
    d->E4 = g->E4;
    d->hubs = g->hubs;
    d->obits = g->obits;
    d->n_hubs = g->n_hubs;
    d->active = g->active;
    d->ix = index_view(g);
    const PhiloxKey key = make_key(q->seed);
    d->k0 = key.k0;
    d->k1 = key.k1;
    d->T = p.T;
    d->n = g->n;
    d->n_active = g->n_active;
    d->s = q->s;
    d->R = p.R;
    d->L = p.L;
    d->vb = g->tuned_vb;
    d->items = items_for(g);
    d->kind = mode == SIMRANK_MODE_STITCHED ? K_STITCHED
              : mode == SIMRANK_MODE_STRATIFIED ? K_STRAT : K_PLAIN;
    d->cost = d->kind == K_STITCHED ? pair_cost(q->c, p.L, d->ix.seg_len) : 1u;
    const int32_t tj = g->tuned_tile_j[d->kind];
    d->tile_nodes = tile_nodes_for(*g, d->kind, p.R, p.L);
    d->tile_j = tj > 0 ? std::min<int32_t>(tj, tile_j_of(d->kind)) : tile_j_of(d->kind);
}

int launch_query_set(const QuerySet &qs, hipStream_t st, const QueryDesc *one) {
    if (qs.nq <= 0) return SIMRANK_OK;
    const unsigned nq = (unsigned)qs.nq;
    const unsigned gx_n = std::min<unsigned>(grid_for(std::max(qs.max_n, 1), 256), 1024u);
    if (one)
        k_init_one<<<gx_n, 256, 0, st>>>(const_cast<QueryDesc *>(qs.desc), *one, qs.counters, CTR_SUMS);
    else
        k_init<<<dim3(gx_n, nq), 256, 0, st>>>(qs.desc, qs.counters, CTR_SUMS);
    if (one)
        k_source_walks_one<<<grid_for(qs.max_R, 256), 256, 0, st>>>(*one, qs.counters);
    else
        k_source_walks<true><<<dim3(grid_for(qs.max_R, 256), nq), 256, 0, st>>>(qs.desc, qs.counters, true);
    if (qs.nq > TILES_IN_UNITS) k_tiles<<<nq, 64, 0, st>>>(qs.desc);
    const uint3 grid = make_uint3((uint32_t)meet_grid_blocks<K_PLAIN, SRK_MEET_SLOTS, false>(),
                                  (uint32_t)meet_grid_blocks<K_STITCHED, SRK_MEET_SLOTS_STITCHED, false>(),
                                  (uint32_t)meet_grid_blocks<K_STRAT, SRK_MEET_SLOTS_STRAT, false>());
    if (one)
        k_units_one<<<1, 64, 0, st>>>(*one, qs.units, grid, qs.counters);
    else
        k_unit_offsets<<<1, 1024, 0, st>>>(qs.desc, qs.nq, qs.units, grid, qs.counters);
    if (qs.units_bound[K_PLAIN] > 0) launch_meet<K_PLAIN, SRK_MEET_SLOTS>(qs, st);
    if (qs.units_bound[K_STITCHED] > 0) launch_meet<K_STITCHED, SRK_MEET_SLOTS_STITCHED>(qs, st);
    if (qs.units_bound[K_STRAT] > 0) launch_meet<K_STRAT, SRK_MEET_SLOTS_STRAT>(qs, st);
    if (qs.groups && qs.groups->ng > 0) {
        const int rc = launch_groups(*qs.groups, qs.counters, st);
        if (rc) return rc;
    }
    k_estimate<<<dim3(gx_n, nq), 256, 0, st>>>(qs.desc, qs.counters);
    SRK_HIP(hipGetLastError());
    return SIMRANK_OK;
}

// Blocks of a kind's persistent serving kernel.
static uint32_t ring_grid(int kind) {
    return (uint32_t)(kind == K_PLAIN      ? meet_grid_blocks<K_PLAIN, SRK_MEET_SLOTS, true>()
                      : kind == K_STITCHED ? meet_grid_blocks<K_STITCHED, SRK_MEET_SLOTS_STITCHED, true>()
                                           : meet_grid_blocks<K_STRAT, SRK_MEET_SLOTS_STRAT, true>());
}

// Preparation of a served request in ring entry `slot`.  Every kernel is
// small (one wave per SIMD at most) so that it fits beside a running
// persistent meet kernel on the same CUs.
int enqueue_ring_request(const QueryDesc &d, const StreamRing &ring, int32_t slot, uint32_t seq,
                         hipStream_t st) {
    QueryDesc *qd = ring.desc + slot;
    unsigned long long *ctr = ring.counters + (size_t)slot * 8;
    const unsigned gx_n = std::min<unsigned>(grid_for(std::max(d.n, 1), 256), 1024u);
    k_init_one<<<gx_n, 256, 0, st>>>(qd, d, ctr, 8);
    k_source_walks<false><<<dim3(grid_for(d.R, 256), 1), 256, 0, st>>>(qd, ctr, false);
    k_publish<<<1, 256, 0, st>>>(ring, slot, seq, ring_grid(d.kind));
    SRK_HIP(hipGetLastError());
    return SIMRANK_OK;
}

int launch_ring_meet(Rows rows, int kind, const StreamRing &ring, hipStream_t st) {
    if (kind == K_PLAIN) launch_meet_ring<K_PLAIN, SRK_MEET_SLOTS>(rows, ring, st);
    else if (kind == K_STITCHED) launch_meet_ring<K_STITCHED, SRK_MEET_SLOTS_STITCHED>(rows, ring, st);
    else launch_meet_ring<K_STRAT, SRK_MEET_SLOTS_STRAT>(rows, ring, st);
    SRK_HIP(hipGetLastError());
    return SIMRANK_OK;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Device bytes of one query's buffers (stratified queries: class table, walk
// classes, weighted sums and the second estimate instead of counts).
size_t request_bytes(const simrank_params &p, int mode, int32_t n) {
    const size_t RL = (size_t)p.R * (size_t)p.L;
    size_t b = align256(4 * RL) + align256((size_t)p.R) + align256(4 * (size_t)p.R) +
               align256(4 * ((size_t)p.R + 1)) + align256(4 * RL) +
               align256(4 * ((size_t)max_tiles_for(p.R, p.L) + 1)) + align256(32) +
               align256(8 * (size_t)n);
    if (mode == SIMRANK_MODE_STRATIFIED)
        b += align256(sizeof(StratTab)) + align256((size_t)p.R) + 2 * align256(8 * (size_t)n);
    else
        b += align256(4 * (size_t)n);
    return b;
}

void carve_request(const simrank_params &p, int mode, int32_t n, char *base, QueryDesc *d) {
    char *cur = base;
    auto take = [&](size_t b) {
        char *r = cur;
        cur += align256(b);
        return r;
    };
    const size_t RL = (size_t)p.R * (size_t)p.L;
    d->sw = (uint32_t *)take(4 * RL);
    d->slen = (uint8_t *)take((size_t)p.R);
    d->jj = (uint32_t *)take(4 * (size_t)p.R);
    d->joff = (uint32_t *)take(4 * ((size_t)p.R + 1));
    d->swc = (uint32_t *)take(4 * RL);
    d->tiles = (uint32_t *)take(4 * ((size_t)max_tiles_for(p.R, p.L) + 1));
    d->meta = (uint32_t *)take(32);
    d->out = (double *)take(8 * (size_t)n);
    if (mode == SIMRANK_MODE_STRATIFIED) {
        d->tab = (const StratTab *)take(sizeof(StratTab));
        d->scls = (uint8_t *)take((size_t)p.R);
        d->wsum = (unsigned long long *)take(8 * (size_t)n);
        d->out_n = (double *)take(8 * (size_t)n);
        d->cnt = nullptr;
    } else {
        d->cnt = (uint32_t *)take(4 * (size_t)n);
    }
}

// ---------------------------------------------------------------- host side

int query_params(const simrank_query *q, int32_t n, simrank_params *out, int *mode) {
    if (!q) return fail(SIMRANK_EINVAL, "query is NULL");
    if (!(q->c > 0.0 && q->c < 1.0)) return fail(SIMRANK_EINVAL, "c must lie in (0, 1)");
    if (!(q->delta > 0.0 && q->delta < 1.0)) return fail(SIMRANK_EINVAL, "delta must lie in (0, 1)");
    if (!(q->eps > 0.0 && q->eps < 1.0)) return fail(SIMRANK_EINVAL, "eps must lie in (0, 1)");
    if (q->mode != SIMRANK_MODE_PLAIN && q->mode != SIMRANK_MODE_STITCHED &&
        q->mode != SIMRANK_MODE_STRATIFIED)
        return fail(SIMRANK_EINVAL, "unknown mode");
    if (q->R_override < 0) return fail(SIMRANK_EINVAL, "R_override must be >= 0");
    if (q->mode == SIMRANK_MODE_STRATIFIED) {
        StratParams sp;
        const int rc = strat_params(q, n, &sp, nullptr);
        if (rc) return rc;
        out->R = sp.N;
        out->L = sp.phi;
        out->T = 0;
        out->reserved = 0;
        if (mode) *mode = q->mode;
        return SIMRANK_OK;
    }
    const int32_t L = q->walk_cap == 0 ? 64 : q->walk_cap;
    if (L < 1 || L > MAX_CAP) return fail(SIMRANK_EINVAL, "walk_cap must lie in [1, 255]");
    if (q->mode == SIMRANK_MODE_STITCHED && L > MAX_STITCH_CAP)
        return fail(SIMRANK_EINVAL, "stitched walks are capped at 64 steps");
    int64_t R;
    if (q->R_override > 0) {
        R = q->R_override;
    } else {
        // Hoeffding: 2 exp(-2 R lambda^2) <= delta (per node) or delta / n
        // (union over n nodes); lambda = eps minus the truncation bias c^(L+1).
        const double lam = q->eps - pow(q->c, (double)(L + 1));
        if (!(lam > 0.0)) return fail(SIMRANK_EINVAL, "eps must exceed c^(L+1)");
        const double num = q->union_bound ? log(2.0 * (double)n / q->delta) : log(2.0 / q->delta);
        const double r = ceil(num / (2.0 * lam * lam));
        if (!(r <= (double)MAX_R)) return fail(SIMRANK_EINVAL, "R exceeds 2^24");
        R = (int64_t)r;
    }
    if (R > MAX_R) return fail(SIMRANK_EINVAL, "R exceeds 2^24");
    out->R = (int32_t)R;
    out->L = L;
    out->T = continue_threshold(q->c);
    out->reserved = 0;
    if (mode) *mode = q->mode;
    return SIMRANK_OK;
}

// Algorithm 1 caps walks at phi = log_{1/sqrt c} n steps (floor) and draws
// N_l = ceil(Z_l) walks of length l from every node, Z_l = z sqrt(c)^l
// (1 - sqrt(c)), with Algorithm 2's z = ln(2n) / (2 (eps - 3/n)^2).  A query
// may fix phi (walk_cap > 0, the longer cap of the error-threshold extension)
// and z (R_override > 0).  sqrt(c)^l is formed by repeated multiplication.
int strat_params(const simrank_query *q, int32_t n, StratParams *sp, StratTab *tab) {
    if (n < 1) return fail(SIMRANK_EINVAL, "n must be >= 1");
    double z;
    if (q->R_override > 0) {
        z = (double)q->R_override;
    } else {
        const double gap = q->eps - 3.0 / (double)n;
        if (!(gap > 0.0)) return fail(SIMRANK_EINVAL, "stratified estimator needs eps > 3/n");
        z = log(2.0 * (double)n) / (2.0 * gap * gap);
    }
    const double r = sqrt(q->c);
    int32_t phi;
    if (q->walk_cap > 0) {
        phi = q->walk_cap;
    } else {
        const double f = floor(log((double)n) / log(1.0 / r));
        if (!(f >= 0.0 && f <= (double)MAX_CAP)) return fail(SIMRANK_EINVAL, "phi beyond 255");
        phi = (int32_t)f;
    }
    if (phi < 1 || phi > MAX_CAP) return fail(SIMRANK_EINVAL, "walk cap phi must lie in [1, 255]");
    double g = 1.0;
    double N = 0.0;
    for (int32_t l = 0; l <= phi; ++l) {
        const double Zl = (z * g) * (1.0 - r);
        const double Zh = ceil(Zl);
        if (tab) {
            tab->ccum[l] = (uint32_t)N;
            tab->a[l] = Zl / Zh;
        }
        N += Zh;
        if (!(N <= (double)MAX_STRAT_N))
            return fail(SIMRANK_EINVAL, "stratified estimator needs fewer than 2^24 walks per node");
        g = g * r;
    }
    if (tab) tab->ccum[phi + 1] = (uint32_t)N;
    sp->z = z;
    sp->N = (int32_t)N;
    sp->phi = phi;
    int32_t bits = 0;
    while ((1 << bits) < sp->N) ++bits;
    sp->sb = (bits + 1) / 2;
    sp->sa = (sp->N + (1 << sp->sb) - 1) >> sp->sb;
    return SIMRANK_OK;
}

int workspace_init(const Graph *g, int32_t max_R, int32_t max_L, Workspace *ws,
                   unsigned long long *counters) {
    if (max_R < 1 || max_R > MAX_R) return fail(SIMRANK_EINVAL, "max_R must lie in [1, 2^24]");
    if (max_L < 1 || max_L > MAX_CAP) return fail(SIMRANK_EINVAL, "max_L must lie in [1, 255]");
    ws->g = g;
    ws->max_R = max_R;
    ws->max_L = max_L;
    ws->max_tiles = max_tiles_for(max_R, max_L);
    const size_t RL = (size_t)max_R * (size_t)max_L;
    int rc;
    if ((rc = device_alloc((void **)&ws->sw, 4 * RL, nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->slen, align256((size_t)max_R), nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->jj, 4 * (size_t)max_R, nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->joff, 4 * ((size_t)max_R + 1), nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->swc, 4 * RL, nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->tiles, 4 * ((size_t)ws->max_tiles + 1), nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->meta, 4 * 8, nullptr))) return rc;
    ws->counters = counters;
    ws->own_counters = !counters;
    if (!counters && (rc = device_alloc((void **)&ws->counters, 8 * CTR_WORDS, nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->desc, sizeof(QueryDesc), nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->units, 4 * units_words(1), nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->scls, (size_t)max_R, nullptr))) return rc;
    if ((rc = device_alloc((void **)&ws->tab, sizeof(StratTab), nullptr))) return rc;
    SRK_HIP(hipEventCreateWithFlags(&ws->ev1, hipEventDisableTiming));
    return SIMRANK_OK;
}

void workspace_release(Workspace *ws) {
    if (!ws) return;
    device_free(ws->sw);
    device_free(ws->slen);
    device_free(ws->jj);
    device_free(ws->joff);
    device_free(ws->swc);
    device_free(ws->tiles);
    device_free(ws->meta);
    if (ws->own_counters) device_free(ws->counters);
    device_free(ws->desc);
    device_free(ws->units);
    device_free(ws->scls);
    device_free(ws->tab);
    if (ws->ev1) (void)hipEventDestroy(ws->ev1);
    *ws = Workspace{};
}

// One query on a workspace: its descriptor, then the whole launch sequence.
static int launch_single(const Graph *g, Workspace *ws, const QueryDesc &d, hipStream_t st) {
    // the meet kernel counts work units (tile x node chunk) in 32 bits
    const int64_t units_bound = units_bound_of(g, d.R, d.L);
    if (units_bound >= (int64_t)0xffffffffu - (1 << 20))
        return fail(SIMRANK_EINVAL, "R * L * n too large for one launch");
    QuerySet qs;
    qs.desc = ws->desc;
    qs.nq = 1;
    qs.max_R = d.R;
    qs.max_n = g->n;
    qs.units_bound[d.kind] = units_bound;
    qs.rows[d.kind] = rows_wish(*g, d);
    qs.units = ws->units;
    qs.counters = ws->counters;
    int rc = launch_query_set(qs, st, &d);
    if (rc) return rc;
    SRK_HIP(hipEventRecord(ws->ev1, st));
    ws->last_stream = st;
    ws->last_params.R = d.R;
    ws->last_params.L = d.L;
    ws->last_params.T = d.T;
    ws->last_params.reserved = 0;
    ws->last_n = g->n;
    ws->pending = true;
    return SIMRANK_OK;
}

static void attach_buffers(Workspace *ws, QueryDesc *d) {
    d->sw = ws->sw;
    d->slen = ws->slen;
    d->jj = ws->jj;
    d->joff = ws->joff;
    d->swc = ws->swc;
    d->tiles = ws->tiles;
    d->meta = ws->meta;
    d->scls = ws->scls;
    d->tab = ws->tab;
}

int enqueue_query(const Graph *g, const simrank_query *q, const simrank_params &p, int mode,
                  Workspace *ws, double *out_dev, uint32_t *counts_dev, hipStream_t st) {
    if (q->s < 0 || q->s >= g->n) return fail(SIMRANK_EINVAL, "source out of range");
    if (mode == SIMRANK_MODE_STRATIFIED)
        return fail(SIMRANK_EINVAL, "stratified queries return weighted sums: use the stratified calls");
    if (p.R > ws->max_R || p.L > ws->max_L)
        return fail(SIMRANK_EINVAL, "query needs R or L beyond the workspace's size");
    if (!counts_dev) return fail(SIMRANK_EINVAL, "counts buffer is NULL");
    const bool stitched = mode == SIMRANK_MODE_STITCHED;
    if (stitched && !g->index) return fail(SIMRANK_ESTATE, "stitched query without an index");
    if (stitched && g->index->T != p.T)
        return fail(SIMRANK_EINVAL, "stitched query's c differs from the index's c");
    QueryDesc d;
    describe_query(g, q, p, mode, &d);
    attach_buffers(ws, &d);
    d.cnt = counts_dev;
    d.out = out_dev;
    return launch_single(g, ws, d, st);
}

int enqueue_stratified(const Graph *g, const simrank_query *q, Workspace *ws, double *out_dev,
                       double *out_n_dev, unsigned long long *wsum_dev, hipStream_t st) {
    if (q->s < 0 || q->s >= g->n) return fail(SIMRANK_EINVAL, "source out of range");
    if (q->mode != SIMRANK_MODE_STRATIFIED) return fail(SIMRANK_EINVAL, "not a stratified query");
    if (!wsum_dev) return fail(SIMRANK_EINVAL, "weighted-sum buffer is NULL");
    StratParams sp;
    StratTab tab{};
    int rc = strat_params(q, g->n, &sp, &tab);
    if (rc) return rc;
    if (sp.N > ws->max_R || sp.phi > ws->max_L)
        return fail(SIMRANK_EINVAL, "query needs N or phi beyond the workspace's size");
    simrank_params p{sp.N, sp.phi, 0u, 0};
    QueryDesc d;
    describe_query(g, q, p, SIMRANK_MODE_STRATIFIED, &d);
    attach_buffers(ws, &d);
    d.wsum = wsum_dev;
    d.out = out_dev;
    d.out_n = out_n_dev;
    d.z = sp.z;
    d.sa = sp.sa;
    d.sb = sp.sb;
    static_assert(sizeof(StratTab) <= 3584, "the class table travels as a kernel argument");
    k_put_tab<<<1, 256, 0, st>>>(ws->tab, tab);
    return launch_single(g, ws, d, st);
}

// Device times of a query, in ms, from its counters and stamps.
static int times_of(const Workspace *ws, const unsigned long long *c, double *ms, double *meet_ms) {
    int khz = 0;   // of the device's constant clock
    SRK_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, ws->g->device));
    const double tick = 1.0 / (double)std::max(khz, 1);
    if (ms) *ms = (double)(c[STAMP_END] - c[STAMP_BEGIN]) * tick;
    if (meet_ms) *meet_ms = (double)(c[STAMP_MET] - c[STAMP_MEET]) * tick;
    return SIMRANK_OK;
}

int query_times(const Workspace *ws, double *ms, double *meet_ms) {
    SRK_HIP(hipEventSynchronize(ws->ev1));
    unsigned long long c[CTR_WORDS];
    SRK_HIP(hipMemcpy(c, ws->counters, sizeof(c), hipMemcpyDeviceToHost));
    return times_of(ws, c, ms, meet_ms);
}

// The last query's statistics from its counters and stamps.
static int fill_stats(Workspace *ws, const unsigned long long *c, simrank_stats *st) {
    ws->pending = false;
    if (!st) return SIMRANK_OK;
    double ms = 0.0, mms = 0.0;
    const int rc = times_of(ws, c, &ms, &mms);
    if (rc) return rc;
    *st = simrank_stats{};
    st->pairs = (uint64_t)(ws->last_n - 1) * (uint64_t)ws->last_params.R;
    st->pairs_walked = c[C_PAIRS];
    st->moves = c[C_MOVES];
    st->draws = c[C_DRAWS];
    st->meets = c[C_MEETS];
    st->tail_steps = c[C_TAIL];
    st->source_moves = c[C_SRC_MOVES];
    st->ms = ms;
    st->meet_ms = mms;
    st->R = ws->last_params.R;
    st->L = ws->last_params.L;
    st->T = ws->last_params.T;
    return SIMRANK_OK;
}

static int read_stats(Workspace *ws, simrank_stats *st) {
    SRK_HIP(hipEventSynchronize(ws->ev1));
    unsigned long long c[CTR_WORDS];   // (one copy: each costs 10 us and more)
    SRK_HIP(hipMemcpy(c, ws->counters, sizeof(c), hipMemcpyDeviceToHost));
    return fill_stats(ws, c, st);
}

// A synchronous call's results: its counters and up to three arrays of n, which
// lie behind one another in device memory.  A copy to the host costs 11 to 13
// us however small, so results of up to 1 MB come in one and are dealt out here;
// larger ones each go where they belong, which costs less than dealing them out.
// A call of hardly any work with one copy and with one for each: n = 500: 61 and
// 93 us; n = 40,000 (484 KB): 95 and 115; n = 80,000 (965 KB): 141 and 154; n =
// 100,000 (1.2 MB): 184 and 165; n = 170,000: 256 and 231.
struct Results {
    char *dev = nullptr;
    size_t at[4] = {0, 0, 0, 0}, bytes[4] = {0, 0, 0, 0}, total = 0;
    void *host[4] = {nullptr, nullptr, nullptr, nullptr};
    unsigned long long ctr[CTR_WORDS];

    ~Results() { device_free(dev); }
    void add(int i, void *to, size_t b) {
        host[i] = to;
        bytes[i] = b;
        at[i] = total;
        total += (b + 255) & ~(size_t)255;
    }
    int alloc() { return device_alloc((void **)&dev, total, nullptr); }
    template <typename T>
    T *at_dev(int i) { return bytes[i] ? reinterpret_cast<T *>(dev + at[i]) : nullptr; }
    // Copies behind the work on st and waits.
    int fetch(hipStream_t st) {
        constexpr size_t SMALL = 1 << 20;
        const std::unique_ptr<char[]> tmp(total <= SMALL ? new (std::nothrow) char[total] : nullptr);
        if (tmp) {
            SRK_HIP(hipMemcpyAsync(tmp.get(), dev, total, hipMemcpyDeviceToHost, st));
            SRK_HIP(hipStreamSynchronize(st));
            for (int i = 0; i < 4; ++i)
                if (host[i]) std::memcpy(host[i], tmp.get() + at[i], bytes[i]);
            return SIMRANK_OK;
        }
        // (synchronous copies: asynchronous ones of each array took 100 us more for
        // 320 and 160 KB)
        SRK_HIP(hipStreamSynchronize(st));
        for (int i = 0; i < 4; ++i)
            if (host[i]) SRK_HIP(hipMemcpy(host[i], dev + at[i], bytes[i], hipMemcpyDeviceToHost));
        return SIMRANK_OK;
    }
};

}  // namespace srk

using namespace srk;


extern "C" int simrank_derive_params(const simrank_query *q, int32_t n, simrank_params *out) {
    clear_error();
    if (!out) return fail(SIMRANK_EINVAL, "out is NULL");
    if (n < 1) return fail(SIMRANK_EINVAL, "n must be >= 1");
    simrank_params p;
    const int rc = query_params(q, n, &p, nullptr);
    if (rc == SIMRANK_OK) *out = p;
    return rc;
}

extern "C" int simrank_workspace_create(const simrank_graph *g, int32_t max_R, int32_t max_L,
                                        simrank_workspace **ws_out) {
    clear_error();
    if (!g || !ws_out) return fail(SIMRANK_EINVAL, "NULL argument");
    *ws_out = nullptr;
    SRK_HIP(hipSetDevice(g->device));
    simrank_workspace *ws = new simrank_workspace();
    const int rc = workspace_init(g, max_R, max_L, ws);
    if (rc != SIMRANK_OK) {
        workspace_release(ws);
        delete ws;
        return rc;
    }
    *ws_out = ws;
    return SIMRANK_OK;
}

extern "C" int simrank_workspace_free(simrank_workspace *ws) {
    clear_error();
    if (!ws) return SIMRANK_OK;
    if (ws->pending && ws->last_stream) (void)hipStreamSynchronize(ws->last_stream);
    workspace_release(ws);
    delete ws;
    return SIMRANK_OK;
}

extern "C" int simrank_single_source_async(const simrank_graph *g, const simrank_query *q,
                                           simrank_workspace *ws, double *out_dev,
                                           uint32_t *counts_dev, void *stream) {
    clear_error();
    if (!g || !q || !ws) return fail(SIMRANK_EINVAL, "NULL argument");
    if (ws->g != g) return fail(SIMRANK_EINVAL, "workspace belongs to another graph");
    simrank_params p;
    int mode;
    int rc = query_params(q, g->n, &p, &mode);
    if (rc) return rc;
    SRK_HIP(hipSetDevice(g->device));
    return enqueue_query(g, q, p, mode, ws, out_dev, counts_dev, (hipStream_t)stream);
}

extern "C" int simrank_workspace_stats(simrank_workspace *ws, simrank_stats *st) {
    clear_error();
    if (!ws) return fail(SIMRANK_EINVAL, "workspace is NULL");
    if (!ws->pending) return fail(SIMRANK_ESTATE, "no call recorded on this workspace");
    return read_stats(ws, st);
}

extern "C" int simrank_single_source_ex(const simrank_graph *g, const simrank_query *q,
                                        double *out_host, uint32_t *counts_host,
                                        simrank_stats *st_opt) {
    clear_error();
    if (!g || !q) return fail(SIMRANK_EINVAL, "NULL argument");
    simrank_params p;
    int mode;
    int rc = query_params(q, g->n, &p, &mode);
    if (rc) return rc;
    if (q->s < 0 || q->s >= g->n) return fail(SIMRANK_EINVAL, "source out of range");
    if (mode == SIMRANK_MODE_STRATIFIED)
        return fail(SIMRANK_EINVAL, "stratified queries: use simrank_single_source_stratified");
    if (mode == SIMRANK_MODE_STITCHED && !g->index)
        return fail(SIMRANK_ESTATE, "stitched query without an index");
    if (mode == SIMRANK_MODE_STITCHED && g->index->T != p.T)
        return fail(SIMRANK_EINVAL, "stitched query's c differs from the index's c");
    SRK_HIP(hipSetDevice(g->device));
    Workspace ws;
    Results res;
    const size_t n = (size_t)g->n;
    res.add(0, res.ctr, sizeof(res.ctr));
    res.add(1, out_host, out_host ? 8 * n : 0);
    res.add(2, counts_host, 4 * n);   // needed on the device in any case
    rc = res.alloc();
    if (!rc) rc = workspace_init(g, p.R, p.L, &ws, res.at_dev<unsigned long long>(0));
    if (!rc) rc = enqueue_query(g, q, p, mode, &ws, res.at_dev<double>(1), res.at_dev<uint32_t>(2), g->stream);
    if (!rc) rc = res.fetch(g->stream);
    if (!rc) rc = fill_stats(&ws, res.ctr, st_opt);
    workspace_release(&ws);
    return rc;
}

extern "C" int simrank_single_source(const simrank_graph *g, int32_t s, double c, double eps,
                                     double delta, double *out) {
    if (!out) {
        clear_error();
        return fail(SIMRANK_EINVAL, "out is NULL");
    }
    simrank_query q{};
    q.s = s;
    q.c = c;
    q.eps = eps;
    q.delta = delta;
    q.seed = 0;
    q.walk_cap = 64;
    q.mode = SIMRANK_MODE_PLAIN;
    return simrank_single_source_ex(g, &q, out, nullptr, nullptr);
}

extern "C" int simrank_walks(const simrank_graph *g, const simrank_query *q, const int32_t *v,
                             const uint32_t *j, int64_t count, int32_t *paths, int32_t *lens) {
    clear_error();
    if (!g || !q || (count > 0 && (!v || !j || !paths || !lens)))
        return fail(SIMRANK_EINVAL, "NULL argument");
    if (count < 0) return fail(SIMRANK_EINVAL, "count < 0");
    simrank_params p;
    int mode;
    int rc = query_params(q, g->n, &p, &mode);
    if (rc) return rc;
    if (mode == SIMRANK_MODE_STRATIFIED)
        return fail(SIMRANK_EINVAL, "stratified walks: use simrank_stratified_walks");
    for (int64_t i = 0; i < count; ++i)
        if (v[i] < 0 || v[i] >= g->n) return fail(SIMRANK_EINVAL, "walk start out of range");
    const bool stitched = mode == SIMRANK_MODE_STITCHED;
    if (stitched && !g->index) return fail(SIMRANK_ESTATE, "stitched walks without an index");
    if (stitched && g->index->T != p.T)
        return fail(SIMRANK_EINVAL, "stitched walks' c differs from the index's c");
    if (count == 0) return SIMRANK_OK;
    SRK_HIP(hipSetDevice(g->device));
    int32_t *dv = nullptr, *dpaths = nullptr, *dlens = nullptr;
    uint32_t *dj = nullptr;
    const size_t rowb = 4 * (size_t)(p.L + 1);
    rc = device_alloc((void **)&dv, 4 * (size_t)count, nullptr);
    if (!rc) rc = device_alloc((void **)&dj, 4 * (size_t)count, nullptr);
    if (!rc) rc = device_alloc((void **)&dpaths, rowb * (size_t)count, nullptr);
    if (!rc) rc = device_alloc((void **)&dlens, 4 * (size_t)count, nullptr);
    hipStream_t st = g->stream;
    if (!rc) {
        hipError_t e = hipMemcpyAsync(dv, v, 4 * (size_t)count, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipMemcpyAsync(dj, j, 4 * (size_t)count, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) {
            WalkArgs wa{g->nodes, g->E, index_view(g), dv, dj, count, dpaths, dlens,
                        make_key(q->seed), p.T, p.L};
            if (stitched)
                k_walks<true><<<grid_for(count, 256), 256, 0, st>>>(wa);
            else
                k_walks<false><<<grid_for(count, 256), 256, 0, st>>>(wa);
            e = hipGetLastError();
        }
        if (e == hipSuccess)
            e = hipMemcpyAsync(paths, dpaths, rowb * (size_t)count, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(lens, dlens, 4 * (size_t)count, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) rc = fail(SIMRANK_EDEVICE, hipGetErrorString(e));
    }
    device_free(dv);
    device_free(dj);
    device_free(dpaths);
    device_free(dlens);
    return rc;
}

// ------------------------------------------------ length-stratified estimator

extern "C" int simrank_derive_stratified(const simrank_query *q, int32_t n,
                                         simrank_strat_params *out) {
    clear_error();
    if (!q || !out) return fail(SIMRANK_EINVAL, "NULL argument");
    simrank_query qq = *q;
    qq.mode = SIMRANK_MODE_STRATIFIED;
    simrank_params p;
    int rc = query_params(&qq, n, &p, nullptr);
    if (rc) return rc;
    StratParams sp;
    rc = strat_params(&qq, n, &sp, nullptr);
    if (rc) return rc;
    *out = simrank_strat_params{sp.z, sp.N, sp.phi, sp.sb, sp.sa};
    return SIMRANK_OK;
}

extern "C" int simrank_stratified_async(const simrank_graph *g, const simrank_query *q,
                                        simrank_workspace *ws, double *out_dev, double *out_n_dev,
                                        uint64_t *wsum_dev, void *stream) {
    clear_error();
    if (!g || !q || !ws) return fail(SIMRANK_EINVAL, "NULL argument");
    if (ws->g != g) return fail(SIMRANK_EINVAL, "workspace belongs to another graph");
    simrank_params p;
    int rc = query_params(q, g->n, &p, nullptr);
    if (rc) return rc;
    SRK_HIP(hipSetDevice(g->device));
    return enqueue_stratified(g, q, ws, out_dev, out_n_dev, (unsigned long long *)wsum_dev,
                              (hipStream_t)stream);
}

extern "C" int simrank_single_source_stratified(const simrank_graph *g, const simrank_query *q,
                                                double *out, double *out_n, uint64_t *wsum,
                                                simrank_stats *st_opt) {
    clear_error();
    if (!g || !q) return fail(SIMRANK_EINVAL, "NULL argument");
    if (q->mode != SIMRANK_MODE_STRATIFIED) return fail(SIMRANK_EINVAL, "not a stratified query");
    simrank_params p;
    int rc = query_params(q, g->n, &p, nullptr);
    if (rc) return rc;
    if (q->s < 0 || q->s >= g->n) return fail(SIMRANK_EINVAL, "source out of range");
    SRK_HIP(hipSetDevice(g->device));
    Workspace ws;
    Results res;
    const size_t n = (size_t)g->n;
    res.add(0, res.ctr, sizeof(res.ctr));
    res.add(1, out, out ? 8 * n : 0);
    res.add(2, out_n, out_n ? 8 * n : 0);
    res.add(3, wsum, 8 * n);   // needed on the device in any case
    rc = res.alloc();
    if (!rc) rc = workspace_init(g, p.R, p.L, &ws, res.at_dev<unsigned long long>(0));
    if (!rc)
        rc = enqueue_stratified(g, q, &ws, res.at_dev<double>(1), res.at_dev<double>(2),
                                res.at_dev<unsigned long long>(3), g->stream);
    if (!rc) rc = res.fetch(g->stream);
    if (!rc) rc = fill_stats(&ws, res.ctr, st_opt);
    workspace_release(&ws);
    return rc;
}

extern "C" int simrank_stratified_walks(const simrank_graph *g, const simrank_query *q,
                                        const int32_t *v, const uint32_t *j, int64_t count,
                                        uint32_t *slot, int32_t *cls, int32_t *paths,
                                        int32_t *lens) {
    clear_error();
    if (!g || !q || (count > 0 && (!v || !j || !slot || !cls)))
        return fail(SIMRANK_EINVAL, "NULL argument");
    if ((paths == nullptr) != (lens == nullptr))
        return fail(SIMRANK_EINVAL, "paths and lens go together");
    if (count < 0) return fail(SIMRANK_EINVAL, "count < 0");
    if (q->mode != SIMRANK_MODE_STRATIFIED) return fail(SIMRANK_EINVAL, "not a stratified query");
    simrank_params p;
    int rc = query_params(q, g->n, &p, nullptr);
    if (rc) return rc;
    StratTab tab;
    StratParams sp;
    rc = strat_params(q, g->n, &sp, &tab);
    if (rc) return rc;
    for (int64_t i = 0; i < count; ++i) {
        if (v[i] < 0 || v[i] >= g->n) return fail(SIMRANK_EINVAL, "walk start out of range");
        if (j[i] >= (uint32_t)sp.N) return fail(SIMRANK_EINVAL, "walk index beyond N");
    }
    if (count == 0) return SIMRANK_OK;
    SRK_HIP(hipSetDevice(g->device));
    int32_t *dv = nullptr, *dpaths = nullptr, *dlens = nullptr, *dcls = nullptr;
    uint32_t *dj = nullptr, *dslot = nullptr;
    StratTab *dtab = nullptr;
    const size_t rowb = 4 * (size_t)(sp.phi + 1), c4 = 4 * (size_t)count;
    rc = device_alloc((void **)&dv, c4, nullptr);
    if (!rc) rc = device_alloc((void **)&dj, c4, nullptr);
    if (!rc) rc = device_alloc((void **)&dslot, c4, nullptr);
    if (!rc) rc = device_alloc((void **)&dcls, c4, nullptr);
    if (!rc) rc = device_alloc((void **)&dtab, sizeof(StratTab), nullptr);
    if (!rc && paths) rc = device_alloc((void **)&dpaths, rowb * (size_t)count, nullptr);
    if (!rc && paths) rc = device_alloc((void **)&dlens, c4, nullptr);
    hipStream_t st = g->stream;
    if (!rc) {
        hipError_t e = hipMemcpy(dv, v, c4, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(dj, j, c4, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(dtab, &tab, sizeof(StratTab), hipMemcpyHostToDevice);
        if (e == hipSuccess) {
            StratWalkArgs wa{g->nodes, g->E, g->node_of, dtab, dv, dj, count, dpaths, dlens,
                             dslot, dcls, make_key(q->seed), (uint32_t)sp.N, (uint32_t)sp.sa,
                             (uint32_t)sp.sb, sp.phi};
            k_walks_strat<<<grid_for(count, 256), 256, 0, st>>>(wa);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess) e = hipMemcpy(slot, dslot, c4, hipMemcpyDeviceToHost);
        if (e == hipSuccess) e = hipMemcpy(cls, dcls, c4, hipMemcpyDeviceToHost);
        if (e == hipSuccess && paths) e = hipMemcpy(paths, dpaths, rowb * (size_t)count, hipMemcpyDeviceToHost);
        if (e == hipSuccess && paths) e = hipMemcpy(lens, dlens, c4, hipMemcpyDeviceToHost);
        if (e != hipSuccess) rc = fail(SIMRANK_EDEVICE, hipGetErrorString(e));
    }
    device_free(dv);
    device_free(dj);
    device_free(dslot);
    device_free(dcls);
    device_free(dtab);
    device_free(dpaths);
    device_free(dlens);
    return rc;
}
