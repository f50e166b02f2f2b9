// Algorithm 2's tuple form of meet detection, for up to 32 sources at once.
//
// Section 3.2 and Algorithm 2: every walk is decomposed into one tuple per
// step after its start, (j, i, node, start); the tuples are sorted on
// (j, i, node) with the sources' tuples first among equal keys; each other
// tuple is linked to the closest source tuple before it (PREDECESSOR), and an
// equal (j, i, node) is a meet of walk j of that source and walk j of the
// tuple's start node, counted once per pair.
//
// The first two parts of the key need no sort: a block takes the walks j of a
// run of start nodes and of the sources, steps them together, and so
// makes the tuples of one (j, i) at a time, of several once fewer walks are
// left (up to 8 steps that fit the buffer).  It sorts those in LDS by
// (i, node), sources first (an LSD radix sort, stable), finds each tuple's predecessor
// among the sources' tuples as a running maximum, and links; the pairs that
// have met are kept in one bit per source and start node.  Tuples never leave
// the CU.  Where no source's walk j has a step i, no tuple of (j, i) can be
// linked: the walks are then only followed to their ends and counted.
//
// What bounds it: at n = 2^14 the LDS passes and their barriers, at n = 2^20 the
// L2 misses of the steps.  The form before it wrote the tuples of a chunk of
// nodes to memory (12 bytes each), sorted them on the whole key in five or six
// passes over memory of 32 bytes a tuple, and took a scan and a link pass more.
// Before and now, 8 sources: n = 2^14, R = 1,521 (5.6e7 tuples) 9.6 and 2.5 ms;
// n = 50,000 23.8 and 7.3 ms; n = 2^20, R = 9,502 (1.73e10 tuples) 2.54 and
// 0.73 s, of which sorting each step by itself took another 0.16 s.
//
// Walks are the same as the fused kernel's (same keys, same steps), but are
// followed to their full length rather than to the first meet, so the counts
// must agree with the fused path: an independent cross-check of it, and the
// paper's own form for several sources that share their walks' key.
#include <algorithm>
#include <string>
#include <vector>

#include "common.hpp"
#include "device_common.hpp"
#include "philox.hpp"

namespace srk {
namespace {

constexpr int MAX_TUPLE_SOURCES = 32;
constexpr int TU_STEP_BITS = 3;                   // steps sorted at once: up to 8
constexpr uint32_t TU_SRC = 0x8000u;              // payload flag of a source's tuple

// Blocks of the tuple kernel: TU_LARGE two to a CU; TU_SMALL of one wave, for few
// start nodes.  A unit of those leaves most of a large block's threads idle, and its
// barriers and passes take as long; of small blocks a CU holds some 25.  Calls
// with large and with small blocks, 8 sources: R = 9,502, n = 10: 1,190 and 294 us, n =
// 250: 1,626 and 341; R = 2,000, c = 0.95, 255 steps, n = 10: 3,019 and 619, n = 250:
// 2,960 and 839.  Where the large blocks take all units at once, a small one's
// four nodes per thread cost more than its barriers save from two per thread on:
// R = 100, n = 120: 138 and 137 us, n = 250: 165 and 177.
template <int BLOCK_, int RPT_>
struct TupleBlock {
    static constexpr int BLOCK = BLOCK_;
    static constexpr int WAVES = BLOCK / 64;
    static constexpr int RPT = RPT_;                          // start nodes per thread
    static constexpr int ROWS = RPT * BLOCK;                  // start nodes per unit
    static constexpr int CAP = ROWS + MAX_TUPLE_SOURCES;      // tuples sorted at once
    static constexpr int ROUNDS = (CAP + BLOCK - 1) / BLOCK;
    static constexpr int DIGIT_BITS = BLOCK == 512 ? 9 : 6;   // of a sort pass, at most
    static_assert(1 << DIGIT_BITS == BLOCK, "one digit per thread");
    static_assert(ROWS < (int)TU_SRC, "payloads in 16 bits");
};
using TU_LARGE = TupleBlock<512, 7>;
using TU_SMALL = TupleBlock<64, 4>;

struct TupleArgs {
    const uint2 *nodes;
    const uint2 *E;
    const int32_t *active;       // start nodes
    int32_t na;                  // their number
    int32_t N, L;                // walks per node; cap (stratified: phi)
    PhiloxKey key;
    uint32_t T;                  // plain: continue threshold
    const StratTab *tab;         // stratified: class table
    uint32_t sa, sb;             // stratified: shuffle grid
    const int32_t *src;          // [k] source nodes
    int32_t k;
    int32_t nb, step_bits;       // bits of an o-value; of a step's number within a sort
    int32_t n;
    int64_t units;               // runs of start nodes x N
    unsigned long long *out;     // [k][n]
    unsigned long long *counters;
};

// Lanes of the wave with the same digit (db bits) as this one.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, int db, bool valid) {
    uint64_t m = __ballot(valid);
    for (int b = 0; b < db; ++b) {
        const uint64_t bb = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bb : ~bb;
    }
    return m;
}

// One walker: the walk j of a start node or source.
struct Walker {
    uint32_t id, o, d;   // start node; current node
    uint32_t r;          // the draws' walk index (stratified: the slot pi(j))
    uint32_t end;        // steps it may take: L, or its class
    bool alive;
};

template <bool STRAT>
__device__ __forceinline__ Walker walker_begin(const TupleArgs &a, uint32_t id, uint32_t j,
                                               const uint32_t *ccum) {
    const uint2 row = a.nodes[id];
    Walker w{id, row.x, row.y, j, (uint32_t)a.L, true};
    if (STRAT) {
        const uint4 fk = philox4x32_10(id, 0u, 0u, DOM_SHUFFLE, a.key);
        w.r = shuffle_slot(j, (uint32_t)a.N, a.sa, a.sb, fk);
        w.end = slot_class(w.r, ccum, a.L);
        w.alive = w.end > 0u;
    }
    return w;
}

// Whether the walker takes step i (its draw in *x1 then picks the neighbour).
template <bool STRAT>
__device__ __forceinline__ bool walker_goes(const TupleArgs &a, const Walker &w, uint32_t i,
                                            uint32_t *x1) {
    if (!w.alive || i > w.end || w.d == 0u) return false;
    const WalkDraws c = walk_draws_begin(w.id, w.r, a.key, STRAT ? DOM_STRAT : DOM_WALK);
    const uint2 x = walk_draw_at(c.j, c.a, c.b, c.cc, (uint64_t)philox_m1() * i, a.key);
    *x1 = x.y;
    return STRAT || x.x < a.T;
}

template <bool STRAT, typename B>
__global__ __launch_bounds__(B::BLOCK) void k_tuples(TupleArgs a) {
    constexpr int TU_BLOCK = B::BLOCK, TU_WAVES = B::WAVES, TU_RPT = B::RPT, TU_ROWS = B::ROWS,
                  TU_CAP = B::CAP, TU_ROUNDS = B::ROUNDS, TU_DIGITS = 1 << B::DIGIT_BITS;
    __shared__ uint32_t s_key[2][TU_CAP];            // tuples: step within the sort, o-value
    __shared__ uint16_t s_val[2][TU_CAP];            // and start node (run-local) or source
    __shared__ uint32_t s_met[TU_ROWS];              // sources that walk (v, j) has met
    __shared__ uint32_t s_cnt[TU_WAVES][TU_DIGITS];  // per wave and digit: count, then start
    __shared__ uint32_t s_ccum[STRAT ? MAX_CAP + 2 : 1];
    __shared__ uint32_t s_srccls[MAX_TUPLE_SOURCES];
    // tuples in the buffer, sources' tuples of the step: of even and odd steps,
    // so that a wave a step ahead leaves the others' alone
    __shared__ uint32_t s_n[2], s_nsrc[2], s_last[TU_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const GlobalPtr<uint64_t> E = (GlobalPtr<uint64_t>)a.E;
    unsigned long long moves = 0, sorted = 0;
    uint32_t meets = 0;   // (in 64 bits 1% slower: n = 50,000 7.00 ms, not 6.93)
    if (STRAT) {
        for (int i = threadIdx.x; i < a.L + 2; i += TU_BLOCK) s_ccum[i] = a.tab->ccum[i];
        __syncthreads();
    }

    for (int64_t unit = blockIdx.x; unit < a.units; unit += gridDim.x) {
        const int64_t run = unit / a.N;
        const uint32_t j = (uint32_t)(unit - run * a.N);
        const int32_t row0 = (int32_t)(run * TU_ROWS);
        Walker w[TU_RPT], sw{};
#pragma unroll
        for (int q = 0; q < TU_RPT; ++q) {
            const int32_t row = q * TU_BLOCK + (int32_t)threadIdx.x;
            s_met[row] = 0u;
            w[q].alive = false;
            if (row0 + row < a.na) w[q] = walker_begin<STRAT>(a, (uint32_t)a.active[row0 + row], j, s_ccum);
        }
        if ((int)threadIdx.x < a.k) {
            sw = walker_begin<STRAT>(a, (uint32_t)a.src[threadIdx.x], j, s_ccum);
            if (STRAT) s_srccls[threadIdx.x] = sw.end;
        }

        uint32_t steps = 0, held = 0;   // steps and tuples in the buffer (uniform)
        for (uint32_t i = 1; i <= (uint32_t)a.L; ++i) {
            // ---- the step: all draws, then all gathers
            bool go[TU_RPT];
            uint2 e[TU_RPT];
#pragma unroll
            for (int q = 0; q < TU_RPT; ++q) {
                uint32_t x1 = 0;
                go[q] = walker_goes<STRAT>(a, w[q], i, &x1);
                w[q].alive = go[q];
                if (go[q]) e[q] = load_edge(E, w[q].o + pick32(x1, w[q].d));
            }
            bool any = false;
#pragma unroll
            for (int q = 0; q < TU_RPT; ++q)
                if (go[q]) {
                    w[q].o = e[q].x;
                    w[q].d = e[q].y;
                    ++moves;
                    any = true;
                }
            // ---- the sources' tuples first
            if (wave == 0) {
                uint32_t x1 = 0;
                const bool sgo = walker_goes<STRAT>(a, sw, i, &x1);
                sw.alive = sgo;
                if (sgo) {
                    const uint2 se = load_edge(E, sw.o + pick32(x1, sw.d));
                    sw.o = se.x;
                    sw.d = se.y;
                }
                const uint64_t m = __ballot(sgo);
                if (sgo) {
                    const uint32_t p = held + lane_rank(m);
                    s_key[0][p] = sw.o | (steps << a.nb);
                    s_val[0][p] = (uint16_t)(TU_SRC | threadIdx.x);
                }
                if (lane == 0) {
                    s_n[i & 1u] = held + (uint32_t)__popcll(m);
                    s_nsrc[i & 1u] = (uint32_t)__popcll(m);
                }
            }
            __syncthreads();
            const uint32_t nsrc = uni(s_nsrc[i & 1u]), before = held + nsrc;
            // ---- then the start nodes' tuples, in any order
            if (nsrc != 0u) {
#pragma unroll
                for (int q = 0; q < TU_RPT; ++q) {
                    const uint64_t m = __ballot(go[q]);
                    uint32_t base = 0;
                    if (m && lane == 0) base = atomicAdd(&s_n[i & 1u], (uint32_t)__popcll(m));
                    base = uni(base);
                    if (go[q]) {
                        const uint32_t p = base + lane_rank(m);
                        s_key[0][p] = w[q].o | (steps << a.nb);
                        s_val[0][p] = (uint16_t)(q * TU_BLOCK + (int)threadIdx.x);
                    }
                }
                ++steps;
            } else {
                // no tuple of this or a later step can be linked: follow the
                // walks to their ends
                for (uint32_t t = i + 1; __ballot(any) != 0ull && t <= (uint32_t)a.L; ++t) {
                    any = false;
#pragma unroll
                    for (int q = 0; q < TU_RPT; ++q) {
                        uint32_t x1 = 0;
                        go[q] = walker_goes<STRAT>(a, w[q], t, &x1);
                        w[q].alive = go[q];
                        if (go[q]) e[q] = load_edge(E, w[q].o + pick32(x1, w[q].d));
                    }
#pragma unroll
                    for (int q = 0; q < TU_RPT; ++q)
                        if (go[q]) {
                            w[q].o = e[q].x;
                            w[q].d = e[q].y;
                            ++moves;
                            any = true;
                        }
                }
            }
            __syncthreads();
            const uint32_t count = uni(s_n[i & 1u]);
            held = count;
            // the walks end when no source or no start node has a step i; the
            // buffer is sorted then, or when the next step (which has no more
            // tuples than this one) may not fit
            const bool ended = nsrc == 0u || count == before || i == (uint32_t)a.L;
            if (!ended && steps < (1u << a.step_bits) && count + (count - before) + nsrc <= (uint32_t)TU_CAP)
                continue;
            if (count == 0u) break;   // (then ended)

            // ---- stable LSD sort by (step, o-value): wave w takes the w-th run of
            // the tuples, so earlier waves, rounds and lanes come first
            const int bits = a.nb + (steps > 1u ? 32 - __builtin_clz(steps - 1u) : 0);
            const int passes = (bits + B::DIGIT_BITS - 1) / B::DIGIT_BITS, digit_bits = (bits + passes - 1) / passes;
            if (threadIdx.x == 0) sorted += (unsigned long long)count * passes;
            const uint32_t rounds = (count + TU_BLOCK - 1) / TU_BLOCK;
            int buf = 0;
            for (int ps = 0; ps < passes; ++ps) {
                const int shift = ps * digit_bits;
                const uint32_t dmask = (1u << digit_bits) - 1u;
                for (int b = threadIdx.x; b < TU_WAVES * TU_DIGITS; b += TU_BLOCK) (&s_cnt[0][0])[b] = 0u;
                __syncthreads();
                uint32_t key[TU_ROUNDS], rank[TU_ROUNDS];
#pragma unroll
                for (int r = 0; r < TU_ROUNDS; ++r) {
                    if ((uint32_t)r >= rounds) break;
                    const uint32_t p = (uint32_t)wave * rounds * 64u + (uint32_t)r * 64u + (uint32_t)lane;
                    const bool valid = p < count;
                    key[r] = valid ? s_key[buf][p] : 0u;
                    const uint32_t dg = (key[r] >> shift) & dmask;
                    const uint64_t m = match_digit(dg, digit_bits, valid);
                    const int leader = valid ? __builtin_ctzll(m) : lane;
                    uint32_t old = 0;
                    if (valid && lane == leader) old = atomicAdd(&s_cnt[wave][dg], (uint32_t)__popcll(m));
                    old = __shfl(old, leader, 64);
                    rank[r] = old + lane_rank(m);
                }
                __syncthreads();
                {
                    uint32_t c[TU_WAVES], sum = 0, total;
#pragma unroll
                    for (int v = 0; v < TU_WAVES; ++v) {
                        c[v] = s_cnt[v][threadIdx.x];
                        sum += c[v];
                    }
                    uint32_t at = block_excl_sum(sum, &total);
#pragma unroll
                    for (int v = 0; v < TU_WAVES; ++v) {
                        s_cnt[v][threadIdx.x] = at;
                        at += c[v];
                    }
                }
                __syncthreads();
#pragma unroll
                for (int r = 0; r < TU_ROUNDS; ++r) {
                    if ((uint32_t)r >= rounds) break;
                    const uint32_t p = (uint32_t)wave * rounds * 64u + (uint32_t)r * 64u + (uint32_t)lane;
                    if (p >= count) continue;
                    const uint32_t to = s_cnt[wave][(key[r] >> shift) & dmask] + rank[r];
                    s_key[buf ^ 1][to] = key[r];
                    s_val[buf ^ 1][to] = s_val[buf][p];
                }
                __syncthreads();
                buf ^= 1;
            }

            // ---- PREDECESSOR: (position + 1) of the last source tuple at or
            // before each position, a running maximum
            const uint32_t p0 = min(count, threadIdx.x * rounds), p1 = min(count, p0 + rounds);
            uint32_t mine = 0;
            for (uint32_t p = p0; p < p1; ++p)
                if (s_val[buf][p] & TU_SRC) mine = p + 1u;
            uint32_t inc = mine;
            for (int dd = 1; dd < 64; dd <<= 1) {
                const uint32_t y = __shfl_up(inc, dd, 64);
                if (lane >= dd) inc = max(inc, y);
            }
            if (lane == 63) s_last[wave] = inc;
            uint32_t last = __shfl_up(inc, 1, 64);
            if (lane == 0) last = 0;
            __syncthreads();
            for (int v = 0; v < wave; ++v) last = max(last, s_last[v]);
            // ---- link: the closest source tuple, and those before it with the
            // same key (the sources' tuples of a key are contiguous, and first)
            for (uint32_t p = p0; p < p1; ++p) {
                const uint32_t val = s_val[buf][p];
                if (val & TU_SRC) {
                    last = p + 1u;
                    continue;
                }
                const uint32_t kp = s_key[buf][p];
                uint32_t bits = 0;
                for (uint32_t q = last; q > 0u && s_key[buf][q - 1u] == kp; --q)
                    bits |= 1u << (s_val[buf][q - 1u] & 31u);
                if (!bits) continue;
                uint32_t fresh = bits & ~atomicOr(&s_met[val], bits);   // a pair counts once
                if (!fresh) continue;
                const uint32_t v = (uint32_t)a.active[row0 + (int32_t)val];
                uint32_t cv = 0;
                if (STRAT) {
                    const uint4 fk = philox4x32_10(v, 0u, 0u, DOM_SHUFFLE, a.key);
                    cv = slot_class(shuffle_slot(j, (uint32_t)a.N, a.sa, a.sb, fk), s_ccum, a.L);
                }
                for (; fresh; fresh &= fresh - 1u) {
                    const int q = __builtin_ctz(fresh);
                    if ((uint32_t)a.src[q] == v) continue;
                    atomicAdd(&a.out[(size_t)q * a.n + v],
                              STRAT ? strat_weight(a.tab->a, s_srccls[q], cv) : 1ull);
                    ++meets;
                }
            }
            if (ended) break;
            steps = held = 0;
            __syncthreads();
        }
        // (a unit adds fewer than 2^17, and the wave's sum below is of 64)
        if (meets >= 1u << 24) {
            atomicAdd(&ctr_set(a.counters)[C_MEETS], (unsigned long long)meets);
            meets = 0;
        }
        __syncthreads();
    }
    for (int dd = 32; dd > 0; dd >>= 1) {
        moves += __shfl_xor(moves, dd, 64);
        meets += __shfl_xor(meets, dd, 64);
    }
    if (lane == 0) {
        unsigned long long *to = ctr_set(a.counters);
        if (moves) atomicAdd(&to[C_MOVES], moves);
        if (meets) atomicAdd(&to[C_MEETS], (unsigned long long)meets);
        if (sorted) atomicAdd(&to[C_SPARE], sorted);
    }
}

// Steps of each start node's walks (grid: x over j, y over nodes, strided), for
// the limit on one node's and the sources' tuples.
__global__ __launch_bounds__(256) void k_row_tuples(TupleArgs a, bool strat, unsigned long long *row_sum) {
    const int32_t j = blockIdx.x * 256 + threadIdx.x;
    for (int32_t row = blockIdx.y; row < a.na; row += gridDim.y) {
        unsigned long long len = 0;
        if (j < a.N) {
            const uint32_t id = (uint32_t)a.active[row];
            Walker w = strat ? walker_begin<true>(a, id, (uint32_t)j, a.tab->ccum)
                             : walker_begin<false>(a, id, (uint32_t)j, nullptr);
            for (uint32_t i = 1; i <= (uint32_t)a.L; ++i) {
                uint32_t x1 = 0;
                if (!(strat ? walker_goes<true>(a, w, i, &x1) : walker_goes<false>(a, w, i, &x1))) break;
                const uint2 e = a.E[w.o + pick32(x1, w.d)];
                w.o = e.x;
                w.d = e.y;
                ++len;
            }
        }
        for (int d = 32; d > 0; d >>= 1) len += __shfl_xor(len, d, 64);
        if ((threadIdx.x & 63) == 0 && len) atomicAdd(&row_sum[row], len);
    }
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// A source's own entry: R (plain: every pair meets at step 0) or 0 (stratified);
// and the folded work counters.
__global__ void k_tuples_end(TupleArgs a, bool strat) {
    const int q = threadIdx.x;
    if (q < a.k) a.out[(size_t)q * a.n + a.src[q]] = strat ? 0ull : (unsigned long long)a.N;
    if (q < 8) {
        unsigned long long sum = 0;
        for (int i = 1; i <= CTR_SETS; ++i) sum += a.counters[8 * i + q];
        a.counters[q] = sum;
    }
}

int bits_for(uint64_t max_value) {
    int b = 1;
    while (b < 64 && (max_value >> b) != 0) ++b;
    return b;
}

struct DevBuf {
    void *p = nullptr;
    ~DevBuf() { device_free(p); }
};

// Blocks of the tuple kernel that are resident at once.
template <bool STRAT, typename B>
int tuple_grid() {
    static const int blocks = [] {
        int dev = 0, cus = 0, per = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_tuples<STRAT, B>, B::BLOCK, 0);
        return (cus > 0 ? cus : 256) * (per > 0 ? per : 1);
    }();
    return blocks;
}

template <bool STRAT, typename B>
void launch_tuples(TupleArgs &a, hipStream_t st) {
    a.units = (int64_t)((a.na + B::ROWS - 1) / B::ROWS) * a.N;
    if (a.units > 0)
        k_tuples<STRAT, B><<<(unsigned)std::min<int64_t>(a.units, tuple_grid<STRAT, B>()), B::BLOCK, 0, st>>>(a);
}

}  // namespace
}  // namespace srk

using namespace srk;

extern "C" int simrank_tuple_meets(const simrank_graph *g, const simrank_query *qs, int32_t k,
                                   uint64_t *sums, simrank_stats *st_opt) {
    clear_error();
    if (!g || !qs || !sums) return fail(SIMRANK_EINVAL, "NULL argument");
    if (k < 1 || k > MAX_TUPLE_SOURCES) return fail(SIMRANK_EINVAL, "k must lie in [1, 32]");
    simrank_params p0;
    int mode0;
    int rc = query_params(&qs[0], g->n, &p0, &mode0);
    if (rc) return rc;
    if (mode0 == SIMRANK_MODE_STITCHED)
        return fail(SIMRANK_EINVAL, "the tuple form takes plain or stratified queries");
    StratTab tab{};
    StratParams sp{};
    const bool strat = mode0 == SIMRANK_MODE_STRATIFIED;
    if (strat && (rc = strat_params(&qs[0], g->n, &sp, &tab))) return rc;
    std::vector<int32_t> srcs(k);
    for (int32_t q = 0; q < k; ++q) {
        simrank_params p;
        int mode;
        if ((rc = query_params(&qs[q], g->n, &p, &mode))) return rc;
        if (qs[q].s < 0 || qs[q].s >= g->n) return fail(SIMRANK_EINVAL, "source out of range");
        if (mode != mode0 || p.R != p0.R || p.L != p0.L || p.T != p0.T || qs[q].seed != qs[0].seed)
            return fail(SIMRANK_EINVAL, "the tuple form's queries must share mode, seed, c, R and L");
        if (strat) {
            StratParams s2;
            if ((rc = strat_params(&qs[q], g->n, &s2, nullptr))) return rc;
            if (s2.z != sp.z) return fail(SIMRANK_EINVAL, "stratified queries must share z");
        }
        srcs[q] = qs[q].s;
    }
    const int32_t N = p0.R, L = p0.L;
    SRK_HIP(hipSetDevice(g->device));
    hipStream_t st = g->stream;
    // e0 / e1 around the call, s0 / s1 around the tuple kernel
    struct EvGuard {
        hipEvent_t e[4] = {nullptr, nullptr, nullptr, nullptr};
        ~EvGuard() {
            for (hipEvent_t x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } evg;
    for (hipEvent_t &x : evg.e) SRK_HIP(hipEventCreate(&x));
    hipEvent_t e0 = evg.e[0], e1 = evg.e[1], s0 = evg.e[2], s1 = evg.e[3];
    SRK_HIP(hipEventRecord(e0, st));

    const size_t n = (size_t)g->n;
    DevBuf d_src, d_tab, d_out, d_cnt;
    if ((rc = device_alloc(&d_src.p, 4 * (size_t)k, nullptr))) return rc;
    if ((rc = device_alloc(&d_tab.p, sizeof(StratTab), nullptr))) return rc;
    if ((rc = device_alloc(&d_out.p, 8 * n * (size_t)k, nullptr))) return rc;
    if ((rc = device_alloc(&d_cnt.p, 8 * CTR_WORDS, nullptr))) return rc;
    SRK_HIP(hipMemcpyAsync(d_src.p, srcs.data(), 4 * (size_t)k, hipMemcpyHostToDevice, st));
    SRK_HIP(hipMemcpyAsync(d_tab.p, &tab, sizeof(StratTab), hipMemcpyHostToDevice, st));
    auto *out = (unsigned long long *)d_out.p;
    auto *counters = (unsigned long long *)d_cnt.p;
    k_fill_u64<<<std::min(grid_for((int64_t)(n * k), 256), 4096u), 256, 0, st>>>(out, (int64_t)(n * k));
    k_fill_u64<<<1, 256, 0, st>>>(counters, CTR_WORDS);

    TupleArgs a{};
    a.nodes = g->nodes;
    a.E = g->E;
    a.active = g->active;
    a.na = g->n_active;
    a.N = N;
    a.L = L;
    a.key = make_key(qs[0].seed);
    a.T = p0.T;
    a.tab = (const StratTab *)d_tab.p;
    a.sa = (uint32_t)sp.sa;
    a.sb = (uint32_t)sp.sb;
    a.src = (const int32_t *)d_src.p;
    a.k = k;
    a.n = g->n;
    a.out = out;
    a.counters = counters;
    a.nb = bits_for((uint64_t)std::max<int64_t>(g->m_slots - 1, 1));   // at most 31
    a.step_bits = std::min(TU_STEP_BITS, 32 - a.nb);

    // Queries whose sources and one start node could have 2^32 - 1 tuples between
    // them are refused: a limit of the interface (simrank.h), which a sort of whole
    // start nodes set; k_tuples itself holds no more than a block's at once.
    const int64_t src_tuples_max = (int64_t)k * N * L;
    if (a.na > 0 && src_tuples_max + (int64_t)N * L >= (int64_t)0xffffffffu) {
        DevBuf rs;
        if ((rc = device_alloc(&rs.p, 8 * (size_t)a.na, nullptr))) return rc;
        k_fill_u64<<<std::min(grid_for(a.na, 256), 4096u), 256, 0, st>>>((unsigned long long *)rs.p, a.na);
        k_row_tuples<<<dim3(grid_for(N, 256), std::min(a.na, 65535)), 256, 0, st>>>(
            a, strat, (unsigned long long *)rs.p);
        SRK_HIP(hipGetLastError());
        std::vector<unsigned long long> row_sum(a.na);
        SRK_HIP(hipMemcpyAsync(row_sum.data(), rs.p, 8 * (size_t)a.na, hipMemcpyDeviceToHost, st));
        SRK_HIP(hipStreamSynchronize(st));
        const int64_t most = (int64_t)*std::max_element(row_sum.begin(), row_sum.end());
        if (src_tuples_max + most >= (int64_t)0xffffffffu)
            return fail(SIMRANK_EINVAL, "one node's and the sources' tuples exceed 2^32 - 2");
    }
    SRK_HIP(hipEventRecord(s0, st));
    const bool small = a.na <= TU_SMALL::ROWS / 2 ||
                       (a.na <= TU_SMALL::ROWS && N > (strat ? tuple_grid<true, TU_LARGE>() : tuple_grid<false, TU_LARGE>()));
    if (strat) {
        if (small) launch_tuples<true, TU_SMALL>(a, st);
        else launch_tuples<true, TU_LARGE>(a, st);
    } else {
        if (small) launch_tuples<false, TU_SMALL>(a, st);
        else launch_tuples<false, TU_LARGE>(a, st);
    }
    SRK_HIP(hipEventRecord(s1, st));
    k_tuples_end<<<1, 64, 0, st>>>(a, strat);
    SRK_HIP(hipGetLastError());
    SRK_HIP(hipEventRecord(e1, st));
    SRK_HIP(hipMemcpyAsync(sums, out, 8 * n * (size_t)k, hipMemcpyDeviceToHost, st));
    unsigned long long c[8];
    SRK_HIP(hipMemcpyAsync(c, counters, sizeof(c), hipMemcpyDeviceToHost, st));
    SRK_HIP(hipStreamSynchronize(st));
    if (st_opt) {
        float ms = 0.f, sms = 0.f;
        SRK_HIP(hipEventElapsedTime(&ms, e0, e1));
        SRK_HIP(hipEventElapsedTime(&sms, s0, s1));
        *st_opt = simrank_stats{};
        st_opt->pairs = (uint64_t)(g->n - 1) * (uint64_t)N * (uint64_t)k;
        st_opt->moves = c[C_MOVES];
        // bytes the sort passes move (see simrank.h): 4 per key a pass counts,
        // 12 per tuple it reads and writes
        st_opt->draws = c[C_SPARE] * 16u;
        st_opt->meet_ms = sms;
        st_opt->meets = c[C_MEETS];
        st_opt->ms = ms;
        st_opt->R = N;
        st_opt->L = L;
        st_opt->T = p0.T;
    }
    return SIMRANK_OK;
}
