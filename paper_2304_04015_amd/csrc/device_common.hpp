// Device helpers shared by the query kernels (single queries and groups).
#pragma once

#include "common.hpp"
#include "philox.hpp"

namespace srk {

__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// Slot entered by walk (v, j) whose private head ended at node y
// (counter (v, j, 0, 2)).
__device__ __forceinline__ uint32_t entry_slot(const IndexView &ix, PhiloxKey key, uint32_t v,
                                               uint32_t j, uint32_t y) {
    const int64_t b = ix.pool_off[y];
    const int64_t P = ix.pool_off[y + 1] - b;
    const uint4 x = philox4x32_10(v, j, 0u, DOM_ENTRY, key);
    return (uint32_t)(b + (int64_t)pick64(x.x, (uint64_t)P));
}

// Set of work counters that this block adds to.
__device__ __forceinline__ unsigned long long *ctr_set(unsigned long long *counters) {
    return counters + 8 * (1 + (blockIdx.x % CTR_SETS));
}

// Adds the lanes' work (moves, draws, meets, tail steps, pairs) to the
// counters at `to`: the waves' sums meet in LDS, so a block makes one atomic
// per counter.  Block-wide (blocks of up to 1024 threads).
__device__ __forceinline__ void add_work(unsigned long long *to, unsigned long long moves,
                                         unsigned long long draws, unsigned long long meets,
                                         unsigned long long tail, unsigned long long pairs) {
    __shared__ unsigned long long part[16][5];
    unsigned long long w[5] = {moves, draws, meets, tail, pairs};
#pragma unroll
    for (int c = 0; c < 5; ++c)
        for (int dd = 32; dd > 0; dd >>= 1) w[c] += __shfl_xor(w[c], dd, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 5; ++c) part[threadIdx.x >> 6][c] = w[c];
    __syncthreads();
    static_assert(C_MOVES == 0 && C_DRAWS == 1 && C_MEETS == 2 && C_TAIL == 3 && C_PAIRS == 4,
                  "one thread per counter");
    if (threadIdx.x < 5) {
        unsigned long long sum = 0;
        for (uint32_t i = 0; i < (blockDim.x >> 6); ++i) sum += part[i][threadIdx.x];
        if (sum) atomicAdd(&to[threadIdx.x], sum);
    }
    __syncthreads();
}

template <typename T>
__device__ __forceinline__ T block_excl_sum(T x, T *total) {
    __shared__ T part[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    T inc = x;
    for (int d = 1; d < 64; d <<= 1) {
        T y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) part[wave] = inc;
    __syncthreads();
    T before = 0, tot = 0;
    for (int w = 0; w < nw; ++w) {
        if (w < wave) before += part[w];
        tot += part[w];
    }
    __syncthreads();
    *total = tot;
    return before + inc - x;
}

// Cuts entries [0, E1), entry e holding words [joff[e], joff[e + 1]), into
// tiles from the front, each the longest run [a, b) with b - a <= TJ and
// joff[b] - joff[a] <= TN; writes the starts to tiles[0 .. count) and returns
// the count.  Every tile but the last is full in walks (TJ) or holds more than
// TN - w words, w the largest entry, so the count stays within 1 + E1 / TJ +
// joff[E1] / (TN - w).  Called by all 64 lanes of one wave (results uniform);
// needs w <= TN.  Each run's end is found by a 64-way search: the lanes probe
// 64 points of the open range at once, so a range of up to 64^2 entries takes
// two rounds of loads.
__device__ inline uint32_t cut_tiles(const uint32_t *joff, uint32_t E1, uint32_t TJ, uint32_t TN,
                                     uint32_t *tiles, int lane) {
    uint32_t a = 0, nt = 0;
    while (a < E1) {
        if (lane == 0) tiles[nt] = a;
        ++nt;
        const uint32_t base = joff[a];
        // the run ends at the largest b in [lo, hi] with joff[b] - base <= TN;
        // lo = a + 1 always qualifies (one entry fits)
        uint32_t lo = a + 1, hi = min(a + TJ, E1);
        while (lo < hi) {
            const uint32_t span = hi - lo;
            const uint32_t p = lo + (uint32_t)(((uint64_t)span * (uint32_t)(lane + 1)) >> 6);
            const bool fits = joff[p] - base <= TN;
            const uint64_t m = __ballot(fits);   // fits holds for a prefix of the lanes
            const uint32_t k = (uint32_t)__popcll(m);
            const uint32_t p_last = uni(__shfl(p, (int)(k ? k - 1 : 0), 64));
            const uint32_t p_next = uni(__shfl(p, (int)(k < 64 ? k : 63), 64));
            if (k == 64) lo = hi;
            else {
                if (k) lo = p_last;
                hi = p_next - 1;
            }
        }
        a = lo;
    }
    return nt;
}

// Pointers read from a descriptor in memory are generic to the compiler, which
// then loads through them with flat instructions: those also go through the
// LDS path and tie the gathers to the LDS counter, so that every LDS read waits
// for them.  gp() states that they point to global memory.  With the gathers
// global and the refill's counts known to be uniform (scalar branches instead
// of exec masks), where the graph sits in the L2 and the meet kernel is bound
// by its instructions: 16 queries on graphs of 4,097 to 150,000 nodes 55.4 ms
// instead of 61.1, a query at n = 40,000 638 us instead of 686, a stratified
// one at n = 2^18 21.8 ms instead of 22.8; none at n = 2^20, bound by the
// L2's misses.
template <typename T>
using GlobalPtr = const __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ GlobalPtr<T> gp(const T *p) {
    return (GlobalPtr<T>)p;
}
// A pointer that is the same in all lanes, kept in scalar registers.
template <typename T>
__device__ __forceinline__ GlobalPtr<T> gp_uni(const T *p) {
    const uint64_t a = (uint64_t)p;
    return (GlobalPtr<T>)(((uint64_t)uni((uint32_t)(a >> 32)) << 32) | uni((uint32_t)a));
}

// The walk's gather of an edge slot.
__device__ __forceinline__ uint2 load_edge(GlobalPtr<uint64_t> E, uint32_t at) {
    const uint64_t v = E[at];
    return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}

// The meet kernels' gathers: packed rows (4 bytes a slot) where the graph has
// them and its hubs' rows fit the kernel's LDS, else load_edge.
struct Gather {
    GlobalPtr<uint64_t> E;
    GlobalPtr<uint32_t> E4;
    uint32_t obits;   // 0: no packed rows
};
template <int HL, typename Desc>   // HL: hubs' rows the kernel's LDS holds
__device__ __forceinline__ Gather gather_of(const Desc &d) {
    return {gp_uni((const uint64_t *)d.E), gp_uni(d.E4),
            uni((uint32_t)d.n_hubs) <= (uint32_t)HL ? uni((uint32_t)d.obits) : 0u};
}
__device__ __forceinline__ uint2 unpack_row(uint32_t r, uint32_t obits, const uint2 *s_hub) {
    const uint32_t d = r >> obits, x = r & ((1u << obits) - 1u);
    return d != 0xffffffffu >> obits ? make_uint2(x, d) : s_hub[x];
}

__device__ __forceinline__ uint32_t lane_rank(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// One pair in flight on a lane.
struct Slot {
    uint32_t at;     // LDS index of the position of walk (s, j) that the next step is tested
                     // against (16 bits); stratified: | class of walk (s, j) << 16
    uint32_t end;    // LDS index of its last one (16 bits) | node index << 16; stitched:
                     // | HEAD_ONLY if the walk goes on beyond it
    uint32_t o, d;   // current node: slot offset in E and in-degree
    WalkDraws rng;
    uint32_t aux;    // stratified: class of walk (v, j); stitched: the tile entry of walk (s, j)
};
constexpr uint32_t HEAD_ONLY = 1u << 31;

// The lanes of a mask that is the same in all lanes.
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Work of a wave: the same in all lanes, but for the tail steps.
struct Work {
    unsigned long long moves = 0, draws = 0, meets = 0, pairs = 0;
    uint32_t tail = 0;
};
__device__ __forceinline__ void add_work(unsigned long long *to, const Work &w) {
    const bool one = (threadIdx.x & 63) == 0;
    add_work(to, one ? w.moves : 0ull, one ? w.draws : 0ull, one ? w.meets : 0ull, w.tail, one ? w.pairs : 0ull);
}

// Items (pairs of a unit) a wave takes from the block's cursor at once: 64, up
// to `most` where the unit has enough of them for its 16 waves.
constexpr uint32_t ITEM_CHUNK = 64;
__device__ __forceinline__ uint32_t item_chunk(uint32_t total, uint32_t most) {
    return min(max((total >> 8) & ~63u, ITEM_CHUNK), most);
}
// Pairs waiting for their stitched tails, per wave: a ring, a power of two
// above 63 + 64 (a wave drains 64 as soon as 64 wait, after each slot's push).
constexpr uint32_t TAIL_Q = 128;

// ------------------------------------------------- walk shuffle (stratified)
//
// Node v's N fixed-length walks are generated class by class (slots
// [ccum[l], ccum[l+1]) hold the walks of length l) and then shuffled: walk j
// is the walk generated in slot pi_v(j).  pi_v is a four-round Feistel
// network over the grid [0, A) x [0, 2^b) (A 2^b >= N, 2^b about sqrt(N)),
// restricted to [0, N) by cycle walking (Black and Rogaway, CT-RSA 2002); its
// round keys are the four words of Philox(v, 0, 0, DOM_SHUFFLE).  Fewer than
// 2/sqrt(N) of the grid's points lie beyond N, so a lane almost never walks a
// second time.

// MurmurHash3's 32-bit finalizer (A. Appleby, public domain), the round function.
__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85ebca6bu;
    h ^= h >> 13;
    h *= 0xc2b2ae35u;
    h ^= h >> 16;
    return h;
}

// Bijection of the grid, point (hi, lo) = hi 2^b + lo: rounds alternately add
// a round-function value scaled into [0, A) to hi modulo A, and XOR lo with
// its low b bits (a mixed-radix Feistel network, as in NIST SP 800-38G FF1).
__device__ __forceinline__ uint32_t feistel4(uint32_t x, uint32_t A, uint32_t b, uint4 k) {
    const uint32_t mb = (1u << b) - 1u;
    uint32_t hi = x >> b, lo = x & mb;
    hi += __umulhi(fmix32(lo ^ k.x), A);
    hi = hi >= A ? hi - A : hi;
    lo ^= fmix32(hi ^ k.y) & mb;
    hi += __umulhi(fmix32(lo ^ k.z), A);
    hi = hi >= A ? hi - A : hi;
    lo ^= fmix32(hi ^ k.w) & mb;
    return (hi << b) | lo;
}

// pi_v(j) for j < N.  The orbit of j under the bijection is a cycle through
// j, so a value below N comes back within A 2^b applications; the loop is
// bounded by that.
__device__ __forceinline__ uint32_t shuffle_slot(uint32_t j, uint32_t N, uint32_t A, uint32_t b,
                                                 uint4 k) {
    uint32_t y = feistel4(j, A, b, k);
    const uint32_t cap = A << b;
    for (uint32_t it = 1; y >= N && it < cap; ++it) y = feistel4(y, A, b, k);
    return y;
}

// Length class of slot r: the largest l <= phi with ccum[l] <= r.
__device__ __forceinline__ uint32_t slot_class(uint32_t r, const uint32_t *ccum, int32_t phi) {
    int32_t lo = 0, hi = phi + 1;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (ccum[mid] <= r) lo = mid; else hi = mid;
    }
    return (uint32_t)lo;
}

// Runs of 2^class_run_log2(N) slots, CLASS_RUNS at most: the class of a run's
// first slot and a step or two up the class starts give a slot's class.
constexpr uint32_t CLASS_RUNS = 4096;
__device__ __forceinline__ uint32_t class_run_log2(uint32_t N) {
    return N <= CLASS_RUNS ? 0u : 20u - (uint32_t)__builtin_clz(N - 1u);
}

// Meet weight of classes (l1, l2) in units of 2^-40 (Lemma 5's ratio
// Z_l1 Z_l2 / (Zhat_l1 Zhat_l2), truncated).
__device__ __forceinline__ unsigned long long strat_weight(const double *a, uint32_t l1, uint32_t l2) {
    return (unsigned long long)((a[l1] * a[l2]) * 1099511627776.0);
}


}  // namespace srk
