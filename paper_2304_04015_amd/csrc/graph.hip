// Graph ingest: the in-edge CSR of G (the reversed graph the walks run on,
// Algorithm 1 "reverse the edges") becomes the library's gather layout.
//
//   nodes[v] = (o(v), deg(v)),  o(v) = sum_{u < v} max(deg(u), 1)
//   E[o(v) + k] = nodes[in_src[in_off[v] + k]]      for k < deg(v)
//   node_of[o(v)] = v
//   E[o(v)] = (NIL, NIL) for a node without in-neighbours (never read by a walk)
//
// A walk at (o, d) picks k < d and reads E[o + k]: one 8-byte gather gives
// the next node's identity o and its degree, so a move never needs a second,
// dependent gather of a row array.  Edge order inside a row is preserved, so
// the k-th in-neighbour is the same as in the caller's CSR.
//
// A graph also has its rows packed in 4 bytes, for the meet kernels: where E is
// larger than an XCD's 4 MB of L2 those are bound by the cache lines their
// gathers fetch from behind it, and of half the footprint the L2 holds twice the
// share.  E4[i] = degree << obits | o with just the bits that o needs; the
// largest degree code stands for a hub, a node whose degree does not fit, with
// its place in `hubs` in place of o.  A graph with more than HUB_CAP hubs has no
// packed rows.  Meet kernel with E and packed: n = 40,000 (5 MB of E), R = 9,502:
// 1,499 and 1,335 us; n = 150,001 (18 MB): 5,949 and 5,093; n = 2^18 (32 MB):
// 11.68 and 9.46 ms; n = 2^19 (66 MB): 24.8 and 21.2; n = 2^20 (133 MB, 6,256
// hubs): 51.9 and 47.8.
#include <vector>

#include "common.hpp"

namespace srk {
namespace {

// Packing of the rows in 4 bytes; E4 NULL: not wanted.
struct PackArgs {
    uint32_t *E4;
    uint32_t obits;
    uint2 *hubs;                  // one for each of them
    uint32_t *hub_at;             // [n] place of a node that is a hub
    unsigned long long *last_hub;   // place of the last hub, -1 before
};

__global__ void k_slot_counts(const int32_t *__restrict__ off, int32_t n,
                              uint32_t *__restrict__ slots, uint32_t *__restrict__ has_in) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int32_t d = off[v + 1] - off[v];
    slots[v] = d > 0 ? (uint32_t)d : 1u;
    has_in[v] = d > 0 ? 1u : 0u;
}

__global__ void k_nodes(const int32_t *__restrict__ off, const int64_t *__restrict__ o, int32_t n,
                        const int64_t *__restrict__ act_pos, uint2 *__restrict__ nodes,
                        uint2 *__restrict__ E, uint32_t *__restrict__ node_of,
                        int32_t *__restrict__ active, PackArgs pk) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int32_t d = off[v + 1] - off[v];
    nodes[v] = make_uint2((uint32_t)o[v], (uint32_t)d);
    node_of[o[v]] = (uint32_t)v;
    if (d > 0) active[act_pos[v]] = (int32_t)v;
    else E[o[v]] = make_uint2(NIL, NIL);
    if (!pk.E4) return;
    if (d == 0) pk.E4[o[v]] = 0u;
    if ((uint32_t)d >= 0xffffffffu >> pk.obits) {
        const unsigned long long k = atomicAdd(pk.last_hub, 1ull) + 1ull;
        pk.hubs[k] = make_uint2((uint32_t)o[v], (uint32_t)d);
        pk.hub_at[v] = (uint32_t)k;
    }
}

__global__ void k_fill_u32(uint32_t *__restrict__ p, int64_t n, uint32_t val) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = val;
}

// A block lays out a tile of consecutive edges.  The row that owns each is found
// for the tile at once: the rows that start in it mark their first edge in LDS,
// and a running maximum over the marks gives every edge its row (empty rows
// share the start of the next and lose to it, the larger).  dbar[u] counts the
// rows that list u (the pool sizes of the stitched index follow it): the tile's
// counts meet in a small LDS hash table first, so that a hub, listed by a great
// many rows, costs an atomic per tile instead of one per edge, all on one cache
// line.  *bad receives the first edge whose source is not a node.
//
// With a binary search over in_off per edge (20 dependent reads), an atomic per
// edge and the sources checked by the host, loading a graph of n = 300,007
// (4.5e6 edges) took 2.23 ms and one of n = 2^22 (6.5e7 edges) 30.8; now 1.35
// and 17.5, k_edges 0.21 and 2.76 of them (257 us and, at n = 2^20, 855 before,
// 713 now: the atomics on distinct nodes remain).
//
// Between the edges of a tile may lie a great many rows without any, which one
// block would go through 256 at a time: with more than EDGE_GAP rows per edge
// (edges counted as 256 at least) each edge's row is searched for among them.
// Loading a graph of 4,096 edges and 2^14 / 2^15 / 2^16 / 2^18 / 2^20 rows in one
// tile: 208 / 234 / 295 / 714 / 2,535 us gone through, 215 / 230 / 263 / 491 / 1,479
// searched; of 1,000 edges and 2^13 / 2^14 / 2^16: 174 / 200 / 290 and 168 / 188 / 243.
//
// A tile is 4,096 edges, or 1,024 up to EDGE_FEW edges, which tiles of 4,096 give to
// too few blocks: loading 4e4 edges took 213 us with these and takes 196 with the
// small ones, 1.6e5 280 and 262, 8e5 456 and 451; 4.5e6 1,546 and 1,572.
constexpr int EDGE_BLOCK = 256;
constexpr int64_t EDGE_FEW = 1 << 20;
constexpr int32_t EDGE_GAP = 16;
constexpr uint32_t EDGE_HASH = 2048;
template <int EDGE_ITEMS>
__global__ __launch_bounds__(EDGE_BLOCK) void k_edges(const int32_t *__restrict__ off,
                                                      const int32_t *__restrict__ src, int32_t n,
                                                      int64_t m, const uint2 *__restrict__ nodes,
                                                      uint2 *__restrict__ E,
                                                      uint32_t *__restrict__ dbar,
                                                      unsigned long long *__restrict__ bad,
                                                      PackArgs pk) {
    constexpr int EDGE_TILE = EDGE_BLOCK * EDGE_ITEMS;
    __shared__ int32_t s_row[EDGE_TILE];
    __shared__ int32_t s_part[EDGE_BLOCK / 64];
    __shared__ uint32_t s_key[EDGE_HASH], s_cnt[EDGE_HASH];
    const int64_t e0 = (int64_t)blockIdx.x * EDGE_TILE;
    const int32_t cnt = (int32_t)min((int64_t)EDGE_TILE, m - e0);
    for (int i = threadIdx.x; i < EDGE_TILE; i += EDGE_BLOCK) s_row[i] = -1;
    for (uint32_t i = threadIdx.x; i < EDGE_HASH; i += EDGE_BLOCK) {
        s_key[i] = NIL;
        s_cnt[i] = 0u;
    }
    // the last row of [lo, hi) that starts at or before edge e
    auto row_of = [&](int64_t e, int32_t lo, int32_t hi) {
        while (hi - lo > 1) {
            const int32_t mid = lo + ((hi - lo) >> 1);
            if ((int64_t)off[mid] <= e) lo = mid; else hi = mid;
        }
        return lo;
    };
    const int32_t v0 = row_of(e0, 0, n), v1 = row_of(e0 + cnt - 1, v0, n);
    __syncthreads();
    if (v1 - v0 > EDGE_GAP * max(cnt, EDGE_BLOCK)) {
        for (int32_t i = threadIdx.x; i < cnt; i += EDGE_BLOCK) s_row[i] = row_of(e0 + i, v0, v1 + 1);
    } else {
        if (threadIdx.x == 0) s_row[0] = v0;
        __syncthreads();
        for (int32_t v = v0 + 1 + (int32_t)threadIdx.x; v <= v1; v += EDGE_BLOCK)
            atomicMax(&s_row[(int64_t)off[v] - e0], v);
        __syncthreads();
        const int b = threadIdx.x * EDGE_ITEMS;
        int32_t r[EDGE_ITEMS], run = -1;
#pragma unroll
        for (int i = 0; i < EDGE_ITEMS; ++i) run = r[i] = max(run, s_row[b + i]);
        int32_t inc = run;
        for (int dd = 1; dd < 64; dd <<= 1) {
            const int32_t y = __shfl_up(inc, dd, 64);
            if ((int)(threadIdx.x & 63) >= dd) inc = max(inc, y);
        }
        if ((threadIdx.x & 63) == 63) s_part[threadIdx.x >> 6] = inc;
        int32_t before = __shfl_up(inc, 1, 64);
        if ((threadIdx.x & 63) == 0) before = -1;
        __syncthreads();
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) before = max(before, s_part[w]);
#pragma unroll
        for (int i = 0; i < EDGE_ITEMS; ++i) s_row[b + i] = max(before, r[i]);
    }
    __syncthreads();
    for (int32_t i = threadIdx.x; i < cnt; i += EDGE_BLOCK) {
        const int64_t e = e0 + i;
        const int32_t v = s_row[i];
        const uint32_t u = (uint32_t)src[e];
        if (u >= (uint32_t)n) {
            atomicMin(bad, (unsigned long long)e);
            continue;
        }
        const int64_t at = (int64_t)nodes[v].x + (e - off[v]);
        const uint2 to = nodes[u];
        E[at] = to;
        if (pk.E4) {
            const uint32_t most = 0xffffffffu >> pk.obits;
            pk.E4[at] = to.y < most ? (to.y << pk.obits) | to.x : (most << pk.obits) | pk.hub_at[u];
        }
        const uint32_t h = (u * 0x9E3779B1u) >> 21;
        static_assert(EDGE_HASH == 1u << 11, "hash bits");
        const uint32_t old = atomicCAS(&s_key[h], NIL, u);
        if (old == NIL || old == u) atomicAdd(&s_cnt[h], 1u);
        else atomicAdd(&dbar[u], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < EDGE_HASH; i += EDGE_BLOCK)
        if (s_cnt[i]) atomicAdd(&dbar[s_key[i]], s_cnt[i]);
}

}  // namespace

int device_alloc(void **p, size_t bytes, int64_t *acct) {
    *p = nullptr;
    if (bytes == 0) bytes = 8;
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return fail(SIMRANK_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed: " +
                                        hipGetErrorString(e));
    }
    if (acct) *acct += (int64_t)bytes;
    return SIMRANK_OK;
}

void device_free(void *p) {
    if (p) (void)hipFree(p);
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Bits of o() in a packed row, or 0 if so few would be left for the degree that
// most nodes were hubs.
static int32_t pack_bits(int64_t m_slots) {
    int32_t b = 1;
    while ((m_slots - 1) >> b) ++b;
    return b <= 26 ? b : 0;
}

static void graph_release(simrank_graph *g) {
    if (!g) return;
    if (g->index) {
        index_free(g->index);
        delete g->index;
        g->index = nullptr;
    }
    device_free(g->nodes);
    device_free(g->E);   // (and node_of, E4 and hubs behind it)
    device_free(g->active);
    device_free(g->dbar);
    if (g->stream) (void)hipStreamDestroy(g->stream);
    delete g;
}

}  // namespace srk

using namespace srk;


extern "C" int simrank_load_graph(int32_t n, int64_t m, const int32_t *in_off,
                                  const int32_t *in_src, simrank_graph **g_out) {
    clear_error();
    if (!g_out) return fail(SIMRANK_EINVAL, "g_out is NULL");
    *g_out = nullptr;
    if (!in_off || (m > 0 && !in_src)) return fail(SIMRANK_EINVAL, "NULL CSR array");
    if (n < 1) return fail(SIMRANK_EINVAL, "n must be >= 1");
    if (m < 0 || m + (int64_t)n >= (int64_t)0x7fffffff)
        return fail(SIMRANK_EINVAL, "need 0 <= m and m + n < 2^31");
    // Host-side validation of the CSR (the copy below trusts it).
    if (in_off[0] != 0) return fail(SIMRANK_EINVAL, "in_off[0] must be 0");
    int32_t max_deg = 0;
    int32_t n_active = 0;
    bool falls = false;
    for (int32_t v = 0; v < n; ++v) {   // (no exit: vectorised)
        const int32_t d = (int32_t)((uint32_t)in_off[v + 1] - (uint32_t)in_off[v]);
        falls |= in_off[v + 1] < in_off[v];
        max_deg = d > max_deg ? d : max_deg;
        n_active += d > 0;
    }
    for (int32_t v = 0; falls && v < n; ++v)
        if (in_off[v + 1] < in_off[v])
            return fail(SIMRANK_EINVAL, "in_off decreases at row " + std::to_string(v));
    if ((int64_t)in_off[n] != m) return fail(SIMRANK_EINVAL, "in_off[n] != m");
    // The sources are checked by the kernel that reads them; here where there
    // is no device to do it.
    auto bad_source = [](int64_t e) {
        return fail(SIMRANK_EINVAL, "in_src[" + std::to_string(e) + "] out of range");
    };
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) {
        (void)hipGetLastError();
        for (int64_t e = 0; e < m; ++e)
            if (in_src[e] < 0 || in_src[e] >= n) return bad_source(e);
    }

    simrank_graph *g = new simrank_graph();
    g->n = n;
    g->m = m;
    g->max_deg = max_deg;
    g->n_active = n_active;
    g->m_slots = m + (int64_t)(n - n_active);
    int rc;
    int32_t *d_off = nullptr, *d_src = nullptr;
    uint32_t *d_slots = nullptr, *d_has = nullptr;
    int64_t *d_o = nullptr, *d_apos = nullptr, *d_tot = nullptr;
#define SRK_TRY(x)                     \
    do {                               \
        rc = (x);                      \
        if (rc != SIMRANK_OK) goto bad; \
    } while (0)
#define SRK_TRYHIP(x)                                                            \
    do {                                                                         \
        hipError_t e_ = (x);                                                     \
        if (e_ != hipSuccess) {                                                  \
            rc = fail(SIMRANK_EDEVICE, std::string(#x) + ": " + hipGetErrorString(e_)); \
            goto bad;                                                            \
        }                                                                        \
    } while (0)
    {
        SRK_TRYHIP(hipGetDevice(&g->device));
        SRK_TRYHIP(hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking));
        hipStream_t st = g->stream;
        SRK_TRY(device_alloc((void **)&g->nodes, sizeof(uint2) * (size_t)n, &g->bytes));
        // E, node_of and the packed rows in one piece (a free of its own for each
        // took 0.3 ms at n = 300,007); a graph that leaves no room for the packed
        // rows does without them
        int32_t obits = pack_bits(g->m_slots);
        int64_t hubs = 0;
        const uint32_t most = 0xffffffffu >> obits;
        if (obits && (uint32_t)max_deg >= most)
            for (int32_t v = 0; v < n; ++v) hubs += (uint32_t)in_off[v + 1] - (uint32_t)in_off[v] >= most;
        if (hubs > (int64_t)HUB_CAP) obits = 0;   // (before memory is taken that nothing would read)
        const size_t sE = align256(sizeof(uint2) * (size_t)g->m_slots);
        const size_t s4 = align256(sizeof(uint32_t) * (size_t)g->m_slots);
        const size_t packed = obits ? s4 + sizeof(uint2) * (size_t)hubs : 0;
        rc = device_alloc((void **)&g->E, sE + s4 + packed, &g->bytes);
        const bool pack = packed && rc == SIMRANK_OK;
        if (packed && !pack) {
            clear_error();
            rc = device_alloc((void **)&g->E, sE + s4, &g->bytes);
        }
        SRK_TRY(rc);
        g->node_of = (uint32_t *)((char *)g->E + sE);
        if (pack) {
            g->E4 = (uint32_t *)((char *)g->node_of + s4);
            g->hubs = (uint2 *)((char *)g->E4 + s4);
        }
        SRK_TRY(device_alloc((void **)&g->active, sizeof(int32_t) * (size_t)(n_active ? n_active : 1),
                             &g->bytes));
        SRK_TRY(device_alloc((void **)&g->dbar, sizeof(uint32_t) * (size_t)n, &g->bytes));
        SRK_TRY(device_alloc((void **)&d_off, sizeof(int32_t) * (size_t)(n + 1), nullptr));
        SRK_TRY(device_alloc((void **)&d_src, sizeof(int32_t) * (size_t)(m ? m : 1), nullptr));
        SRK_TRY(device_alloc((void **)&d_slots, sizeof(uint32_t) * (size_t)n, nullptr));
        SRK_TRY(device_alloc((void **)&d_has, sizeof(uint32_t) * (size_t)n, nullptr));
        SRK_TRY(device_alloc((void **)&d_o, sizeof(int64_t) * (size_t)n, nullptr));
        SRK_TRY(device_alloc((void **)&d_apos, sizeof(int64_t) * (size_t)n, nullptr));
        // totals, first bad edge, hubs
        SRK_TRY(device_alloc((void **)&d_tot, sizeof(int64_t) * 4, nullptr));
        const PackArgs pk{g->E4, (uint32_t)obits, g->hubs, d_slots, (unsigned long long *)(d_tot + 3)};
        SRK_TRYHIP(hipMemcpyAsync(d_off, in_off, sizeof(int32_t) * (size_t)(n + 1),
                                  hipMemcpyHostToDevice, st));
        k_slot_counts<<<grid_for(n, 256), 256, 0, st>>>(d_off, n, d_slots, d_has);
        SRK_TRY(scan_exclusive_u32_to_i64(d_slots, n, d_o, d_tot, st));
        SRK_TRY(scan_exclusive_u32_to_i64(d_has, n, d_apos, d_tot + 1, st));
        k_fill_u32<<<1024, 256, 0, st>>>(g->node_of, g->m_slots, NIL);
        k_fill_u32<<<1, 64, 0, st>>>((uint32_t *)(d_tot + 2), 4, NIL);
        k_fill_u32<<<1024, 256, 0, st>>>(g->dbar, n, 0u);
        k_nodes<<<grid_for(n, 256), 256, 0, st>>>(d_off, d_o, n, d_apos, g->nodes, g->E, g->node_of,
                                                   g->active, pk);
        if (m) {
            SRK_TRYHIP(hipMemcpyAsync(d_src, in_src, sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice, st));
            const int items = m <= EDGE_FEW ? 4 : 16;
            const auto kernel = m <= EDGE_FEW ? k_edges<4> : k_edges<16>;
            kernel<<<grid_for(m, EDGE_BLOCK * items), EDGE_BLOCK, 0, st>>>(
                d_off, d_src, n, m, g->nodes, g->E, g->dbar, (unsigned long long *)(d_tot + 2), pk);
        }
        SRK_TRYHIP(hipGetLastError());
        int64_t tot[4];
        SRK_TRYHIP(hipMemcpyAsync(tot, d_tot, sizeof(tot), hipMemcpyDeviceToHost, st));
        SRK_TRYHIP(hipStreamSynchronize(st));
        if (tot[2] != -1) {
            rc = bad_source(tot[2]);
            goto bad;
        }
        if (tot[0] != g->m_slots || tot[1] != n_active) {
            rc = fail(SIMRANK_EDEVICE, "ingest totals disagree with the host count");
            goto bad;
        }
        if (pack) {
            if (tot[3] + 1 != hubs) {
                rc = fail(SIMRANK_EDEVICE, "ingest hubs disagree with the host count");
                goto bad;
            }
            g->obits = obits;
            g->n_hubs = (int32_t)hubs;
        }
    }
    device_free(d_off); device_free(d_src); device_free(d_slots); device_free(d_has);
    device_free(d_o); device_free(d_apos); device_free(d_tot);
    *g_out = g;
    return SIMRANK_OK;
bad:
    device_free(d_off); device_free(d_src); device_free(d_slots); device_free(d_has);
    device_free(d_o); device_free(d_apos); device_free(d_tot);
    graph_release(g);
    return rc;
#undef SRK_TRY
#undef SRK_TRYHIP
}

extern "C" int simrank_free_graph(simrank_graph *g) {
    clear_error();
    if (!g) return SIMRANK_OK;
    (void)hipSetDevice(g->device);
    if (g->stream) (void)hipStreamSynchronize(g->stream);
    graph_release(g);
    return SIMRANK_OK;
}

extern "C" int simrank_graph_info(const simrank_graph *g, int32_t *n, int64_t *m,
                                  int32_t *n_active, int64_t *device_bytes) {
    clear_error();
    if (!g) return fail(SIMRANK_EINVAL, "graph is NULL");
    if (n) *n = g->n;
    if (m) *m = g->m;
    if (n_active) *n_active = g->n_active;
    if (device_bytes) *device_bytes = g->bytes + (g->index ? g->index->bytes : 0);
    return SIMRANK_OK;
}
