// A5 -- compliant-path existence and hop distance: breadth-first search
// restricted to the switches whose jurisdiction an intent allows.
//
// The paper's path scheduler searches the live topology for a
// constraint-respecting path (weighted Dijkstra with a BFS fallback;
// Network orchestration); as a validator check the question is whether a
// path exists that never leaves the allowed jurisdictions, and how long the
// shortest one is.  Vertex v is allowed for query q iff bit region[v] of
// allowed[q] is set; distances are hop counts in the allowed-induced
// subgraph, -1 when unreachable or when the source is not allowed.
//
// Design (gfx950):
//   bitset : graphs that fit in LDS (27 bytes per vertex): 64 queries per
//            workgroup, one bit each, level-synchronous frontier bitsets
//            (visited / frontier / next) in LDS, push expansion of a
//            compacted frontier list (a few lanes per vertex, coalesced
//            adjacency reads) with 64-bit LDS atomic OR, the per-query
//            allowed mask applied per vertex as a precomputed 64-bit region
//            mask; stops when every query's target is resolved or no
//            frontier bit is left.  The per-vertex words sit in XOR-swizzled
//            slots: vertices 16 apart map to different LDS banks (unswizzled,
//            a fat-tree core's pushes to its per-pod peers, 48 apart, all
//            hit one bank pair).
//   map    : larger graphs whose visited bits fit in LDS (1.2 million
//            vertices): one workgroup per query.  Narrow frontiers, which a
//            sparse graph has for hundreds of levels, are one wavefront's work
//            without barriers, one memory latency per level: a vertex's first
//            16 neighbours and their regions sit in one 64-byte record.
//            Meanwhile the other wavefronts write the row's -1s.  Wide
//            frontiers take the whole workgroup.
//   queue  : still larger graphs: one workgroup per query, frontier queue in
//            scratch, the distance row itself (or a scratch row, with
//            targets) as the visited set claimed with compare-and-swap.
#include <algorithm>

#include "pc_internal.h"

namespace {

constexpr int kBitsetThreads = 1024;  // two workgroups per CU fill all 32 wave slots
constexpr int kQueueThreads = 256;
constexpr int kMaxBitsetV = 6016;  // 3 x 8 B + 1 B + 2 B per vertex, plus masks, within 160 KB of LDS
constexpr int kBitsetStatic = 1024;  // LDS of the bitset search besides these, at most

__device__ __forceinline__ bool allowed_v(const uint8_t *region, uint32_t A, int32_t v)
{
    const uint32_t r = region[v];
    return r < 32 && ((A >> r) & 1u);
}

// Is v in the forbidden list of one query (Kf entries, -1 = unused)?
__device__ __forceinline__ bool forbidden_v(const int32_t *__restrict__ fl, int32_t Kf, int32_t v)
{
    for (int32_t k = 0; k < Kf; ++k)
        if (fl[k] == v) return true;
    return false;
}

// Everything a search checks about its inputs, in one launch (a small call is
// its launches: with one kernel per check and a fill of the flag, 64 queries
// on 20 vertices took 41 us, now 24).  The data errors: regions, offsets, adjacency
// entries, sources, targets, waypoint and forbidden lists (every entry -1 or
// a vertex).  And, for a gen other than 0, the graph's symmetry: *asym becomes gen
// unless every adjacency list is sorted and every valid entry u -> v has its
// reverse v -> u (a vertex whose offsets are invalid has no entries, so no
// valid list may name it).  Then the search from v reaches u exactly when the
// search from u reaches v, at the same distance.  One wavefront per vertex, its
// lanes over the vertex's entries.  The caller numbers its calls, so that
// the flag needs no clearing.
struct Checks {
    int32_t V;
    const int32_t *adj_off, *adj;
    int64_t n_adj;
    const uint8_t *region;
    int32_t Q;
    const int32_t *src, *target;
    int64_t nv, nf;
    const int32_t *via, *forbid;
    int32_t *asym;
    int32_t gen;
    uint32_t *d_err;
};

__device__ __forceinline__ bool bad_vertices(const int32_t *__restrict__ ids, int64_t n, int32_t lowest, int32_t V,
                                             int64_t i0, int64_t stride)
{
    bool bad = false;
    for (int64_t i = i0; i < n; i += stride) bad |= ids[i] < lowest || ids[i] >= V;
    return bad;
}

__global__ __launch_bounds__(256) void k_rc_checks(Checks c)
{
    uint32_t errs = 0;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t i0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    for (int64_t v = i0; v < c.V; v += stride) {
        if (c.region[v] >= 32) errs |= PC_DERR_JUR;
        if (!pc_range_ok(c.adj_off[v], c.adj_off[v + 1], c.n_adj)) errs |= PC_DERR_OFFSETS;
    }
    if (bad_vertices(c.adj, c.n_adj, 0, c.V, i0, stride)) errs |= PC_DERR_GRAPH;
    if (bad_vertices(c.src, c.Q, 0, c.V, i0, stride) ||
        bad_vertices(c.target, c.target ? c.Q : 0, 0, c.V, i0, stride) ||
        bad_vertices(c.via, c.nv, -1, c.V, i0, stride) || bad_vertices(c.forbid, c.nf, -1, c.V, i0, stride))
        errs |= PC_DERR_SWITCH;
    if (errs) atomicOr(c.d_err, errs);
    if (c.gen == 0) return;
    const int lane = threadIdx.x & 63;
    const int32_t waves = gridDim.x * 4;
    bool bad = false;
    for (int32_t u = blockIdx.x * 4 + (threadIdx.x >> 6); u < c.V; u += waves) {
        const int64_t b = c.adj_off[u], e = c.adj_off[u + 1];
        if (!pc_range_ok(b, e, c.n_adj)) continue;
        for (int64_t p = b + lane; p < e; p += 64) {
            const int32_t v = c.adj[p];
            if (p > b && c.adj[p - 1] > v) bad = true;
            if (v < 0 || v >= c.V) continue;
            int64_t lo = c.adj_off[v], hi = c.adj_off[v + 1];
            if (!pc_range_ok(lo, hi, c.n_adj)) {
                bad = true;
                continue;
            }
            const int64_t end = hi;
            while (lo < hi) {  // first entry >= u
                const int64_t mid = (lo + hi) >> 1;
                if (c.adj[mid] < u) lo = mid + 1;
                else hi = mid;
            }
            if (lo >= end || c.adj[lo] != u) bad = true;
        }
    }
    if (__ballot(bad) && lane == 0) *c.asym = c.gen;
}

// Append v to an LDS list when `add`, one counter update per wavefront
// (every active lane of the wavefront calls this together).
__device__ __forceinline__ void wave_append(bool add, uint16_t v, int32_t *count, uint16_t *list)
{
    const uint64_t b = __ballot(add);
    if (b == 0) return;
    const int leader = __builtin_ctzll(b);
    const int lane = threadIdx.x & 63;
    int32_t base = 0;
    if (lane == leader) base = atomicAdd(count, static_cast<int32_t>(__popcll(b)));
    base = __shfl(base, leader, 64);
    if (add) {
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u));
        list[base + static_cast<int32_t>(below)] = v;
    }
}

// Queries ordered by source for the bitset search: a counting sort (the
// order among queries of one source is arbitrary; every result is per
// query).  A workgroup's 64 queries then share few sources, so their
// frontiers overlap and one push along an edge serves many of them.
// Sources outside [0, V) go to bucket V.  Counting: each workgroup ranks its
// queries within their buckets in LDS and reserves its share of every
// bucket it meets with one global atomic (a few thousand instead of one
// per query on the same few counters); pos[q] = the query's place within
// its bucket.
constexpr int kSortThreads = 1024;
constexpr int kSortPer = 4096;  // queries per counting workgroup

__global__ __launch_bounds__(kSortThreads) void k_rc_src_count(int32_t Q, const int32_t *__restrict__ src, int32_t V,
                                                               int32_t *__restrict__ cnt, int32_t *__restrict__ pos)
{
    extern __shared__ int32_t loc[];  // [V + 1] per-bucket counts, then the workgroup's bases
    for (int32_t b = threadIdx.x; b <= V; b += kSortThreads) loc[b] = 0;
    __syncthreads();
    const int32_t q0 = blockIdx.x * kSortPer;
    const int32_t q1 = min(Q, q0 + kSortPer);
    for (int32_t q = q0 + threadIdx.x; q < q1; q += kSortThreads) {
        const int32_t s = src[q];
        pos[q] = atomicAdd(loc + ((s >= 0 && s < V) ? s : V), 1);
    }
    __syncthreads();
    for (int32_t b = threadIdx.x; b <= V; b += kSortThreads) {
        const int32_t n = loc[b];
        loc[b] = n ? atomicAdd(cnt + b, n) : 0;
    }
    __syncthreads();
    for (int32_t q = q0 + threadIdx.x; q < q1; q += kSortThreads) {
        const int32_t s = src[q];
        pos[q] += loc[(s >= 0 && s < V) ? s : V];
    }
}

__global__ void k_rc_src_place(int32_t Q, const int32_t *__restrict__ src, int32_t V, const int32_t *__restrict__ off,
                               const int32_t *__restrict__ pos, int32_t *__restrict__ perm)
{
    for (int32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < Q; q += gridDim.x * blockDim.x) {
        const int32_t s = src[q];
        perm[off[(s >= 0 && s < V) ? s : V] + pos[q]] = q;
    }
}

// Leg k of query q (k <= m, m = waypoints before the first -1) runs from the
// previous waypoint (or src) to the next one (or target); legs past m are
// inactive (-1 to -1).  On a symmetric graph (flip) legs 0, 2, 4, ... are
// searched from their far end, so that legs 2j and 2j + 1 start at the same
// waypoint and share their frontiers in the workgroup's bitsets.
struct Leg {
    int32_t from, to;
    bool last;  // the walk ends with it
};

__device__ __forceinline__ Leg leg_of(const int32_t *__restrict__ src, const int32_t *__restrict__ target,
                                      const int32_t *__restrict__ w, int32_t Kv, int32_t q, int32_t k, bool flip)
{
    int32_t from = src[q];
    for (int32_t i = 0; i < k; ++i) {
        from = w[i];
        if (from == -1) return {-1, -1, true};
    }
    const int32_t nxt = k < Kv ? w[k] : -1;
    const int32_t to = nxt == -1 ? target[q] : nxt;
    return flip && (k & 1) == 0 ? Leg{to, from, nxt == -1} : Leg{from, to, nxt == -1};
}

// Sum of the distances of a walk's legs up to the last, -1 if any is
// unreachable (saturating at INT32_MAX).
struct WalkLength {
    int64_t total = 0;
    bool open = true;
    __device__ __forceinline__ void add(int32_t d, bool last)
    {
        if (!open) return;
        total = d < 0 ? -1 : total + d;
        open = d >= 0 && !last;
    }
    __device__ __forceinline__ int32_t length() const
    {
        return static_cast<int32_t>(total > 0x7FFFFFFF ? 0x7FFFFFFF : total);
    }
};

// 64 queries per workgroup; dist is [Q][V] (target == nullptr) or [Q].
// Each level pushes the frontier along its edges: the frontier vertices are
// kept as a list in LDS and GS lanes share one vertex's adjacency, so the
// adjacency loads are coalesced and the vertex's frontier word is a
// broadcast; the next frontier is built (and the list rewritten) in one
// pass over the vertices.
// kLegs: a query is Kv + 1 legs of one walk (leg_of), a workgroup takes as
// many whole queries as fit 64 legs, and dist[q] is the walk's length.
template <int GS, bool kLegs>
__global__ __launch_bounds__(kBitsetThreads) void k_rc_bitset(int32_t V, const int32_t *__restrict__ adj_off,
                                                              const int32_t *__restrict__ adj, int64_t n_adj,
                                                              const uint8_t *__restrict__ region, int32_t Q,
                                                              const int32_t *__restrict__ src,
                                                              const uint32_t *__restrict__ allowed,
                                                              const int32_t *__restrict__ target,
                                                              int32_t *__restrict__ dist,
                                                              const int32_t *__restrict__ forbid, int32_t Kf,
                                                              int32_t qdiv, const int32_t *__restrict__ asym,
                                                              int32_t gen, const int32_t *__restrict__ perm,
                                                              const int32_t *__restrict__ via, int32_t Kv)
{
    extern __shared__ uint64_t lds[];
    // visited / frontier / next words of vertex v sit in slot sl(v) =
    // v ^ ((v >> 4) & 15), a permutation of each block of 16, so that
    // vertices a multiple of 16 apart (a core switch's aggregation peers,
    // one per pod) fall in different LDS banks; Vp slots each
    const int32_t Vp = (V + 15) & ~15;
    auto sl = [](int32_t v) { return v ^ ((v >> 4) & 15); };
    uint64_t *vis = lds;
    uint64_t *fr = vis + Vp;
    uint64_t *nx = fr + Vp;
    uint64_t *rmask = nx + Vp;                                              // [32]
    uint8_t *reg = reinterpret_cast<uint8_t *>(rmask + 32);                 // [V]
    uint16_t *flist = reinterpret_cast<uint16_t *>(reg + ((V + 3) & ~3));  // [V] frontier vertices
    __shared__ int32_t nfr[2];                                              // list lengths, by level parity
    __shared__ int flag_done;
    // target look-ahead: each query's target's adjacency list
    __shared__ int32_t tbeg[64], tdeg[64];
    __shared__ unsigned long long found, act;
    // queries still searching (target mode): resolved queries' frontier
    // bits are dropped, so their searches stop spreading
    __shared__ unsigned long long live;
    // query of bit k: qid[k] (queries taken in perm order when given)
    __shared__ int32_t qid[64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t legs = kLegs ? Kv + 1 : 1;
    const int32_t per = 64 / legs;  // queries of this workgroup
    const int32_t q0 = blockIdx.x * per;
    const int32_t nq = min(per, Q - q0) * legs;
    if (tid < 64) qid[lane] = lane < nq ? (perm ? perm[q0 + lane] : q0 + lane / legs) : 0;
    for (int32_t v = tid; v < Vp; v += kBitsetThreads) {
        vis[v] = 0;
        fr[v] = 0;
        nx[v] = 0;
        if (v < V) reg[v] = region[v];
    }
    if (tid < 64) {
        const uint32_t A = lane < nq ? allowed[qid[lane] / qdiv] : 0u;
        for (int r = 0; r < 32; ++r) {
            const uint64_t m = __ballot((A >> r) & 1u);
            if (lane == 0) rmask[r] = m;
        }
    }
    if (tid == 0) nfr[0] = nfr[1] = 0;
    __syncthreads();
    // forbidden vertices start out visited, so they are never entered
    if (Kf > 0) {
        if (tid < 64 && lane < nq) {
            const int32_t *fl = forbid + static_cast<int64_t>(qid[lane] / qdiv) * Kf;
            for (int32_t k = 0; k < Kf; ++k) {
                const int32_t f = fl[k];
                if (f >= 0 && f < V) atomicOr(reinterpret_cast<unsigned long long *>(&vis[sl(f)]), 1ull << lane);
            }
        }
        __syncthreads();
    }
    // sources; per-query result state lives in wave 0, lane = query
    int32_t res = -1, tgt = -1;
    bool done = true, last = true;
    if (tid < 64 && lane < nq) {
        const int32_t q = qid[lane];
        int32_t s;
        if (kLegs) {
            const Leg leg = leg_of(src, target, via + static_cast<int64_t>(q) * Kv, Kv, q, lane % legs, *asym != gen);
            s = leg.from;
            tgt = leg.to;
            last = leg.last;
        } else {
            s = src[q];
        }
        const bool s_ok = s >= 0 && s < V && allowed_v(reg, allowed[q / qdiv], s) && !((vis[sl(s)] >> lane) & 1);
        if (target) {
            // a target that is not allowed, or forbidden, is never reached:
            // the query is resolved (-1) without a search
            if (!kLegs) tgt = target[q];
            done = !(s_ok && tgt >= 0 && tgt < V && allowed_v(reg, allowed[q / qdiv], tgt) &&
                     !((vis[sl(tgt)] >> lane) & 1));
        }
        if (s_ok) {
            atomicOr(reinterpret_cast<unsigned long long *>(&fr[sl(s)]), 1ull << lane);
            atomicOr(reinterpret_cast<unsigned long long *>(&vis[sl(s)]), 1ull << lane);
            if (!target) dist[static_cast<int64_t>(q) * V + s] = 0;
        }
    }
    __syncthreads();
    for (int32_t v = tid; v < V; v += kBitsetThreads)
        wave_append(fr[sl(v)] != 0, static_cast<uint16_t>(v), &nfr[0], flist);
    if (tid < 64) {
        if (!done && ((vis[sl(tgt)] >> lane) & 1)) {
            res = 0;
            done = true;
        }
        // A query whose target is allowed and has a neighbour in its
        // frontier at distance d is resolved at d + 1 without expanding
        // that frontier: list each such target's adjacency once.  Only on
        // a symmetric graph (*asym != gen), where the target's list names
        // exactly the vertices whose lists name the target.
        int32_t deg = 0, b = 0;
        bool t_allowed = false;
        if (target && !done && *asym != gen) {
            const int64_t b64 = adj_off[tgt], e64 = adj_off[tgt + 1];
            t_allowed = allowed_v(reg, allowed[qid[lane] / qdiv], tgt);
            if (t_allowed && pc_range_ok(b64, e64, n_adj)) {
                b = static_cast<int32_t>(b64);
                deg = static_cast<int32_t>(e64 - b64);
            }
        }
        tbeg[lane] = b;
        tdeg[lane] = deg;
        const uint64_t a = __ballot(deg > 0);
        if (lane == 0) act = a;
        const uint64_t lv = target ? __ballot(!done) : ~0ull;
        if (lane == 0) live = lv;
    }
    __syncthreads();
    // the look-ahead has kAheadLanes lanes per query, each with two of its
    // target's neighbours in registers (a search for the query of every list entry
    // at every level: 174,763 queries on 2,880
    // switches 654 us, now 520; 200 queries there 38, now 32)
    constexpr int kAheadLanes = kBitsetThreads / 64;
    const int aq = tid / kAheadLanes, al = tid % kAheadLanes;
    const int32_t a_beg = target ? tbeg[aq] : 0, a_deg = target ? tdeg[aq] : 0;
    auto neighbour = [&](int32_t k) {
        const int32_t u = k < a_deg ? adj[a_beg + k] : -1;
        return u >= 0 && u < V ? sl(u) : -1;
    };
    const int32_t near0 = neighbour(al), near1 = neighbour(al + kAheadLanes);
    const int grp = tid / GS, gl = tid % GS;
    constexpr int kNG = kBitsetThreads / GS;  // groups
    for (int32_t d = 1;; ++d) {
        const int cur = (d - 1) & 1;
        const int32_t nf = nfr[cur];
        if (tid == 0) nfr[cur ^ 1] = 0;  // last read at the start of the previous level
        // A group takes GS frontier entries at a time: lane k loads entry k's
        // adjacency range and frontier word in one round (no dependent load
        // chain per vertex), then the group walks the GS entries, taking
        // each range and word from lane k by shuffle.
        for (int32_t i0 = grp; i0 < nf; i0 += kNG * GS) {
            const int32_t my = i0 + kNG * gl;
            int32_t b = 0, e = 0;
            uint32_t flo = 0, fhi = 0;
            if (my < nf) {
                const int32_t u = flist[my];
                const int64_t b64 = adj_off[u], e64 = adj_off[u + 1];
                if (pc_range_ok(b64, e64, n_adj)) {
                    b = static_cast<int32_t>(b64);
                    e = static_cast<int32_t>(e64);
                    const uint64_t f = fr[sl(u)];
                    flo = static_cast<uint32_t>(f);
                    fhi = static_cast<uint32_t>(f >> 32);
                }
            }
            const int32_t nk = min(GS, (nf - i0 + kNG - 1) / kNG);
            for (int k = 0; k < nk; ++k) {
                const int32_t bk = __shfl(b, k, GS), ek = __shfl(e, k, GS);
                const uint64_t fk = static_cast<uint64_t>(static_cast<uint32_t>(__shfl(fhi, k, GS))) << 32 |
                                    static_cast<uint32_t>(__shfl(flo, k, GS));
                for (int32_t p = bk + gl; p < ek; p += GS) {
                    const int32_t v = adj[p];
                    if (v >= 0 && v < V) atomicOr(reinterpret_cast<unsigned long long *>(&nx[sl(v)]), fk);
                }
            }
        }
        __syncthreads();
        for (int32_t v = tid; v < V; v += kBitsetThreads) {
            const int32_t x = sl(v);
            uint64_t n = nx[x];
            if (n) {
                nx[x] = 0;
                const uint32_t r = reg[v];
                n &= (r < 32 ? rmask[r] : 0ull) & ~vis[x] & live;
                vis[x] |= n;
                if (!target) {
                    uint64_t m = n;
                    while (m) {
                        const int q = __builtin_ctzll(m);
                        m &= m - 1;
                        dist[static_cast<int64_t>(qid[q]) * V + v] = d;
                    }
                }
            }
            fr[x] = n;
            wave_append(n != 0, static_cast<uint16_t>(v), &nfr[cur ^ 1], flist);
        }
        if (tid == 0) found = 0;
        __syncthreads();
        if (target) {
            if ((act >> aq) & 1) {
                uint64_t hit = (near0 >= 0 ? fr[near0] : 0) | (near1 >= 0 ? fr[near1] : 0);
                for (int32_t k = al + 2 * kAheadLanes; k < a_deg; k += kAheadLanes) {
                    const int32_t u = neighbour(k);
                    hit |= u >= 0 ? fr[u] : 0;
                }
                if ((hit >> aq) & 1) atomicOr(&found, 1ull << aq);
            }
            __syncthreads();
        }
        if (tid < 64) {
            if (!done && ((fr[sl(tgt)] >> lane) & 1)) {
                res = d;
                done = true;
            } else if (!done && target && ((found >> lane) & 1)) {
                res = d + 1;
                done = true;
            }
            const uint64_t still = __ballot(!done);
            if (tid == 0) {
                flag_done = target ? still == 0 : 0;
                act &= still;
                if (target) live = still;
            }
        }
        __syncthreads();
        // nfr[cur ^ 1] is reset only two levels on; flag_done is rewritten
        // only after the next level's second barrier
        if (nfr[cur ^ 1] == 0 || flag_done) break;
    }
    if (kLegs) {
        if (tid < 64) {
            WalkLength w;
            for (int32_t k = 0; k < legs; ++k) w.add(__shfl(res, (lane + k) & 63, 64), __shfl(last, (lane + k) & 63, 64));
            if (lane < nq && lane % legs == 0) dist[qid[lane]] = w.length();
        }
    } else if (target && tid < 64 && lane < nq) {
        dist[qid[lane]] = res;
    }
}

// Neighbour records for the map search: word j of a vertex's 64 bytes is
// its j-th neighbour and that neighbour's region (vertex | region << 26; kHole
// where there is none, or none that any query may enter).  A vertex of more
// than kEll entries has kUseLists in word 0.
constexpr int kEll = 16;
constexpr int kVertexBits = 26;
constexpr uint32_t kHole = 0xFFFFFFFFu, kUseLists = 0xFFFFFFFEu;

__global__ __launch_bounds__(256) void k_rc_records(int32_t V, const int32_t *__restrict__ adj_off,
                                                    const int32_t *__restrict__ adj, int64_t n_adj,
                                                    const uint8_t *__restrict__ region, uint32_t *__restrict__ ell)
{
    // four lanes per vertex, four words each
    const int64_t x = blockIdx.x * 256ll + threadIdx.x;
    const int32_t v = static_cast<int32_t>(x / 4), j0 = static_cast<int32_t>(x % 4) * 4;
    if (v >= V) return;
    const int64_t b = adj_off[v], e = adj_off[v + 1];
    uint32_t r[4] = {kHole, kHole, kHole, kHole};
    if (pc_range_ok(b, e, n_adj)) {
        if (e - b > kEll) {
            if (j0 == 0) r[0] = kUseLists;
        } else {
            int32_t u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = b + j0 + k < e ? adj[b + j0 + k] : -1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t g = u[k] >= 0 && u[k] < V ? region[u[k]] : 32u;
                if (g < 32) r[k] = static_cast<uint32_t>(u[k]) | g << kVertexBits;
            }
        }
    }
    reinterpret_cast<uint4 *>(ell)[x] = make_uint4(r[0], r[1], r[2], r[3]);
}

// One workgroup per query (grid-stride over queries).  LDS: a visited bit
// per vertex (forbidden vertices start out visited).  list: every visited
// vertex of the query in BFS order, so a level is a range of it.
// While wavefront 0 walks the first levels, whose vertices it only lists
// (and the levels' starts), the others fill the row with -1; then the listed
// vertices get their distances.  After that a frontier of at most kNarrow
// vertices is again wavefront 0's, from an LDS copy, and a wider one takes a
// barrier per level.
// GS lanes share a vertex: with the records (kRecords) four, each reading 16 bytes.
// Bound by the deepest query's levels, one record latency each, and by
// the -1 fill: 256 rows of a million vertices (mean degree 4, deepest search
// 196 levels) in 325 us, the -1s alone about 200 us; the queue search took
// 1,210 us after a fill of 207 us.  At mean degree 6 (one component, 1,800
// levels) 8.4 ms against 39 ms; 8,191 vertices of mean degree 60, 256 rows
// 0.28 ms against 2.0 ms.
constexpr int kMapThreads = 1024;
constexpr int kNarrow = 256;
// Vertices of more than kHubDegree entries wait, up to kHubs at a time, for the whole
// workgroup (5,000 vertices joined to four of them: one query with a target 132 us with
// a hub's entries by the wavefront that takes its level, 27 so; 1,000 rows 812 and 155).
// Marked as unlikely, which keeps it out of the way of graphs without (256 rows of a
// million vertices 392 us in line, 389 so and without it).
constexpr int kHubs = 64;
constexpr int kHubDegree = 256;
constexpr int kDeferred = 1023 - kHubs;    // levels walked at most while the row is filled
template <int GS, bool kRecords>
__global__ __launch_bounds__(kMapThreads) void k_rc_map(int32_t V, const int32_t *__restrict__ adj_off,
                                                        const int32_t *__restrict__ adj, int64_t n_adj,
                                                        const uint8_t *__restrict__ region,
                                                        const uint32_t *__restrict__ ell, int32_t Q,
                                                        const int32_t *__restrict__ src,
                                                        const uint32_t *__restrict__ allowed,
                                                        const int32_t *__restrict__ target, int32_t *__restrict__ dist,
                                                        int32_t *__restrict__ list_all,
                                                        const int32_t *__restrict__ forbid, int32_t Kf, int32_t qdiv)
{
    static_assert(!kRecords || GS == 4, "four lanes read a record");
    extern __shared__ uint4 map_lds[];
    uint32_t *bm = reinterpret_cast<uint32_t *>(map_lds);  // [ceil(V / 128) * 4]
    __shared__ int32_t near_q[2][kNarrow];  // a narrow frontier and the next one
    __shared__ int32_t starts[kDeferred + 1];
    __shared__ int32_t hubs[kHubs];  // with their entries not yet looked at
    __shared__ int32_t s_lo, s_hi, s_d, s_tail, s_hubs;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool rows = target == nullptr;
    int32_t *list = list_all + static_cast<int64_t>(blockIdx.x) * V;
    auto bit = [&](int32_t v) { return (bm[v >> 5] >> (v & 31)) & 1u; };
    auto rank_in = [](uint64_t m) {
        return static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
            static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
    };
    for (int32_t q = blockIdx.x; q < Q; q += gridDim.x) {
        int32_t *row = rows ? dist + static_cast<int64_t>(q) * V : nullptr;
        const uint32_t A = allowed[q / qdiv];
        const int32_t s = src[q];
        const int32_t tgt = rows ? -1 : target[q];
        for (int32_t i = tid; i < (V + 127) / 128; i += kMapThreads) map_lds[i] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        if (tid < Kf) {
            const int32_t f = forbid[static_cast<int64_t>(q / qdiv) * Kf + tid];
            if (f >= 0 && f < V) atomicOr(&bm[f >> 5], 1u << (f & 31));
        }
        __syncthreads();
        // a target that is not allowed, or forbidden, is never reached
        const bool go = s >= 0 && s < V && allowed_v(region, A, s) && !bit(s) &&
                        (rows || (tgt >= 0 && tgt < V && allowed_v(region, A, tgt) && !bit(tgt)));
        __syncthreads();
        if (tid == 0) {
            s_lo = 0;
            s_hi = go ? 1 : 0;
            s_d = 0;
            s_hubs = 0;
            starts[0] = 0;
            if (go) {
                list[0] = s;
                near_q[0][0] = s;
                atomicOr(&bm[s >> 5], 1u << (s & 31));
            }
        }
        __syncthreads();
        // Narrow levels, by wavefront 0: the frontier in near_q[0], ids
        // list[lo .. hi).  Ends with the frontier empty, too wide, the target
        // reached, (deferred) kDeferred levels behind it, or hubs among the
        // last level's vertices.
        auto narrow = [&](bool deferred) {
            int32_t lo = s_lo, hi = s_hi, d = s_d, cur = 0, nh = 0;
            while (hi > lo && hi - lo <= kNarrow && !(deferred && d >= kDeferred) && !(!rows && bit(tgt))) {
                const int32_t n = hi - lo;
                int32_t *nq = near_q[cur ^ 1];
                int32_t nn = 0;
                auto claim = [&](uint32_t r) {
                    const bool ok = !(r >> 31) && ((A >> (r >> kVertexBits)) & 1u);
                    const uint32_t u = r & ((1u << kVertexBits) - 1);
                    if (!__ballot(ok)) return;
                    bool fresh = false;
                    if (ok) fresh = !((atomicOr(&bm[u >> 5], 1u << (u & 31)) >> (u & 31)) & 1u);
                    const uint64_t m = __ballot(fresh);
                    if (fresh) {
                        const int32_t pos = nn + rank_in(m);
                        list[hi + pos] = static_cast<int32_t>(u);
                        if (pos < kNarrow) nq[pos] = static_cast<int32_t>(u);
                        if (rows && !deferred) row[u] = d + 1;
                    }
                    nn += static_cast<int32_t>(__popcll(m));
                };
                constexpr int kSteps = 4;  // 16 vertices each, their records in flight together
                for (int32_t i0 = 0; i0 < n; i0 += 16 * kSteps) {
                    uint4 R[kSteps];
                    int32_t v[kSteps];
#pragma unroll
                    for (int k = 0; k < kSteps; ++k) {
                        const int32_t i = i0 + 16 * k + lane / 4;
                        v[k] = i < n ? near_q[cur][i] : -1;
                        R[k] = make_uint4(kHole, kHole, kHole, kHole);
                        if (v[k] >= 0) R[k] = reinterpret_cast<const uint4 *>(ell)[static_cast<int64_t>(v[k]) * 4 + (lane & 3)];
                    }
#pragma unroll
                    for (int k = 0; k < kSteps; ++k) {
                        if (i0 + 16 * k >= n) break;
                        uint64_t big = __ballot((lane & 3) == 0 && R[k].x == kUseLists);
                        claim(R[k].x);
                        claim(R[k].y);
                        claim(R[k].z);
                        claim(R[k].w);
                        while (__builtin_expect(big != 0, 0)) {  // a vertex of many entries: its list, across the wavefront
                            const int32_t w = __builtin_amdgcn_readlane(v[k], static_cast<int>(__builtin_ctzll(big)));
                            big &= big - 1;
                            const int64_t e = adj_off[w + 1];
                            int64_t p = adj_off[w];
                            if (__builtin_expect(e - p > kHubDegree && nh < kHubs, 0)) {
                                if (lane == 0) hubs[nh] = w;
                                ++nh;
                                continue;
                            }
                            for (; p < e; p += 64) {
                                const int32_t u = p + lane < e ? adj[p + lane] : -1;
                                const uint32_t g = u >= 0 && u < V ? region[u] : 32u;
                                claim(g < 32 ? static_cast<uint32_t>(u) | g << kVertexBits : kHole);
                            }
                        }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                lo = hi;
                hi += nn;
                ++d;
                if (deferred && lane == 0) starts[d] = lo;
                if (nh) break;
                cur ^= 1;
            }
            if (lane == 0) {
                s_lo = lo;
                s_hi = hi;
                s_d = d;
                s_hubs = nh;
            }
        };
        // the whole workgroup's: r's vertex is on level d unless it was reached before
        auto claim_wide = [&](uint32_t r, int32_t d) {
            const bool ok = !(r >> 31) && ((A >> (r >> kVertexBits)) & 1u);
            const uint32_t u = r & ((1u << kVertexBits) - 1);
            if (!__ballot(ok)) return;
            bool fresh = false;
            if (ok && !bit(static_cast<int32_t>(u)))
                fresh = !((atomicOr(&bm[u >> 5], 1u << (u & 31)) >> (u & 31)) & 1u);
            const uint64_t m = __ballot(fresh);
            if (!m) return;
            const int lead = static_cast<int>(__builtin_ctzll(m));
            int32_t at = 0;
            if (lane == lead) at = atomicAdd(&s_tail, static_cast<int32_t>(__popcll(m)));
            at = __builtin_amdgcn_readlane(at, lead);
            if (fresh) {
                list[at + rank_in(m)] = static_cast<int32_t>(u);
                if (rows) row[u] = d;
            }
        };
        // the waiting hubs' neighbours, on level d (between barriers)
        auto expand_hubs = [&](int32_t n, int32_t d) {
            for (int32_t h = 0; h < min(n, kHubs); ++h) {
                const int32_t w = hubs[h];
                const int64_t e = adj_off[w + 1];
                for (int64_t p = adj_off[w] + wave * 64; p < e; p += kMapThreads) {
                    const int32_t u = p + lane < e ? adj[p + lane] : -1;
                    const uint32_t g = u >= 0 && u < V ? region[u] : 32u;
                    claim_wide(g < 32 ? static_cast<uint32_t>(u) | g << kVertexBits : kHole, d);
                }
            }
        };
        auto fill = [&](int32_t first, int32_t step) {  // -1 over the row: 16-byte stores between its unaligned ends
            const int32_t head = min(V, static_cast<int32_t>((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15) / 4);
            const int32_t quads = (V - head) / 4;
            typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
            i32x4 *body = reinterpret_cast<i32x4 *>(row + head);
            // (non-temporal: the records stay in L2, 389 -> 325 us at a million vertices)
            for (int32_t i = first; i < quads; i += step) __builtin_nontemporal_store(i32x4{-1, -1, -1, -1}, body + i);
            for (int32_t i = first; i < head; i += step) row[i] = -1;
            for (int32_t i = head + quads * 4 + first; i < V; i += step) row[i] = -1;
        };
        if (rows) {
            if (!kRecords) fill(tid, kMapThreads);
            else if (wave == 0) narrow(true);
            else fill(tid - 64, kMapThreads - 64);
            __syncthreads();
            const int32_t hi = s_hi, d_end = s_d;
            for (int32_t i = tid; i < hi; i += kMapThreads) {  // level of entry i: the last d with starts[d] <= i
                int32_t a = 0, b = d_end + 1;
                while (b - a > 1) {
                    const int32_t mid = (a + b) >> 1;
                    if (starts[mid] <= i) a = mid;
                    else b = mid;
                }
                row[list[i]] = a;
            }
            __syncthreads();
        }
        while (true) {
            const int32_t lo = s_lo, d = s_d, waiting = kRecords ? s_hubs : 0;
            int32_t hi = s_hi;
            if (__builtin_expect(waiting != 0, 0)) {  // left by narrow()
                if (tid == 0) s_tail = hi;
                __syncthreads();
                expand_hubs(waiting, d);
                __syncthreads();
                hi = s_tail;
                if (tid == 0) {
                    s_hi = hi;
                    s_hubs = 0;
                }
            }
            if (hi <= lo || (!rows && bit(tgt))) break;
            __syncthreads();
            if (kRecords && hi - lo <= kNarrow / 2) {
                if (wave == 0) {
                    for (int32_t i = lane; i < hi - lo; i += 64) near_q[0][i] = list[lo + i];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    narrow(false);
                }
                __syncthreads();
                continue;
            }
            if (tid == 0) s_tail = hi;
            __syncthreads();
            constexpr int kPerWave = 64 / GS;
            for (int32_t i0 = lo + wave * kPerWave; i0 < hi; i0 += kMapThreads / GS) {
                const int32_t i = i0 + lane / GS;
                const int32_t w = i < hi ? list[i] : -1;
                bool lists = !kRecords && w >= 0;
                if constexpr (kRecords) {
                    uint4 R = make_uint4(kHole, kHole, kHole, kHole);
                    if (w >= 0) R = reinterpret_cast<const uint4 *>(ell)[static_cast<int64_t>(w) * 4 + (lane & 3)];
                    lists = __shfl(R.x == kUseLists ? 1 : 0, lane & ~3, 64) != 0;
                    claim_wide(R.x, d + 1);
                    claim_wide(R.y, d + 1);
                    claim_wide(R.z, d + 1);
                    claim_wide(R.w, d + 1);
                }
                int64_t p = 0, e = 0;
                if (lists) {
                    p = adj_off[w];
                    e = adj_off[w + 1];
                    if (!pc_range_ok(p, e, n_adj)) e = p;
                }
                if (kRecords && __ballot(e - p > kHubDegree)) {
                    int32_t at = kHubs;
                    if (e - p > kHubDegree && (lane & 3) == 0) at = atomicAdd(&s_hubs, 1);
                    if (at < kHubs) hubs[at] = w;
                    if (__shfl(at, lane & ~3, 64) < kHubs) e = p;  // (all four lanes')
                }
                for (p += lane % GS; __ballot(p < e); p += GS) {
                    const int32_t u = p < e ? adj[p] : -1;
                    const uint32_t g = u >= 0 && u < V ? region[u] : 32u;
                    claim_wide(g < 32 ? static_cast<uint32_t>(u) | g << kVertexBits : kHole, d + 1);
                }
            }
            __syncthreads();
            if (kRecords) {
                const int32_t found = s_hubs;
                if (found) {
                    expand_hubs(found, d + 1);
                    __syncthreads();
                }
            }
            if (tid == 0) {
                s_lo = hi;
                s_hi = s_tail;
                s_d = d + 1;
                s_hubs = 0;
            }
            __syncthreads();
        }
        if (!rows && tid == 0) dist[q] = go && bit(tgt) ? s_d : -1;
        __syncthreads();
    }
}

// One workgroup per query (grid-stride over queries).
__global__ __launch_bounds__(kQueueThreads) void k_rc_queue(int32_t V, const int32_t *__restrict__ adj_off,
                                                            const int32_t *__restrict__ adj, int64_t n_adj,
                                                            const uint8_t *__restrict__ region, int32_t Q,
                                                            const int32_t *__restrict__ src,
                                                            const uint32_t *__restrict__ allowed,
                                                            const int32_t *__restrict__ target,
                                                            int32_t *__restrict__ dist, int32_t *__restrict__ qbuf_all,
                                                            int32_t *__restrict__ rows_all,
                                                            const int32_t *__restrict__ forbid, int32_t Kf,
                                                            int32_t qdiv)
{
    __shared__ int32_t tail_s;
    const int tid = threadIdx.x;
    int32_t *qbuf = qbuf_all + static_cast<int64_t>(blockIdx.x) * V;
    for (int32_t q = blockIdx.x; q < Q; q += gridDim.x) {
        int32_t *drow = target ? rows_all + static_cast<int64_t>(blockIdx.x) * V : dist + static_cast<int64_t>(q) * V;
        const uint32_t A = allowed[q / qdiv];
        const int32_t s = src[q];
        const int32_t tgt = target ? target[q] : -1;
        const int32_t *fl = Kf > 0 ? forbid + static_cast<int64_t>(q / qdiv) * Kf : nullptr;
        const bool s_ok = s >= 0 && s < V && allowed_v(region, A, s) && !forbidden_v(fl, Kf, s);
        // a target that is not allowed, or forbidden, is never reached
        const bool t_ok =
            !target || (tgt >= 0 && tgt < V && allowed_v(region, A, tgt) && !forbidden_v(fl, Kf, tgt));
        if (tid == 0) {
            tail_s = 0;
            if (s_ok && t_ok) {
                drow[s] = 0;
                qbuf[0] = s;
                tail_s = 1;
            }
        }
        __syncthreads();
        int32_t lo = 0, hi = tail_s;
        for (int32_t d = 0; lo < hi; ++d) {
            if (target && t_ok && drow[tgt] != -1) break;
            for (int32_t i = lo + tid; i < hi; i += kQueueThreads) {
                const int32_t u = qbuf[i];
                const int64_t b = adj_off[u], e = adj_off[u + 1];
                if (!pc_range_ok(b, e, n_adj)) continue;
                for (int64_t p = b; p < e; ++p) {
                    const int32_t v = adj[p];
                    if (v < 0 || v >= V || !allowed_v(region, A, v) || forbidden_v(fl, Kf, v)) continue;
                    if (atomicCAS(&drow[v], -1, d + 1) == -1) qbuf[atomicAdd(&tail_s, 1)] = v;
                }
            }
            __syncthreads();
            lo = hi;
            hi = tail_s;
            __syncthreads();
        }
        if (target) {
            __syncthreads();
            if (tid == 0) dist[q] = (s_ok && t_ok) ? drow[tgt] : -1;
            __syncthreads();
            const int32_t n = tail_s;
            for (int32_t i = tid; i < n; i += kQueueThreads) drow[qbuf[i]] = -1;
        }
        __syncthreads();
    }
}

}  // namespace

namespace {

// Data errors and, with sym, the graph's symmetry (see k_rc_checks): it is
// symmetric unless *asym(ctx) holds the number returned.
int32_t checks(pc_ctx *ctx, int32_t V, const int32_t *adj_off, const int32_t *adj, int64_t n_adj,
               const uint8_t *region, int32_t Q, const int32_t *src, const int32_t *target, const int32_t *via,
               int32_t Kv, const int32_t *forbid, int32_t Kf, bool sym, hipStream_t stream)
{
    if (sym) ctx->reach_gen = ctx->reach_gen == INT32_MAX ? 1 : ctx->reach_gen + 1;
    const Checks c{V, adj_off, adj, n_adj, region, Q, src, target, static_cast<int64_t>(Q) * Kv,
                   static_cast<int64_t>(Q) * Kf, via, forbid, ctx->d_small + 4, sym ? ctx->reach_gen : 0, ctx->d_err};
    const int64_t n = std::max<int64_t>({V, Q, n_adj, c.nv, c.nf});
    int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
    if (sym) blocks = std::max<int64_t>(blocks, std::min<int64_t>((V + 3) / 4, 8192));
    if (blocks > 0)
        PC_TIMED(ctx, "k_rc_checks", stream,
                 hipLaunchKernelGGL(k_rc_checks, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, c));
    return c.gen;
}

// Does the bitset search take Q queries (rows, or targets and legs)?  The graph
// has to fit its LDS.  Few queries on a sparse graph would leave most of the chip
// idle and pass over every vertex on each of many levels; the map search pays for
// every query, and past 512 workgroups a second round.  How many levels there are
// the host does not know.  Bitset / map on geometric graphs of mean degree 4 (many
// levels) and random ones of mean degree 8 (few): rows, 256 queries on 1,000
// vertices 86 / 49 and 55 / 38 us, 512 there 91 / 83 and 55 / 62, 512 on 2,000
// 149 / 89 and 95 / 70, 1,024 on 6,000 436 / 252 and 265 / 240; past the limit 1,024 on
// 1,000 92 / 148 and 57 / 101.  Targets, 256 queries on 1,000 vertices 86 / 50 and
// 23 / 32, 512 on 6,000 387 / 144 and 102 / 95; past the limit 512 on 1,000 88 / 85
// and 23 / 45, 1,024 on 6,000 386 / 231 and 76 / 166.  Denser graphs have few levels
// (1,280 switches of degree 32, 64 queries 41 / 36; 2,880 of degree 48 80 / 84):
// the bitset search keeps them.
size_t bitset_lds(int32_t V)
{
    // visited / frontier / next (8 B each), region (1 B) and list (2 B) per vertex
    return ((static_cast<size_t>(V) + 15) & ~size_t(15)) * 3 * 8 + 32 * 8 + ((static_cast<size_t>(V) + 3) & ~size_t(3)) +
           static_cast<size_t>(V) * 2;
}

bool takes_bitset(int32_t V, int64_t n_adj, int64_t Q, bool rows)
{
    static_assert(kMaxBitsetV * 27 + 256 + kBitsetStatic <= 160 * 1024, "within a workgroup's LDS");
    const int64_t few = std::min(std::max(V / (rows ? 4 : 12), 256), 1024);
    return V > 0 && V <= kMaxBitsetV && !(n_adj / V <= kEll / 2 && V >= 512 && Q <= few);
}

// The search of Q queries (legs).  bits: the bitset search.  Else, with map:
// the map search, its workgroups, whether neighbour records are formed (up to a
// mean of kEll / 2 entries nearly all vertices fit one) and its scratch, in the
// arena.  Else the queue search.
struct Search {
    bool bits = false, map = false, records = false;
    size_t lds = 0;
    int32_t grid = 0;
    int32_t *list = nullptr;
    uint32_t *ell = nullptr;
};

// The map search asks for more scratch than the others (up to 512 lists and the
// records): where that is refused, graphs that fit the bitset search take
// it, which may need none, and larger ones the queue search.  Chosen before the
// checks: only the bitset search asks for the graph's symmetry.
// (Targets close to their sources do not repay the records of a large graph: one
// query two hops away on a million vertices 36 us, by the queue search 21; but
// where they are is not known, and sixteen queries anywhere 242, by the queue
// search 864.)
int choose_search(pc_ctx *ctx, int32_t V, int64_t n_adj, int64_t Q, bool rows, Search &s)
{
    s.bits = takes_bitset(V, n_adj, Q, rows);
    if (s.bits || V == 0 || Q == 0 || Q > INT32_MAX) return PC_OK;
    int max_lds = 0;
    PC_HIP(ctx, hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, ctx->device));
    s.lds = (static_cast<size_t>(V) + 127) / 128 * 16;
    hipFuncAttributes fm{};
    PC_HIP(ctx, hipFuncGetAttributes(&fm, reinterpret_cast<const void *>(k_rc_map<4, true>)));
    if (V >= (1 << kVertexBits) || s.lds + fm.sharedSizeBytes > static_cast<size_t>(max_lds)) return PC_OK;
    s.records = n_adj / V <= kEll / 2;
    const int per_cu = 2 * (s.lds + fm.sharedSizeBytes) <= static_cast<size_t>(max_lds) ? 2 : 1;
    s.grid = static_cast<int32_t>(std::min<int64_t>(Q, 256 * per_cu));
    auto carve = [&](Carver &c) {
        s.list = c.take<int32_t>(static_cast<size_t>(s.grid) * V);
        s.ell = c.take<uint32_t>(s.records ? static_cast<size_t>(V) * kEll : 1);
    };
    Carver dry{nullptr, 0};
    carve(dry);
    const int rc = pc_ensure_arena(ctx, dry.off);
    if (rc == PC_ENOMEM) {
        ctx->msg[0] = 0;
        s.bits = V <= kMaxBitsetV;
        return PC_OK;
    }
    if (rc) return rc;
    Carver real{ctx->arena, 0};
    carve(real);
    s.map = true;
    return PC_OK;
}

// Are the queries (legs) ordered by source?  Workgroups then share
// frontiers and expand each for more of their queries, which pays for the
// four launches of the sort only with enough workgroups and vertices.
// Sorted / unsorted, targets: 20,000 queries on 1,280 vertices 40 / 31 us,
// 266,666 on 80 143 / 114, 66,666 on 1,280 62 / 72, 20,000 on 2,880 49 / 55.
// Legs (unsorted they are computed and summed in the search, and the two
// legs of a waypoint share its workgroup): 6,000 walks of two legs on 1,280
// vertices 56 / 43, 20,000 on 320 55 / 44, 66,666 on 320 90 / 103, 4,000 on
// 2,880 82 / 90.  Rows: 20,000 queries on 320 vertices 53 / 38, 6,000 on
// 2,880 103 / 96, 20,000 on 1,280 85 / 75.
bool sorts(int32_t V, int64_t Q, bool legs)
{
    return Q > 64 && Q * V > (legs ? int64_t(1) << 24 : int64_t(1) << 25);
}

// BFS of Q queries; query j's allowed mask is allowed[j / qdiv] and its
// forbidden list forbid[(j / qdiv) * Kf ...] (Kf = 0: none).  m: choose_search's.
// gen: what checks() returned.  via (bitset search, no sort): the queries are walks of
// Kv + 1 legs.  Takes the context's arena when it needs scratch.
int bfs(pc_ctx *ctx, int32_t V, const int32_t *adj_off, const int32_t *adj, int64_t n_adj, const uint8_t *region,
        int32_t Q, const int32_t *src, const uint32_t *allowed, const int32_t *target, int32_t *dist,
        const int32_t *forbid, int32_t Kf, int32_t qdiv, const Search &m, int32_t gen, const int32_t *via, int32_t Kv,
        hipStream_t stream)
{
    if (V == 0) {
        if (target) launch_fill_u32(reinterpret_cast<uint32_t *>(dist), static_cast<size_t>(Q), 0xFFFFFFFFu, stream);
        PC_LAUNCH_CHECK(ctx);
        return PC_OK;
    }
    const int64_t avg = n_adj / V;
    if (m.bits) {
        const size_t lds = bitset_lds(V);
        if (!target) launch_fill_u32(reinterpret_cast<uint32_t *>(dist), static_cast<size_t>(Q) * V, 0xFFFFFFFFu, stream);
        PC_LAUNCH_CHECK(ctx);
        int32_t *perm = nullptr;
        if (!via && sorts(V, Q, qdiv > 1)) {
            int32_t *cnt, *off, *pos;
            auto carve = [&](Carver &c) {
                cnt = c.take<int32_t>(static_cast<size_t>(V) + 2);
                off = c.take<int32_t>(static_cast<size_t>(V) + 2);
                pos = c.take<int32_t>(static_cast<size_t>(Q));
                perm = c.take<int32_t>(static_cast<size_t>(Q));
            };
            Carver dry{nullptr, 0};
            carve(dry);
            int rc = pc_ensure_arena(ctx, dry.off);
            if (rc) return rc;
            Carver real{ctx->arena, 0};
            carve(real);
            launch_fill_u32(reinterpret_cast<uint32_t *>(cnt), static_cast<size_t>(V) + 1, 0, stream);
            PC_TIMED(ctx, "k_rc_src_count", stream,
                     hipLaunchKernelGGL(k_rc_src_count, dim3(static_cast<unsigned>((Q + kSortPer - 1) / kSortPer)),
                                        dim3(kSortThreads), (static_cast<size_t>(V) + 1) * sizeof(int32_t), stream, Q,
                                        src, V, cnt, pos));
            launch_scan_i32(cnt, V + 1, off, nullptr, nullptr, stream);
            PC_TIMED(ctx, "k_rc_src_place", stream,
                     hipLaunchKernelGGL(k_rc_src_place, dim3(static_cast<unsigned>(std::min<int64_t>((Q + 255) / 256, 4096))),
                                        dim3(256), 0, stream, Q, src, V, off, pos, perm));
            PC_LAUNCH_CHECK(ctx);
        }
        // lanes per vertex: a power of two near a third of the mean degree
        const int gs = avg <= 12 ? 4 : avg <= 24 ? 8 : avg <= 48 ? 16 : 32;
        const int32_t per = via ? 64 / (Kv + 1) : 64;
        const dim3 grid_b(static_cast<unsigned>((static_cast<int64_t>(Q) + per - 1) / per));
        auto launch = [&](auto kern) -> int {
            if (lds > 48 * 1024)
                PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
            PC_TIMED(ctx, "k_rc_bitset", stream,
                     hipLaunchKernelGGL(kern, grid_b, dim3(kBitsetThreads), lds, stream, V, adj_off, adj, n_adj,
                                        region, Q, src, allowed, target, dist, forbid, Kf, qdiv, ctx->d_small + 4, gen,
                                        perm, via, Kv));
            PC_LAUNCH_CHECK(ctx);
            return PC_OK;
        };
        if (via) {
            if (gs == 4) return launch(k_rc_bitset<4, true>);
            if (gs == 8) return launch(k_rc_bitset<8, true>);
            if (gs == 16) return launch(k_rc_bitset<16, true>);
            return launch(k_rc_bitset<32, true>);
        }
        if (gs == 4) return launch(k_rc_bitset<4, false>);
        if (gs == 8) return launch(k_rc_bitset<8, false>);
        if (gs == 16) return launch(k_rc_bitset<16, false>);
        return launch(k_rc_bitset<32, false>);
    }
    if (m.map) {
        if (m.records)
            PC_TIMED(ctx, "k_rc_records", stream,
                     hipLaunchKernelGGL(k_rc_records, dim3(static_cast<unsigned>((static_cast<int64_t>(V) * 4 + 255) / 256)), dim3(256), 0,
                                        stream, V, adj_off, adj, n_adj, region, m.ell));
        auto launch = [&](auto kern) -> int {
            PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(m.lds)));
            PC_TIMED(ctx, "k_rc_map", stream,
                     hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(m.grid)), dim3(kMapThreads), m.lds, stream, V,
                                        adj_off, adj, n_adj, region, m.ell, Q, src, allowed, target, dist, m.list, forbid,
                                        Kf, qdiv));
            PC_LAUNCH_CHECK(ctx);
            return PC_OK;
        };
        if (m.records) return launch(k_rc_map<4, true>);
        return avg <= 24 ? launch(k_rc_map<8, false>) : launch(k_rc_map<32, false>);
    }
    if (!target) launch_fill_u32(reinterpret_cast<uint32_t *>(dist), static_cast<size_t>(Q) * V, 0xFFFFFFFFu, stream);
    int32_t grid = Q < 256 ? Q : 256;
    int32_t *qbuf, *rows;
    auto carve = [&](Carver &c) {
        qbuf = c.take<int32_t>(static_cast<size_t>(grid) * V);
        rows = c.take<int32_t>(target ? static_cast<size_t>(grid) * V : 1);
    };
    Carver dry{nullptr, 0};
    carve(dry);
    const int rc = pc_ensure_arena(ctx, dry.off);
    if (rc) return rc;
    Carver real{ctx->arena, 0};
    carve(real);
    if (target) launch_fill_u32(reinterpret_cast<uint32_t *>(rows), static_cast<size_t>(grid) * V, 0xFFFFFFFFu, stream);
    PC_TIMED(ctx, "k_rc_queue", stream, hipLaunchKernelGGL(k_rc_queue, dim3(static_cast<unsigned>(grid)), dim3(kQueueThreads), 0, stream, V, adj_off, adj,
                       n_adj, region, Q, src, allowed, target, dist, qbuf, rows, forbid, Kf, qdiv));
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}

__global__ void k_rc_legs(int32_t Q, const int32_t *__restrict__ src, const int32_t *__restrict__ target,
                          const int32_t *__restrict__ via, int32_t Kv, const int32_t *__restrict__ asym, int32_t gen,
                          int32_t *__restrict__ leg_src, int32_t *__restrict__ leg_tgt)
{
    const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= Q) return;
    const bool flip = *asym != gen;
    for (int32_t k = 0; k <= Kv; ++k) {
        const Leg leg = leg_of(src, target, via + static_cast<int64_t>(q) * Kv, Kv, q, k, flip);
        leg_src[static_cast<int64_t>(q) * (Kv + 1) + k] = leg.from;
        leg_tgt[static_cast<int64_t>(q) * (Kv + 1) + k] = leg.to;
    }
}

__global__ void k_rc_via_sum(int32_t Q, const int32_t *__restrict__ via, int32_t Kv,
                             const int32_t *__restrict__ leg_dist, int32_t *__restrict__ dist)
{
    const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= Q) return;
    WalkLength w;
    for (int32_t k = 0; k <= Kv && w.open; ++k)
        w.add(leg_dist[static_cast<int64_t>(q) * (Kv + 1) + k], k == Kv || via[static_cast<int64_t>(q) * Kv + k] == -1);
    dist[q] = w.length();
}

}  // namespace

int run_reach(pc_ctx *ctx, int32_t V, const int32_t *adj_off, const int32_t *adj, int64_t n_adj,
              const uint8_t *region, int32_t Q, const int32_t *src, const uint32_t *allowed, const int32_t *target,
              int32_t *dist, hipStream_t stream)
{
    Search m;
    const int rc = choose_search(ctx, V, n_adj, Q, target == nullptr, m);
    if (rc) return rc;
    const int32_t gen = checks(ctx, V, adj_off, adj, n_adj, region, Q, src, target, nullptr, 0, nullptr, 0,
                               target && m.bits, stream);
    PC_LAUNCH_CHECK(ctx);
    return bfs(ctx, V, adj_off, adj, n_adj, region, Q, src, allowed, target, dist, nullptr, 0, 1, m, gen, nullptr, 0,
               stream);
}

int run_reach_via(pc_ctx *ctx, int32_t V, const int32_t *adj_off, const int32_t *adj, int64_t n_adj,
                  const uint8_t *region, int32_t Q, const int32_t *src, const uint32_t *allowed,
                  const int32_t *target, const int32_t *via, int32_t Kv, const int32_t *forbid, int32_t Kf,
                  int32_t *dist, hipStream_t stream)
{
    const int64_t nl = static_cast<int64_t>(Q) * (Kv + 1);
    Search m;
    int rc = choose_search(ctx, V, n_adj, nl, false, m);
    if (rc) return rc;
    const int32_t gen = checks(ctx, V, adj_off, adj, n_adj, region, Q, src, target, via, Kv, forbid, Kf,
                               Q > 0 && (Kv > 0 || m.bits), stream);
    PC_LAUNCH_CHECK(ctx);
    if (Q == 0) return PC_OK;
    if (Kv == 0 || (m.bits && !sorts(V, nl, true)))
        return bfs(ctx, V, adj_off, adj, n_adj, region, Q, src, allowed, target, dist, forbid, Kf, 1, m, gen,
                   Kv == 0 ? nullptr : via, Kv, stream);
    // legs [Q][Kv + 1] (sources, targets, distances) in the auxiliary
    // buffer; leg j belongs to query j / (Kv + 1)
    if (nl > 0x7FFFFFFF) return pc_set_error(ctx, PC_EINVAL, "pc_masked_reach_via: Q*(Kv+1) over 2^31 legs");
    int32_t *leg_src, *leg_tgt, *leg_dist;
    auto carve = [&](Carver &c) {
        leg_src = c.take<int32_t>(static_cast<size_t>(nl));
        leg_tgt = c.take<int32_t>(static_cast<size_t>(nl));
        leg_dist = c.take<int32_t>(static_cast<size_t>(nl));
    };
    Carver dry{nullptr, 0};
    carve(dry);
    rc = pc_ensure_aux(ctx, dry.off);
    if (rc) return rc;
    Carver real{ctx->aux, 0};
    carve(real);
    const unsigned qb = static_cast<unsigned>((Q + 255) / 256);
    PC_TIMED(ctx, "k_rc_legs", stream,
             hipLaunchKernelGGL(k_rc_legs, dim3(qb), dim3(256), 0, stream, Q, src, target, via, Kv, ctx->d_small + 4,
                                gen, leg_src, leg_tgt));
    PC_LAUNCH_CHECK(ctx);
    rc = bfs(ctx, V, adj_off, adj, n_adj, region, static_cast<int32_t>(nl), leg_src, allowed, leg_tgt, leg_dist,
             forbid, Kf, Kv + 1, m, gen, nullptr, 0, stream);
    if (rc) return rc;
    PC_TIMED(ctx, "k_rc_via_sum", stream,
             hipLaunchKernelGGL(k_rc_via_sum, dim3(qb), dim3(256), 0, stream, Q, via, Kv, leg_dist, dist));
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}
