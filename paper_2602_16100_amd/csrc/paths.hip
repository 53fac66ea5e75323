// NEXT-2 -- compliant path synthesis: the path scheduler's search for a
// minimum-weight walk through allowed, non-forbidden switches via ordered
// waypoints (weighted Dijkstra, BFS when every link weighs 1), and the
// walk's compilation into one exact-match flow rule per switch (paper,
// Network orchestration).
//
// Design (gfx950):
//   1. validate : the data-error flags, a sweep over the whole input.
//   2. in-links : the reverse of the port graph -- per switch v the (u, port)
//                 pairs of the links u -> v -- counted, scanned and filled --
//                 and packed link records for the directed search.
//   3. bounds   : with many more legs than switches and weights that differ
//                 (one_weight), for every switch that a leg ends at, a lower
//                 bound of every switch's distance to it: the distances of
//                 the whole port graph, which no request's restrictions can
//                 shorten, in units taken from a sample of the weights
//                 (bound_form), 16 or 32 bits each.
//   4. goal     : one wavefront per request.  A leg relaxes only switches
//                 whose distance plus bound stays within a limit, which starts
//                 at the bound of the leg's source and grows until the leg's
//                 end is reached; the few dozen switches that pass it live in
//                 a small LDS hash table.  A request that outgrows its table or
//                 its work limit is left for 5.
//   5. search   : one workgroup per request.  Its usable-switch bitset,
//                 distances and frontier queues live in LDS.  Each leg is
//                 a chaotic relaxation in rounds: a wavefront takes 64
//                 frontier switches at a time (one lane each reads the
//                 port range), then relaxes them one after another, its
//                 lanes over a switch's ports with LDS atomic minima,
//                 loading the next switch's links while the current one's
//                 are relaxed; a switch whose distance drops joins the next
//                 round's frontier once (a flag bit per switch).  A frontier
//                 switch at or beyond the target's current distance is
//                 skipped: with weights >= 1 it cannot shorten the target's
//                 path, so every switch nearer than the target ends with its
//                 exact distance.  The leg is then
//                 walked back from its end by one wavefront: the
//                 predecessor of v is the lowest-numbered u among v's
//                 in-links with dist(u) + w = dist(v) (a wavefront minimum;
//                 the in-link lists carry each link's weight).
//                 The legs' switches collect in an LDS walk; the rules are
//                 written from it, one wavefront per switch finding the port
//                 of least (weight, index) to the next switch.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "pc_internal.h"

namespace {

constexpr int kPsThreads = 512;  // 8 wavefronts: four such workgroups fit a CU's LDS at fat-tree sizes
constexpr int kPsWaves = kPsThreads / 64;
constexpr int32_t kInf = INT32_MAX;

__device__ __forceinline__ int32_t wave_min_i32(int32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
    return v;
}

// Data-error flags, each a property of the whole input, and *span += the ports of
// all valid ranges, which overlapping ranges count more than once.
__global__ __launch_bounds__(256) void k_ps_validate(int32_t V, const int32_t *__restrict__ port_off,
                                                     const int32_t *__restrict__ port_peer, int64_t n_ports,
                                                     const uint32_t *__restrict__ weight,
                                                     const uint8_t *__restrict__ region, int32_t Q,
                                                     const int32_t *__restrict__ src,
                                                     const int32_t *__restrict__ target,
                                                     const int32_t *__restrict__ out_port,
                                                     const int32_t *__restrict__ via, int32_t Kv,
                                                     const int32_t *__restrict__ forbid, int32_t Kf,
                                                     unsigned long long *__restrict__ span,
                                                     uint32_t *__restrict__ d_err)
{
    uint32_t errs = 0;
    unsigned long long mine = 0;
    const int64_t per_q = Kv > Kf ? (Kv > 1 ? Kv : 1) : (Kf > 1 ? Kf : 1);
    int64_t tot = static_cast<int64_t>(Q) * per_q;
    if (n_ports > tot) tot = n_ports;
    if (V > tot) tot = V;
    for (int64_t x = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; x < tot;
         x += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (x < V) {
            if (region[x] >= 32) errs |= PC_DERR_JUR;
            if (!pc_range_ok(port_off[x], port_off[x + 1], n_ports)) errs |= PC_DERR_OFFSETS;
            else mine += static_cast<uint32_t>(port_off[x + 1] - port_off[x]);
        }
        if (x < n_ports) {
            if (port_peer[x] < -1 || port_peer[x] >= V) errs |= PC_DERR_SWITCH;
            if (weight && weight[x] == 0) errs |= PC_DERR_GRAPH;
        }
        if (x < Q) {
            const int32_t t = target[x];
            if (src[x] < 0 || src[x] >= V || t < 0 || t >= V) {
                errs |= PC_DERR_SWITCH;
            } else if (pc_range_ok(port_off[t], port_off[t + 1], n_ports) &&
                       (out_port[x] < 0 || out_port[x] >= port_off[t + 1] - port_off[t])) {
                errs |= PC_DERR_ACTION;
            }
        }
        if (x < static_cast<int64_t>(Q) * Kv && (via[x] < -1 || via[x] >= V)) errs |= PC_DERR_SWITCH;
        if (x < static_cast<int64_t>(Q) * Kf && (forbid[x] < -1 || forbid[x] >= V)) errs |= PC_DERR_SWITCH;
    }
    if (errs) atomicOr(d_err, errs);
    if (span != nullptr && __ballot(mine != 0)) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
        if ((threadIdx.x & 63) == 0) atomicAdd(span, mine);
    }
}

// Weight of port p as a link, or 0 when it is none.
__device__ __forceinline__ uint32_t link_weight(const int32_t *__restrict__ port_peer,
                                                const uint32_t *__restrict__ weight, int32_t V, int64_t p)
{
    const int32_t v = port_peer[p];
    if (v < 0 || v >= V) return 0;
    return weight ? weight[p] : 1u;
}

// Lanes per switch of the in-link kernels: a switch's ports are read
// together (one thread per switch walked 48 ports one after another: 181 and
// 162 us for 138,240 ports, against 15 and 20 us).
constexpr int kInLanes = 16;

// Do the in-link lists serve?  They hold n_ports entries, and switches whose
// port ranges overlap can have more links than that, even more than 32 bits count:
// then no list is written, and the walk-back looks through the switches.
__device__ __forceinline__ bool in_lists(const unsigned long long *span, int64_t n_ports)
{
    return *span <= static_cast<unsigned long long>(n_ports);
}

// In-link counts: kInLanes lanes per switch u, +1 at the peer of each link.
__global__ __launch_bounds__(256) void k_ps_in_count(int32_t V, const int32_t *__restrict__ port_off,
                                                     const int32_t *__restrict__ port_peer, int64_t n_ports,
                                                     const uint32_t *__restrict__ weight,
                                                     const unsigned long long *__restrict__ span,
                                                     int32_t *__restrict__ cnt)
{
    if (!in_lists(span, n_ports)) return;
    const int32_t u = (blockIdx.x * blockDim.x + threadIdx.x) / kInLanes;
    if (u >= V) return;
    const int64_t b = port_off[u], e = port_off[u + 1];
    if (!pc_range_ok(b, e, n_ports)) return;
    for (int64_t p = b + threadIdx.x % kInLanes; p < e; p += kInLanes)
        if (link_weight(port_peer, weight, V, p)) atomicAdd(&cnt[port_peer[p]], 1);
}

// In-link lists: (u, link weight) pairs in rin[rin_off[v] ..); cursor starts as a
// copy of rin_off.  The order within a list is arbitrary (only minima are
// taken over it).
__global__ __launch_bounds__(256) void k_ps_in_fill(int32_t V, const int32_t *__restrict__ port_off,
                                                    const int32_t *__restrict__ port_peer, int64_t n_ports,
                                                    const uint32_t *__restrict__ weight,
                                                    const unsigned long long *__restrict__ span,
                                                    int32_t *__restrict__ cursor, int2 *__restrict__ rin)
{
    if (!in_lists(span, n_ports)) return;
    const int32_t u = (blockIdx.x * blockDim.x + threadIdx.x) / kInLanes;
    if (u >= V) return;
    const int64_t b = port_off[u], e = port_off[u + 1];
    if (!pc_range_ok(b, e, n_ports)) return;
    for (int64_t p = b + threadIdx.x % kInLanes; p < e; p += kInLanes) {
        const uint32_t w = link_weight(port_peer, weight, V, p);
        if (w) {
            const int32_t pos = atomicAdd(&cursor[port_peer[p]], 1);
            rin[pos] = make_int2(u, static_cast<int32_t>(w));  // the weight's bits
        }
    }
}

// ---------------------------------------------------------------- directed search
constexpr uint32_t kNoLink = 0xFFFF0000u;  // bounds' links: slot 0 at the weight that saturates every sum
constexpr uint32_t kNoPeer = 0xFFFFu;  // packed links: the port is no link (switch ids stay below 12,288)

// How the bounds are kept, from a sorted sample of n link weights: in 16 bits
// and units of 2^shift, where nineteen links in twenty have at most twelve
// bits left (sixteen such links before a bound saturates), and the heavier
// ones count no more than a saturated bound.  Weights are rounded down and
// clamped, so the sums stay lower bounds.  Where a unit would be coarse for the
// lighter links (less than sixteen of them in the lowest quarter's weight),
// which the search would then wander along at no cost: kWideBounds, 32 bits and the
// weights as they are.
// (32,768 requests over 2,880 switches.  One drained link of 65,535 among
// weights 1-10: 6.8 ms with the largest weight's scale, whose bounds are all 0,
// 5.3 by the workgroup search alone, 0.68 so, as without that link; a fifth of
// the links drained 7.4 / 5.7 / 1.6; weights up to 2^20, their logarithms
// uniform, 10.9 / 9.4 / 2.5.)
constexpr uint32_t kWideBounds = 256;
__device__ __forceinline__ uint32_t bound_form(const uint32_t *sorted, int n)
{
    if (n == 0) return kWideBounds;
    const uint32_t heavy = sorted[(n - 1) * 19 / 20], light = sorted[n / 4];
    const int bits = 32 - __builtin_clz(heavy | 1u);
    const uint32_t shift = bits > 12 ? static_cast<uint32_t>(bits - 12) : 0u;
    return shift == 0 || (light >> shift) >= 16 ? shift : kWideBounds;
}

// A sample of the links' weights, a port from every stretch of n_ports /
// kSample, sorted (bitonic, two values a thread; non-links last); returns the
// number of links.  A step within 128 values is one wavefront's and needs no
// barrier.
constexpr int kSample = 512;
__device__ __forceinline__ int sample_weights(int32_t V, const int32_t *__restrict__ port_peer, int64_t n_ports,
                                              const uint32_t *__restrict__ weight, uint32_t *sorted)
{
    __shared__ int n;
    const int tid = threadIdx.x;
    if (tid == 0) n = 0;
    __syncthreads();
    const int64_t per = (n_ports + kSample - 1) / kSample;
    for (int i = tid; i < kSample; i += kSample / 2) {
        const int64_t p = i * per + (static_cast<uint32_t>(i) * 2654435761u >> 8) % per;
        const uint32_t w = p < n_ports ? link_weight(port_peer, weight, V, p) : 0u;
        sorted[i] = w ? w : ~0u;
        if (w) atomicAdd(&n, 1);
    }
    __syncthreads();
    for (int k = 2; k <= kSample; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int a = (tid & ~(j - 1)) << 1 | (tid & (j - 1)), b = a + j;
            const uint32_t x = sorted[a], y = sorted[b];
            if ((x > y) == ((a & k) == 0)) {
                sorted[a] = y;
                sorted[b] = x;
            }
            if (j > 64 || (j == 1 && k >= 128)) {  // the step is, or the next one will be, across wavefronts
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
    return n;
}

// The links' largest weight and the complement of their smallest
// (wspan[0], wspan[1], both maxima), and the switches that some leg ends at
// (every target and waypoint that is a switch).  Meanwhile the last workgroup
// chooses the bounds' form (wspan[2]) from a sample, and names the sample's lightest
// weight if 99 links in 100 have it (wspan[3], else 0).
__global__ __launch_bounds__(256) void k_ps_survey(int32_t V, const int32_t *__restrict__ port_peer, int64_t n_ports,
                                                   const uint32_t *__restrict__ weight, int32_t Q,
                                                   const int32_t *__restrict__ target, const int32_t *__restrict__ via,
                                                   int32_t Kv, int32_t *__restrict__ need,
                                                   uint32_t *__restrict__ wspan)
{
    __shared__ uint32_t top[2], sorted[kSample];
    const unsigned blocks = gridDim.x - 1;
    if (blockIdx.x == blocks) {
        const int n = sample_weights(V, port_peer, n_ports, weight, sorted);
        if (threadIdx.x == 0) {
            wspan[2] = bound_form(sorted, n);
            wspan[3] = n > 0 && sorted[n * 99 / 100] == sorted[0] ? sorted[0] : 0u;
        }
        return;
    }
    if (threadIdx.x < 2) top[threadIdx.x] = 0;
    __syncthreads();
    const int64_t nv = static_cast<int64_t>(Q) * Kv;
    int64_t tot = n_ports > nv ? n_ports : nv;
    if (Q > tot) tot = Q;
    uint32_t mine = 0, least = ~0u;
    for (int64_t x = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; x < tot;
         x += static_cast<int64_t>(blocks) * blockDim.x) {
        if (x < n_ports) {
            const uint32_t w = link_weight(port_peer, weight, V, x);
            mine = mine > w ? mine : w;
            if (w) least = least < w ? least : w;
        }
        if (x < Q && target[x] >= 0 && target[x] < V) need[target[x]] = 1;
        if (x < nv && via[x] >= 0 && via[x] < V) need[via[x]] = 1;
    }
    if (mine) {
        atomicMax(&top[0], mine);
        atomicMax(&top[1], ~least);
    }
    __syncthreads();
    if (threadIdx.x < 2 && top[threadIdx.x]) atomicMax(wspan + threadIdx.x, top[threadIdx.x]);
}

// Links of one weight (or none at all), or nearly all of the lightest:
// equally short paths are the rule then, a fat-tree's edge switches have one
// through every core, and a directed search would keep most of the graph.
// The workgroup search takes every request.  2,880 switches, 32,768 requests,
// workgroup search / directed: weight 10 and one link of 11 or 65,535 2.4 / 2.6 ms,
// one link in 1,000 2.4 / 2.6, in 100 2.4 / 2.4, in 33 2.4 / 2.3, in 10 2.5 / 1.6
// (of 65,535 2.6 / 2.1).  A few lighter links break the ties: one in 1,000 of
// weight 1 2.6 / 2.1, in 100 2.8 / 1.0.
__device__ __forceinline__ bool one_weight(const uint32_t *wspan)
{
    const uint32_t most = wspan[0], least = ~wspan[1];
    return most == 0 || most == least || wspan[3] == least;
}

// Does the workgroup search take every request?
__device__ __forceinline__ bool undirected(const uint32_t *wspan, const unsigned long long *span, int64_t n_ports)
{
    return one_weight(wspan) || !in_lists(span, n_ports);
}

__device__ __forceinline__ bool wide_bounds(const uint32_t *wspan) { return wspan[2] == kWideBounds; }
__device__ __forceinline__ uint32_t bound_shift(const uint32_t *wspan) { return wspan[2] & 31u; }

// The LDS slot of switch v in the bounds kernel: switches 16 apart fall in
// different banks (the peers of a fat-tree's core are a pod apart).
__device__ __forceinline__ int32_t bslot(int32_t v) { return v ^ ((v >> 4) & 15); }

// Packed forms of the port graph: per port (peer | region << 16, weight)
// and (peer's slot | scaled weight << 16, for 16-bit bounds), per switch its port range (empty when
// its offsets are bad), and the list of the switches that legs end at.
__global__ __launch_bounds__(256) void k_ps_links(int32_t V, const int32_t *__restrict__ port_off,
                                                  const int32_t *__restrict__ port_peer, int64_t n_ports,
                                                  const uint32_t *__restrict__ weight,
                                                  const uint8_t *__restrict__ region,
                                                  const int32_t *__restrict__ need, const int32_t *__restrict__ row,
                                                  const uint32_t *__restrict__ wspan, int2 *__restrict__ link,
                                                  uint32_t *__restrict__ blink, int2 *__restrict__ range,
                                                  int32_t *__restrict__ ends)
{
    const uint32_t shift = bound_shift(wspan);
    const int64_t tot = n_ports > V ? n_ports : V;
    for (int64_t x = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; x < tot;
         x += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (x < n_ports) {
            const uint32_t w = link_weight(port_peer, weight, V, x);
            const uint32_t u = w ? static_cast<uint32_t>(port_peer[x]) : kNoPeer;
            const uint32_t r = w ? region[u] : 32u;
            const uint32_t ws = w >> shift;
            link[x] = make_int2(static_cast<int>(u | (r < 32 ? r : 32u) << 16), static_cast<int>(w));
            blink[x] = w ? static_cast<uint32_t>(bslot(static_cast<int32_t>(u))) | (ws < 0xFFFFu ? ws : 0xFFFFu) << 16 : kNoLink;
        }
        if (x < V) {
            const int64_t b = port_off[x], e = port_off[x + 1];
            range[x] = pc_range_ok(b, e, n_ports) ? make_int2(static_cast<int>(b), static_cast<int>(e)) : make_int2(0, 0);
            if (need[x]) ends[row[x]] = static_cast<int32_t>(x);
        }
    }
}

// Distances of the whole port graph to 2 * kW of the listed switches per
// workgroup, two 16-bit values a word, or to kW of them in 32 bits: every
// switch takes the minimum over its links of weight + the peer's values until
// nothing changes.  A quad of
// lanes shares a switch's links, kBv switches and kBu links of each in flight
// at once, the next switches' ranges read ahead (wider groups spend more
// instructions on the minimum over the group than on the links: 0.63 ms with
// 16 lanes instead of 0.34 ms).  Values only fall, and each entry is written by one
// lane, so sweeps read whatever is newest.  Saturated sums are lower
// bounds like the rest.  A graph that needs more than kSweeps sweeps is too
// long for this: its rows are marked as missing.
// Bound by the chains link -> LDS words -> packed add and minimum of each link and
// word: of 315 us the vector units issue 28 % of what they could, and waves wait 45 %
// of their cycles, 31 % for an operand.  2,880 rows over 138,240 links, 7-8 sweeps,
// in 0.31 ms with eight rows per workgroup, 0.33 ms with four; in 32 bits, over weights
// of a range that needs them, 0.53-1.2 ms.
constexpr int kSweeps = 40;
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
template <class T>
__device__ __forceinline__ T pk_min(T a, T b)
{
    return __builtin_elementwise_min(a, b);
}

// Minimum over a quad of lanes, in each of them.
template <class T>
__device__ __forceinline__ T quad_pk_min(T x)
{
    const auto dpp = [](T a, auto ctrl) {
        const int v = __builtin_bit_cast(int, a);
        return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(v, v, decltype(ctrl)::value, 0xF, 0xF, false));
    };
    x = pk_min(x, dpp(x, std::integral_constant<int, 0xB1>{}));     // quad_perm 1,0,3,2
    return pk_min(x, dpp(x, std::integral_constant<int, 0x4E>{}));  // quad_perm 2,3,0,1
}

template <class T, int kW>
struct __align__(4 * kW) BoundWords {
    T w[kW];
};

// A link as a sweep reads it: the peer's slot and the weight (no link: slot 0 at
// the weight that saturates every sum).
__device__ __forceinline__ uint32_t bound_link(const uint32_t *__restrict__ links, int32_t p, bool in)
{
    return in ? links[p] : kNoLink;
}
__device__ __forceinline__ int2 bound_link(const int2 *__restrict__ links, int32_t p, bool in)
{
    const int2 x = in ? links[p] : make_int2(static_cast<int>(kNoPeer), 0);
    const int32_t u = x.x & 0xFFFF;
    return u == static_cast<int32_t>(kNoPeer) ? make_int2(0, -1) : make_int2(bslot(u), x.y);
}
__device__ __forceinline__ uint32_t link_slot(uint32_t link) { return link & 0xFFFFu; }
__device__ __forceinline__ uint32_t link_slot(int2 link) { return static_cast<uint32_t>(link.x); }
__device__ __forceinline__ u16x2 link_cost(uint32_t link)
{
    const uint16_t w = static_cast<uint16_t>(link >> 16);
    return u16x2{w, w};
}
__device__ __forceinline__ uint32_t link_cost(int2 link) { return static_cast<uint32_t>(link.y); }

// The rows from r0 on.  T: a word of values (u16x2 or uint32_t), Out: a value.
template <int kBv, int kBu, int kW, class T, class Out, class Link>
__device__ __forceinline__ void bound_rows(int32_t V, const int2 *__restrict__ range, const Link *__restrict__ links,
                                           const int32_t *__restrict__ ends, int32_t n, int32_t r0, uint4 *lds,
                                           Out *__restrict__ bound, int32_t *__restrict__ row_ok)
{
    using Words = BoundWords<T, kW>;
    constexpr int kRows = static_cast<int>(sizeof(Words) / sizeof(Out)), kBoundThreads = 256 * kW;
    Words *dd = reinterpret_cast<Words *>(lds);  // [V rounded up to 16], at bslot(v)
    const int tid = threadIdx.x;
    Words none;
#pragma unroll
    for (int k = 0; k < kW; ++k) none.w[k] = __builtin_bit_cast(T, ~0u);
    for (int32_t v = tid; v < ((V + 15) & ~15); v += kBoundThreads) dd[v] = none;
    __syncthreads();
    if (tid < kRows && r0 + tid < n) reinterpret_cast<Out *>(&dd[bslot(ends[r0 + tid])])[tid] = 0;
    __syncthreads();
    constexpr int GS = 4, kStep = kBoundThreads / GS * kBv;
    const int grp = tid / GS, gl = tid % GS;
    auto ranges = [&](int32_t v0, int2 (&r)[kBv]) {
#pragma unroll
        for (int k = 0; k < kBv; ++k) r[k] = range[min(v0 + k, V - 1)];
    };
    bool done = false;
    for (int sweep = 0; sweep < kSweeps && !done; ++sweep) {
        bool changed = false;
        int2 rn[kBv];
        ranges(grp * kBv, rn);
        for (int32_t v0 = grp * kBv; v0 < V; v0 += kStep) {
            int2 r[kBv];
#pragma unroll
            for (int k = 0; k < kBv; ++k) r[k] = rn[k];
            Link L[kBv][kBu];
#pragma unroll
            for (int k = 0; k < kBv; ++k)
#pragma unroll
                for (int j = 0; j < kBu; ++j) {
                    const int32_t p = r[k].x + j * GS + gl;
                    L[k][j] = bound_link(links, p, p < r[k].y);
                }
            ranges(v0 + kStep, rn);
#pragma unroll
            for (int k = 0; k < kBv; ++k) {
                if (v0 + k >= V) break;
                Words acc = none;
                auto take = [&](Link link) {
                    const Words x = dd[link_slot(link)];
                    const T w = link_cost(link);
#pragma unroll
                    for (int i = 0; i < kW; ++i) acc.w[i] = pk_min(acc.w[i], __builtin_elementwise_add_sat(x.w[i], w));
                };
#pragma unroll
                for (int j = 0; j < kBu; ++j) take(L[k][j]);
                for (int32_t p = r[k].x + kBu * GS; p < r[k].y; p += GS) take(bound_link(links, p + gl, p + gl < r[k].y));
#pragma unroll
                for (int i = 0; i < kW; ++i) acc.w[i] = quad_pk_min(acc.w[i]);
                if (gl == 0) {
                    const Words old = dd[bslot(v0 + k)];
                    bool less = false;
#pragma unroll
                    for (int i = 0; i < kW; ++i) {
                        acc.w[i] = pk_min(acc.w[i], old.w[i]);
                        less |= __builtin_bit_cast(uint32_t, acc.w[i]) != __builtin_bit_cast(uint32_t, old.w[i]);
                    }
                    if (less) {
                        dd[bslot(v0 + k)] = acc;
                        changed = true;
                    }
                }
            }
        }
        done = !__syncthreads_or(changed);
    }
    for (int k = 0; k < kRows; ++k) {
        if (r0 + k >= n) break;
        Out *row = bound + static_cast<int64_t>(r0 + k) * V;
        for (int32_t v = tid; v < V; v += kBoundThreads) row[v] = reinterpret_cast<const Out *>(&dd[bslot(v)])[k];
        if (tid == 0) row_ok[r0 + k] = done;
    }
}

// (A grid of V / kW workgroups: half of them end at once with 16-bit values.  The
// 32-bit form has half as many switches in flight where that is several: its
// links take twice the registers, and a second workgroup has to fit a CU.)
template <int kBv, int kBu, int kW>
__global__ __launch_bounds__(256 * kW) void k_ps_bound(int32_t V, const int2 *__restrict__ range,
                                                            const uint32_t *__restrict__ blink,
                                                            const int2 *__restrict__ link,
                                                            const int32_t *__restrict__ ends,
                                                            const int32_t *__restrict__ n_ends,
                                                            const uint32_t *__restrict__ wspan,
                                                            const unsigned long long *__restrict__ span, int64_t n_ports,
                                                            uint32_t *__restrict__ bound, int32_t *__restrict__ row_ok)
{
    extern __shared__ uint4 ps_bound_lds[];
    const int32_t n = *n_ends;
    const bool wide = wide_bounds(wspan);
    const int32_t r0 = blockIdx.x * (wide ? kW : 2 * kW);
    if (r0 >= n || undirected(wspan, span, n_ports)) return;
    if (wide)
        bound_rows<(kBv + 1) / 2, kBu, kW, uint32_t, uint32_t>(V, range, link, ends, n, r0, ps_bound_lds, bound, row_ok);
    else
        bound_rows<kBv, kBu, kW, u16x2, uint16_t>(V, range, blink, ends, n, r0, ps_bound_lds,
                                                  reinterpret_cast<uint16_t *>(bound), row_ok);
}

// One wavefront per request, directed by the bounds.  A switch u relaxed to
// distance d is kept only while d + bound(u) <= limit, the smaller of B and
// the distance found for the leg's end.  Every switch on a minimum-weight
// path of the request's own graph passes that test once B reaches the path's
// weight, with its exact distance, since the bounds never exceed the
// restricted distances; so do all of its equally short predecessors, which
// is what the walk-back compares.  B starts at the source's bound; while
// the end lies beyond it, every kept switch is relaxed again with B raised to
// the smallest value that was turned away, and at least by half of its excess
// over the start, so that the passes stay few under weights of any size
// (doubling the excess kept so many more switches that about 1 request in 50
// outgrew its table: 597 + 207 us instead of 541 + 6 for both searches).
// Kept switches: an LDS hash table of distance << 16 | switch (forbidden
// switches sit in it with bit 15 set) and a ring of the slots to relax.  GS
// lanes share a switch's links, so 64 / GS switches are relaxed at once, kUn
// links per lane in flight.  Requests that need more than kFull slots or
// max_steps rounds of links go to the list `hard`.
// Bound by the latency of the link and bound reads (waves wait 61 % of their
// cycles; vector units 22 %, scalar units 41 % of their issue rates), so the wave slots have
// to fill: 512 slots keep 5 KB of LDS per wavefront (1,024 slots: 0.96 ms
// instead of 0.60 at the time).  Three links per lane in flight and 16 lanes a
// switch fit 48-port switches (0.51 ms; four links 0.54, 8 lanes 0.64, 32 lanes
// 0.52).  65,536 weighted requests with a waypoint each over 2,880 switches:
// 10.44 ms by the workgroup search, 0.51 + 0.31 ms (bounds) directed.
constexpr int kSlots = 512;
constexpr int kFull = 384;
constexpr uint32_t kForbid = 0x8000u;
constexpr int kUn = 3;

template <int GS>
__global__ __launch_bounds__(64) void k_ps_goal(
    int32_t V, int64_t n_ports, const int2 *__restrict__ range, const int2 *__restrict__ link, const uint8_t *__restrict__ region,
    const int32_t *__restrict__ rin_off, const int2 *__restrict__ rin, const int32_t *__restrict__ row,
    const int32_t *__restrict__ row_ok, const uint32_t *__restrict__ bound, const uint32_t *__restrict__ wspan,
    const int32_t *__restrict__ src, const int32_t *__restrict__ target, const uint32_t *__restrict__ allowed,
    const int32_t *__restrict__ via, int32_t Kv, const int32_t *__restrict__ forbid, int32_t Kf,
    const pc_key *__restrict__ key, const int32_t *__restrict__ out_port, int32_t prio, int32_t max_hops,
    int32_t *__restrict__ hops_out, int32_t *__restrict__ path_out, pc_rule *__restrict__ rules_out,
    const unsigned long long *__restrict__ span, int32_t max_steps,
    int32_t *__restrict__ hard, int32_t *__restrict__ n_hard)
{
    constexpr unsigned long long kEmpty = ~0ull;
    __shared__ __align__(16) unsigned long long tab[kSlots];
    __shared__ uint32_t inq[kSlots / 32];
    __shared__ uint16_t ring[kSlots];
    extern __shared__ uint16_t ps_walk[];  // the walk, one leg backwards, the walk's ports: max_hops + 2 each
    uint16_t *walk = ps_walk, *leg = walk + max_hops + 2, *act = leg + max_hops + 2;
    const int lane = threadIdx.x, grp = lane / GS, gl = lane % GS;
    constexpr int kNG = 64 / GS;
    auto wave_sync = [] {  // LDS written by other lanes of this wavefront
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto slot_of = [](uint32_t u) { return (u * 40503u >> 7) & (kSlots - 1); };
    if (undirected(wspan, span, n_ports)) return;
    const int32_t q = blockIdx.x;
    const int32_t s = src[q], t = target[q];
    bool fail = s < 0 || s >= V || t < 0 || t >= V;
    if (!fail) {
        const int2 r = range[t];
        fail = out_port[q] < 0 || out_port[q] >= r.y - r.x;
    }
    const uint32_t A = allowed[q];
    const int32_t *fl = forbid + static_cast<int64_t>(q) * Kf;
    const int32_t *vl = via + static_cast<int64_t>(q) * Kv;
    auto usable = [&](int32_t v) {
        const uint32_t r = region[v];
        if (r >= 32 || !((A >> r) & 1u)) return false;
        for (int32_t k = 0; k < Kf; ++k)
            if (fl[k] == v) return false;
        return true;
    };
    int32_t m = 0;  // waypoints: the list ends at its first -1
    while (m < Kv && vl[m] != -1) ++m;
    const bool wide = wide_bounds(wspan);
    const uint32_t shift = bound_shift(wspan);
    // every stop is a usable switch, or the request fails before any search
    if (!fail) fail = !usable(s) || !usable(t);
    for (int32_t k = 0; k < m && !fail; ++k) fail = vl[k] < 0 || vl[k] >= V || !usable(vl[k]);

    int32_t total = 0, steps = 0;
    bool hard_q = false;
    int32_t from = s;
    if (lane == 0 && !fail) walk[0] = static_cast<uint16_t>(s);
    for (int32_t li = 0; li <= m && !fail && !hard_q; ++li) {
        const int32_t to = li < m ? vl[li] : t;
        const int32_t rw = row[to];
        if (!row_ok[rw]) {
            hard_q = true;
            break;
        }
        const uint32_t *bt32 = bound + static_cast<int64_t>(rw) * V;
        const uint16_t *bt16 = reinterpret_cast<const uint16_t *>(bound) + static_cast<int64_t>(rw) * V;
        auto bound_of = [&](uint32_t v) -> uint32_t { return wide ? bt32[v] : bt16[v]; };  // in units of 2^shift
        // the empty table with the forbidden switches and the leg's source
        for (int i = lane; i < kSlots / 2; i += 64) reinterpret_cast<ulonglong2 *>(tab)[i] = make_ulonglong2(kEmpty, kEmpty);
        if (lane < kSlots / 32) inq[lane] = 0;
        wave_sync();
        int32_t stored = 1;
        if (lane < Kf && fl[lane] >= 0 && fl[lane] < V) {
            const uint32_t f = static_cast<uint32_t>(fl[lane]);
            uint32_t h = slot_of(f);
            while (true) {
                const unsigned long long o = atomicCAS(&tab[h], kEmpty, static_cast<unsigned long long>(f | kForbid));
                if (o == kEmpty || (o & 0x7FFFu) == f) break;
                h = (h + 1) & (kSlots - 1);
            }
        }
        wave_sync();
        stored += Kf;
        uint32_t s_slot = slot_of(static_cast<uint32_t>(from));
        while (tab[s_slot] != kEmpty) s_slot = (s_slot + 1) & (kSlots - 1);
        wave_sync();
        if (lane == 0) {
            tab[s_slot] = static_cast<unsigned long long>(from);
            ring[0] = static_cast<uint16_t>(s_slot);
            inq[s_slot >> 5] = 1u << (s_slot & 31);
        }
        wave_sync();
        uint32_t head = 0, tail = 1;
        const uint64_t base = static_cast<uint64_t>(bound_of(static_cast<uint32_t>(from))) << shift;
        uint64_t B = base;  // limits and sums in 64 bits: a bound may exceed 2^31 (then the leg has no path)
        uint32_t dto = from == to ? 0u : static_cast<uint32_t>(kInf);
        while (true) {
            uint32_t turned = ~0u;  // the smallest distance + bound beyond B (below 2^32 - 1, or saturated)
            while (head != tail && !hard_q) {
                // 64 / GS switches of the ring; one lane group each
                const uint32_t n = tail - head;
                const bool mine = static_cast<uint32_t>(grp) < n;
                uint32_t v = 0, dv = 0;
                int2 r = make_int2(0, 0);
                if (mine) {
                    const uint32_t sl = ring[(head + grp) & (kSlots - 1)];
                    if (gl == 0) atomicAnd(&inq[sl >> 5], ~(1u << (sl & 31)));
                    const unsigned long long e = tab[sl];
                    v = static_cast<uint32_t>(e & 0x7FFFu);
                    dv = static_cast<uint32_t>(e >> 16);
                    r = range[v];
                }
                head += n < kNG ? n : kNG;
                wave_sync();
                for (int32_t p0 = 0; __ballot(r.x + p0 < r.y) != 0; p0 += GS * kUn) {
                    ++steps;
                    int2 L[kUn];
                    uint32_t hb[kUn];
#pragma unroll
                    for (int k = 0; k < kUn; ++k) {
                        const int32_t p = r.x + p0 + k * GS + gl;
                        L[k] = p < r.y ? link[p] : make_int2(static_cast<int>(kNoPeer | 32u << 16), 0);
                    }
#pragma unroll
                    for (int k = 0; k < kUn; ++k) {
                        const uint32_t x = static_cast<uint32_t>(L[k].x), g = x >> 16;
                        const bool ok = g < 32 && ((A >> (g & 31)) & 1u);
                        if (!ok) L[k].x = static_cast<int>(kNoPeer);
                        hb[k] = ok ? bound_of(x & 0xFFFFu) : 0u;
                    }
#pragma unroll
                    for (int k = 0; k < kUn; ++k) {
                        const uint32_t u = static_cast<uint32_t>(L[k].x) & 0xFFFFu;
                        // distances are below 2^31 - 1; a heavier sum is no path
                        const uint32_t nd = dv + min(static_cast<uint32_t>(L[k].y), static_cast<uint32_t>(kInf));
                        const uint64_t f = static_cast<uint64_t>(nd) + (static_cast<uint64_t>(hb[k]) << shift);
                        bool keep = u != kNoPeer && nd < static_cast<uint32_t>(kInf) && f <= dto;
                        if (keep && f > B) {
                            turned = min(turned, static_cast<uint32_t>(f < 0xFFFFFFFEull ? f : 0xFFFFFFFEull));
                            keep = false;
                        }
                        bool fresh = false, push = false;
                        uint32_t h = 0;
                        if (keep) {
                            const unsigned long long want = static_cast<unsigned long long>(nd) << 16 | u;
                            h = slot_of(u);
                            while (true) {
                                unsigned long long e = tab[h];
                                if (e == kEmpty) {
                                    e = atomicCAS(&tab[h], kEmpty, want);
                                    if (e == kEmpty) {
                                        fresh = push = true;
                                        break;
                                    }
                                }
                                if ((e & 0x7FFFu) == u) {
                                    // (a forbidden switch's entry is below every distance)
                                    if (!(e & kForbid) && want < e) push = atomicMin(&tab[h], want) > want;
                                    break;
                                }
                                h = (h + 1) & (kSlots - 1);
                            }
                        }
                        if (push) push = !((atomicOr(&inq[h >> 5], 1u << (h & 31)) >> (h & 31)) & 1u);
                        if (__ballot(keep && u == static_cast<uint32_t>(to))) {
                            uint32_t d = keep && u == static_cast<uint32_t>(to) ? nd : static_cast<uint32_t>(kInf);
#pragma unroll
                            for (int off = 32; off > 0; off >>= 1) d = min(d, static_cast<uint32_t>(__shfl_xor(d, off, 64)));
                            dto = min(dto, d);
                        }
                        const uint64_t pm = __ballot(push);
                        if (push) {
                            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                                static_cast<uint32_t>(pm >> 32),
                                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(pm), 0u));
                            ring[(tail + below) & (kSlots - 1)] = static_cast<uint16_t>(h);
                        }
                        tail += static_cast<uint32_t>(__popcll(pm));
                        stored += static_cast<int32_t>(__popcll(__ballot(fresh)));
                        if (stored > kFull) break;  // room for one more round of 64 is left either way
                    }
                    wave_sync();
                    if (stored > kFull || steps > max_steps) {
                        hard_q = true;
                        break;
                    }
                }
            }
            if (hard_q || dto <= B) break;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) turned = min(turned, static_cast<uint32_t>(__shfl_xor(turned, off, 64)));
            if (turned == ~0u) break;  // nothing was turned away: no path (or the end's distance stands)
            const uint64_t wider = B + (B - base) / 2;
            B = turned > wider ? turned : wider;
            // every kept switch again, with the wider limit
            head = 0;
            tail = 0;
            for (int i = 0; i < kSlots / 64; ++i) {
                const int sl = i * 64 + lane;
                const unsigned long long e = tab[sl];
                const bool in = e != kEmpty && !(e & kForbid);
                const uint64_t pm = __ballot(in);
                if (in) {
                    const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                        static_cast<uint32_t>(pm >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(pm), 0u));
                    ring[tail + below] = static_cast<uint16_t>(sl);
                }
                if (lane < 2) inq[2 * i + lane] = static_cast<uint32_t>(pm >> (32 * lane));
                tail += static_cast<uint32_t>(__popcll(pm));
            }
            wave_sync();
        }
        if (hard_q) break;
        if (dto == static_cast<uint32_t>(kInf)) {
            fail = true;
            break;
        }
        // walk back from `to`: the lowest-numbered predecessor on a minimum-weight path
        int32_t c = to, n = 1;
        uint32_t dc = dto;
        if (lane == 0) leg[0] = static_cast<uint16_t>(to);
        while (c != from) {
            if (total + n > max_hops) {
                fail = true;
                break;
            }
            int32_t best = INT32_MAX;
            uint32_t bd = 0;
            for (int32_t k = rin_off[c] + lane; k < rin_off[c + 1]; k += 64) {
                const int2 in = rin[k];
                const uint32_t w = min(static_cast<uint32_t>(in.y), static_cast<uint32_t>(kInf));
                if (w > dc || in.x >= best) continue;
                uint32_t h = slot_of(static_cast<uint32_t>(in.x));
                while (true) {
                    const unsigned long long e = tab[h];
                    if (e == kEmpty) break;
                    if ((e & 0x7FFFu) == static_cast<uint32_t>(in.x)) {
                        if (!(e & kForbid) && static_cast<uint32_t>(e >> 16) + w == dc) {
                            best = in.x;
                            bd = dc - w;
                        }
                        break;
                    }
                    h = (h + 1) & (kSlots - 1);
                }
            }
            const int32_t least = wave_min_i32(best);
            if (least == INT32_MAX) {
                fail = true;
                break;
            }
            const int who = static_cast<int>(__builtin_ctzll(__ballot(best == least)));
            c = least;
            dc = __builtin_amdgcn_readlane(bd, who);
            if (lane == 0) leg[n] = static_cast<uint16_t>(c);
            ++n;
        }
        wave_sync();
        if (fail) break;
        for (int32_t i = 1 + lane; i < n; i += 64) walk[total + i] = leg[n - 1 - i];
        total += n - 1;
        wave_sync();
        from = to;
    }
    if (hard_q) {
        if (lane == 0) hard[atomicAdd(n_hard, 1)] = q;
        return;
    }
    const int32_t slots = max_hops + 1;
    if (lane == 0) hops_out[q] = fail ? -1 : total;
    int32_t *pq = path_out + static_cast<int64_t>(q) * slots;
    for (int32_t k = lane; k < slots; k += 64) pq[k] = (!fail && k <= total) ? walk[k] : -1;
    // the port of least (weight, index) to the next switch: one lane group per switch of the walk
    for (int32_t k0 = 0; !fail && k0 < total; k0 += kNG) {
        const int32_t k = k0 + grp;
        uint64_t best = UINT64_MAX;  // (weight << 32) | local port
        if (k < total) {
            const int2 r = range[walk[k]];
            const uint32_t nx = walk[k + 1];
            for (int32_t p = r.x + gl; p < r.y; p += GS) {
                const int2 L = link[p];
                if ((static_cast<uint32_t>(L.x) & 0xFFFFu) == nx) {
                    const uint64_t x = static_cast<uint64_t>(static_cast<uint32_t>(L.y)) << 32 |
                                       static_cast<uint32_t>(p - r.x);
                    best = x < best ? x : best;
                }
            }
        }
#pragma unroll
        for (int off = GS / 2; off > 0; off >>= 1) {
            const uint64_t o = __shfl_xor(best, off, 64);
            best = o < best ? o : best;
        }
        if (gl == 0 && k < total) act[k] = static_cast<uint16_t>(best & 0xFFFFu);
    }
    if (lane == 0 && !fail) act[total] = static_cast<uint16_t>(out_port[q]);
    wave_sync();
    // 10 dwords per slot: value[4], mask[4], priority | action << 16, rsv
    const pc_key kq = key[q];
    uint32_t *rq = reinterpret_cast<uint32_t *>(rules_out + static_cast<int64_t>(q) * slots);
    for (int32_t i = lane; i < slots * 10; i += 64) {
        const int32_t k = i / 10, d = i - 10 * k;
        uint32_t x = 0;
        if (!fail && k <= total) {
            x = d < 4 ? (d < 2 ? (d ? kq.w[1] : kq.w[0]) : (d == 2 ? kq.w[2] : kq.w[3]))
              : d < 7 ? 0xFFFFFFFFu
              : d == 7 ? 0xFFu
              : d == 8 ? static_cast<uint32_t>(prio) | static_cast<uint32_t>(act[k]) << 16
                       : 0u;
        }
        rq[i] = x;
    }
}

// One workgroup per request (see the file header).  Dynamic LDS: dist,
// two frontier queues (V each), the round flags and the usable bits
// (ceil(V/32) words each), the walk and one leg (max_hops + 2 each).
__global__ __launch_bounds__(kPsThreads) void k_ps_search(
    int32_t V, const int32_t *__restrict__ port_off, const int32_t *__restrict__ port_peer, int64_t n_ports,
    const uint32_t *__restrict__ weight, const uint8_t *__restrict__ region, const int32_t *__restrict__ rin_off,
    const int2 *__restrict__ rin, const int32_t *__restrict__ src, const int32_t *__restrict__ target,
    const uint32_t *__restrict__ allowed, const int32_t *__restrict__ via, int32_t Kv,
    const int32_t *__restrict__ forbid, int32_t Kf, const pc_key *__restrict__ key,
    const int32_t *__restrict__ out_port, int32_t prio, int32_t max_hops, int32_t *__restrict__ hops_out,
    int32_t *__restrict__ path_out, pc_rule *__restrict__ rules_out, int32_t Q,
    const unsigned long long *__restrict__ span, const int32_t *__restrict__ list, const int32_t *__restrict__ n_list, const uint32_t *__restrict__ wspan)
{
    extern __shared__ int32_t ps_lds[];
    const int32_t VW = (V + 31) >> 5;
    int32_t *dist = ps_lds;
    int32_t *qa = dist + V;
    int32_t *qb = qa + V;
    uint32_t *inflag = reinterpret_cast<uint32_t *>(qb + V);
    uint32_t *usable = inflag + VW;
    int32_t *walk = reinterpret_cast<int32_t *>(usable + VW);
    int32_t *leg = walk + max_hops + 2;
    __shared__ int32_t s_nf, s_fail, s_total;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t slots = max_hops + 1;
    const bool lists = in_lists(span, n_ports);
    if (list && undirected(wspan, span, n_ports)) list = nullptr;  // the directed search took none
    const int32_t n_req = list ? *n_list : Q;
    for (int32_t at = blockIdx.x; at < n_req; at += gridDim.x) {
    const int32_t q = list ? list[at] : at;
    const int32_t s = src[q], t = target[q];
    bool fail = s < 0 || s >= V || t < 0 || t >= V;
    if (!fail) {
        const int64_t tb = port_off[t], te = port_off[t + 1];
        fail = !pc_range_ok(tb, te, n_ports) || out_port[q] < 0 || out_port[q] >= te - tb;
    }
    const uint32_t A = allowed[q];
    // usable bits: each wavefront takes 64 switches (two words) at a time
    for (int32_t v0 = wave * 64; v0 < V; v0 += kPsWaves * 64) {
        const int32_t v = v0 + lane;
        const uint32_t r = v < V ? region[v] : 32u;
        const uint64_t m = __ballot(r < 32 && ((A >> r) & 1u));
        if (lane < 2 && (v0 >> 5) + lane < VW) usable[(v0 >> 5) + lane] = static_cast<uint32_t>(m >> (32 * lane));
    }
    __syncthreads();
    if (tid < Kf) {
        const int32_t f = forbid[static_cast<int64_t>(q) * Kf + tid];
        if (f >= 0 && f < V) atomicAnd(&usable[f >> 5], ~(1u << (f & 31)));
    }
    if (tid == 0) {
        s_fail = fail;
        s_total = 0;
        if (!fail) walk[0] = s;
    }
    __syncthreads();
    int32_t m = 0;  // waypoints: the list ends at its first -1
    while (m < Kv && via[static_cast<int64_t>(q) * Kv + m] != -1) ++m;
    auto is_usable = [&](int32_t v) { return (usable[v >> 5] >> (v & 31)) & 1u; };

    int32_t from = s;
    for (int32_t li = 0; li <= m && !s_fail; ++li) {
        const int32_t to = li < m ? via[static_cast<int64_t>(q) * Kv + li] : t;
        if (to < 0 || to >= V || !is_usable(from) || !is_usable(to)) break;  // uniform: s_fail set below
        for (int32_t v = tid; v < V; v += kPsThreads) dist[v] = kInf;
        for (int32_t w = tid; w < VW; w += kPsThreads) inflag[w] = 0;
        __syncthreads();
        if (tid == 0) {
            dist[from] = 0;
            qa[0] = from;
            s_nf = 0;
        }
        __syncthreads();
        int32_t nf = 1;
        int32_t *cur = qa, *nxt = qb;
        // Port p's peer and weight: unconditional loads (an index past the
        // switch's last port is clamped to it; the caller drops that lane),
        // whose results nothing touches before relax, so that a wavefront's
        // next switch is fetched while the current one is relaxed.
        const uint32_t *wsrc = weight ? weight : reinterpret_cast<const uint32_t *>(port_peer);
        auto fetch = [&](int64_t p, int64_t e, int32_t &u, uint32_t &w) {
            const int64_t pc = p < e ? p : e - 1;
            u = port_peer[pc];
            w = wsrc[pc];
        };
        // (dto: the target's distance when the switch was taken, an upper
        // bound of the current one, so the pruning stays safe)
        auto relax = [&](int32_t u, uint32_t w, int32_t dv, int32_t dto, int32_t *nxt) {
            if (!weight) w = 1u;
            const bool link = u >= 0 && u < V && w;
            const int32_t uc = link ? u : 0;
            const uint32_t ubits = usable[uc >> 5];  // both LDS reads issued together
            const int32_t du = dist[uc];
            // 32-bit unsigned: distances are below kInf = 2^31 - 1 and a weight
            // of 2^31 - 1 or more cannot shorten any path, so clamping it
            // keeps the sum exact where it matters and below 2^32
            const uint32_t nd32 = static_cast<uint32_t>(dv) + min(w, static_cast<uint32_t>(kInf));
            if (!link || !((ubits >> (uc & 31)) & 1u) || nd32 >= static_cast<uint32_t>(du) ||
                nd32 >= static_cast<uint32_t>(dto))
                return;
            const int32_t nd = static_cast<int32_t>(nd32);
            const int32_t old = atomicMin(&dist[u], nd);
            if (nd < old) {
                const uint32_t bit = 1u << (u & 31);
                if (!(atomicOr(&inflag[u >> 5], bit) & bit)) nxt[atomicAdd(&s_nf, 1)] = u;
            }
        };
        while (nf > 0) {
            // Wavefront `wave` takes frontier entries wave, wave + kPsWaves, ...
            // in batches of 64: each lane reads one entry's port range (one
            // round of loads for 64 switches), then the switches are
            // relaxed one after another, each one's first 64 links loaded
            // while the previous one's are relaxed (two register sets, A
            // and B, in turn).
            for (int32_t base = wave; base < nf; base += kPsWaves * 64) {
                const int32_t idx = base + lane * kPsWaves;
                int32_t vl = 0, bl = 0, el = 0;
                if (idx < nf) {
                    vl = cur[idx];
                    if (dist[vl] < dist[to]) {  // else it cannot shorten the target's path
                        const int32_t b = port_off[vl], e = port_off[vl + 1];
                        if (pc_range_ok(b, e, n_ports)) {
                            bl = b;
                            el = e;
                        }
                    }
                }
                uint64_t live = __ballot(el > bl);
                if (!live) continue;
                // the next switch of the batch (none left: `prev` again, with more = false)
                auto take = [&](int32_t prev, bool &more, int32_t &b, int32_t &e) {
                    more = live != 0;
                    const int32_t jj = more ? static_cast<int32_t>(__builtin_ctzll(live)) : prev;
                    live &= live - 1;
                    b = __builtin_amdgcn_readlane(bl, jj);
                    e = __builtin_amdgcn_readlane(el, jj);
                    return jj;
                };
                auto expand = [&](int32_t jj, int32_t b, int32_t e, int32_t u, uint32_t w) {
                    const int32_t dv = dist[__builtin_amdgcn_readlane(vl, jj)];  // current: it may have dropped
                    const int32_t dto = dist[to];
                    if (static_cast<int64_t>(b) + lane < e) relax(u, w, dv, dto, nxt);
                    for (int64_t p = static_cast<int64_t>(b) + 64 + lane; p < e; p += 64) {
                        int32_t u2;
                        uint32_t w2;
                        fetch(p, e, u2, w2);
                        relax(u2, w2, dv, dto, nxt);
                    }
                };
                bool more;
                int32_t bA, eA, bB, eB, uA, uB;
                uint32_t wA, wB;
                int32_t jA = take(0, more, bA, eA);
                fetch(static_cast<int64_t>(bA) + lane, eA, uA, wA);
                while (true) {
                    const int32_t jB = take(jA, more, bB, eB);
                    fetch(static_cast<int64_t>(bB) + lane, eB, uB, wB);
                    expand(jA, bA, eA, uA, wA);
                    if (!more) break;
                    jA = take(jB, more, bA, eA);
                    fetch(static_cast<int64_t>(bA) + lane, eA, uA, wA);
                    expand(jB, bB, eB, uB, wB);
                    if (!more) break;
                }
            }
            __syncthreads();
            nf = s_nf;
            __syncthreads();
            for (int32_t i = tid; i < nf; i += kPsThreads) {
                const int32_t u = nxt[i];
                atomicAnd(&inflag[u >> 5], ~(1u << (u & 31)));
            }
            if (tid == 0) s_nf = 0;
            int32_t *tmp = cur;
            cur = nxt;
            nxt = tmp;
            __syncthreads();
        }
        if (dist[to] == kInf) break;  // no path: s_fail set below
        if (wave == 0) {
            // walk back from `to`: the lowest-numbered predecessor on a minimum-weight path
            const int32_t total = s_total;
            int32_t c = to, n = 1;
            bool bad = false;
            if (lane == 0) leg[0] = to;
            while (c != from) {
                if (total + n > max_hops) {
                    bad = true;
                    break;
                }
                int32_t best = INT32_MAX;
                const int32_t dc = dist[c];
                auto pred = [&](int32_t u, uint32_t w) {
                    const int32_t du = dist[u];
                    if (du != kInf && static_cast<uint32_t>(du) + min(w, static_cast<uint32_t>(kInf)) ==
                                          static_cast<uint32_t>(dc))
                        best = min(best, u);
                };
                if (lists) {
                    for (int32_t k = rin_off[c] + lane; k < rin_off[c + 1]; k += 64) {
                        const int2 in = rin[k];
                        pred(in.x, static_cast<uint32_t>(in.y));
                    }
                } else {  // overlapping port ranges: the links of every switch the leg has reached
                    for (int32_t u = lane; u < V; u += 64) {
                        if (dist[u] == kInf) continue;
                        const int64_t b = port_off[u], e = port_off[u + 1];
                        if (!pc_range_ok(b, e, n_ports)) continue;
                        for (int64_t p = b; p < e; ++p) {
                            const uint32_t w = link_weight(port_peer, weight, V, p);
                            if (w && port_peer[p] == c) pred(u, w);
                        }
                    }
                }
                best = wave_min_i32(best);
                if (best == INT32_MAX) {
                    bad = true;
                    break;
                }
                c = best;
                if (lane == 0) leg[n] = c;
                ++n;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (bad) {
                if (lane == 0) s_fail = 1;
            } else {
                for (int32_t i = 1 + lane; i < n; i += 64) walk[total + i] = leg[n - 1 - i];
                if (lane == 0) s_total = total + n - 1;
            }
        }
        __syncthreads();
        from = to;
        if (li == m && !s_fail) from = -1;  // the walk reached the target
    }
    // a leg that broke off before its walk (bad stop or no path) leaves from != -1
    if (tid == 0 && from != -1) s_fail = 1;
    __syncthreads();

    const bool ok = !s_fail;
    const int32_t total = s_total;
    if (tid == 0) hops_out[q] = ok ? total : -1;
    int32_t *pq = path_out + static_cast<int64_t>(q) * slots;
    for (int32_t k = tid; k < slots; k += kPsThreads) pq[k] = (ok && k <= total) ? walk[k] : -1;
    // rules: one wavefront per switch of the walk finds its port to the next switch
    uint32_t *rq = reinterpret_cast<uint32_t *>(rules_out + static_cast<int64_t>(q) * slots);
    for (int32_t k = wave; k < slots; k += kPsWaves) {
        uint32_t action = 0;
        const bool live = ok && k <= total;
        if (live && k < total) {
            const int32_t a = walk[k], bnext = walk[k + 1];
            const int64_t pb = port_off[a], pe = port_off[a + 1];
            uint64_t best = UINT64_MAX;  // (weight << 32) | local port
            for (int64_t p = pb + lane; p < pe; p += 64) {
                const uint32_t w = link_weight(port_peer, weight, V, p);
                if (w && port_peer[p] == bnext) {
                    const uint64_t c = (static_cast<uint64_t>(w) << 32) | static_cast<uint64_t>(p - pb);
                    best = c < best ? c : best;
                }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const uint64_t o = __shfl_xor(best, off, 64);
                best = o < best ? o : best;
            }
            action = static_cast<uint32_t>(best & 0xFFFFu);
        } else if (live) {
            action = static_cast<uint32_t>(out_port[q]) & 0xFFFFu;
        }
        // 10 dwords: value[4], mask[4], priority | action << 16, rsv
        if (lane < 10) {
            uint32_t d = 0;
            if (live) {
                if (lane < 4)
                    d = key[q].w[lane];
                else if (lane < 7)
                    d = 0xFFFFFFFFu;
                else if (lane == 7)
                    d = 0xFFu;
                else if (lane == 8)
                    d = static_cast<uint32_t>(prio) | (action << 16);
            }
            rq[static_cast<int64_t>(k) * 10 + lane] = d;
        }
    }
    __syncthreads();  // the next request reuses the LDS
    }
}

}  // namespace

int run_synthesize(pc_ctx *ctx, int32_t V, const int32_t *port_off, const int32_t *port_peer, int64_t n_ports,
                   const uint32_t *weight, const uint8_t *region, int32_t Q, const int32_t *src, const int32_t *target,
                   const uint32_t *allowed, const int32_t *via, int32_t Kv, const int32_t *forbid, int32_t Kf,
                   const pc_key *key, const int32_t *out_port, int32_t prio, int32_t max_hops, int32_t *hops,
                   int32_t *path, pc_rule *rules, hipStream_t stream)
{
    // The directed search pays for its bounds (a row per switch that legs end
    // at, at most V, each about as dear as one undirected leg) and for four
    // more launches, about 25 million links' worth of undirected search.
    // Undirected / directed at weights 1-10, one leg per request: 138,240
    // ports and 1,440 legs 357 / 328 us, 5,760 legs 939 / 343 us; 17,280 ports
    // and 720 legs 87 / 139 us, 1,440 legs 132 / 144 us, 2,880 legs 201 / 160 us;
    // 2,160 ports and 1,440 legs 65 / 106 us.
    const int64_t legs = static_cast<int64_t>(Q) * (Kv + 1);
    bool directed = weight != nullptr && V > 0 && n_ports > 0 && n_ports < (int64_t(1) << 30) &&
                    legs >= V + 25'000'000 / n_ports;
    const size_t n_rows = directed ? static_cast<size_t>(V) : 0;
    // zeroed together: the valid ranges' ports, in-link counts, needed rows, the hard requests' count, the weights' span
    unsigned long long *span;
    int32_t *cnt, *need, *n_hard, *rin_off, *cursor, *row, *ends, *row_ok, *hard;
    int2 *rin, *link, *range;
    uint32_t *blink, *wspan, *bound;
    const size_t n_zero = static_cast<size_t>(V) * 2 + 8;
    auto carve = [&](Carver &cv, bool with) {
        span = reinterpret_cast<unsigned long long *>(cv.take<int32_t>(n_zero));
        cnt = reinterpret_cast<int32_t *>(span + 1);
        rin_off = cv.take<int32_t>(static_cast<size_t>(V) + 1);
        cursor = cv.take<int32_t>(static_cast<size_t>(V) + 1);
        rin = cv.take<int2>(static_cast<size_t>(n_ports) + 1);
        if (!with) return;
        need = cnt + V + 1;
        n_hard = need + V;
        wspan = reinterpret_cast<uint32_t *>(n_hard + 1);
        row = cv.take<int32_t>(static_cast<size_t>(V) + 1);
        ends = cv.take<int32_t>(static_cast<size_t>(V));
        row_ok = cv.take<int32_t>(static_cast<size_t>(V));
        hard = cv.take<int32_t>(static_cast<size_t>(Q));
        link = cv.take<int2>(static_cast<size_t>(n_ports) + 1);
        blink = cv.take<uint32_t>(static_cast<size_t>(n_ports) + 1);
        range = cv.take<int2>(static_cast<size_t>(V));
        bound = cv.take<uint32_t>(n_rows * V);
    };
    Carver dry{nullptr, 0};
    carve(dry, directed);
    int rc = pc_ensure_arena(ctx, dry.off);
    if (rc == PC_ENOMEM && directed) {  // no room for the bounds: the undirected search needs none
        directed = false;
        dry.off = 0;
        carve(dry, false);
        rc = pc_ensure_arena(ctx, dry.off);
        if (rc == PC_OK) ctx->msg[0] = 0;
    }
    if (rc) return rc;
    Carver real{ctx->arena, 0};
    carve(real, directed);

    int64_t tot = std::max<int64_t>({static_cast<int64_t>(V), n_ports, static_cast<int64_t>(Q) * std::max(Kv, 1),
                                     static_cast<int64_t>(Q) * std::max(Kf, 1)});
    if (Q > 0) launch_fill_u32(reinterpret_cast<uint32_t *>(span), n_zero, 0, stream);
    PC_LAUNCH_CHECK(ctx);
    const unsigned g_all = static_cast<unsigned>(std::min<int64_t>((tot + 255) / 256, 8192));
    if (tot > 0) {
        PC_TIMED(ctx, "k_ps_validate", stream,
                 hipLaunchKernelGGL(k_ps_validate, dim3(g_all), dim3(256), 0, stream, V, port_off, port_peer, n_ports,
                                    weight, region, Q, src, target, out_port, via, Kv, forbid, Kf,
                                    Q > 0 ? span : nullptr, ctx->d_err));
        PC_LAUNCH_CHECK(ctx);
    }
    if (Q == 0) return PC_OK;
    if (V > 0) {
        const unsigned g = static_cast<unsigned>((static_cast<int64_t>(V) * kInLanes + 255) / 256);
        PC_TIMED(ctx, "k_ps_in_count", stream,
                 hipLaunchKernelGGL(k_ps_in_count, dim3(g), dim3(256), 0, stream, V, port_off, port_peer, n_ports,
                                    weight, span, cnt));
        PC_LAUNCH_CHECK(ctx);
        launch_scan_i32(cnt, V, rin_off, cursor, nullptr, stream);
        PC_LAUNCH_CHECK(ctx);
        PC_TIMED(ctx, "k_ps_in_fill", stream,
                 hipLaunchKernelGGL(k_ps_in_fill, dim3(g), dim3(256), 0, stream, V, port_off, port_peer, n_ports,
                                    weight, span, cursor, rin));
        PC_LAUNCH_CHECK(ctx);
    }
    if (directed) {
        const unsigned g = static_cast<unsigned>(std::min<int64_t>((std::max<int64_t>(n_ports, V) + 255) / 256, 4096));
        PC_TIMED(ctx, "k_ps_survey", stream,
                 hipLaunchKernelGGL(k_ps_survey, dim3(std::min(g_all, 1024u) + 1), dim3(256), 0, stream, V, port_peer,
                                    n_ports, weight, Q, target, via, Kv, need, wspan));
        launch_scan_i32(need, V, row, nullptr, nullptr, stream);
        PC_TIMED(ctx, "k_ps_links", stream,
                 hipLaunchKernelGGL(k_ps_links, dim3(g), dim3(256), 0, stream, V, port_off, port_peer, n_ports,
                                    weight, region, need, row, wspan, link, blink,
                                    range, ends));
        PC_LAUNCH_CHECK(ctx);
        // lanes per switch: a power of two near a third of the mean degree
        const int64_t avg = n_ports / V;
        const int gs = avg <= 12 ? 4 : avg <= 24 ? 8 : 16;
        // eight rows per workgroup where two such workgroups fit a CU's LDS and
        // enough of them remain to fill the chip, else four
        const int words = V > 1024 && V <= 4800 ? 4 : 2;
        const size_t lds_b = ((static_cast<size_t>(V) + 15) & ~size_t(15)) * 4 * words;
        const size_t lds_g = static_cast<size_t>(max_hops + 2) * 3 * sizeof(uint16_t);
        // a request that relaxes more links than the whole graph holds (a few
        // times over) is not being directed: the workgroup search takes it
        const int32_t max_steps = static_cast<int32_t>(std::min<int64_t>(64 + n_ports / 64, INT32_MAX / 2));
        auto launch = [&](auto bk, auto gk) -> int {
            PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(bk),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_b)));
            PC_TIMED(ctx, "k_ps_bound", stream,
                     hipLaunchKernelGGL(bk, dim3(static_cast<unsigned>((V + words - 1) / words)), dim3(256 * words), lds_b,
                                        stream, V, range, blink, link, ends, row + V, wspan, span, n_ports, bound,
                                        row_ok));
            PC_TIMED(ctx, "k_ps_goal", stream,
                     hipLaunchKernelGGL(gk, dim3(static_cast<unsigned>(Q)), dim3(64), lds_g, stream, V, n_ports, range,
                                        link, region, rin_off, rin, row, row_ok, bound,
                                        wspan, src, target, allowed, via, Kv,
                                        forbid, Kf, key, out_port, prio, max_hops, hops, path, rules, span, max_steps,
                                        hard, n_hard));
            PC_LAUNCH_CHECK(ctx);
            return PC_OK;
        };
        const auto goal = gs == 4 ? k_ps_goal<4> : gs == 8 ? k_ps_goal<8> : k_ps_goal<16>;
        rc = avg <= 12 ? (words == 4 ? launch(k_ps_bound<4, 3, 4>, goal) : launch(k_ps_bound<4, 3, 2>, goal))
                       : (words == 4 ? launch(k_ps_bound<1, 12, 4>, goal) : launch(k_ps_bound<1, 12, 2>, goal));
        if (rc) return rc;
    }
    const int32_t VW = (V + 31) / 32;
    const size_t lds = (static_cast<size_t>(V) * 3 + static_cast<size_t>(VW) * 2 +
                        2 * static_cast<size_t>(max_hops + 2)) * 4;
    PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(k_ps_search),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
    // after the directed search: the requests it left, by a grid that walks their list
    const unsigned grid = static_cast<unsigned>(directed ? std::min(Q, 16384) : Q);
    PC_TIMED(ctx, "k_ps_search", stream,
             hipLaunchKernelGGL(k_ps_search, dim3(grid), dim3(kPsThreads), lds, stream, V,
                                port_off, port_peer, n_ports, weight, region, rin_off, rin, src, target, allowed, via,
                                Kv, forbid, Kf, key, out_port, prio, max_hops, hops, path, rules,
                                Q, span, directed ? hard : nullptr, directed ? n_hard : nullptr,
                                directed ? wspan : nullptr));
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}
