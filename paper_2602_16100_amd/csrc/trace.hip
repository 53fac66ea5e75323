// A2-A4 -- routing constraints on the realised paths: trace every header
// hop by hop through the per-switch, priority-ordered ternary flow tables
// and collect the jurisdictions visited.
//
// The paper compiles every path into one flow rule per hop (Network
// orchestration), and a routing constraint is judged on the paths those
// rules actually realise (Formal Model and Satisfaction, condition (ii)); the
// validator checks that realised paths avoid forbidden switches (validator
// check definition).  The first-match rule order (larger priority, then
// lower index), table miss, drop, egress and TTL are the readings written in
// include/pc.h.
//
// Design (gfx950):
//   prep   : per switch, kChunks 4-bit chunks of the 104-bit key chosen from
//            a sample of its rules and of the headers (the chunks on which
//            its rules discriminate most among the headers seen); per
//            32-rule group, for each chunk and each of the 16 chunk values,
//            the 32-bit set of rules whose mask/value admit that value (per-
//            rule admit sets from an LDS table, then a bit transpose across
//            the half-wavefront).  Stored plane-major per switch so a
//            wavefront loads 64 groups with coalesced reads.  Also validates
//            ports, jurisdictions, offsets and actions (the data-error sweep).
//   levels : level-synchronous walk.  Live traces are bucketed by their
//            current switch: a plan pass scans the per-switch counts, a
//            scatter pass writes each trace's 32-byte bucket record (trace,
//            jurisdiction mask, header) at its switch's offset plus its
//            rank.  One workgroup per work item (a switch and a balanced
//            share of its bucket) keeps the switch's chunk sets in LDS
//            (4,096 rules a slice) or, few lookups per table, in VGPRs,
//            and filters every lookup with kChunks reads and ANDs; the
//            survivors of the highest priorities are verified against the full
//            104-bit rule and the first match is the minimum of (0xFFFF -
//            priority, index) (LDS 64-bit atomic min).  The same workgroup then
//            applies the match with the switch's ports staged in LDS, counts
//            the moving traces per forwarding port (one count update per
//            port and workgroup, which also gives each trace its rank in its
//            next switch's bucket) and writes their live-list entries in its
//            own share of the list, grouped by port.
//   tail   : once few traces are left in flight (walk_most), one workgroup per
//            trace walks it to its end, reading only the chunk-set words its
//            header selects, and skipping whole turns of a loop.
//   direct : few traces over small tables are walked rule by rule in one
//            launch, without chunk sets.
#include <stdlib.h>

#include <algorithm>

#include "pc_internal.h"

namespace {

constexpr int kChunks = 6;                 // 4-bit chunks of the key used by the filter (chosen per switch)
constexpr int kKeyNibbles = 26;            // the 104-bit key: 8 nibbles in each of w0..w2, 2 in w3's low byte
constexpr int kChooseSample = 256;         // rules per switch sampled to choose its filter chunks
constexpr int kPlaneWords = kChunks * 16;  // words per 32-rule group
constexpr int kMatchWaves = 8;
constexpr int kMatchThreads = kMatchWaves * 64;
constexpr int kSliceGroups = 128;            // groups whose chunk sets a match workgroup holds in LDS (48 KB)
constexpr int kChunk = kMatchThreads;        // lookups matched together at most (one epilogue thread each)
constexpr int kItemMax = kChunk;             // lookups per work item at most
constexpr int kItemLeast = 384;              // the same of a small level
constexpr int64_t kItemsWanted = 4096;       // work items of a large level
constexpr int kQueue = 128;                  // queued filter survivors per wavefront (>= 64)
constexpr int kWideWaves = 4;                // k_tr_match_wide: a group (32 rules) per lane, its sets in registers
constexpr int kWideThreads = kWideWaves * 64;
constexpr int kWideItem = 192;               // lookups per work item
constexpr int kWideChunk = 256;              // the same, padded, at most
constexpr int kWideQueue = 512;              // queued filter survivors per wavefront (>= 4 x 64)
constexpr int kItemMin = kWideItem;          // lookups per work item, of either form, unless it is its switch's only one
constexpr int kPrepGroups = 128;             // groups per prep workgroup (16 wavefronts x 4 rounds x 2 groups)
constexpr uint64_t kNoMatch = ~0ull;
static_assert(kItemMin <= kChunk && kChunk <= kMatchWaves * 64, "a wavefront's lookups fit its lanes");
static_assert((kWideItem + 3) / 4 * 4 <= kWideChunk && kWideChunk <= kWideThreads, "one epilogue thread per lookup");
constexpr int kCountPad = 32;  // live-trace counters are 128 bytes apart: contended atomics on one line serialise
constexpr int32_t kDirectRules = 1024;               // mean rules per switch that a walk may match one by one,
constexpr int64_t kDirectWork = 5000000;             // traces times mean rules,
constexpr int64_t kDirectWorst = int64_t(1) << 26;   // traces times all rules,
constexpr int64_t kDirectTable = 40960;              // rules of one table,
constexpr int64_t kDirectTableWork = int64_t(3) << 23;  // and traces times these
constexpr int kDirectThreads = 256;                  // k_tr_direct's workgroup
constexpr int kPortSlots = 64;  // forwarding ports whose moves a match workgroup counts in LDS

// Bit k set iff slot k of trace t's watch list names switch s (K = 0: none).
__device__ __forceinline__ uint32_t watch_bits(const int32_t *__restrict__ watch, int32_t K, int32_t t, int32_t s)
{
    uint32_t m = 0;
    const int32_t *w = watch + static_cast<int64_t>(t) * K;
    for (int32_t k = 0; k < K; ++k)
        if (w[k] == s) m |= 1u << k;
    return m;
}

// Nibble n (0..25) of a 104-bit key or mask: bits 4(n mod 8) .. +3 of word n / 8.
__device__ __forceinline__ uint32_t key_nibble(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t n)
{
    const uint32_t w = n < 8 ? w0 : n < 16 ? w1 : n < 24 ? w2 : w3;
    return (w >> ((n & 7u) * 4u)) & 15u;
}

// Filter chunk c of a switch whose chunk positions are packed in cp (5 bits each).
__device__ __forceinline__ uint32_t chunk_pos(uint32_t cp, int c) { return (cp >> (5 * c)) & 31u; }

// Bit of switch s in a visited-switch summary.
__device__ __forceinline__ uint64_t sum_bit(int32_t s) { return 1ull << (s & 63); }

constexpr int kWalkSlots = 8;  // walk records: the first 8 switches of a walk

__device__ __forceinline__ uint32_t jur_bit(const uint8_t *jur, int32_t s)
{
    const uint32_t j = jur[s];
    return j < 32 ? (1u << j) : 0u;
}

// Per switch: validate offsets / jurisdiction, count 32-rule groups and prep
// blocks; *largest (cleared): the groups of the largest table.
__global__ void k_tr_switch_info(int32_t S, const int32_t *__restrict__ port_off, int64_t n_ports,
                                 const uint8_t *__restrict__ jur, const int32_t *__restrict__ rule_off,
                                 int64_t n_rules, int32_t *__restrict__ gcount, int32_t *__restrict__ bcount,
                                 int32_t *__restrict__ largest, uint32_t *__restrict__ d_err)
{
    uint32_t errs = 0;
    int32_t most = 0;
    for (int32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < S; s += gridDim.x * blockDim.x) {
        if (jur[s] >= 32) errs |= PC_DERR_JUR;
        const bool pok = pc_range_ok(port_off[s], port_off[s + 1], n_ports);
        const int64_t rb = rule_off[s], re = rule_off[s + 1];
        const bool rok = pc_range_ok(rb, re, n_rules);
        if (!pok || !rok) errs |= PC_DERR_OFFSETS;
        const int64_t g = rok ? (re - rb + 31) / 32 : 0;
        gcount[s] = static_cast<int32_t>(g);
        bcount[s] = static_cast<int32_t>((g + kPrepGroups - 1) / kPrepGroups);
        most = max(most, static_cast<int32_t>(g));
    }
    if (errs) atomicOr(d_err, errs);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, 64));
    if ((threadIdx.x & 63) == 0 && most > 0) atomicMax(largest, most);
}

// What a lookup at a switch starts from, in one 32-byte record.
struct __align__(32) SwInfo {
    int32_t G;        // 32-rule groups
    int32_t gofs;     // the first one's place in the chunk sets
    uint32_t cpos;    // filter chunks
    int32_t rb;       // first rule
    int32_t pb;       // first port
    int32_t np;       // ports, -1 when the port range is invalid
    int32_t R;        // rules
    int32_t pad;
};

__device__ __forceinline__ SwInfo make_info(int32_t s, const int32_t *__restrict__ port_off, int64_t n_ports,
                                            const int32_t *__restrict__ rule_off, int64_t n_rules, int32_t gofs,
                                            uint32_t cpos)
{
    const int64_t pb = port_off[s], pe = port_off[s + 1], rb = rule_off[s], re = rule_off[s + 1];
    const bool rok = pc_range_ok(rb, re, n_rules);
    SwInfo x;
    x.R = rok ? static_cast<int32_t>(re - rb) : 0;
    x.G = rok ? static_cast<int32_t>((re - rb + 31) / 32) : 0;
    x.gofs = gofs;
    x.cpos = cpos;
    x.rb = rok ? static_cast<int32_t>(rb) : 0;
    x.pb = static_cast<int32_t>(pb);
    x.np = pc_range_ok(pb, pe, n_ports) ? static_cast<int32_t>(pe - pb) : -1;
    x.pad = 0;
    return x;
}

// A port's peer and the peer's jurisdiction bit (0 unless the peer is a switch).
__device__ __forceinline__ int2 make_port(int32_t peer, int32_t S, const uint8_t *__restrict__ jur)
{
    const uint32_t j = peer >= 0 && peer < S ? jur[peer] : 32u;
    return make_int2(peer, j < 32 ? static_cast<int32_t>(1u << j) : 0);
}

// Per port and per switch the records above, of tables prepared by an
// earlier call.
__device__ __forceinline__ void port_infos(int64_t n_ports, const int32_t *__restrict__ port_off,
                                           const int32_t *__restrict__ port_peer, int32_t S,
                                           const uint8_t *__restrict__ jur, const int32_t *__restrict__ rule_off,
                                           int64_t n_rules, const int32_t *__restrict__ gofs,
                                           const uint32_t *__restrict__ cpos, int2 *__restrict__ pinfo,
                                           SwInfo *__restrict__ sinfo)
{
    const int64_t tot = n_ports > S ? n_ports : S;
    for (int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; p < tot;
         p += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (p < n_ports) pinfo[p] = make_port(port_peer[p], S, jur);
        if (p < S) {
            const int32_t s = static_cast<int32_t>(p);
            sinfo[s] = make_info(s, port_off, n_ports, rule_off, n_rules, gofs[s], cpos[s]);
        }
    }
}

__global__ void k_tr_port_info(int64_t n_ports, const int32_t *__restrict__ port_off,
                               const int32_t *__restrict__ port_peer, int32_t S, const uint8_t *__restrict__ jur,
                               const int32_t *__restrict__ rule_off, int64_t n_rules,
                               const int32_t *__restrict__ gofs, const uint32_t *__restrict__ cpos,
                               int2 *__restrict__ pinfo, SwInfo *__restrict__ sinfo)
{
    port_infos(n_ports, port_off, port_peer, S, jur, rule_off, n_rules, gofs, cpos, pinfo, sinfo);
}

// Input sweeps in one launch: ports (every peer -1 or a switch), watch
// lists (n_watch ids) and, with hh, the header histogram below.
__device__ __forceinline__ bool bad_ids(int64_t n, const int32_t *__restrict__ ids, int32_t S)
{
    bool bad = false;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int32_t v = ids[i];
        bad |= v < -1 || v >= S;
    }
    return bad;
}

// Histogram of the headers' nibble values over a strided sample of at most
// kHeaderSample headers: hh[n][x] = sampled headers whose nibble n is x.
// hh must be zero on entry.
constexpr int kHeaderSample = 65536;
constexpr size_t kHistWords = kKeyNibbles * 16 + 1;  // and the groups of the largest table (layout)
__global__ __launch_bounds__(256) void k_tr_sweep(int64_t n_ports, const int32_t *__restrict__ port_peer, int32_t S,
                                                  int64_t n_watch, const int32_t *__restrict__ watch,
                                                  const pc_key *__restrict__ hdr, int32_t T,
                                                  uint32_t *__restrict__ hh, uint32_t *__restrict__ d_err)
{
    __shared__ uint32_t loc[kKeyNibbles * 16];
    const bool bad_port = bad_ids(n_ports, port_peer, S), bad_watch = bad_ids(n_watch, watch, S);
    const bool bad = bad_port || bad_watch;
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(d_err, PC_DERR_SWITCH);
    if (hh == nullptr) return;
    for (int i = threadIdx.x; i < kKeyNibbles * 16; i += 256) loc[i] = 0;
    __syncthreads();
    const int64_t stride = T > kHeaderSample ? (static_cast<int64_t>(T) + kHeaderSample - 1) / kHeaderSample : 1;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i * stride < T; i += static_cast<int64_t>(gridDim.x) * 256) {
        const pc_key h = hdr[i * stride];
        for (uint32_t n = 0; n < kKeyNibbles; ++n)
            atomicAdd(&loc[n * 16 + key_nibble(h.w[0], h.w[1], h.w[2], h.w[3], n)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kKeyNibbles * 16; i += 256)
        if (loc[i]) atomicAdd(hh + i, loc[i]);
}

// Per switch the group count and the exclusive scans of group counts
// (gofs) and prep blocks (bofs), their totals at [S]; offsets and
// jurisdictions validated; the header histogram cleared for k_tr_sweep; the
// totals and the groups of the largest table to host memory.  One workgroup: with the separate kernels, three
// launches, a clear and two copies.
constexpr int32_t kLayoutS = 16384;  // switches at most
__global__ __launch_bounds__(1024) void k_tr_layout(int32_t S, const int32_t *__restrict__ port_off, int64_t n_ports,
                                                    const uint8_t *__restrict__ jur,
                                                    const int32_t *__restrict__ rule_off, int64_t n_rules,
                                                    int32_t *__restrict__ gcount, int32_t *__restrict__ gofs,
                                                    int32_t *__restrict__ bofs, uint32_t *__restrict__ hh,
                                                    int32_t *__restrict__ host, uint32_t *__restrict__ d_err)
{
    constexpr int kPer = 4;  // consecutive switches per thread and pass
    __shared__ int32_t wsum[2][16];
    __shared__ int32_t carry_s[2], most_s;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (tid < 2) carry_s[tid] = 0;
    if (tid == 2) most_s = 0;
    for (int i = tid; i < kKeyNibbles * 16; i += 1024) hh[i] = 0;
    __syncthreads();
    uint32_t errs = 0;
    int32_t most = 0;
    for (int32_t base = 0; base < S; base += 1024 * kPer) {
        const int32_t i0 = base + tid * kPer;
        int32_t g[kPer], b[kPer];
        int32_t s0 = 0, s1 = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            g[k] = b[k] = 0;
            const int32_t s = i0 + k;
            if (s >= S) continue;
            const int64_t rb = rule_off[s], re = rule_off[s + 1];
            const bool rok = pc_range_ok(rb, re, n_rules);
            if (jur[s] >= 32) errs |= PC_DERR_JUR;
            if (!rok || !pc_range_ok(port_off[s], port_off[s + 1], n_ports)) errs |= PC_DERR_OFFSETS;
            g[k] = rok ? static_cast<int32_t>((re - rb + 31) / 32) : 0;
            b[k] = (g[k] + kPrepGroups - 1) / kPrepGroups;
            gcount[s] = g[k];
            s0 += g[k];
            s1 += b[k];
            most = max(most, g[k]);
        }
        int32_t x0 = s0, x1 = s1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y0 = __shfl_up(x0, off, 64), y1 = __shfl_up(x1, off, 64);
            if (lane >= off) {
                x0 += y0;
                x1 += y1;
            }
        }
        if (lane == 63) {
            wsum[0][wid] = x0;
            wsum[1][wid] = x1;
        }
        __syncthreads();
        if (wid < 2) {
            int32_t w = lane < 16 ? wsum[wid][lane] : 0;
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                const int32_t y = __shfl_up(w, off, 64);
                if (lane >= off) w += y;
            }
            if (lane < 16) wsum[wid][lane] = w;
        }
        __syncthreads();
        int32_t e0 = carry_s[0] + (wid ? wsum[0][wid - 1] : 0) + x0 - s0;
        int32_t e1 = carry_s[1] + (wid ? wsum[1][wid - 1] : 0) + x1 - s1;
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (i0 + k < S) {
                gofs[i0 + k] = e0;
                bofs[i0 + k] = e1;
                e0 += g[k];
                e1 += b[k];
            }
        __syncthreads();
        if (tid < 2) carry_s[tid] += wsum[tid][15];
        __syncthreads();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, 64));
    if (lane == 0) atomicMax(&most_s, most);
    __syncthreads();
    if (tid == 0) {
        gofs[S] = carry_s[0];
        bofs[S] = carry_s[1];
        host[0] = carry_s[0];
        host[1] = carry_s[1];
        host[2] = most_s;
        __threadfence_system();
    }
    if (errs) atomicOr(d_err, errs);
}

// What k_tr_choose needs to write the switches' and ports' records as well
// (sinfo nullptr: it does not).
struct Infos {
    SwInfo *sinfo;
    int2 *pinfo;
    const int32_t *port_off, *port_peer;
    int64_t n_ports;
    const uint8_t *jur;
    const int32_t *gofs;
    uint32_t *d_err;

    // the ports' records of switch s, by n threads
    __device__ __forceinline__ void ports(int32_t s, int32_t S, int32_t thread, int32_t n) const
    {
        const int64_t pb = port_off[s], pe = port_off[s + 1];
        if (pc_range_ok(pb, pe, n_ports))
            for (int64_t p = pb + thread; p < pe; p += n) pinfo[p] = make_port(port_peer[p], S, jur);
    }
    // the action flag of a switch without chunk sets (else k_tr_prep raises it)
    __device__ __forceinline__ void sweep_actions(int32_t s, const pc_rule *__restrict__ r, int64_t R) const
    {
        const int64_t pb = port_off[s], pe = port_off[s + 1];
        const int64_t np = pc_range_ok(pb, pe, n_ports) ? pe - pb : 0;
        bool bad = false;
        for (int64_t i = threadIdx.x; i < R; i += blockDim.x) {
            const uint32_t act = r[i].action;
            bad |= act != PC_ACTION_DROP && static_cast<int64_t>(act) >= np;
        }
        if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(d_err, PC_DERR_ACTION);
    }
};

// The condition of a walk rule by rule on the longest table (word nullptr:
// none): k_tr_direct sets *word to the call's number if a table has more than
// most rules (so that nothing is cleared), and the walk ends at once then.  The
// number and the answer go to the host as early as they are known: from k_tr_direct's
// first workgroup, which looks at every table (early), else from the walk as it starts.
struct Guard {
    uint32_t *word;
    uint32_t call;
    int32_t most;
    unsigned long long *host;  // call << 32 | (1: too long)
    bool early;

    __device__ __forceinline__ bool too_long(const int32_t *__restrict__ rule_off, int64_t n_rules, int32_t s) const
    {
        const int64_t rb = rule_off[s], re = rule_off[s + 1];
        return word != nullptr && pc_range_ok(rb, re, n_rules) && re - rb > most;
    }
    __device__ __forceinline__ void tell(bool stop) const
    {
        __hip_atomic_store(host, static_cast<unsigned long long>(call) << 32 | (stop ? 1u : 0u), __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
};

// Small tables, whose rules a walk matches one by one: everything a trace
// call prepares, in one launch: a workgroup per switch, the sweeps of the ports and
// the watch lists spread over these and further workgroups.  (A table that is too
// long is swept by k_tr_prep.)
__global__ __launch_bounds__(kDirectThreads) void k_tr_direct(int32_t S, const int32_t *__restrict__ rule_off,
                                                              int64_t n_rules, const pc_rule *__restrict__ rules,
                                                              int64_t n_watch, const int32_t *__restrict__ watch,
                                                              Infos inf, Guard guard)
{
    const int32_t s = blockIdx.x;
    if (guard.early && s == 0) {
        bool stop = false;
        for (int32_t i = threadIdx.x; i < S; i += kDirectThreads) stop |= guard.too_long(rule_off, n_rules, i);
        stop = __syncthreads_or(stop);
        if (threadIdx.x == 0) {
            if (stop) *guard.word = guard.call;
            guard.tell(stop);
        }
    }
    uint32_t errs = 0;
    if (bad_ids(inf.n_ports, inf.port_peer, S) || bad_ids(n_watch, watch, S)) errs |= PC_DERR_SWITCH;
    bool rok = false;
    int64_t rb = 0, re = 0;
    if (s < S) {
        rb = rule_off[s];
        re = rule_off[s + 1];
        rok = pc_range_ok(rb, re, n_rules);
        if (inf.jur[s] >= 32) errs |= PC_DERR_JUR;
        if (!rok || !pc_range_ok(inf.port_off[s], inf.port_off[s + 1], inf.n_ports)) errs |= PC_DERR_OFFSETS;
    }
    if (errs) atomicOr(inf.d_err, errs);
    if (s >= S) return;
    if (guard.too_long(rule_off, n_rules, s)) {
        if (!guard.early && threadIdx.x == 0) *guard.word = guard.call;
        return;
    }
    if (threadIdx.x == 0) inf.sinfo[s] = make_info(s, inf.port_off, inf.n_ports, rule_off, n_rules, 0, 0);
    inf.ports(s, S, threadIdx.x, kDirectThreads);
    if (rok) inf.sweep_actions(s, rules + rb, re - rb);
}

// The filter chunks of each switch (one workgroup per switch).  From a
// sample of at most kChooseSample of its rules (every ceil(R / sample)-th):
// for each of the key's 26 nibbles and each chunk value x, the number A[x]
// of sampled rules whose value/mask admit x.  With hh the headers' nibble
// histogram, score = sum_x (hh[x] + 1) A[x] is proportional to the chance
// that a header drawn like the traced ones (smoothed towards uniform)
// passes the nibble's filter against a rule drawn like the switch's.  The
// kChunks nibbles of smallest score (ties: lower nibble) filter out the
// most: nibbles the rules wildcard, or where headers and rules agree on a
// few values, score high.  Any choice gives the same results; it only
// decides how many rules reach the full 104-bit check.
__global__ __launch_bounds__(256) void k_tr_choose(int32_t S, const int32_t *__restrict__ rule_off, int64_t n_rules,
                                                   const pc_rule *__restrict__ rules,
                                                   const uint32_t *__restrict__ hh, uint32_t *__restrict__ cpos,
                                                   Infos inf)
{
    __shared__ uint32_t hist[kKeyNibbles][256];  // (value & mask, mask) patterns per nibble
    __shared__ unsigned long long score[kKeyNibbles];
    const int32_t s = blockIdx.x;
    if (s >= S) return;
    for (int i = threadIdx.x; i < kKeyNibbles * 256; i += 256) (&hist[0][0])[i] = 0;
    if (threadIdx.x < kKeyNibbles) score[threadIdx.x] = 0;
    __syncthreads();
    const int64_t rb = rule_off[s], re = rule_off[s + 1];
    const int64_t R = pc_range_ok(rb, re, n_rules) ? re - rb : 0;
    const int64_t stride = R > kChooseSample ? (R + kChooseSample - 1) / kChooseSample : 1;
    for (int64_t i = threadIdx.x; i * stride < R && i < kChooseSample; i += 256) {
        const pc_rule *r = rules + rb + i * stride;
        const uint32_t v0 = r->value.w[0], v1 = r->value.w[1], v2 = r->value.w[2], v3 = r->value.w[3];
        const uint32_t m0 = r->mask.w[0], m1 = r->mask.w[1], m2 = r->mask.w[2], m3 = r->mask.w[3];
        for (uint32_t n = 0; n < kKeyNibbles; ++n) {
            const uint32_t m = key_nibble(m0, m1, m2, m3, n);
            const uint32_t v = key_nibble(v0, v1, v2, v3, n) & m;
            // rules that wildcard the nibble share one count: added by one lane
            const uint64_t any = __ballot(m == 0);
            if (m != 0) atomicAdd(&hist[n][m << 4 | v], 1u);
            else if (static_cast<int>(threadIdx.x & 63) == __builtin_ctzll(any)) atomicAdd(&hist[n][0], static_cast<uint32_t>(__popcll(any)));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kKeyNibbles * 16; i += 256) {
        const int n = i >> 4;
        const uint32_t x = i & 15;
        uint64_t a = 0;  // sampled rules admitting chunk value x: (x & m) == (v & m)
        for (uint32_t m = 0; m < 16; ++m) a += hist[n][m << 4 | (x & m)];
        atomicAdd(&score[n], static_cast<unsigned long long>(a * (static_cast<uint64_t>(hh[n * 16 + x]) + 1)));
    }
    __syncthreads();
    // the first wavefront ranks the scores, a nibble per lane (a thread that
    // picked them one after the other read 156 in a chain); the others write
    // the ports' records
    if (threadIdx.x >= 64) {
        if (inf.sinfo != nullptr) inf.ports(s, S, threadIdx.x - 64, 192);
        return;
    }
    const int n = threadIdx.x;
    int rank = kChunks;
    if (n < kKeyNibbles) {
        rank = 0;
        for (int k = 0; k < kKeyNibbles; ++k) rank += score[k] < score[n] || (score[k] == score[n] && k < n);
    }
    uint32_t cp = rank < kChunks ? static_cast<uint32_t>(n) << (5 * rank) : 0u;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) cp |= __shfl_xor(cp, off, 64);
    if (n == 0) {
        cpos[s] = cp;
        if (inf.sinfo != nullptr)
            inf.sinfo[s] = make_info(s, inf.port_off, inf.n_ports, rule_off, n_rules, inf.gofs[s], cp);
    }
}

// Rows r of a 32-lane half hold 32-bit words x_r; afterwards lane i holds
// column i (bit r = bit i of the old x_r).  Five block-swap stages, one per
// lane-index bit j: the partner's word (lane i ^ j) is rotated so that its
// blocks land where this lane takes them, then merged under the lane's keep
// mask.  The stages commute; each costs one cross-lane move and two VALU ops.
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x)
{
    const int v = static_cast<int>(x);
    if constexpr (J == 1) return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
    if constexpr (J == 2) return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false));  // quad_perm 2,3,0,1
    if constexpr (J == 4) {
        // banks 0 and 2 of each row read lane + 4 (row_shl:4), banks 1 and 3 read lane - 4 (row_shr:4)
        const int lo = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false);
        return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(lo, v, 0x114, 0xF, 0xA, false));
    }
    if constexpr (J == 8) return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0x128, 0xF, 0xF, false));  // row_ror:8
    if constexpr (J == 16) return static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(v, 0x401F));  // 32-lane groups, xor 16
    return x;
}

template <int J>
__device__ __forceinline__ uint32_t swap_stage(uint32_t x, uint32_t keep, uint32_t rot)
{
    const uint32_t y = lane_xor<J>(x);
    const uint32_t t = __builtin_amdgcn_alignbit(y, y, rot);  // rotate right
    return (x & keep) | (t & ~keep);
}

__device__ __forceinline__ uint32_t transpose32(uint32_t x, const uint32_t (&keep)[5], const uint32_t (&rot)[5])
{
    x = swap_stage<1>(x, keep[0], rot[0]);
    x = swap_stage<2>(x, keep[1], rot[1]);
    x = swap_stage<4>(x, keep[2], rot[2]);
    x = swap_stage<8>(x, keep[3], rot[3]);
    return swap_stage<16>(x, keep[4], rot[4]);
}

constexpr int kPrepWaves = 16;
constexpr int kPrepRounds = 4;                          // 64-rule rounds per wavefront, loads issued up front
constexpr int kTileStride = kPrepGroups + 2;            // LDS row pitch (spreads a half-wave's rows over banks)
static_assert(kPrepGroups == 2 * kPrepWaves * kPrepRounds, "two groups per wavefront round");

// Build the chunk sets of kPrepGroups groups (block b) of switch s, and with
// prio the rules' priorities (0xFFFF - priority, 32 a group); validate actions.
// Lane r of a half-wave holds rule r of a group and looks up, for each chunk,
// the 16-bit set of chunk values its value/mask admit (a 256-entry LDS table
// indexed by the chunk's value & mask and mask).  Two chunks share a word;
// a 32 x 32 bit transpose over the half-wave turns the rules' admit sets
// into the group's per-value rule sets: word (chunk c, value x) lands in lane
// (c % 2) * 16 + x of the transpose of word c / 2.
__device__ __forceinline__ void prep_block(int32_t s, int32_t b, uint32_t *tile, uint16_t *admit,
                                           const int32_t *__restrict__ port_off, int64_t n_ports,
                                           const int32_t *__restrict__ rule_off, const pc_rule *__restrict__ rules,
                                           const int32_t *__restrict__ gcount, const int32_t *__restrict__ gofs,
                                           uint32_t *__restrict__ filt, uint16_t *__restrict__ prio,
                                           uint32_t *__restrict__ d_err, uint32_t *__restrict__ sw_bad,
                                           const uint32_t *__restrict__ cpos)
{
    const int32_t G = gcount[s];
    const int32_t g0 = b * kPrepGroups;
    const int64_t rb = rule_off[s];
    const int64_t R = rule_off[s + 1] - rb;
    const bool pok = pc_range_ok(port_off[s], port_off[s + 1], n_ports);
    const int64_t np = pok ? port_off[s + 1] - port_off[s] : 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t cp = cpos[s];
    // issue every round's loads before any use
    uint4 vv[kPrepRounds], mm[kPrepRounds];
    uint32_t act[kPrepRounds];
    bool ok[kPrepRounds];
#pragma unroll
    for (int k = 0; k < kPrepRounds; ++k) {
        const int32_t gl = 2 * (wave * kPrepRounds + k) + (lane >> 5);
        const int64_t local = static_cast<int64_t>(g0 + gl - (lane >> 5)) * 32 + lane;  // rule index within the switch
        ok[k] = local < R && g0 + gl < G;
        vv[k] = mm[k] = make_uint4(0, 0, 0, 0);
        act[k] = 0;
        if (ok[k]) {
            const pc_rule *r = rules + rb + local;
            vv[k] = make_uint4(r->value.w[0], r->value.w[1], r->value.w[2], r->value.w[3]);
            mm[k] = make_uint4(r->mask.w[0], r->mask.w[1], r->mask.w[2], r->mask.w[3]);
            act[k] = r->action;
            if (prio != nullptr) prio[static_cast<int64_t>(gofs[s]) * 32 + local] = static_cast<uint16_t>(0xFFFFu - r->priority);
        }
    }
    // admit[(v & m) | m << 4] = set of 4-bit values y with (y & m) == (v & m)
    if (threadIdx.x < 256) {
        const uint32_t m = threadIdx.x >> 4, t = threadIdx.x & 15;
        uint32_t set = 0;
        for (uint32_t y = 0; y < 16; ++y) set |= static_cast<uint32_t>((y & m) == t) << y;
        admit[threadIdx.x] = static_cast<uint16_t>(set);
    }
    // per-stage keep masks and rotations of this lane (stage j = 1, 2, 4, 8, 16)
    uint32_t keep[5], rot[5];
    {
        const uint32_t blk[5] = {0x55555555u, 0x33333333u, 0x0F0F0F0Fu, 0x00FF00FFu, 0x0000FFFFu};
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const bool up = (lane >> q) & 1;
            keep[q] = up ? ~blk[q] : blk[q];
            rot[q] = up ? (1u << q) : 32u - (1u << q);
        }
    }
    __syncthreads();
    bool bad_action = false;
#pragma unroll
    for (int k = 0; k < kPrepRounds; ++k) {
        uint32_t w[kChunks / 2];
#pragma unroll
        for (int d = 0; d < kChunks / 2; ++d) {
            const uint32_t n0 = chunk_pos(cp, 2 * d), n1 = chunk_pos(cp, 2 * d + 1);
            const uint32_t ma = key_nibble(mm[k].x, mm[k].y, mm[k].z, mm[k].w, n0);
            const uint32_t mb = key_nibble(mm[k].x, mm[k].y, mm[k].z, mm[k].w, n1);
            const uint32_t i0 = (key_nibble(vv[k].x, vv[k].y, vv[k].z, vv[k].w, n0) & ma) | (ma << 4);
            const uint32_t i1 = (key_nibble(vv[k].x, vv[k].y, vv[k].z, vv[k].w, n1) & mb) | (mb << 4);
            const uint32_t a0 = ok[k] ? admit[i0] : 0u, a1 = ok[k] ? admit[i1] : 0u;
            w[d] = transpose32(a0 | (a1 << 16), keep, rot);
        }
        bad_action |= ok[k] && act[k] != PC_ACTION_DROP && static_cast<int64_t>(act[k]) >= np;
        const int gl = 2 * (wave * kPrepRounds + k) + (lane >> 5);
#pragma unroll
        for (int d = 0; d < kChunks / 2; ++d) tile[(32 * d + (lane & 31)) * kTileStride + gl] = w[d];
    }
    if (__ballot(bad_action) && lane == 0) {
        atomicOr(d_err, PC_DERR_ACTION);
        if (sw_bad != nullptr) atomicOr(sw_bad + s, 1u);
    }
    __syncthreads();
    uint32_t *dst = filt + static_cast<int64_t>(gofs[s]) * kPlaneWords;
    for (int i = threadIdx.x; i < kPlaneWords * kPrepGroups; i += blockDim.x) {
        const int row = i / kPrepGroups, gl = i % kPrepGroups;
        const int32_t g = g0 + gl;
        if (g < G) dst[static_cast<int64_t>(row) * G + g] = tile[row * kTileStride + gl];
    }
}

// The switch that owns prep block b: the largest s with bofs[s] <= b (b < bofs[S]).
__device__ __forceinline__ int32_t block_owner(const int32_t *__restrict__ bofs, int32_t S, int32_t b)
{
    int32_t lo = 0, hi = S;  // invariant: bofs[lo] <= b < bofs[hi]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (bofs[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(1024) void k_tr_prep(int32_t S, const int32_t *__restrict__ port_off, int64_t n_ports,
                                                  const int32_t *__restrict__ rule_off,
                                                  const pc_rule *__restrict__ rules,
                                                  const int32_t *__restrict__ gcount,
                                                  const int32_t *__restrict__ gofs, const int32_t *__restrict__ bofs,
                                                  uint32_t *__restrict__ filt, uint16_t *__restrict__ prio,
                                                  uint32_t *__restrict__ d_err, uint32_t *__restrict__ sw_bad,
                                                  const uint32_t *__restrict__ cpos)
{
    __shared__ uint32_t tile[kPlaneWords * kTileStride];
    __shared__ uint16_t admit[256];
    const int32_t b = blockIdx.x;
    if (b >= bofs[S]) return;
    const int32_t s = block_owner(bofs, S, b);
    prep_block(s, b - bofs[s], tile, admit, port_off, n_ports, rule_off, rules, gcount, gofs, filt, prio, d_err,
               sw_bad, cpos);
}

// The same for the switches marked in a bitmap, unless *skip.
__global__ __launch_bounds__(1024) void k_tr_prep_marked(int32_t S, const int32_t *__restrict__ port_off,
                                                         int64_t n_ports, const int32_t *__restrict__ rule_off,
                                                         const pc_rule *__restrict__ rules,
                                                         const int32_t *__restrict__ gcount,
                                                         const int32_t *__restrict__ gofs,
                                                         const int32_t *__restrict__ bofs,
                                                         uint32_t *__restrict__ filt, uint16_t *__restrict__ prio,
                                                         uint32_t *__restrict__ d_err, uint32_t *__restrict__ sw_bad,
                                                         const uint32_t *__restrict__ cpos,
                                                         const uint32_t *__restrict__ marked,
                                                         const uint32_t *__restrict__ skip)
{
    __shared__ uint32_t tile[kPlaneWords * kTileStride];
    __shared__ uint16_t admit[256];
    const int32_t b = blockIdx.x;
    if (*skip || b >= bofs[S]) return;
    const int32_t s = block_owner(bofs, S, b);
    if (!((marked[s >> 5] >> (s & 31)) & 1u)) return;
    prep_block(s, b - bofs[s], tile, admit, port_off, n_ports, rule_off, rules, gcount, gofs, filt, prio, d_err,
               sw_bad, cpos);
}

// The same for listed switches, unless *skip: list entry blockIdx.y, its
// block blockIdx.x (a repeated switch is done twice, alike).
__global__ __launch_bounds__(1024) void k_tr_prep_listed(int32_t S, const int32_t *__restrict__ port_off,
                                                         int64_t n_ports, const int32_t *__restrict__ rule_off,
                                                         const pc_rule *__restrict__ rules,
                                                         const int32_t *__restrict__ gcount,
                                                         const int32_t *__restrict__ gofs,
                                                         const int32_t *__restrict__ bofs,
                                                         uint32_t *__restrict__ filt, uint16_t *__restrict__ prio,
                                                         uint32_t *__restrict__ d_err, uint32_t *__restrict__ sw_bad,
                                                         const uint32_t *__restrict__ cpos,
                                                         const int32_t *__restrict__ listed,
                                                         const uint32_t *__restrict__ skip)
{
    __shared__ uint32_t tile[kPlaneWords * kTileStride];
    __shared__ uint16_t admit[256];
    if (*skip) return;
    const int32_t s = listed[blockIdx.y], b = blockIdx.x;
    if (s < 0 || s >= S || b >= bofs[s + 1] - bofs[s]) return;
    prep_block(s, b, tile, admit, port_off, n_ports, rule_off, rules, gcount, gofs, filt, prio, d_err, sw_bad, cpos);
}

// Level 0: every trace starts at its ingress switch (an invalid ingress
// ends it at once as MISS).  A workgroup takes kInitPer traces, kInitPer /
// 1024 per thread: with kLds (S small enough) it counts them per switch in
// LDS and reserves each switch's share with one global count update, a
// trace's rank being that share's base plus its rank in the workgroup;
// otherwise every trace updates its switch's count itself.  Live-list slots
// are reserved once per workgroup.
// A bucketed lookup: the trace, its jurisdiction mask so far and its
// header, gathered when the trace is bucketed so that the match stages its
// lookups with contiguous loads.
struct __align__(16) BRec {
    int32_t t;
    uint32_t jm;
    uint32_t pad[2];
    pc_key key;
};

// A live-list entry: a trace in flight, the switch it is at, its rank in
// that switch's bucket, its jurisdiction mask so far and its header (next
// = -1: the slot of a trace that has ended).
struct __align__(16) LRec {
    int32_t t;
    int32_t next;
    int32_t rk;
    uint32_t jm;
    pc_key key;
};

constexpr int kInitThreads = 1024;
constexpr int kInitRounds = 4;
constexpr int kInitPer = kInitThreads * kInitRounds;
constexpr int kInitLdsS = 8192;  // switches counted in LDS at most (32 KB)
template <bool kLds>
__global__ __launch_bounds__(kInitThreads) void k_tr_init(int32_t S, const uint8_t *__restrict__ jur,
                                                          const int32_t *__restrict__ ingress,
                                                          const pc_key *__restrict__ hdr, int32_t T,
                                                          LRec *__restrict__ live,
                                                          int32_t *__restrict__ nlive,
                                                          int32_t *__restrict__ counts, pc_trace_out *__restrict__ out,
                                                          const int32_t *__restrict__ watch, int32_t K,
                                                          uint32_t *__restrict__ visit, uint64_t *__restrict__ vsum,
                                                          int32_t *__restrict__ walk, uint32_t *__restrict__ d_err)
{
    extern __shared__ int32_t lcnt[];  // [S] with kLds
    __shared__ int32_t nloc, base;
    if (threadIdx.x == 0) nloc = 0;
    if constexpr (kLds)
        for (int32_t b = threadIdx.x; b < S; b += kInitThreads) lcnt[b] = 0;
    __syncthreads();
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kInitPer;
    int32_t sw[kInitRounds], rk[kInitRounds], slot[kInitRounds];
    uint32_t jb[kInitRounds];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kInitRounds; ++k) {
        const int64_t t64 = t0 + k * kInitThreads + threadIdx.x;
        const int32_t t = static_cast<int32_t>(t64);
        sw[k] = -1;
        rk[k] = 0;
        jb[k] = 0;
        if (t64 < T) {
            const int32_t s = ingress[t];
            if (s < 0 || s >= S) {
                bad = true;
                pc_trace_out o;
                o.jmask = 0;
                o.last_switch = s;
                o.last_port = PC_NO_PORT;
                o.hops = 0;
                o.state = PC_MISS;
                out[t] = o;
                if (visit) visit[t] = 0;
                if (vsum) vsum[t] = 0;
                if (walk)
                    for (int j = 0; j < kWalkSlots; ++j) walk[static_cast<int64_t>(t) * kWalkSlots + j] = -1;
            } else {
                jb[k] = jur_bit(jur, s);
                if (visit) visit[t] = watch_bits(watch, K, t, s);
                if (vsum) vsum[t] = sum_bit(s);
                if (walk)
                    for (int j = 0; j < kWalkSlots; ++j) walk[static_cast<int64_t>(t) * kWalkSlots + j] = j ? -1 : s;
                sw[k] = s;
                if constexpr (kLds) rk[k] = atomicAdd(&lcnt[s], 1);
                else rk[k] = atomicAdd(&counts[static_cast<int64_t>(s) * kCountPad], 1);
            }
        }
        // a slot in the workgroup's share of the live list: one LDS update per wavefront
        const uint64_t m = __ballot(sw[k] >= 0);
        int32_t wb = 0;
        if ((threadIdx.x & 63) == 0 && m) wb = atomicAdd(&nloc, static_cast<int32_t>(__popcll(m)));
        wb = __shfl(wb, 0, 64);
        slot[k] = sw[k] >= 0 ? wb + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                                        static_cast<uint32_t>(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)))
                             : -1;
    }
    __syncthreads();
    if constexpr (kLds)
        for (int32_t b = threadIdx.x; b < S; b += kInitThreads) {
            const int32_t n = lcnt[b];
            lcnt[b] = n ? atomicAdd(&counts[static_cast<int64_t>(b) * kCountPad], n) : 0;
        }
    if (threadIdx.x == 0) base = nloc ? atomicAdd(nlive, nloc) : 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kInitRounds; ++k)
        if (slot[k] >= 0) {
            const int32_t t = static_cast<int32_t>(t0 + k * kInitThreads + threadIdx.x);
            LRec e;
            e.t = t;
            e.next = sw[k];
            e.rk = kLds ? lcnt[sw[k]] + rk[k] : rk[k];
            e.jm = jb[k];
            e.key = hdr[t];
            live[base + slot[k]] = e;
        }
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(d_err, PC_DERR_SWITCH);
}

// Bucket the live traces by current switch: a live entry puts its trace at
// slot boff[switch] + rank, its rank having been taken when it was counted.
// The list holds *len entries; traces that ended leave entries with switch
// -1.  Also maps each match work item to (its switch, its index among the
// switch's items): the switch is the last s with ioff[s] <= item.
__global__ void k_tr_scatter(const LRec *__restrict__ live, const int32_t *__restrict__ len, int32_t T, int32_t S,
                             const int32_t *__restrict__ boff, BRec *__restrict__ bucket,
                             const int32_t *__restrict__ ioff, int2 *__restrict__ imap, int32_t icap)
{
    const int32_t n_items = min(ioff[S], icap);
    for (int32_t it = blockIdx.x * blockDim.x + threadIdx.x; it < n_items; it += gridDim.x * blockDim.x) {
        int32_t lo = 0, hi = S;
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (ioff[mid] <= it) lo = mid;
            else hi = mid;
        }
        imap[it] = make_int2(lo, it - ioff[lo]);
    }
    const int32_t n = min(*len, T);
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int4 e = reinterpret_cast<const int4 *>(live)[2 * i];  // (t, next, rk, jm)
        if (e.y < 0 || e.y >= S || static_cast<uint32_t>(e.x) >= static_cast<uint32_t>(T)) continue;
        const int32_t pos = boff[e.y] + e.z;
        if (pos >= 0 && pos < T) {
            BRec r;
            r.t = e.x;
            r.jm = static_cast<uint32_t>(e.w);
            r.pad[0] = r.pad[1] = 0;
            r.key = live[i].key;
            bucket[pos] = r;
        }
    }
}

__device__ __forceinline__ bool rule_matches(const pc_rule *r, uint32_t h0, uint32_t h1, uint32_t h2, uint32_t h3)
{
    return (((h0 ^ r->value.w[0]) & r->mask.w[0]) | ((h1 ^ r->value.w[1]) & r->mask.w[1]) |
            ((h2 ^ r->value.w[2]) & r->mask.w[2]) | ((h3 ^ r->value.w[3]) & r->mask.w[3])) == 0;
}

// First-match key of a rule: (0xFFFF - priority) << 48 | local index << 16 |
// action.  The smallest key is the highest priority, ties to the lower
// index; the action rides along, so applying the match reads no rule.
__device__ __forceinline__ uint64_t rule_key(const pc_rule *r, uint32_t local)
{
    return (static_cast<uint64_t>(0xFFFFu - r->priority) << 48) | (static_cast<uint64_t>(local) << 16) | r->action;
}

// Verify the surviving rules of one 32-rule group against the full header
// and fold their (priority, index) keys into *best.
__device__ __forceinline__ void verify_group(uint32_t surv, const pc_rule *grp, uint32_t local0, const pc_key &h,
                                             unsigned long long *best)
{
    while (surv) {
        const int bit = __builtin_ctz(surv);
        surv &= surv - 1;
        const pc_rule *r = grp + bit;
        if (rule_matches(r, h.w[0], h.w[1], h.w[2], h.w[3]))
            atomicMin(best, static_cast<unsigned long long>(rule_key(r, local0 + bit)));
    }
}

// Apply the chosen rule (its key, see rule_key) at a switch of np ports (np
// < 0: the switch's port range is invalid) whose port a leads to
// peer_of(a): returns the terminal state, or -1 when the trace moves on to
// *next through port *port.
template <class PeerOf>
__device__ __forceinline__ int apply_key(int32_t S, int32_t ttl, int64_t np, const PeerOf &peer_of, uint64_t key,
                                         int32_t hops, int32_t *next, uint16_t *port)
{
    if (key == kNoMatch) return PC_MISS;
    const uint32_t a = static_cast<uint32_t>(key & 0xFFFFu);
    if (a == PC_ACTION_DROP) return PC_DROP;
    if (np < 0 || static_cast<int64_t>(a) >= np) return PC_MISS;
    const int32_t peer = peer_of(a);
    if (peer == -1) {
        *port = static_cast<uint16_t>(a);
        return PC_EGRESS;
    }
    if (peer < -1 || peer >= S) return PC_MISS;
    if (hops == ttl) return PC_TTL;
    *next = peer;
    *port = static_cast<uint16_t>(a);  // the forwarding port
    return -1;
}

__device__ __forceinline__ void write_out(pc_trace_out *out, int32_t t, uint32_t jm, int32_t s, uint16_t port,
                                          int32_t hops, int state)
{
    pc_trace_out o;
    o.jmask = jm;
    o.last_switch = s;
    o.last_port = port;
    o.hops = static_cast<uint8_t>(hops);
    o.state = static_cast<uint8_t>(state);
    out[t] = o;
}

// Per-trace state of the level loop and where a level's results go.
struct Level {
    int32_t S;
    int32_t T;              // capacity of the live list
    const int32_t *port_peer;
    const int2 *pinfo;      // per port: (peer, the peer's jurisdiction bit)
    const uint8_t *jur;
    int32_t ttl;
    int32_t cap;            // lookups per work item at most
    int32_t hops;           // hops every trace of this level has made (the level's index)
    LRec *live_next;        // one entry per lookup of this level, at its bucket slot (switch -1: the trace ended)
    int32_t *nlive_next;    // traces in flight after this level
    int32_t *counts_next;   // live traces per switch after this level
    pc_trace_out *out;
    const int32_t *watch;   // [T][K] switches whose visit is recorded
    int32_t K;
    uint32_t *visit;        // [T] or nullptr
    uint64_t *vsum;         // [T] visited-switch summaries or nullptr
    int32_t *walk;          // [T][kWalkSlots] walk records or nullptr
};

// Lookups per match work item of a switch with n lookups in this level: the
// switch's lookups split evenly over as few items as hold at most cap each;
// and of the parts an item of n lookups is matched in.
__device__ __forceinline__ int32_t even_parts(int32_t n, int32_t cap)
{
    const int32_t parts = max(1, (n + cap - 1) / cap);
    return max(1, (n + parts - 1) / parts);
}

// Per level: bucket offsets boff = exclusive scan of counts (which are
// cleared for reuse), work-item offsets ioff = exclusive scan of
// ceil(counts / even_parts(counts, cap)), *total = the level's lookups (the
// length of the live list its match writes) and *host, and *nlive_next = 0 for
// the match to count the traces that move on.  One workgroup of 1024 threads;
// each thread takes kPlanPer consecutive switches per pass, so a pass
// covers 4,096 switches with all of its loads in flight together.
constexpr int kPlanPer = 4;
__global__ __launch_bounds__(1024) void k_tr_plan(int32_t *__restrict__ counts, int32_t S, int32_t *__restrict__ boff,
                                                  int32_t *__restrict__ ioff, int32_t cap,
                                                  int32_t *__restrict__ total, int32_t *__restrict__ nlive_next,
                                                  int32_t *__restrict__ host)
{
    __shared__ int32_t wsum[2][16];
    __shared__ int32_t carry_s[2];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (tid < 2) carry_s[tid] = 0;
    if (tid == 0) *nlive_next = 0;
    __syncthreads();
    for (int32_t base = 0; base < S; base += 1024 * kPlanPer) {
        const int32_t i0 = base + tid * kPlanPer;
        int32_t v0[kPlanPer], v1[kPlanPer];
#pragma unroll
        for (int k = 0; k < kPlanPer; ++k) v0[k] = i0 + k < S ? counts[static_cast<int64_t>(i0 + k) * kCountPad] : 0;
        int32_t s0 = 0, s1 = 0;
#pragma unroll
        for (int k = 0; k < kPlanPer; ++k) {
            const int32_t ch = even_parts(v0[k], cap);
            v1[k] = (v0[k] + ch - 1) / ch;
            s0 += v0[k];
            s1 += v1[k];
        }
        int32_t x0 = s0, x1 = s1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y0 = __shfl_up(x0, off, 64), y1 = __shfl_up(x1, off, 64);
            if (lane >= off) {
                x0 += y0;
                x1 += y1;
            }
        }
        if (lane == 63) {
            wsum[0][wid] = x0;
            wsum[1][wid] = x1;
        }
        __syncthreads();
        if (wid < 2) {
            int32_t w = lane < 16 ? wsum[wid][lane] : 0;
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                const int32_t y = __shfl_up(w, off, 64);
                if (lane >= off) w += y;
            }
            if (lane < 16) wsum[wid][lane] = w;
        }
        __syncthreads();
        const int32_t c0 = carry_s[0], c1 = carry_s[1];
        int32_t e0 = c0 + (wid ? wsum[0][wid - 1] : 0) + x0 - s0;
        int32_t e1 = c1 + (wid ? wsum[1][wid - 1] : 0) + x1 - s1;
#pragma unroll
        for (int k = 0; k < kPlanPer; ++k)
            if (i0 + k < S) {
                boff[i0 + k] = e0;
                ioff[i0 + k] = e1;
                counts[static_cast<int64_t>(i0 + k) * kCountPad] = 0;
                e0 += v0[k];
                e1 += v1[k];
            }
        __syncthreads();
        if (tid == 0) {
            carry_s[0] = c0 + wsum[0][15];
            carry_s[1] = c1 + wsum[1][15];
        }
        __syncthreads();
    }
    if (tid == 0) {
        boff[S] = carry_s[0];
        ioff[S] = carry_s[1];
        *total = carry_s[0];
        *host = carry_s[0];
        __threadfence_system();
    }
}

// What a match workgroup keeps of its switch's first kPortSlots ports: peer,
// the peer's jurisdiction bit, and the item's traces that leave through the port
// (count, then the base of their ranks in the peer's bucket).  The item's live
// entries are ordered by forwarding port: port p's run starts at run[p], the run
// of the other ports at run[kPortSlots].
struct PortMoves {
    int32_t peer[kPortSlots], count[kPortSlots], base[kPortSlots];
    uint32_t jbit[kPortSlots];
    int32_t run[kPortSlots + 1];
    int32_t nother, nmove;  // traces leaving through the other ports; all that move on
};

// The end of a match workgroup: every lookup's first match is in best (all in
// LDS; behind a barrier); at most a lookup per thread.
__device__ __forceinline__ void apply_matches(const Level &lv, int32_t s, int64_t pb, int64_t np, int32_t bb,
                                              int32_t tn, const int32_t *tids, const uint32_t *tjm,
                                              const uint64_t *best, const pc_key *keys, PortMoves &ports)
{
    const int lane = threadIdx.x & 63;
    // apply the first match.  A trace that moves on is counted in its next
    // switch's bucket (one count update per forwarding port and workgroup;
    // its rank there is the port's base plus its rank in the item) and gets
    // an entry in the item's share of the live list, grouped by port so that
    // the bucketing pass writes runs; the slots after the item's moving
    // traces are marked as ended (switch -1).
    const int32_t h = lv.hops;
    int32_t t = -1, lrank = -1, orank = -1, next = -1, rk = 0;
    uint32_t jm_next = 0;
    uint16_t port = PC_NO_PORT;
    if (threadIdx.x < tn) {  // (at most a lookup per thread)
        t = tids[threadIdx.x];
        if (t >= 0) {
            const uint32_t jmv = tjm[threadIdx.x];
            const int state = apply_key(
                lv.S, lv.ttl, np,
                [&](uint32_t a) { return a < kPortSlots ? ports.peer[a] : lv.port_peer[pb + a]; },
                best[threadIdx.x], h, &next, &port);
            if (state >= 0) {
                write_out(lv.out, t, jmv, s, port, h, state);
                t = -1;
            } else {
                jm_next = jmv | (port < kPortSlots ? ports.jbit[port] : jur_bit(lv.jur, next));
                if (lv.visit) lv.visit[t] |= watch_bits(lv.watch, lv.K, t, next);
                if (lv.vsum) lv.vsum[t] |= sum_bit(next);
                if (lv.walk && h + 1 < kWalkSlots) lv.walk[static_cast<int64_t>(t) * kWalkSlots + h + 1] = next;
                if (port < kPortSlots) {
                    lrank = atomicAdd(&ports.count[port], 1);
                } else {
                    rk = atomicAdd(&lv.counts_next[static_cast<int64_t>(next) * kCountPad], 1);
                    orank = atomicAdd(&ports.nother, 1);
                }
            }
        }
    }
    __syncthreads();
    static_assert(kPortSlots == 64, "one wavefront scans the port counts");
    if (threadIdx.x < kPortSlots) {
        const int32_t c = ports.count[threadIdx.x];
        // a port some trace forwarded through: its peer is a valid switch
        if (c > 0) ports.base[threadIdx.x] = atomicAdd(&lv.counts_next[static_cast<int64_t>(ports.peer[threadIdx.x]) * kCountPad], c);
        int32_t x = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        ports.run[threadIdx.x] = x - c;
        if (threadIdx.x == kPortSlots - 1) {
            ports.run[kPortSlots] = x;
            const int32_t m = x + ports.nother;
            ports.nmove = m;
            if (m) atomicAdd(lv.nlive_next, m);  // the traces in flight after this level
        }
    }
    __syncthreads();
    int32_t slot = -1;
    if (lrank >= 0) {
        rk = ports.base[port] + lrank;
        slot = ports.run[port] + lrank;
    } else if (orank >= 0) {
        slot = ports.run[kPortSlots] + orank;
    }
    if (slot >= 0) {
        LRec e;
        e.t = t;
        e.next = next;
        e.rk = rk;
        e.jm = jm_next;
        e.key = keys[threadIdx.x];
        lv.live_next[bb + slot] = e;
    }
    if (threadIdx.x >= ports.nmove && threadIdx.x < tn)
        *reinterpret_cast<int4 *>(lv.live_next + bb + threadIdx.x) = make_int4(-1, -1, 0, 0);
}

typedef uint32_t v16u __attribute__((ext_vector_type(16)));

// Filter four lookups: sv[k] = AND over the six chunks c of F[c][x[c][k]].
// GPR index mode stays on while only its index changes, and every indexed
// read feeds its lookup's AND directly; the four lookups' ANDs alternate, so
// consecutive vector instructions do not depend on each other.  The chunk
// sets sit in fixed registers v32..v127 (chunk c at v[32 + 16c .. 47 + 16c]);
// indices are below 16, so every indexed read stays inside its chunk's
// sixteen registers.  Two blocks of three chunks keep the operand lists short.
// Index mode keeps its index in M0, which each block declares clobbered.
#define PC_IDX(a, b, c, d, base, op)                        \
    "s_set_gpr_idx_idx %" #a "\n\t"                          \
    "v_" op "_b32 %0, v" #base ", %0\n\t"                    \
    "s_set_gpr_idx_idx %" #b "\n\t"                          \
    "v_" op "_b32 %1, v" #base ", %1\n\t"                    \
    "s_set_gpr_idx_idx %" #c "\n\t"                          \
    "v_" op "_b32 %2, v" #base ", %2\n\t"                    \
    "s_set_gpr_idx_idx %" #d "\n\t"                          \
    "v_" op "_b32 %3, v" #base ", %3\n\t"
__device__ __forceinline__ void filter_quad(const uint32_t (&x)[kChunks][4], const v16u (&F)[kChunks],
                                            uint32_t (&sv)[4])
{
    uint32_t a0, a1, a2, a3;
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
        "v_mov_b32 %0, v32\n\t"
        "s_set_gpr_idx_idx %5\n\t"
        "v_mov_b32 %1, v32\n\t"
        "s_set_gpr_idx_idx %6\n\t"
        "v_mov_b32 %2, v32\n\t"
        "s_set_gpr_idx_idx %7\n\t"
        "v_mov_b32 %3, v32\n\t"
        PC_IDX(8, 9, 10, 11, 48, "and")
        PC_IDX(12, 13, 14, 15, 64, "and")
        "s_set_gpr_idx_off"
        : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3)
        : "s"(x[0][0]), "s"(x[0][1]), "s"(x[0][2]), "s"(x[0][3]), "s"(x[1][0]), "s"(x[1][1]), "s"(x[1][2]),
          "s"(x[1][3]), "s"(x[2][0]), "s"(x[2][1]), "s"(x[2][2]), "s"(x[2][3]), "{v[32:47]}"(F[0]),
          "{v[48:63]}"(F[1]), "{v[64:79]}"(F[2])
        : "m0");
    asm volatile(
        "s_set_gpr_idx_on %4, gpr_idx(SRC0)\n\t"
        "v_and_b32 %0, v80, %0\n\t"
        "s_set_gpr_idx_idx %5\n\t"
        "v_and_b32 %1, v80, %1\n\t"
        "s_set_gpr_idx_idx %6\n\t"
        "v_and_b32 %2, v80, %2\n\t"
        "s_set_gpr_idx_idx %7\n\t"
        "v_and_b32 %3, v80, %3\n\t"
        PC_IDX(8, 9, 10, 11, 96, "and")
        PC_IDX(12, 13, 14, 15, 112, "and")
        "s_set_gpr_idx_off"
        : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3)
        : "s"(x[3][0]), "s"(x[3][1]), "s"(x[3][2]), "s"(x[3][3]), "s"(x[4][0]), "s"(x[4][1]), "s"(x[4][2]),
          "s"(x[4][3]), "s"(x[5][0]), "s"(x[5][1]), "s"(x[5][2]), "s"(x[5][3]), "{v[80:95]}"(F[3]),
          "{v[96:111]}"(F[4]), "{v[112:127]}"(F[5])
        : "m0");
    sv[0] = a0;
    sv[1] = a1;
    sv[2] = a2;
    sv[3] = a3;
}
#undef PC_IDX

// One workgroup per work item = (switch, an even share of at most lv.cap
// lookups of its bucket).  Items are dealt to XCDs in contiguous ranges, so
// the shares of one switch share an L2.  The chunk sets are in registers, a
// group per lane and 256 groups per workgroup: for levels of few lookups per
// table (see wide_level), where no barrier between the parts of a table and smaller
// items count for more than k_tr_match's cheaper filter.
__global__ __launch_bounds__(kWideThreads, 4) void k_tr_match_wide(
    int32_t S, const SwInfo *__restrict__ sinfo, const pc_rule *__restrict__ rules, const uint32_t *__restrict__ filt,
    const int32_t *__restrict__ boff, const int32_t *__restrict__ ioff, const int2 *__restrict__ imap,
    const BRec *__restrict__ bucket, Level lv)
{
    __shared__ uint64_t best[kWideChunk];
    __shared__ __align__(16) uint32_t cidx[kChunks][kWideChunk];  // each lookup's values of the switch's filter chunks
    __shared__ __align__(16) pc_key keys[kWideChunk];
    __shared__ int32_t tids[kWideChunk];
    __shared__ uint32_t tjm[kWideChunk];  // each lookup's trace: jurisdiction mask so far
    __shared__ uint2 queue[kWideWaves][kWideQueue];  // per wavefront: (survivor set, lookup << 6 | lane)
    __shared__ PortMoves ports;
    // the grid was sized from an upper bound on the item count: blocks past
    // the real count's per-XCD share return at once
    const int32_t n_items = ioff[S];
    const int32_t per = (n_items + 7) / 8;
    const int32_t kx = static_cast<int32_t>(blockIdx.x >> 3);
    if (kx >= per) return;
    const int32_t item = static_cast<int32_t>(blockIdx.x & 7) * per + kx;
    if (item >= n_items) return;
    // the item's switch and its index among the switch's items
    const int2 im = imap[item];
    const int32_t s = im.x;
    if (static_cast<uint32_t>(s) >= static_cast<uint32_t>(S)) return;
    const SwInfo si = sinfo[s];
    const int32_t b0 = boff[s], b1 = boff[s + 1];
    const int32_t chunk = even_parts(b1 - b0, lv.cap);
    const int32_t bb = b0 + im.y * chunk;
    const int32_t tn = min(chunk, min(b1, lv.T) - bb);  // bucket holds at most T entries
    if (tn <= 0) return;
    const int32_t tn4 = (tn + 3) & ~3;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t G = si.G;
    const int64_t rb = si.rb;
    const uint32_t *fs = filt + static_cast<int64_t>(si.gofs) * kPlaneWords;
    const int32_t nslices = max(1, (G + kWideThreads - 1) / kWideThreads);
    const uint32_t cp = si.cpos;
    uint2 *q = queue[wave];
    // A table of fewer than kWideThreads groups fills gws wavefronts; the
    // workgroup's other wavefronts take further shares of the lookups: wave
    // = stream * gws + gwi holds groups gwi * 64 .. and filters the lookups
    // of its stream (contiguous quads).  Waves past the last stream idle.
    const int32_t gws = G >= kWideThreads ? kWideWaves : max(1, (G + 63) / 64);
    const int32_t streams = kWideWaves / gws;
    const int32_t gwi = wave % gws, st = wave / gws;
    const int32_t nquads = tn4 / 4;
    const int32_t per_stream = (nquads + streams - 1) / streams;
    const int32_t jb = st < streams ? min(tn4, 4 * st * per_stream) : tn4;
    const int32_t je = st < streams ? min(tn4, 4 * (st + 1) * per_stream) : tn4;
    // the switch's ports (np < 0: its port range is invalid)
    const int64_t pb = si.pb, np = si.np;
    // A lane's chunk sets of group g: buffer loads with the lane's group as
    // the vector offset (clamped into the table) and the plane as a scalar
    // offset; an opaque copy of the plane stride keeps the 96 offsets from
    // being hoisted out of the loops (and spilled) as invariants.  A lane past
    // the last group gets empty chunk sets, so it never survives the filter;
    // a switch without rules (G = 0) reads offset 0 of an empty buffer, which
    // returns zeros.
    auto load_sets = [&](int32_t g, v16u (&F)[kChunks]) {
        uint32_t pstride = static_cast<uint32_t>(G) * 4u;
        asm volatile("" : "+s"(pstride));
        const __amdgpu_buffer_rsrc_t frs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint32_t *>(fs), static_cast<short>(0), kPlaneWords * G * 4, 0x00020000);
        const uint32_t voff = static_cast<uint32_t>(max(0, min(g, G - 1))) * 4u;
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
#pragma unroll
            for (int x = 0; x < 16; ++x)
                F[c][x] = __builtin_amdgcn_raw_buffer_load_b32(frs, voff, static_cast<uint32_t>(c * 16 + x) * pstride, 0);
        if (g >= G) {
#pragma unroll
            for (int x = 0; x < 16; ++x) F[0][x] = 0u;
        }
    };
    // stage the chunk (at most one lookup per thread: tn4 <= kWideChunk <=
    // kWideThreads); pad to a multiple of 4 lookups with copies of the last
    const int i = static_cast<int>(threadIdx.x);
    BRec r{};
    if (i < tn4) r = bucket[bb + min(i, tn - 1)];
    // the first slice's chunk sets load while the lookups are staged
    // (whether or not this wavefront filters: the loads are clamped into the
    // table, and a branch would leave the sets undefined on one path)
    v16u F0[kChunks];
    load_sets(gwi * 64 + lane, F0);
    if (i < tn4) {
        int32_t t = r.t;
        pc_key h = r.key;
        uint32_t jmv = r.jm;
        if (static_cast<uint32_t>(t) >= static_cast<uint32_t>(lv.T)) {  // not a trace id: skipped
            t = -1;
            h = pc_key{};
            jmv = 0;
        }
        tids[i] = t;
        keys[i] = h;
        tjm[i] = jmv;
        best[i] = kNoMatch;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) cidx[c][i] = key_nibble(h.w[0], h.w[1], h.w[2], h.w[3], chunk_pos(cp, c));
    }
    if (threadIdx.x < kPortSlots) {
        const int2 pi = static_cast<int64_t>(threadIdx.x) < np ? lv.pinfo[pb + threadIdx.x] : make_int2(-2, 0);
        ports.peer[threadIdx.x] = pi.x;
        ports.jbit[threadIdx.x] = static_cast<uint32_t>(pi.y);
        ports.count[threadIdx.x] = 0;
        if (threadIdx.x == 0) ports.nother = 0;
    }
    __syncthreads();
    // Filter phase: survivors of the chunk filter are queued (per wavefront)
    // until the queue could overflow.  Verify phase: the queued survivors are
    // checked against their full rules, 64 at a time, with the chunk sets
    // dead.  Then filtering resumes with the sets loaded again.  A quad of
    // lookups queues at most 256 entries, so every round advances.  gw is
    // the group of lane 0.
    auto round = [&](int32_t gw, int32_t &jr, const v16u (&F)[kChunks]) {
        int32_t qn = 0;
        int32_t j0 = jr;
        for (; j0 < je; j0 += 4) {
            uint4 X[kChunks];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) X[c] = reinterpret_cast<const uint4 *>(cidx[c])[j0 >> 2];
            uint32_t sv[4];
            uint32_t xi[kChunks][4];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                xi[c][0] = __builtin_amdgcn_readfirstlane(X[c].x);
                xi[c][1] = __builtin_amdgcn_readfirstlane(X[c].y);
                xi[c][2] = __builtin_amdgcn_readfirstlane(X[c].z);
                xi[c][3] = __builtin_amdgcn_readfirstlane(X[c].w);
            }
            filter_quad(xi, F, sv);
            if (__ballot((sv[0] | sv[1] | sv[2] | sv[3]) != 0)) {
                uint64_t m[4];
                int32_t n = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    m[k] = __ballot(sv[k] != 0);
                    n += __popcll(m[k]);
                }
                if (qn + n > kWideQueue) break;  // resume at this quad after verifying
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (sv[k]) {
                        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                            static_cast<uint32_t>(m[k] >> 32),
                            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m[k]), 0u));
                        q[qn + below] = make_uint2(sv[k], static_cast<uint32_t>(j0 + k) << 6 | lane);
                    }
                    qn += __popcll(m[k]);
                }
            }
        }
        jr = j0;
        // the queue entries were written by other lanes of this wavefront
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int32_t e = lane; e < qn; e += 64) {
            const uint2 en = q[e];
            const int32_t j = static_cast<int32_t>(en.y >> 6);
            const int32_t gg = gw + static_cast<int32_t>(en.y & 63u);
            verify_group(en.x, rules + rb + static_cast<int64_t>(gg) * 32, static_cast<uint32_t>(gg) * 32,
                         keys[j], reinterpret_cast<unsigned long long *>(&best[j]));
        }
        __builtin_amdgcn_wave_barrier();
    };
    // one slice of kWideThreads groups at a time, one group per lane, its
    // chunk sets held in VGPRs while the chunk's lookups stream past.  The
    // first round of the first slice uses the sets loaded with the staging;
    // it runs outside the slice loop, so those sets are dead after it and
    // never live beside a later round's (inside the loop they would be, and
    // the 192 registers would spill)
    int32_t jr0 = jb;
    if (jb < je) round(gwi * 64, jr0, F0);
    for (int32_t sl = 0; sl < nslices; ++sl) {
        const int32_t g = sl * kWideThreads + gwi * 64 + lane;
        const int32_t gw = sl * kWideThreads + gwi * 64;
        int32_t jr = sl == 0 ? jr0 : jb;
        while (jr < je) {
            v16u F[kChunks];
            load_sets(g, F);
            round(gw, jr, F);
        }
    }
    // every wavefront's matches are in best[] (a lookup's matches come from
    // the wavefronts that hold its groups, its epilogue thread may be another)
    __syncthreads();
    apply_matches(lv, s, pb, np, bb, tn, tids, tjm, best, keys, ports);
}

// The survivors of a lookup in four groups: bit r of s[k] is rule r of group
// k.  at: the groups' chunk sets of value 0 of chunk 0, rows of 16 << kLg bytes
// (row c * 16 + x: chunk c, value x); nib: the lookup's values, four bits each.
template <int kLg>
__device__ __forceinline__ void load_sets(const char *at, uint32_t nib, uint4 (&v)[kChunks])
{
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
        v[c] = *reinterpret_cast<const uint4 *>(at + (c * 16 << (kLg + 4)) + (((nib >> (4 * c)) & 15) << (kLg + 4)));
}

__device__ __forceinline__ void and_sets(const uint4 (&v)[kChunks], uint32_t (&s)[4])
{
    s[0] = v[0].x & v[1].x & v[2].x & v[3].x & v[4].x & v[5].x;
    s[1] = v[0].y & v[1].y & v[2].y & v[3].y & v[4].y & v[5].y;
    s[2] = v[0].z & v[1].z & v[2].z & v[3].z & v[4].z & v[5].z;
    s[3] = v[0].w & v[1].w & v[2].w & v[3].w & v[4].w & v[5].w;
    static_assert(kChunks == 6, "every chunk's set");
}

// One wavefront matches its nw <= 64 lookups (lane j's packed: lookup j's values
// of the chunks) against the slice whose chunk sets and priorities (0xFFFF -
// priority) are in LDS.  1 << kLg lanes take a lookup, four groups a lane, so
// that a read is 16 bytes a lane; two passes' reads go out together.  A pass only
// asks which lanes have survivors and queues these; 64 queued at a time, their sets are
// formed again and cand[j], cand2[j] become lookup j's first two survivors by (priority,
// index).  Only these rules are checked in full (lane j: verify(lookup, rule)): where
// many rules admit a header, as with prefixes, nearly every survivor matches.
// A lookup whose candidates both fail checks all its survivors.
template <int kLg, class Verify>
__device__ __forceinline__ void filter_slice(const uint4 *sets, const uint16_t *prio, uint32_t packed, int32_t nw,
                                             uint16_t *q, uint32_t *cand, uint32_t *cand2,
                                             Verify &&verify)
{
    constexpr int kPer = 64 >> kLg;  // lookups per pass
    const int lane = threadIdx.x & 63, sub = lane >> kLg, l = lane & ((1 << kLg) - 1);
    const char *base = reinterpret_cast<const char *>(sets);
    auto of_lane = [&](int32_t j, uint32_t x) {
        return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(4 * j, static_cast<int>(x)));
    };
    auto settle = [&]() {  // what other lanes of this wavefront wrote to LDS
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    int32_t qn = 0;
    auto push = [&](bool any, uint32_t entry, auto &&drain) {
        const uint64_t m = __ballot(any);
        const int n = __popcll(m);
        if (qn + n > kQueue) drain();
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
        if (any) q[qn + below] = static_cast<uint16_t>(entry);
        qn += n;
    };
    // queued: lookup << 5 | lane of its groups
    auto rank = [&]() {
        settle();
        for (int32_t e0 = 0; e0 < qn; e0 += 64) {
            const uint32_t en = q[min(e0 + lane, qn - 1)];
            const int32_t j = static_cast<int32_t>(en >> 5), ql = static_cast<int32_t>(en & 31);
            uint4 v[kChunks];
            uint32_t s[4], first = ~0u, second = ~0u;
            load_sets<kLg>(base + 16 * ql, of_lane(j, packed), v);
            and_sets(v, s);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                for (uint32_t m = s[k]; m; m &= m - 1) {
                    const uint32_t at = 128 * ql + 32 * k + __builtin_ctz(m);
                    const uint32_t key = static_cast<uint32_t>(prio[at]) << 12 | at;
                    second = min(second, max(first, key));
                    first = min(first, key);
                }
            // what does not stay the first competes for the second place
            if (e0 + lane < qn) second = min(second, max(first, atomicMin(cand + j, first)));
            if (e0 + lane < qn && second != ~0u) atomicMin(cand2 + j, second);
        }
        settle();
        qn = 0;
    };
    if (lane < nw) cand[lane] = cand2[lane] = ~0u;
    for (int32_t j0 = 0; j0 < nw; j0 += 2 * kPer) {
        uint4 a[kChunks], b[kChunks];
        uint32_t s[4];
        load_sets<kLg>(base + 16 * l, of_lane(min(j0 + sub, nw - 1), packed), a);
        load_sets<kLg>(base + 16 * l, of_lane(min(j0 + kPer + sub, nw - 1), packed), b);
        and_sets(a, s);
        push((s[0] | s[1] | s[2] | s[3]) != 0 && j0 + sub < nw, (j0 + sub) << 5 | l, rank);
        and_sets(b, s);
        push((s[0] | s[1] | s[2] | s[3]) != 0 && j0 + kPer + sub < nw, (j0 + kPer + sub) << 5 | l, rank);
    }
    rank();
    const uint32_t first = lane < nw ? cand[lane] : ~0u, second = lane < nw ? cand2[lane] : ~0u;
    const bool one = first != ~0u && verify(lane, static_cast<int32_t>(first & 4095));
    const bool two = second != ~0u && verify(lane, static_cast<int32_t>(second & 4095));
    const bool failed = second != ~0u && !one && !two;
    const uint64_t fm = __ballot(failed);
    if (fm == 0) return;
    // the failed lookups again, compacted; queued: place << 7 | lane << 2 | word
    const int32_t nf = __popcll(fm);
    if (failed) q[__popcll(fm & ((1ull << lane) - 1))] = static_cast<uint16_t>(lane);
    settle();
    const uint32_t which = q[min(lane, nf - 1)];
    const uint32_t again = of_lane(static_cast<int32_t>(which), packed);
    settle();
    auto check = [&]() {
        settle();
        for (int32_t e0 = 0; e0 < qn; e0 += 64) {
            const uint32_t en = q[min(e0 + lane, qn - 1)];
            const int32_t j = static_cast<int32_t>(en >> 7), ql = static_cast<int32_t>((en >> 2) & 31);
            uint4 v[kChunks];
            uint32_t s[4];
            load_sets<kLg>(base + 16 * ql, of_lane(j, again), v);
            and_sets(v, s);
            const uint32_t k = en & 3, to = of_lane(j, which);
            if (e0 + lane < qn)
                for (uint32_t m = k == 0 ? s[0] : k == 1 ? s[1] : k == 2 ? s[2] : s[3]; m; m &= m - 1)
                    (void)verify(static_cast<int32_t>(to), static_cast<int32_t>(128 * ql + 32 * k + __builtin_ctz(m)));
        }
        settle();
        qn = 0;
    };
    for (int32_t j0 = 0; j0 < nf; j0 += kPer) {
        uint4 a[kChunks];
        uint32_t s[4];
        load_sets<kLg>(base + 16 * l, of_lane(min(j0 + sub, nf - 1), again), a);
        and_sets(a, s);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            push(s[k] != 0 && j0 + sub < nf, (j0 + sub) << 7 | l << 2 | k, check);
    }
    check();
}

// The same with the chunk sets read from LDS, a slice of 4,096 rules at a time, which takes half the instructions of
// k_tr_match_wide's register indexing (a level of 4.2 million lookups in 1,280
// tables of 4,096 rules: 42 vector and 35 scalar instructions per lookup there,
// 31 and 15 here).  Bound by staging and moving the lookups, 155 of such a level's 340
// us, then by the vector instructions of the filter, 130.  4,194,304 traces
// over these tables 1,757 us in k_tr_match_wide, now 1,417; 500,009 over
// 720 routing tables of 2,048 prefixes, where a lookup has dozens of matching
// rules, 935 and 470 (842 with every survivor checked).
__global__ __launch_bounds__(kMatchThreads, 4) void k_tr_match(
    int32_t S, const SwInfo *__restrict__ sinfo, const pc_rule *__restrict__ rules, const uint32_t *__restrict__ filt,
    const uint16_t *__restrict__ prios, const int32_t *__restrict__ boff, const int32_t *__restrict__ ioff,
    const int2 *__restrict__ imap, const BRec *__restrict__ bucket, Level lv)
{
    __shared__ uint4 sets[kPlaneWords * kSliceGroups / 4];
    __shared__ uint64_t best[kChunk];
    __shared__ __align__(16) pc_key keys[kChunk];
    __shared__ uint32_t cidx[kChunk];  // each lookup's values of the switch's filter chunks, four bits each; then its
                                       // candidate (a wavefront's own lookups only)
    __shared__ uint32_t cand2[kChunk];
    __shared__ int32_t tids[kChunk];
    __shared__ uint32_t tjm[kChunk];   // each lookup's trace: jurisdiction mask so far
    __shared__ uint16_t prio[kSliceGroups * 32] __attribute__((aligned(16)));
    __shared__ uint16_t queue[kMatchWaves][kQueue];  // per wavefront (see filter_slice)
    __shared__ PortMoves ports;
    // the grid was sized from an upper bound on the item count: blocks past
    // the real count's per-XCD share return at once
    const int32_t n_items = ioff[S];
    const int32_t per = (n_items + 7) / 8;
    const int32_t kx = static_cast<int32_t>(blockIdx.x >> 3);
    if (kx >= per) return;
    const int32_t item = static_cast<int32_t>(blockIdx.x & 7) * per + kx;
    if (item >= n_items) return;
    // the item's switch and its index among the switch's items
    const int2 im = imap[item];
    const int32_t s = im.x;
    if (static_cast<uint32_t>(s) >= static_cast<uint32_t>(S)) return;
    const SwInfo si = sinfo[s];
    const int32_t b0 = boff[s], b1 = boff[s + 1];
    const int32_t share = even_parts(b1 - b0, lv.cap);
    const int32_t bb = b0 + im.y * share;
    const int32_t tn = min(share, min(b1, lv.T) - bb);  // bucket holds at most T entries
    if (tn <= 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t G = si.G;
    const int64_t rb = si.rb;
    const uint32_t *fs = filt + static_cast<int64_t>(si.gofs) * kPlaneWords;
    const uint32_t cp = si.cpos;
    // the switch's ports (np < 0: its port range is invalid)
    const int64_t pb = si.pb, np = si.np;
    // lanes that take a lookup: a slice's groups, four a lane
    const int32_t quads = (min(G, kSliceGroups) + 3) / 4;
    const int lpl_bits = quads <= 1 ? 0 : 32 - __builtin_clz(static_cast<uint32_t>(quads - 1)), lpl = 1 << lpl_bits;
    // a slice's chunk sets into LDS (no survivors past the last group)
    auto fill = [&](int32_t g0) {
        const int32_t ng = min(G - g0, kSliceGroups);
        constexpr int kFills = kPlaneWords * kSliceGroups / 4 / kMatchThreads;
        static_assert(kSliceGroups * 4 == kMatchThreads, "16 bytes of priorities per thread");
        uint4 v[kFills], pr = make_uint4(0, 0, 0, 0);
        if (static_cast<int32_t>(threadIdx.x) < ng * 4)
            pr = reinterpret_cast<const uint4 *>(prios + (static_cast<int64_t>(si.gofs) + g0) * 32)[threadIdx.x];
#pragma unroll
        for (int k = 0; k < kFills; ++k) {
            const int x = static_cast<int>(threadIdx.x) + k * kMatchThreads;
            const int32_t row = x >> lpl_bits, g = 4 * (x & (lpl - 1));
            v[k] = make_uint4(0, 0, 0, 0);
            if (row < kPlaneWords) {
                const uint32_t *src = fs + static_cast<int64_t>(row) * G + g0 + g;
                if (g + 4 <= ng) {
                    __builtin_memcpy(&v[k], src, 16);
                } else {
                    if (g < ng) v[k].x = src[0];
                    if (g + 1 < ng) v[k].y = src[1];
                    if (g + 2 < ng) v[k].z = src[2];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kFills; ++k) {
            const int x = static_cast<int>(threadIdx.x) + k * kMatchThreads;
            if (x < kPlaneWords * lpl) sets[x] = v[k];
        }
        reinterpret_cast<uint4 *>(prio)[threadIdx.x] = pr;
    };
    // stage the lookups (one per thread) and the first slice's sets
    const int i = static_cast<int>(threadIdx.x);
    BRec r{};
    if (i < tn) r = bucket[bb + i];
    fill(0);
    if (threadIdx.x < kPortSlots) {
        const int2 pi = static_cast<int64_t>(threadIdx.x) < np ? lv.pinfo[pb + threadIdx.x] : make_int2(-2, 0);
        ports.peer[threadIdx.x] = pi.x;
        ports.jbit[threadIdx.x] = static_cast<uint32_t>(pi.y);
        ports.count[threadIdx.x] = 0;
        if (threadIdx.x == 0) ports.nother = 0;
    }
    if (i < tn) {
        int32_t t = r.t;
        pc_key h = r.key;
        uint32_t jmv = r.jm;
        if (static_cast<uint32_t>(t) >= static_cast<uint32_t>(lv.T)) {  // not a trace id: skipped
            t = -1;
            h = pc_key{};
            jmv = 0;
        }
        tids[i] = t;
        keys[i] = h;
        tjm[i] = jmv;
        best[i] = kNoMatch;
        uint32_t x = 0;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) x |= key_nibble(h.w[0], h.w[1], h.w[2], h.w[3], chunk_pos(cp, c)) << (4 * c);
        cidx[i] = x;
    }
    __syncthreads();
    const int32_t per_wave = (tn + kMatchWaves - 1) / kMatchWaves;  // the wavefront's lookups
    const int32_t jw = wave * per_wave, nw = min(per_wave, tn - jw);
    const uint32_t packed = nw > 0 ? cidx[jw + min(lane, nw - 1)] : 0u;
    for (int32_t g0 = 0; g0 < G; g0 += kSliceGroups) {
        if (g0 > 0) {
            __syncthreads();  // the slice before is no longer read
            fill(g0);
            __syncthreads();
        }
        auto verify = [&](int32_t j, int32_t at) {
            const uint32_t local = static_cast<uint32_t>(g0) * 32 + static_cast<uint32_t>(at);
            const pc_rule x = rules[rb + local];
            const pc_key &h = keys[jw + j];
            const bool ok = rule_matches(&x, h.w[0], h.w[1], h.w[2], h.w[3]);
            if (ok)
                atomicMin(reinterpret_cast<unsigned long long *>(&best[jw + j]),
                          static_cast<unsigned long long>(rule_key(&x, local)));
            return ok;
        };
        if (lpl_bits == 5) filter_slice<5>(sets, prio, packed, nw, queue[wave], cidx + jw, cand2 + jw, verify);
        else if (lpl_bits == 4) filter_slice<4>(sets, prio, packed, nw, queue[wave], cidx + jw, cand2 + jw, verify);
        else if (lpl_bits == 3) filter_slice<3>(sets, prio, packed, nw, queue[wave], cidx + jw, cand2 + jw, verify);
        else if (lpl_bits == 2) filter_slice<2>(sets, prio, packed, nw, queue[wave], cidx + jw, cand2 + jw, verify);
        else if (lpl_bits == 1) filter_slice<1>(sets, prio, packed, nw, queue[wave], cidx + jw, cand2 + jw, verify);
        else filter_slice<0>(sets, prio, packed, nw, queue[wave], cidx + jw, cand2 + jw, verify);
    }
    // every wavefront's matches are in best[]
    __syncthreads();
    apply_matches(lv, s, pb, np, bb, tn, tids, tjm, best, keys, ports);
}

// What every walk of a launch shares.
struct WalkArgs {
    int32_t S;
    const SwInfo *sinfo;
    const int2 *pinfo;
    const pc_rule *rules;
    const uint32_t *filt;
    int32_t ttl;
    pc_trace_out *out;
    const int32_t *watch;
    int32_t K;
    uint32_t *visit;
    uint64_t *vsum;
    int32_t *walk;
};

// One workgroup walks trace t (header h) from switch s to its end, filtering
// each switch's rule groups with only the kChunks chunk-set words its
// header selects (coalesced over groups) and reducing the first match in
// LDS; without chunk sets (kDirect) the rules are matched one per lane.
// Bound by the latency of a hop: the switch's record, its ports
// together with the chunk-set words of two groups per lane, the survivors'
// rules.  Where 5,200 of 500,009 traces loop until a TTL of 32, 329 us with a hop
// per link, now 46; 6,001 traces over 777 rules per switch 54 us, now 22.
template <bool kDirect>
__device__ __forceinline__ void walk_trace(const WalkArgs &w, unsigned long long *best, int32_t t, const pc_key &h,
                                           int32_t s, uint32_t jm, uint32_t vis, uint64_t vs, int32_t hops)
{
    const int lane = threadIdx.x & 63;
    // A walk is a function of the switch (its header does not change): once
    // a switch comes again, the walk repeats until its TTL, and whole
    // turns of the cycle are skipped, their switches being in every mask
    // already.  The switch two hops back finds the ping-pong of two
    // switches at once, an anchor that moves on at doubled distances
    // (Brent) any other cycle.
    int32_t back1 = -1, back2 = -1, anchor = s, anchor_hops = hops, span = 1;
    for (;;) {
        if (threadIdx.x == 0) *best = kNoMatch;
        __syncthreads();
        const SwInfo si = w.sinfo[s];
        const int32_t G = si.G;
        const pc_rule *rs = w.rules + si.rb;
        // this lane's of the switch's first 64 ports
        const int2 port_lane = lane < si.np ? w.pinfo[si.pb + lane] : make_int2(-2, 0);
        if constexpr (!kDirect) {
            const uint32_t *fs = w.filt + static_cast<int64_t>(si.gofs) * kPlaneWords;
            int64_t row[kChunks];
#pragma unroll
            for (int c = 0; c < kChunks; ++c)
                row[c] = static_cast<int64_t>(c * 16 + key_nibble(h.w[0], h.w[1], h.w[2], h.w[3], chunk_pos(si.cpos, c))) * G;
            for (int32_t g = threadIdx.x; g < G; g += 2 * blockDim.x) {
                const int32_t g2 = g + static_cast<int32_t>(blockDim.x);
                uint32_t surv = ~0u, surv2 = g2 < G ? ~0u : 0u;
#pragma unroll
                for (int c = 0; c < kChunks; ++c) {
                    surv &= fs[row[c] + g];
                    surv2 &= fs[row[c] + min(g2, G - 1)];
                }
                if (surv) verify_group(surv, rs + static_cast<int64_t>(g) * 32, static_cast<uint32_t>(g) * 32, h, best);
                if (surv2)
                    verify_group(surv2, rs + static_cast<int64_t>(g2) * 32, static_cast<uint32_t>(g2) * 32, h, best);
            }
        } else {
            // four rules of a longer table in flight per lane
            constexpr int kAhead = 4;
            const int32_t step = static_cast<int32_t>(blockDim.x);
            auto check = [&](int32_t r, bool hit) {
                if (hit) atomicMin(best, static_cast<unsigned long long>(rule_key(rs + r, static_cast<uint32_t>(r))));
            };
            auto matches = [&](int32_t r) { return rule_matches(rs + r, h.w[0], h.w[1], h.w[2], h.w[3]); };
            int32_t r = threadIdx.x;
            for (int32_t left = si.R; left >= kAhead * step; left -= kAhead * step, r += kAhead * step) {
                bool hit[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; ++k) hit[k] = matches(r + k * step);
#pragma unroll
                for (int k = 0; k < kAhead; ++k) check(r + k * step, hit[k]);
            }
            for (; r < si.R; r += step) check(r, matches(r));
        }
        __syncthreads();
        const uint64_t key = *best;
        int32_t next = -1;
        uint32_t jb = 0;
        uint16_t port = PC_NO_PORT;
        const int state = apply_key(w.S, w.ttl, si.np, [&](uint32_t a) {
            const uint32_t ua = __builtin_amdgcn_readfirstlane(a);
            const int2 p = ua < 64 ? make_int2(__builtin_amdgcn_readlane(port_lane.x, static_cast<int>(ua)),
                                               __builtin_amdgcn_readlane(port_lane.y, static_cast<int>(ua)))
                                   : w.pinfo[si.pb + static_cast<int64_t>(ua)];
            jb = static_cast<uint32_t>(p.y);
            return p.x;
        }, key, hops, &next, &port);
        __syncthreads();  // everyone has read *best before it is reset
        if (state >= 0) {
            if (threadIdx.x == 0) {
                write_out(w.out, t, jm, s, port, hops, state);
                if (w.visit) w.visit[t] = vis;
                if (w.vsum) w.vsum[t] = vs;
            }
            break;
        }
        back2 = back1;
        back1 = s;
        s = __builtin_amdgcn_readfirstlane(next);
        hops += 1;
        jm |= jb;
        if (w.visit) vis |= watch_bits(w.watch, w.K, t, s);
        if (w.vsum) vs |= sum_bit(s);
        if (w.walk && hops < kWalkSlots && threadIdx.x == 0) w.walk[static_cast<int64_t>(t) * kWalkSlots + hops] = s;
        const int32_t period = s == back2 ? 2 : s == anchor ? hops - anchor_hops : 0;
        if (period > 0 && !(w.walk && hops < kWalkSlots)) {
            hops += (w.ttl - hops) / period * period;  // (hops <= ttl: a forward at hops == ttl has ended the walk)
            back2 = anchor = -1;                        // less than a turn is left
            span = INT32_MAX;
        } else if (hops - anchor_hops >= span) {
            anchor = s;
            anchor_hops = hops;
            span = span < (1 << 20) ? 2 * span : span;
        }
    }
}

// Sparse tail: every trace of a level's list that is still in flight.
__global__ __launch_bounds__(256) void k_tr_walk(WalkArgs w, const LRec *__restrict__ live,
                                                 const int32_t *__restrict__ len, int32_t hops0)
{
    __shared__ unsigned long long best;
    const int32_t n = *len;
    const int lane = threadIdx.x & 63;
    // Every gridDim-th entry is this workgroup's, 64 of them looked at
    // together (most are the slots of traces that have ended).
    const int64_t grid = gridDim.x;
    for (int64_t i0 = blockIdx.x; i0 < n; i0 += 64 * grid) {
        const int64_t il = i0 + lane * grid;
        const int32_t at = il < n ? live[il].next : -1;
        uint64_t flying = __ballot(at >= 0 && at < w.S);
        while (flying) {
            const LRec e = live[i0 + __builtin_ctzll(flying) * grid];
            flying &= flying - 1;
            walk_trace<false>(w, &best, e.t, e.key, __builtin_amdgcn_readfirstlane(e.next), e.jm, w.visit ? w.visit[e.t] : 0u,
                              w.vsum ? w.vsum[e.t] : 0ull, hops0);
        }
    }
}

// Few traces: every one (or those of a list) from its ingress (an invalid
// ingress ends it at once as MISS), without levels or counts.  None if the
// guard found a table too long.
template <bool kDirect>
__global__ __launch_bounds__(256) void k_tr_walk_all(WalkArgs w, int32_t T, const pc_key *__restrict__ hdr,
                                                     const int32_t *__restrict__ ingress,
                                                     const uint8_t *__restrict__ jur, uint32_t *__restrict__ d_err,
                                                     const int32_t *__restrict__ list, Guard guard)
{
    __shared__ unsigned long long best;
    if (guard.word != nullptr) {
        const bool stop = *guard.word == guard.call;
        if (!guard.early && blockIdx.x == 0 && threadIdx.x == 0) guard.tell(stop);
        if (stop) return;
    }
    for (int32_t i = blockIdx.x; i < T; i += gridDim.x) {
        const int32_t t = list != nullptr ? list[i] : i;
        const int32_t s = __builtin_amdgcn_readfirstlane(ingress[t]);
        const bool in = s >= 0 && s < w.S;
        if (w.walk && threadIdx.x < kWalkSlots)
            w.walk[static_cast<int64_t>(t) * kWalkSlots + threadIdx.x] = in && threadIdx.x == 0 ? s : -1;
        if (in) {
            walk_trace<kDirect>(w, &best, t, hdr[t], s, jur_bit(jur, s), w.visit ? watch_bits(w.watch, w.K, t, s) : 0u,
                                sum_bit(s), 0);
        } else if (threadIdx.x == 0) {
            write_out(w.out, t, 0, s, PC_NO_PORT, 0, PC_MISS);
            if (w.visit) w.visit[t] = 0;
            if (w.vsum) w.vsum[t] = 0;
            atomicOr(d_err, PC_DERR_SWITCH);
        }
    }
}

// ---------------------------------------------------------------- deltas
// The state of a delta call on the device: cleared words, then the bitmap of
// the changed switches.
struct DeltaState {
    unsigned long long mask;  // summary bits of the changed switches
    uint32_t n;               // traces to trace again
    uint32_t differs;         // the kept tables have another switch's group count
};

// Summary bits and the bitmap of the changed switches (ids outside [0, S)
// are ignored and raise SWITCH).  With kept tables (gold, sw_bad): offsets and
// jurisdictions validated, the group counts compared with the kept ones
// (then no chunk set moves), the changed switches' action flags cleared.  A
// single workgroup (up to kLayoutS switches) clears the state itself;
// the bitmap's clearing has returned before its setting starts.
__global__ __launch_bounds__(1024) void k_delta_plan(const int32_t *__restrict__ changed, int32_t C, int32_t S,
                                                     DeltaState *__restrict__ state, uint32_t *__restrict__ bitmap,
                                                     int32_t words, const int32_t *__restrict__ port_off,
                                                     int64_t n_ports, const uint8_t *__restrict__ jur,
                                                     const int32_t *__restrict__ rule_off, int64_t n_rules,
                                                     const int32_t *__restrict__ gold, uint32_t *__restrict__ sw_bad,
                                                     uint32_t *__restrict__ d_err)
{
    __shared__ unsigned long long m;
    __shared__ uint32_t differs;
    const int32_t i0 = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    if (threadIdx.x == 0) {
        m = 0;
        differs = 0;
    }
    uint32_t seen = 0;
    if (gridDim.x == 1)
        for (int32_t i = threadIdx.x; i < words; i += blockDim.x) seen |= atomicExch(bitmap + i, 0u);
    asm volatile("" ::"v"(seen) : "memory");
    __syncthreads();
    uint64_t mine = 0;
    uint32_t errs = 0;
    for (int32_t i = i0; i < C; i += stride) {
        const int32_t s = changed[i];
        if (s < 0 || s >= S) {
            errs |= PC_DERR_SWITCH;
        } else {
            mine |= sum_bit(s);
            atomicOr(bitmap + (s >> 5), 1u << (s & 31));
            if (sw_bad != nullptr) sw_bad[s] = 0;
        }
    }
    if (mine) atomicOr(&m, static_cast<unsigned long long>(mine));
    bool d = false;
    if (gold != nullptr)
        for (int32_t s = i0; s < S; s += stride) {
            const int64_t rb = rule_off[s], re = rule_off[s + 1];
            const bool rok = pc_range_ok(rb, re, n_rules);
            if (jur[s] >= 32) errs |= PC_DERR_JUR;
            if (!rok || !pc_range_ok(port_off[s], port_off[s + 1], n_ports)) errs |= PC_DERR_OFFSETS;
            d |= (rok ? static_cast<int32_t>((re - rb + 31) / 32) : 0) != gold[s];
        }
    if (d) differs = 1;
    if (errs) atomicOr(d_err, errs);
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (gridDim.x == 1) {
        *state = DeltaState{m, 0u, differs};
    } else {
        if (m) atomicOr(&state->mask, m);
        if (differs) atomicOr(&state->differs, 1u);
    }
}

// What follows the selection: the counts to the host and the caller, the
// ports' sweep and, where the kept tables serve, their switch and port
// records and the ACTION flag of the unchanged switches (k_tr_prep raises it
// for the others).
__global__ __launch_bounds__(256) void k_delta_post(const DeltaState *__restrict__ state, int32_t *__restrict__ host,
                                                    int32_t *__restrict__ n_out, bool kept, int64_t n_ports,
                                                    const int32_t *__restrict__ port_off,
                                                    const int32_t *__restrict__ port_peer, int32_t S,
                                                    const uint8_t *__restrict__ jur,
                                                    const int32_t *__restrict__ rule_off, int64_t n_rules,
                                                    const int32_t *__restrict__ gofs,
                                                    const uint32_t *__restrict__ cpos, int2 *__restrict__ pinfo,
                                                    SwInfo *__restrict__ sinfo, const uint32_t *__restrict__ sw_bad,
                                                    uint32_t *__restrict__ d_err)
{
    const DeltaState d = *state;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *n_out = static_cast<int32_t>(d.n);
        host[0] = static_cast<int32_t>(d.n);
        host[1] = static_cast<int32_t>(d.differs);
        __threadfence_system();
    }
    if (!kept || d.differs) return;
    uint32_t errs = bad_ids(n_ports, port_peer, S) ? PC_DERR_SWITCH : 0;
    port_infos(n_ports, port_off, port_peer, S, jur, rule_off, n_rules, gofs, cpos, pinfo, sinfo);
    for (int32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < S; s += gridDim.x * blockDim.x)
        if (sw_bad[s]) errs |= PC_DERR_ACTION;
    if (errs) atomicOr(d_err, errs);
}

// The traces to trace again, in a list (one counter update per workgroup
// of 1,024 traces): with walk records, a walk of at most kWalkSlots
// switches (hops + 1 of its record) is selected iff one of them changed;
// otherwise, iff its summary meets the mask.  Also the ingress sweep of the
// SWITCH flag over every trace.
__global__ __launch_bounds__(1024) void k_delta_select(const uint64_t *__restrict__ vsum,
                                                       const int32_t *__restrict__ walk,
                                                       const pc_trace_out *__restrict__ out,
                                                       const uint32_t *__restrict__ bitmap,
                                                       const int32_t *__restrict__ ingress, int32_t T, int32_t S,
                                                       DeltaState *__restrict__ state, int32_t *__restrict__ list,
                                                       uint32_t *__restrict__ d_err)
{
    __shared__ uint32_t wcount[16], wbase[16];
    const uint64_t m = state->mask;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t base = static_cast<int64_t>(blockIdx.x) * blockDim.x; base < T;
         base += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t t = base + threadIdx.x;
        const bool in = t < T;
        bool sel = false;
        if (in) {
            const int32_t len = static_cast<int32_t>(out[t].hops) + 1;
            if (walk != nullptr && len <= kWalkSlots) {
                const int32_t *w = walk + t * kWalkSlots;
                for (int j = 0; j < len; ++j) {
                    const int32_t v = w[j];
                    if (v >= 0 && v < S && ((bitmap[v >> 5] >> (v & 31)) & 1u)) sel = true;
                }
            } else {
                sel = (vsum[t] & m) != 0;
            }
        }
        const int32_t s = in ? ingress[t] : 0;
        if (__ballot(in && (s < 0 || s >= S)) && lane == 0) atomicOr(d_err, PC_DERR_SWITCH);
        const uint64_t b = __ballot(sel);
        if (lane == 0) wcount[wave] = static_cast<uint32_t>(__popcll(b));
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int w = 0; w < 16; ++w) {
                wbase[w] = tot;
                tot += wcount[w];
            }
            const uint32_t off = tot ? atomicAdd(&state->n, tot) : 0u;
            for (int w = 0; w < 16; ++w) wbase[w] += off;
        }
        __syncthreads();
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u));
        if (sel) list[wbase[wave] + below] = static_cast<int32_t>(t);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_delta_gather(const int32_t *__restrict__ list, int32_t n,
                                                      const pc_key *__restrict__ hdr,
                                                      const int32_t *__restrict__ ingress, pc_key *__restrict__ hdr_c,
                                                      int32_t *__restrict__ ing_c)
{
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int32_t t = list[i];
        hdr_c[i] = hdr[t];
        ing_c[i] = ingress[t];
    }
}

__global__ __launch_bounds__(256) void k_delta_scatter(const int32_t *__restrict__ list, int32_t n,
                                                       const pc_trace_out *__restrict__ out_c,
                                                       const uint64_t *__restrict__ vsum_c,
                                                       const int32_t *__restrict__ walk_c,
                                                       pc_trace_out *__restrict__ out, uint64_t *__restrict__ vsum,
                                                       int32_t *__restrict__ walk)
{
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int32_t t = list[i];
        out[t] = out_c[i];
        vsum[t] = vsum_c[i];
        if (walk)
            for (int j = 0; j < kWalkSlots; ++j)
                walk[static_cast<int64_t>(t) * kWalkSlots + j] = walk_c[static_cast<int64_t>(i) * kWalkSlots + j];
    }
}

// Levels with few traces in flight are cheaper as independent walks than as
// bucketed passes (tunable with PC_TRACE_WALK_MAX, 0 = never walk): a walk
// skips its loops, a level costs three launches and a pass over its
// tables.  Large tables make a walk's hop dearer (24 bytes per 32 rules).
// Calls that walk from the start / from 8,192 traces on: 60,000 traces over
// 512 rules per switch (k = 16) 231 / 258 us, over 2,048 (k = 32) 275 / 302,
// over 32,768 (k = 16) 908 / 835, 30,000 traces there 527 / 803; 4,194,304
// traces, of which 8,900 loop until their TTL, 2.4 / 3.2 ms; 30,000 over 500,000
// (k = 4) 4.9 / 7.8 ms.
// Nor may the walks' passes over the largest table take much longer than the levels'
// at their worst, one switch of 320 with nearly all rules where every trace enters
// (in brackets a fifth of them, then none more than elsewhere): 16,000 traces, two
// million rules 1,351 / 3,234 us; 30,000, 1.1 million 1,306 / 1,842; 60,000, half a
// million 1,157 / 886 (492 / 872, 164 / 650); past the limit 60,000, 1.1 million
// 3,216 / 1,760 (1,190 / 1,749, 280 / 1,286); 30,000, two million 3,132 / 3,243; 60,000
// there 7,679 / 3,742 (2,331 / 3,699, 462 / 1,869).
constexpr int64_t kWalkLeast = 8192;
constexpr int64_t kWalkGroups = int64_t(1) << 30;  // traces times the groups of the largest table
int64_t walk_most(int64_t mean_groups, int64_t largest)
{
    if (const char *env = getenv("PC_TRACE_WALK_MAX")) return atoll(env);
    return std::max(std::min<int64_t>(mean_groups <= 128 ? 65536 : 32768, kWalkGroups / std::max<int64_t>(largest, 1)),
                    kWalkLeast);
}

// The walks' workgroup: about two rule groups per lane of a mean table; all of it
// for few walks where the largest table is long (1.1 million rules on one of 320
// switches, where every / no more than its share of the traces enter, 64 / 256 threads:
// 300 traces 169 / 84 us and 155 / 78, 2,000 170 / 151 and 162 / 81; past the
// limit 4,000 195 / 267 and 162 / 83; 60,000 rules there, 2,000 traces 49 / 47).
int walk_threads(int64_t walks, int64_t mean_groups, int64_t largest)
{
    if (walks <= 2048 && largest > 1024) return 256;
    return mean_groups <= 128 ? 64 : mean_groups <= 256 ? 128 : 256;
}

// The chunk sets' buffer: the sets of every group, then (for levels matched
// by candidate) the rules' priorities.
size_t chunk_set_bytes(int64_t groups, bool prio)
{
    return static_cast<size_t>(groups + 1) * (kPlaneWords * sizeof(uint32_t) + (prio ? 32 * sizeof(uint16_t) : 0));
}

uint16_t *priorities(void *filt, int64_t groups)
{
    return reinterpret_cast<uint16_t *>(static_cast<uint32_t *>(filt) + groups * kPlaneWords);
}

// Is a level of n lookups matched by k_tr_match_wide?  It spreads a large table
// over the registers of its wavefronts; k_tr_match reads the table's sets into LDS
// slice by slice, which pays with enough lookups per table.  Wide / not, us of
// all levels (rpath unless noted): tables of one slice, 78 lookups a table 156 / 191,
// 234 238 / 226, 3,276 1,882 / 1,412, prefixes 694 896 / 458; two slices, 277
// 288 / 327, 1,388 776 / 697; four slices, 347 1,530 / 1,958, 781 1,463 / 1,796,
// 1,250 652 / 650, 1,388 1,323 / 1,263.
bool wide_level(int64_t n, int32_t S, int64_t mean_groups)
{
    const int64_t slices = std::max<int64_t>((mean_groups + kSliceGroups - 1) / kSliceGroups, 1);
    return n < S * (slices == 1 ? 128 : 320 * slices);
}

unsigned grid_for(int64_t n, int threads)
{
    int64_t b = (n + threads - 1) / threads;
    if (b > 65536) b = 65536;
    return b > 0 ? static_cast<unsigned>(b) : 1u;
}

// The input sweeps with the header histogram (hh zeroed), then each switch's
// filter chunks and, when inf names them, the switches' and ports' records.
int sweep_and_choose(pc_ctx *ctx, int32_t S, const int32_t *port_peer, int64_t n_ports, const int32_t *rule_off,
                     int64_t n_rules, const pc_rule *rules, const pc_key *hdr, int32_t T, int64_t n_watch,
                     const int32_t *watch, uint32_t *hh, uint32_t *cpos, const Infos &inf, hipStream_t stream)
{
    const int64_t n = std::max<int64_t>({n_ports, n_watch, std::min<int64_t>(T, kHeaderSample)});
    const unsigned blocks = static_cast<unsigned>(std::min<int64_t>(std::max<int64_t>((n + 255) / 256, 1), 256));
    PC_TIMED(ctx, "k_tr_sweep", stream,
             hipLaunchKernelGGL(k_tr_sweep, dim3(blocks), dim3(256), 0, stream, n_ports, port_peer, S, n_watch, watch,
                                hdr, T, hh, ctx->d_err));
    PC_TIMED(ctx, "k_tr_choose", stream,
             hipLaunchKernelGGL(k_tr_choose, dim3(static_cast<unsigned>(S)), dim3(256), 0, stream, S, rule_off,
                                n_rules, rules, hh, cpos, inf));
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}

// Group counts and offsets, prep-block offsets (bcount: scratch of the form
// for many switches) and the zeroed header histogram; the two totals and the groups
// of the largest table in ctx->h_small[0..2] once the stream has come so far.
int layout(pc_ctx *ctx, int32_t S, const int32_t *port_off, int64_t n_ports, const uint8_t *jur,
           const int32_t *rule_off, int64_t n_rules, int32_t *gcount, int32_t *bcount, int32_t *gofs, int32_t *bofs,
           uint32_t *hh, hipStream_t stream)
{
    if (S <= kLayoutS) {
        PC_TIMED(ctx, "k_tr_layout", stream,
                 hipLaunchKernelGGL(k_tr_layout, dim3(1), dim3(1024), 0, stream, S, port_off, n_ports, jur, rule_off,
                                    n_rules, gcount, gofs, bofs, hh, ctx->h_small, ctx->d_err));
    } else {
        int32_t *largest = reinterpret_cast<int32_t *>(hh + kKeyNibbles * 16);
        launch_fill_u32(hh, kHistWords, 0, stream);
        PC_TIMED(ctx, "k_tr_switch_info", stream,
                 hipLaunchKernelGGL(k_tr_switch_info, dim3(grid_for(S, 256)), dim3(256), 0, stream, S, port_off,
                                    n_ports, jur, rule_off, n_rules, gcount, bcount, largest, ctx->d_err));
        launch_scan_i32(gcount, S, gofs, nullptr, nullptr, stream);
        launch_scan_i32(bcount, S, bofs, nullptr, nullptr, stream);
        PC_HIP(ctx, hipMemcpyAsync(ctx->h_small + 2, largest, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        PC_HIP(ctx, hipMemcpyAsync(ctx->h_small, gofs + S, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        PC_HIP(ctx, hipMemcpyAsync(ctx->h_small + 1, bofs + S, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
    }
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}

bool capturing(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) (void)hipGetLastError();
    return status != hipStreamCaptureStatusNone;
}

// Waits for the guard's answer: the host goes on as the walk starts (waiting for
// its end takes 25 us a call).  Ends at the latest with the stream's work.
int wait_guard(pc_ctx *ctx, const Guard &g, hipStream_t stream, bool *too_long)
{
    for (unsigned n = 1;; ++n) {
        // (seldom: a query puts a marker into the stream)
        const bool over = n % (1u << 20) == 0 && hipStreamQuery(stream) != hipErrorNotReady;
        const unsigned long long x = __atomic_load_n(g.host, __ATOMIC_ACQUIRE);
        *too_long = x & 1;
        if (x >> 32 == g.call) return PC_OK;
        if (over) {
            PC_HIP(ctx, hipStreamSynchronize(stream));
            return pc_set_error(ctx, PC_EDEVICE, "pc_trace_flows: no word from the device");
        }
    }
}

}  // namespace

int run_trace(pc_ctx *ctx, int32_t S, const int32_t *port_off, const int32_t *port_peer, int64_t n_ports,
              const uint8_t *jur, const int32_t *rule_off, const pc_rule *rules, int64_t n_rules,
              const pc_key *hdr, const int32_t *ingress, int32_t T, int32_t ttl, const int32_t *watch, int32_t K,
              pc_trace_out *out, uint32_t *visit, uint64_t *vsum, int32_t *walk, hipStream_t stream,
              const TracePrep *pre)
{
    struct Bufs {
        int32_t *gcount, *bcount, *gofs, *bofs, *counts0, *counts1, *boff, *ioff;
        BRec *bucket;
        LRec *live0, *live1;
        int2 *pinfo, *imap;
        SwInfo *sinfo;
        uint32_t *filt, *cpos, *hh;
        uint16_t *prio;
    } B;
    const int64_t mean_groups = S > 0 ? (pre != nullptr ? pre->groups : (n_rules + 31) / 32) / S : 0;
    // (until the largest table is known, the rule without it)
    int64_t largest = pre != nullptr ? pre->largest : 0;
    int64_t most_walks = walk_most(mean_groups, largest);
    bool levels = T > most_walks;
    bool may_level = pre != nullptr ? levels : T > walk_most(mean_groups, kWalkGroups);
    // Few enough traces over tables this small are matched rule by rule: no
    // chunk sets, no wait for their count, two launches.  Chunk sets / rule by
    // rule: 1,000 traces over 16 rules per switch 46 / 23 us (k = 16), 4,000
    // over 1,024 rules 61 / 55, 60,000 over 64 rules 145 / 68, 16,000 over 256
    // rules 89 / 54; past the limit 16,000 over 512 rules 93 / 100, over 1,024
    // 96 / 189.
    bool direct = pre == nullptr && !levels && S > 0 && (T > 0 || n_rules <= kDirectTable) &&
                  n_rules <= static_cast<int64_t>(kDirectRules) * S &&
                  static_cast<int64_t>(T) * (n_rules / S + 1) <= kDirectWork &&
                  static_cast<int64_t>(T) * n_rules <= kDirectWorst;
    // The host knows the mean table only, and a wavefront takes a hop's rules in
    // turn: where one table could hold too many, the preparation looks for such a
    // table, the walk goes on only if there is none, and the host waits for the
    // answer to see whether the call needs chunk sets after all.  All but 16 rules a switch
    // (k = 16) in the table that every trace enters, rule by rule / found too long:
    // 16,384 rules, one trace 29 / 48 us, 1,000 traces 45 / 57; 55,000, one trace
    // 70 / 49, 1,000 traces 110 / 58; 262,144, one trace 1,989 (the table's
    // actions swept by one wavefront too) / 69.  Asking costs 0-4 us: 3,000 traces
    // over 64 rules a switch (k = 16) 15 / 17, 500 over 100 (k = 32) 13 / 17.
    const int64_t longest = std::min(kDirectTable, kDirectTableWork / std::max(T, 1));
    // (A stream under capture cannot be waited for: no question then.)
    const bool guarded = direct && n_rules > longest && !capturing(stream);
    // work items of a level: at most T / kItemMin + S (see the match launch)
    const int32_t icap = static_cast<int32_t>(std::min<int64_t>(static_cast<int64_t>(T) / kItemMin + S + 1, INT32_MAX));
    auto carve = [&](Carver &c) {
        B.pinfo = c.take<int2>(static_cast<size_t>(n_ports) + 1);
        B.sinfo = c.take<SwInfo>(static_cast<size_t>(S) + 1);
        if (direct) return;
        B.cpos = c.take<uint32_t>(S + 1);
        B.hh = c.take<uint32_t>(kHistWords);
        B.gcount = c.take<int32_t>(S + 1);
        B.bcount = c.take<int32_t>(S + 1);
        B.gofs = c.take<int32_t>(S + 1);
        B.bofs = c.take<int32_t>(S + 1);
        if (!may_level) return;
        B.counts0 = c.take<int32_t>(2 * static_cast<size_t>(S + 1) * kCountPad);
        B.counts1 = B.counts0 + static_cast<size_t>(S + 1) * kCountPad;
        B.boff = c.take<int32_t>(S + 1);
        B.ioff = c.take<int32_t>(S + 1);
        B.live0 = c.take<LRec>(T + 1);
        B.live1 = c.take<LRec>(T + 1);
        B.bucket = c.take<BRec>(T + 1);
        B.imap = c.take<int2>(static_cast<size_t>(icap));
    };
    auto reserve = [&]() -> int {
        Carver dry{nullptr, 0};
        carve(dry);
        const int rc = pc_ensure_arena(ctx, dry.off);
        Carver real{ctx->arena, 0};
        if (rc == PC_OK) carve(real);
        return rc;
    };
    int rc = reserve();
    if (rc == PC_ENOMEM && may_level && T <= walk_most(mean_groups, 0)) {
        // no room for levels, which only the largest table asks for: walks, which need none
        may_level = levels = false;
        rc = reserve();
        if (rc == PC_OK) ctx->msg[0] = 0;
    }
    if (rc) return rc;
    if (!visit) K = 0;
    const int64_t n_watch = static_cast<int64_t>(T) * K;
    Infos inf{B.sinfo, B.pinfo, port_off, port_peer, n_ports, jur, nullptr, ctx->d_err};
    B.filt = nullptr;
    B.prio = nullptr;
    auto walk_args = [&]() { return WalkArgs{S, B.sinfo, B.pinfo, rules, B.filt, ttl, out, watch, K, visit, vsum, walk}; };
    auto walk_all = [&](int threads, const Guard &guard) -> int {
        PC_TIMED(ctx, "k_tr_walk", stream,
                 hipLaunchKernelGGL(direct ? k_tr_walk_all<true> : k_tr_walk_all<false>,
                                    dim3(static_cast<unsigned>(std::min(T, 8192))), dim3(threads), 0, stream, walk_args(), T, hdr, ingress, jur, ctx->d_err, nullptr, guard));
        PC_LAUNCH_CHECK(ctx);
        return PC_OK;
    };

    // ---- rule by rule
    auto by_rule = [&](const Guard &guard) -> int {
        const int64_t sweep = (std::max(n_ports, n_watch) + 4 * kDirectThreads - 1) / (4 * kDirectThreads);
        const int64_t blocks = std::max<int64_t>(S, std::min<int64_t>(sweep, 1024));
        PC_TIMED(ctx, "k_tr_direct", stream,
                 hipLaunchKernelGGL(k_tr_direct, dim3(static_cast<unsigned>(blocks)), dim3(kDirectThreads), 0, stream, S,
                                    rule_off, n_rules, rules, n_watch, watch, inf, guard));
        PC_LAUNCH_CHECK(ctx);
        return T > 0 ? walk_all(64, guard) : PC_OK;
    };
    // where the chunk sets of a call whose longest table asks for them are
    // refused, its rules are matched one by one all the same
    auto refused = [&](int rc) -> int {
        if (rc != PC_ENOMEM || !guarded) return rc;
        direct = true;
        rc = reserve();
        if (rc) return rc;
        ctx->msg[0] = 0;
        inf.sinfo = B.sinfo;
        inf.pinfo = B.pinfo;
        return by_rule(Guard{});
    };
    if (direct) {
        Guard guard{};
        if (guarded) {
            ctx->direct_call = ctx->direct_call == UINT32_MAX ? 1 : ctx->direct_call + 1;
            guard = Guard{reinterpret_cast<uint32_t *>(ctx->d_small + 8), ctx->direct_call,
                          static_cast<int32_t>(longest), reinterpret_cast<unsigned long long *>(ctx->h_small + 16),
                          S <= kLayoutS};
            *guard.host = 0;  // (the last guarded call's has been read)
        }
        rc = by_rule(guard);
        if (rc || !guarded) return rc;
        bool too_long = false;
        rc = wait_guard(ctx, guard, stream, &too_long);
        if (rc || !too_long) return rc;
        direct = false;
        rc = reserve();
        if (rc) return refused(rc);
        inf.sinfo = B.sinfo;
        inf.pinfo = B.pinfo;
    }

    // ---- prep: per-switch sizes, offsets, chunk sets, data-error sweep
    // (done by the caller when it passes prepared tables)
    if (pre != nullptr) {
        B.filt = const_cast<uint32_t *>(pre->filt);
        B.prio = pre->prio;
        B.gcount = const_cast<int32_t *>(pre->gcount);
        const int64_t n_info = std::max<int64_t>(n_ports, S);
        if (n_info > 0)
            PC_TIMED(ctx, "k_tr_port_info", stream,
                     hipLaunchKernelGGL(k_tr_port_info, dim3(static_cast<unsigned>(std::min<int64_t>((n_info + 255) / 256, 4096))),
                                        dim3(256), 0, stream, n_ports, port_off, port_peer, S, jur, rule_off, n_rules,
                                        pre->gofs, pre->cpos, B.pinfo, B.sinfo));
        if (n_watch > 0)
            PC_TIMED(ctx, "k_tr_sweep", stream,
                     hipLaunchKernelGGL(k_tr_sweep, dim3(256), dim3(256), 0, stream, int64_t(0), nullptr, S, n_watch,
                                        watch, nullptr, 0, nullptr, ctx->d_err));
        PC_LAUNCH_CHECK(ctx);
    } else if (S > 0) {
        rc = layout(ctx, S, port_off, n_ports, jur, rule_off, n_rules, B.gcount, B.bcount, B.gofs, B.bofs, B.hh, stream);
        if (rc) return rc;
        inf.gofs = B.gofs;
        // exact sizes of the chunk-set buffer and of the prep grid (switch
        // ranges may overlap, so no host-side bound from n_rules holds);
        // the host waits for these two counts only, while the sweeps and
        // the chunk choice, queued behind them, keep the GPU busy
        PC_HIP(ctx, hipEventRecord(ctx->lvl_ev[0], stream));
        rc = sweep_and_choose(ctx, S, port_peer, n_ports, rule_off, n_rules, rules, hdr, T, n_watch, watch, B.hh,
                              B.cpos, inf, stream);
        if (rc) return rc;
        PC_HIP(ctx, hipEventSynchronize(ctx->lvl_ev[0]));
        const int64_t groups = ctx->h_small[0], prep_blocks = ctx->h_small[1];
        if (groups < 0 || prep_blocks < 0)
            return pc_set_error(ctx, PC_EINVAL, "pc_trace_flows: more than 2^31 rule groups");
        largest = ctx->h_small[2];
        most_walks = walk_most(mean_groups, largest);
        levels = may_level && T > most_walks;
        bool ranked = levels && !wide_level(T, S, mean_groups);  // (levels only shrink)
        rc = pc_ensure_aux(ctx, chunk_set_bytes(groups, ranked));
        if (rc == PC_ENOMEM && ranked) {  // no room for the priorities: k_tr_match_wide needs none
            ranked = false;
            rc = pc_ensure_aux(ctx, chunk_set_bytes(groups, false));
            if (rc == PC_OK) ctx->msg[0] = 0;
        }
        if (rc) return refused(rc);
        B.filt = reinterpret_cast<uint32_t *>(ctx->aux);
        if (ranked) B.prio = priorities(ctx->aux, groups);
        if (prep_blocks > 0 && n_rules > 0) {
            PC_TIMED(ctx, "k_tr_prep", stream, hipLaunchKernelGGL(k_tr_prep, dim3(static_cast<unsigned>(prep_blocks)), dim3(kPrepWaves * 64), 0, stream, S,
                               port_off, n_ports, rule_off, rules, B.gcount, B.gofs, B.bofs, B.filt,
                               B.prio, ctx->d_err, nullptr, B.cpos));
            PC_LAUNCH_CHECK(ctx);
        }
    }
    if (T == 0) return PC_OK;
    if (!levels) return walk_all(walk_threads(T, mean_groups, largest), Guard{});
    const WalkArgs wa = walk_args();

    // ---- level-synchronous walk
    int32_t *d_n = ctx->d_small;  // [0], [1]: live counts of the two live lists ([4], [5]: the reach kernels')
    launch_fill_u32(reinterpret_cast<uint32_t *>(d_n), 2, 0, stream);
    if (S > 0)
        launch_fill_u32(reinterpret_cast<uint32_t *>(B.counts0), 2 * static_cast<size_t>(S + 1) * kCountPad, 0, stream);
    {
        const dim3 ig(static_cast<unsigned>((static_cast<int64_t>(T) + kInitPer - 1) / kInitPer));
        if (S <= kInitLdsS)
            PC_TIMED(ctx, "k_tr_init", stream,
                     hipLaunchKernelGGL(k_tr_init<true>, ig, dim3(kInitThreads), static_cast<size_t>(S) * 4, stream, S,
                                        jur, ingress, hdr, T, B.live0, d_n, B.counts0, out, watch, K, visit, vsum,
                                        walk, ctx->d_err));
        else
            PC_TIMED(ctx, "k_tr_init", stream,
                     hipLaunchKernelGGL(k_tr_init<false>, ig, dim3(kInitThreads), 0, stream, S, jur, ingress, hdr, T,
                                        B.live0, d_n, B.counts0, out, watch, K, visit, vsum, walk, ctx->d_err));
    }
    PC_LAUNCH_CHECK(ctx);
    LRec *live_cur = B.live0, *live_nxt = B.live1;
    int32_t *cnt_cur = B.counts0, *cnt_nxt = B.counts1;
    int32_t *n_cur = d_n, *n_nxt = d_n + 1;
    // The host does not wait for a level before queueing the next one: live
    // counts only shrink, so level L is launched with the latest count the
    // host has (exact for level 0, else the count entering level L - 1) as
    // the bound for its grids, and the kernels read the exact count on the
    // device.  Level L's plan writes the count entering it to host memory,
    // and the host waits for that plan while level L runs.
    int32_t *h_cnt = ctx->h_small + 8;  // two pinned slots, by level parity
    int32_t *d_len = ctx->d_small + 6;  // two slots, by level parity: each level's lookups (its live list's length)
    // An upper bound on the count entering the next level (T for level 0:
    // the host does not wait for the initial count); from level 2 on, also
    // the exact length of the live list the previous level wrote (every
    // lookup of a level leaves an entry, the traces that ended included).
    int64_t known = T;
    for (int level = 0;; ++level) {
        if (level > ttl + 2)
            return pc_set_error(ctx, PC_EDEVICE, "pc_trace_flows: level loop exceeded ttl+2 levels");
        if (known == 0) break;
        // the live list this level reads: from k_tr_init (as many entries as
        // traces in flight) or from the previous level's match
        const int32_t *len_cur = level == 0 ? n_cur : d_len + ((level - 1) & 1);
        if (known <= most_walks) {
            const unsigned wb = static_cast<unsigned>(known < 8192 ? known : 8192);
            PC_TIMED(ctx, "k_tr_walk", stream,
                     hipLaunchKernelGGL(k_tr_walk, dim3(wb), dim3(walk_threads(known, mean_groups, largest)), 0, stream, wa,
                                        live_cur, len_cur, level));
            PC_LAUNCH_CHECK(ctx);
            break;
        }
        const int32_t nlive = static_cast<int32_t>(known);
        const bool wide = B.prio == nullptr || wide_level(known, S, mean_groups);
        // Larger items read a table's sets less often, as long as there are enough
        // of them (192 / 256 / 384 lookups: a million over 320 tables of 1,024
        // rules 254 / 232 / 199 us, over 720 of 8,192 816 / 772 / 697).
        const int32_t cap = wide ? kWideItem
                                 : static_cast<int32_t>(std::min<int64_t>(std::max<int64_t>(known / kItemsWanted, kItemLeast), kItemMax));
        PC_TIMED(ctx, "k_tr_plan", stream,
                 hipLaunchKernelGGL(k_tr_plan, dim3(1), dim3(1024), 0, stream, cnt_cur, S, B.boff, B.ioff, cap, d_len + (level & 1), n_nxt, h_cnt + (level & 1)));
        PC_HIP(ctx, hipEventRecord(ctx->lvl_ev[level & 1], stream));
        PC_TIMED(ctx, "k_tr_scatter", stream,
                 hipLaunchKernelGGL(k_tr_scatter, dim3(grid_for(nlive, 256)), dim3(256), 0, stream, live_cur, len_cur,
                                    T, S, B.boff, B.bucket, B.ioff, B.imap, icap));
        const Level lv{S,        T,     port_peer, B.pinfo, jur,   ttl, cap, level, live_nxt, n_nxt,
                       cnt_nxt, out,   watch,     K,       visit, vsum, walk};
        // at most nlive / kItemMin + S items: a switch of n lookups takes ceil(n / cap) items with cap >= kItemMin
        const int64_t max_items = std::min<int64_t>(static_cast<int64_t>(nlive) / kItemMin + S, nlive);
        const dim3 mgrid(static_cast<unsigned>(8 * ((max_items + 7) / 8)));
        if (wide)
            PC_TIMED(ctx, "k_tr_match_wide", stream,
                     hipLaunchKernelGGL(k_tr_match_wide, mgrid, dim3(kWideThreads), 0, stream, S, B.sinfo, rules,
                                        B.filt, B.boff, B.ioff, B.imap, B.bucket, lv));
        else
            PC_TIMED(ctx, "k_tr_match", stream,
                     hipLaunchKernelGGL(k_tr_match, mgrid, dim3(kMatchThreads), 0, stream, S, B.sinfo, rules, B.filt,
                                        B.prio, B.boff, B.ioff, B.imap, B.bucket, lv));
        PC_LAUNCH_CHECK(ctx);
        if (level == 0) {
            known = nlive;  // the bound for level 1; its exact count is learned after level 0 completes
        } else {
            // the count entering this level, written by its plan
            PC_HIP(ctx, hipEventSynchronize(ctx->lvl_ev[level & 1]));
            known = h_cnt[level & 1];
        }
        std::swap(live_cur, live_nxt);
        int32_t *tmp;
        tmp = cnt_cur; cnt_cur = cnt_nxt; cnt_nxt = tmp;
        tmp = n_cur; n_cur = n_nxt; n_nxt = tmp;
    }
    return PC_OK;
}

namespace {

// Per-switch arrays of the cached prepared tables in ctx->tc_meta.
struct TcMeta {
    int32_t *gcount, *bcount, *gofs, *bofs;
    uint32_t *sw_bad, *cpos, *hh;
};

TcMeta tc_meta(pc_ctx *ctx, int32_t S)
{
    Carver c{ctx->tc_meta, 0};
    TcMeta m;
    m.gcount = c.take<int32_t>(static_cast<size_t>(S) + 1);
    m.bcount = c.take<int32_t>(static_cast<size_t>(S) + 1);
    m.gofs = c.take<int32_t>(static_cast<size_t>(S) + 1);
    m.bofs = c.take<int32_t>(static_cast<size_t>(S) + 1);
    m.sw_bad = c.take<uint32_t>(static_cast<size_t>(S) + 1);
    m.cpos = c.take<uint32_t>(static_cast<size_t>(S) + 1);
    m.hh = c.take<uint32_t>(kHistWords);
    return m;
}

size_t tc_meta_bytes(int32_t S) { return 7 * (256 + (static_cast<size_t>(S) + 1) * 4) + kHistWords * 4; }

// The kept tables' priorities (nullptr: there was no room for them).
uint16_t *kept_priorities(pc_ctx *ctx)
{
    return ctx->tc_ranked ? priorities(ctx->tc_filt, ctx->tc_groups) : nullptr;
}

// Prepare every switch's tables into the context's cache (and sweep them
// for data errors); the cache then describes these tables.
int tc_prepare_all(pc_ctx *ctx, int32_t S, const int32_t *port_off, const int32_t *port_peer, int64_t n_ports,
                   const uint8_t *jur, const int32_t *rule_off, const pc_rule *rules, int64_t n_rules,
                   const pc_key *hdr, int32_t T, hipStream_t stream)
{
    ctx->tc_S = -1;
    int rc = pc_ensure_tc_meta(ctx, tc_meta_bytes(S));
    if (rc) return rc;
    const TcMeta m = tc_meta(ctx, S);
    int64_t groups = 0, blocks = 0, largest = 0;
    if (S > 0) {
        rc = layout(ctx, S, port_off, n_ports, jur, rule_off, n_rules, m.gcount, m.bcount, m.gofs, m.bofs, m.hh, stream);
        if (rc) return rc;
        PC_HIP(ctx, hipEventRecord(ctx->lvl_ev[0], stream));
        // queued while the host waits for the two counts
        launch_fill_u32(m.sw_bad, static_cast<size_t>(S), 0, stream);
        rc = sweep_and_choose(ctx, S, port_peer, n_ports, rule_off, n_rules, rules, hdr, T, 0, nullptr, m.hh, m.cpos,
                              Infos{}, stream);
        if (rc) return rc;
        PC_HIP(ctx, hipEventSynchronize(ctx->lvl_ev[0]));
        groups = ctx->h_small[0];
        blocks = ctx->h_small[1];
        largest = ctx->h_small[2];
        if (groups < 0 || blocks < 0)
            return pc_set_error(ctx, PC_EINVAL, "pc_trace_flows_delta: more than 2^31 rule groups");
    }
    ctx->tc_ranked = true;
    rc = pc_ensure_tc_filt(ctx, chunk_set_bytes(groups, true));
    if (rc == PC_ENOMEM) {  // no room for the priorities: k_tr_match_wide needs none
        ctx->tc_ranked = false;
        rc = pc_ensure_tc_filt(ctx, chunk_set_bytes(groups, false));
        if (rc == PC_OK) ctx->msg[0] = 0;
    }
    if (rc) return rc;
    if (S > 0) {
        if (blocks > 0) {
            PC_TIMED(ctx, "k_tr_prep", stream,
                     hipLaunchKernelGGL(k_tr_prep, dim3(static_cast<unsigned>(blocks)), dim3(kPrepWaves * 64), 0,
                                        stream, S, port_off, n_ports, rule_off, rules, m.gcount, m.gofs, m.bofs,
                                        reinterpret_cast<uint32_t *>(ctx->tc_filt),
                                        ctx->tc_ranked ? priorities(ctx->tc_filt, groups) : nullptr, ctx->d_err,
                                        m.sw_bad, m.cpos));
            PC_LAUNCH_CHECK(ctx);
        }
    }
    ctx->tc_S = S;
    ctx->tc_groups = groups;
    ctx->tc_blocks = blocks;
    ctx->tc_largest = largest;
    return PC_OK;
}

}  // namespace

int run_trace_delta(pc_ctx *ctx, int32_t S, const int32_t *port_off, const int32_t *port_peer, int64_t n_ports,
                    const uint8_t *jur, const int32_t *rule_off, const pc_rule *rules, int64_t n_rules,
                    const pc_key *hdr, const int32_t *ingress, int32_t T, int32_t ttl, const int32_t *changed,
                    int32_t C, pc_trace_out *out, uint64_t *vsum, int32_t *walk, int32_t *n_retraced,
                    hipStream_t stream)
{
    if (C < 0) {  // every trace, from scratch; the prepared tables are kept for later deltas
        launch_fill_u32(reinterpret_cast<uint32_t *>(n_retraced), 1, static_cast<uint32_t>(T), stream);
        int rc = tc_prepare_all(ctx, S, port_off, port_peer, n_ports, jur, rule_off, rules, n_rules, hdr, T, stream);
        if (rc) return rc;
        if (T == 0) return PC_OK;
        const TcMeta m = tc_meta(ctx, S);
        const TracePrep pre{reinterpret_cast<const uint32_t *>(ctx->tc_filt), m.gcount, m.gofs, m.cpos,
                            ctx->tc_groups, ctx->tc_largest, kept_priorities(ctx)};
        return run_trace(ctx, S, port_off, port_peer, n_ports, jur, rule_off, rules, n_rules, hdr, ingress, T, ttl,
                         nullptr, 0, out, nullptr, vsum, walk, stream, &pre);
    }
    // compacted traces live in their own buffer: run_trace carves the arena
    const size_t Tn = static_cast<size_t>(T) + 1;
    const size_t words = (static_cast<size_t>(S) + 31) / 32 + 1;
    const size_t need = 256 * 9 + words * 4 +
                        Tn * (sizeof(int32_t) * 2 + sizeof(pc_key) + sizeof(pc_trace_out) + 8 + 4 * kWalkSlots);
    int rc = pc_ensure_delta(ctx, need);
    if (rc) return rc;
    Carver cv{ctx->delta, 0};
    DeltaState *state = cv.take<DeltaState>(1);
    uint32_t *bitmap = cv.take<uint32_t>(words);
    int32_t *list = cv.take<int32_t>(Tn);
    pc_key *hdr_c = cv.take<pc_key>(Tn);
    int32_t *ing_c = cv.take<int32_t>(Tn);
    pc_trace_out *out_c = cv.take<pc_trace_out>(Tn);
    uint64_t *vsum_c = cv.take<uint64_t>(Tn);
    int32_t *walk_c = cv.take<int32_t>(Tn * kWalkSlots);
    int2 *pinfo;
    SwInfo *sinfo;
    auto carve = [&](Carver &c) {
        pinfo = c.take<int2>(static_cast<size_t>(n_ports) + 1);
        sinfo = c.take<SwInfo>(static_cast<size_t>(S) + 1);
    };
    Carver dry{nullptr, 0};
    carve(dry);
    rc = pc_ensure_arena(ctx, dry.off);
    if (rc) return rc;
    Carver real{ctx->arena, 0};
    carve(real);

    // with reuse declared (pc_trace_keep_tables) the cache holds the previous
    // tables when its switch count matches; it serves the new ones when no
    // switch's group count changed.  Without it every call prepares anew.
    const bool cached = ctx->tc_keep && ctx->tc_S == S && S > 0;
    const TcMeta kept = cached ? tc_meta(ctx, S) : TcMeta{};
    const bool one = S <= kLayoutS && C <= kLayoutS;
    if (!one) {
        launch_fill_u32(reinterpret_cast<uint32_t *>(state), sizeof(DeltaState) / 4, 0, stream);
        launch_fill_u32(bitmap, words, 0, stream);
    }
    PC_TIMED(ctx, "k_delta_plan", stream,
             hipLaunchKernelGGL(k_delta_plan, dim3(one ? 1 : grid_for(std::max(S, C), 1024)), dim3(1024), 0, stream,
                                changed, C, S, state, bitmap, static_cast<int32_t>(words), port_off, n_ports, jur,
                                rule_off, n_rules, kept.gcount, kept.sw_bad, ctx->d_err));
    if (T > 0)
        PC_TIMED(ctx, "k_delta_select", stream,
                 hipLaunchKernelGGL(k_delta_select, dim3(grid_for(T, 1024)), dim3(1024), 0, stream, vsum, walk, out,
                                    bitmap, ingress, T, S, state, list, ctx->d_err));
    PC_TIMED(ctx, "k_delta_post", stream,
             hipLaunchKernelGGL(k_delta_post,
                                dim3(cached ? grid_for(std::min<int64_t>(std::max<int64_t>(n_ports, S), 1 << 20), 256) : 1),
                                dim3(256), 0, stream, state, ctx->h_small, n_retraced, cached, n_ports, port_off,
                                port_peer, S, jur, rule_off, n_rules, kept.gofs, kept.cpos, pinfo, sinfo, kept.sw_bad,
                                ctx->d_err));
    PC_LAUNCH_CHECK(ctx);
    PC_HIP(ctx, hipEventRecord(ctx->lvl_ev[0], stream));
    // while the host waits for the counts: the changed switches are prepared
    // again if the kept tables serve (they keep their filter chunks: any choice is exact)
    if (cached && ctx->tc_blocks > 0 && C > 0) {
        // By the list with a workgroup for every block of the largest table, unless that
        // is more than all tables' blocks (an empty workgroup costs some 10 ns).  One of
        // 320 switches with 1.1 million rules, 16 on the others, 1 / 16 / 320 changed, it
        // among them: 24 / 31 / 25 us, with workgroups for the mean table's blocks 1,132; 16
        // rules on each of 1,280, 16 / 1,280 changed: 9 / 22 us.
        const int64_t most = (ctx->tc_largest + kPrepGroups - 1) / kPrepGroups;
        uint32_t *filt = reinterpret_cast<uint32_t *>(ctx->tc_filt);
        uint16_t *prio = kept_priorities(ctx);
        if (C <= 65535 && C * most <= ctx->tc_blocks)
            PC_TIMED(ctx, "k_tr_prep_listed", stream,
                     hipLaunchKernelGGL(k_tr_prep_listed, dim3(static_cast<unsigned>(most), static_cast<unsigned>(C)),
                                        dim3(kPrepWaves * 64), 0, stream, S, port_off, n_ports, rule_off, rules,
                                        kept.gcount, kept.gofs, kept.bofs, filt, prio, ctx->d_err, kept.sw_bad,
                                        kept.cpos, changed, &state->differs));
        else
            PC_TIMED(ctx, "k_tr_prep_marked", stream,
                     hipLaunchKernelGGL(k_tr_prep_marked, dim3(static_cast<unsigned>(ctx->tc_blocks)),
                                        dim3(kPrepWaves * 64), 0, stream, S, port_off, n_ports, rule_off, rules,
                                        kept.gcount, kept.gofs, kept.bofs, filt, prio, ctx->d_err, kept.sw_bad,
                                        kept.cpos, bitmap, &state->differs));
        PC_LAUNCH_CHECK(ctx);
    }
    PC_HIP(ctx, hipEventSynchronize(ctx->lvl_ev[0]));
    const int32_t n = ctx->h_small[0];
    const bool serves = cached && ctx->h_small[1] == 0;
    if (!serves) {
        rc = tc_prepare_all(ctx, S, port_off, port_peer, n_ports, jur, rule_off, rules, n_rules, hdr, T, stream);
        if (rc) return rc;
    }
    if (n == 0) return PC_OK;
    const TcMeta m = tc_meta(ctx, S);
    const int64_t mean_groups = S > 0 ? ctx->tc_groups / S : 0;
    if (n <= walk_most(mean_groups, ctx->tc_largest)) {  // walked in place
        const int64_t n_info = std::max<int64_t>(n_ports, S);
        if (!serves && n_info > 0)
            PC_TIMED(ctx, "k_tr_port_info", stream,
                     hipLaunchKernelGGL(k_tr_port_info, dim3(static_cast<unsigned>(std::min<int64_t>((n_info + 255) / 256, 4096))),
                                        dim3(256), 0, stream, n_ports, port_off, port_peer, S, jur, rule_off, n_rules,
                                        m.gofs, m.cpos, pinfo, sinfo));
        const WalkArgs wa{S, sinfo, pinfo, rules, reinterpret_cast<const uint32_t *>(ctx->tc_filt), ttl, out, nullptr,
                          0, nullptr, vsum, walk};
        PC_TIMED(ctx, "k_tr_walk", stream,
                 hipLaunchKernelGGL(k_tr_walk_all<false>, dim3(static_cast<unsigned>(std::min(n, 8192))),
                                    dim3(walk_threads(n, mean_groups, ctx->tc_largest)), 0, stream, wa, n, hdr, ingress, jur, ctx->d_err, list, Guard{}));
        PC_LAUNCH_CHECK(ctx);
        return PC_OK;
    }
    PC_TIMED(ctx, "k_delta_gather", stream,
             hipLaunchKernelGGL(k_delta_gather, dim3(grid_for(n, 256)), dim3(256), 0, stream, list, n, hdr, ingress,
                                hdr_c, ing_c));
    PC_LAUNCH_CHECK(ctx);
    const TracePrep pre{reinterpret_cast<const uint32_t *>(ctx->tc_filt), m.gcount, m.gofs, m.cpos,
                        ctx->tc_groups, ctx->tc_largest, kept_priorities(ctx)};
    rc = run_trace(ctx, S, port_off, port_peer, n_ports, jur, rule_off, rules, n_rules, hdr_c, ing_c, n, ttl, nullptr,
                   0, out_c, nullptr, vsum_c, walk ? walk_c : nullptr, stream, &pre);
    if (rc) return rc;
    PC_TIMED(ctx, "k_delta_scatter", stream,
             hipLaunchKernelGGL(k_delta_scatter, dim3(grid_for(n, 256)), dim3(256), 0, stream, list, n, out_c, vsum_c,
                                walk_c, out, vsum, walk));
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}
