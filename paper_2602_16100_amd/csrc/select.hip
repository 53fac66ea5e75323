// A1 -- placement constraints: node-selector evaluation for every selector
// row x node, emitting a feasible-node bitset and a popcount per row.
//
// The operators are Kubernetes node-affinity's (In / NotIn / Exists over a
// label), which is how the paper compiles a placement constraint such as a
// residency region that the pod's node must carry as a label (Formal Model
// and Satisfaction, example; Service Placement Module).
//
// Design (gfx950):
//   1. presence  : which values of each label occur at all.
//   2. label scan: plane numbering -- one plane per present (label, value);
//                  on small inputs by the last presence workgroup.
//   3. planes    : one 64-bit node set per (plane, 64-node word), built with
//                  a ballot per present value; row-major, Wp words a plane.
//                  For the affinity paths also the prefix planes.
//   4. compile   : eight lanes per row turn its predicates into a clause
//                  program over plane ids (In S = OR of S's planes or NOT OR
//                  of the rest, whichever is shorter; NotIn the reverse;
//                  Exists = NOT the absent-value plane), validate it, and
//                  write a 64-byte row record holding programs of up to 15
//                  entries inline.
//   5. eval      : one row at a time per wavefront over a tile of 128 words
//                  (two per lane, 16-byte loads and stores).  The row's
//                  record arrives through scalar loads, so its plane loads
//                  (L2 hits: a tile of every plane is P KiB), exactly as
//                  many as its program has entries, all go out together
//                  with scalar offsets, followed by one output store.  A
//                  row's tiles are shifted so that stores cover whole
//                  128-byte lines.  Per-lane popcounts are collected as
//                  bytes in LDS and summed once per 64 rows; a last pass
//                  sums the tiles.
// Small clusters take none of these: k_sel_small.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "pc_internal.h"

namespace {

constexpr int kEvalThreads = 256;  // 4 wavefronts, one row at a time each
constexpr int kEvalWaves = kEvalThreads / 64;
constexpr int kWpl = 2;            // 64-bit words per lane
constexpr int kTileW = 64 * kWpl;  // words per tile
constexpr int kRecWords = 16;      // row record: header + 15 inline entries
constexpr int kInline = kRecWords - 1;
constexpr int kGroup = 8;          // plane loads in flight together
constexpr int kPad = 16;           // plane rows: words before column 0 (a row's shift is at most 15 words)

__device__ __forceinline__ uint64_t uniform_u64(uint64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// What a call clears before it counts, merges or reads: its presence sets,
// the all-zero plane, its counters.  One launch, or the validation's.
struct Clears {
    uint64_t *p[4];
    int64_t n[4];
    uint64_t v[4];
    __device__ __forceinline__ void run() const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n[k];
                 i += static_cast<int64_t>(gridDim.x) * blockDim.x)
                p[k][i] = v[k];
    }
};

__global__ __launch_bounds__(256) void k_sel_clear(Clears c) { c.run(); }

// A call's counters (64-bit words, cleared): workgroups done with the
// presence sets, the entries of prog used, the class lists' lengths.
constexpr int kCtlDone = 0, kCtlProg = 1, kCtlLists = 2, kCtlWords = 4;

// Exclusive scan of per-label plane counts -> wbase[l][k] = id of the first
// plane of label l whose value lies in 64-value word k.  One workgroup of kT threads.
template <int kT, class Load>
__device__ __forceinline__ void scan_labels(int32_t L, uint32_t *__restrict__ wbase, Load &&present)
{
    constexpr int kW = kT / 64;
    __shared__ uint32_t wsum[kW];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    uint32_t carry = 0;
    for (int32_t base = 0; base < L; base += kT) {
        const int32_t l = base + tid;
        uint32_t c[4] = {0, 0, 0, 0};
        if (l < L)
            for (int k = 0; k < 4; ++k) c[k] = __popcll(present(static_cast<int64_t>(l) * 4 + k));
        const uint32_t v = c[0] + c[1] + c[2] + c[3];
        uint32_t x = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        uint32_t excl = carry + x - v;
        for (int w = 0; w < kW; ++w) {
            if (w < wid) excl += wsum[w];
            carry += wsum[w];
        }
        if (l < L) {
            for (int k = 0; k < 4; ++k) {
                wbase[static_cast<int64_t>(l) * 4 + k] = excl;
                excl += c[k];
            }
        }
        __syncthreads();
    }
}

// Which values each label has: labels is read as one flat array in 16-byte
// pieces (from the first 16-byte boundary on; the bytes before it and after
// the last piece one by one), a byte at a time tested against, and if new
// OR-ed into, the workgroup's LDS table (L x 256 bits), which is OR-ed into
// present32 at the end.  After the first nodes nearly every byte is only an
// LDS read.  100,000 nodes x 64 labels (6.4 MB): 38 us by single bytes, now 16.
// With done, the last workgroup to finish (no workgroup waits) numbers the planes.
constexpr int32_t kPresenceLdsL = 1024;  // labels whose table fits 32 KB
__global__ __launch_bounds__(256) void k_sel_presence_flat(const uint8_t *__restrict__ labels, int64_t n_bytes,
                                                           int32_t L, uint32_t *present32,
                                                           uint32_t *__restrict__ wbase, uint64_t *done)
{
    extern __shared__ uint32_t ptab[];  // [L][8]
    for (int32_t i = threadIdx.x; i < L * 8; i += 256) ptab[i] = 0;
    __syncthreads();
    auto put = [&](uint32_t l, uint32_t x) {
        uint32_t *w = ptab + l * 8 + (x >> 5);
        const uint32_t bit = 1u << (x & 31);
        if (!(*w & bit)) atomicOr(w, bit);
    };
    const int64_t head = min(n_bytes, static_cast<int64_t>((16 - (reinterpret_cast<uintptr_t>(labels) & 15)) & 15));
    const int64_t pieces = (n_bytes - head) / 16;
    const uint4 *body = reinterpret_cast<const uint4 *>(labels + head);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    constexpr int kAhead = 4;
    for (int64_t i0 = blockIdx.x * 256ll + threadIdx.x; i0 < pieces; i0 += stride * kAhead) {
        uint4 v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (i0 + k * stride < pieces) v[k] = body[i0 + k * stride];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (i0 + k * stride >= pieces) break;
            uint32_t l = static_cast<uint32_t>((head + (i0 + k * stride) * 16) % L);
            const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                put(l, (w[j / 4] >> (8 * (j % 4))) & 0xFFu);
                l = l + 1 == static_cast<uint32_t>(L) ? 0 : l + 1;
            }
        }
    }
    if (blockIdx.x == 0) {
        const int64_t tail = head + pieces * 16;
        for (int64_t o = threadIdx.x; o < head; o += 256) put(static_cast<uint32_t>(o % L), labels[o]);
        for (int64_t o = tail + threadIdx.x; o < n_bytes; o += 256) put(static_cast<uint32_t>(o % L), labels[o]);
    }
    __syncthreads();
    if (done == nullptr) {
        for (int32_t i = threadIdx.x; i < L * 8; i += 256)
            if (ptab[i] & ~present32[i]) atomicOr(&present32[i], ptab[i]);  // (mostly known by then: no contended atomics)
        return;
    }
    // An atomic that has returned its old value has been performed, so the
    // count below comes after this workgroup's sets without a fence (an
    // agent-wide release writes the L2 back: 100,000 nodes 89 us with one).
    // That is how this hardware orders them, not a release and an acquire: what
    // the last workgroup reads here it must read with atomic loads, and other
    // kernels read it only after this launch has ended.
    uint32_t seen = 0;
    for (int32_t i = threadIdx.x; i < L * 8; i += 256)
        if (ptab[i] & ~present32[i]) seen |= atomicOr(&present32[i], ptab[i]);
    asm volatile("" ::"v"(seen) : "memory");
    __shared__ bool last;
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(reinterpret_cast<unsigned long long *>(done), 1ull) + 1 == gridDim.x;
    __syncthreads();
    if (!last) return;
    const uint64_t *present = reinterpret_cast<const uint64_t *>(present32);
    scan_labels<256>(L, wbase, [&](int64_t i) {
        return __hip_atomic_load(present + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
}

// The same for more labels than the table holds: a tile of 64 labels per workgroup column.
__global__ __launch_bounds__(256) void k_sel_presence(const uint8_t *__restrict__ labels, int32_t N, int32_t L,
                                                      int64_t chunk, uint32_t *__restrict__ present32)
{
    __shared__ uint32_t tab[64 * 8];
    const int tid = threadIdx.x;
    for (int i = tid; i < 512; i += 256) tab[i] = 0;
    __syncthreads();
    const int lt = tid & 63, sub = tid >> 6;
    const int32_t l = blockIdx.x * 64 + lt;
    const int64_t n0 = static_cast<int64_t>(blockIdx.y) * chunk;
    const int64_t n1 = min(static_cast<int64_t>(N), n0 + chunk);
    uint32_t m[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // this thread's 256-bit value set, in registers
    if (l < L) {
        for (int64_t n = n0 + sub; n < n1; n += 4) {
            const uint32_t x = labels[n * L + l];
            const uint32_t word = x >> 5, bit = 1u << (x & 31);
#pragma unroll
            for (int k = 0; k < 8; ++k) m[k] |= word == static_cast<uint32_t>(k) ? bit : 0u;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (m[k]) atomicOr(&tab[lt * 8 + k], m[k]);
    }
    __syncthreads();
    for (int i = tid; i < 512; i += 256) {
        const int32_t ll = blockIdx.x * 64 + (i >> 3);
        if (ll < L && tab[i]) atomicOr(&present32[static_cast<int64_t>(ll) * 8 + (i & 7)], tab[i]);
    }
}

__global__ __launch_bounds__(1024) void k_sel_label_scan(const uint64_t *__restrict__ present, int32_t L,
                                                         uint32_t *__restrict__ wbase)
{
    scan_labels<1024>(L, wbase, [&](int64_t i) { return present[i]; });
}

// A wavefront builds kPlaneWords words (1,024 nodes) of one label's planes, so
// that what it writes of a plane is a whole 128-byte line, four values'
// lines to a store.  A lane keeps its nodes' values of the label.  Few
// values: per value and word a ballot gives the word, which moves into the
// lane that stores it.  More than kBallots of a 64-value word: every node sets
// its bit in an LDS tile (one atomic per node and label instead of a ballot
// per value).  A workgroup's wavefronts take four neighbouring labels, whose
// bytes arrive together (kWide: as one aligned word, L a multiple of 4).
// Word w of plane p lives at planes[p * Wp + kPad + w].
// 100,000 nodes x 64 labels: 78 us with a word per wavefront (8 bytes of a line
// written at a time), now 25; 50,000 nodes 44 us, now 16.
// kPrefix (the affinity paths): also plane pfx0 + p for each plane p of value v
// (not the absent value's) = OR of the label's planes of present values <= v, so that
// Gt / Lt take at most two entries (cmp_clause): an OR scan over the four values of
// a store, carried from store to store.  64 labels over 5,037 nodes: planes 11 us
// and, reading them again, prefix planes 11 in a launch of its own, now 13 together.
constexpr int kPlaneWords = 16;
constexpr int kBallots = 8;
template <bool kWide, bool kPrefix>
__global__ __launch_bounds__(256) void k_sel_planes(const uint8_t *__restrict__ labels, int32_t N, int32_t L,
                                                    const uint64_t *__restrict__ present,
                                                    const uint32_t *__restrict__ wbase, uint64_t *__restrict__ planes,
                                                    int64_t Wp, uint32_t pfx0)
{
    constexpr int kRow = 2 * kPlaneWords + 2;  // dwords per value of the tile: neighbouring values in other banks
    __shared__ __align__(8) uint32_t tiles[4][64 * kRow];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t w0 = blockIdx.x * kPlaneWords;
    const int32_t l = blockIdx.y * 4 + wave;
    if (l >= L) return;
    const int32_t W = static_cast<int32_t>((static_cast<int64_t>(N) + 63) / 64);
    uint32_t *tile = tiles[wave];
    uint32_t x[kPlaneWords];
#pragma unroll
    for (int k = 0; k < kPlaneWords; ++k) {
        const int64_t n = static_cast<int64_t>(w0 + k) * 64 + lane;
        x[k] = 0x100u;  // equals no value
        if (n < N) {
            if constexpr (kWide)
                x[k] = (*reinterpret_cast<const uint32_t *>(labels + n * L + blockIdx.y * 4) >> (8 * wave)) & 0xFFu;
            else
                x[k] = labels[n * L + l];
        }
    }
    const int col = lane & (kPlaneWords - 1), slot = lane / kPlaneWords;
    const bool store = w0 + col < W;
    uint64_t acc = 0;  // column col of the label's last prefix plane
    // words col of values v0 + slot of k4 (word 0 past the last) to their planes
    auto put = [&](uint64_t *out, int v0, int n, bool absent_last, uint64_t word) {
        const bool here = store && v0 + slot < n;
        if (here) out[static_cast<int64_t>(v0 + slot) * Wp + col] = word;
        if constexpr (kPrefix) {
            const uint64_t one = __shfl_up(word, kPlaneWords, 64);
            uint64_t x = word | (slot >= 1 ? one : 0);
            const uint64_t two = __shfl_up(x, 2 * kPlaneWords, 64);
            x |= (slot >= 2 ? two : 0) | acc;
            if (here && !(absent_last && v0 + slot == n - 1))
                out[(static_cast<int64_t>(pfx0) + v0 + slot) * Wp + col] = x;
            acc = __shfl(x, 3 * kPlaneWords + col, 64);
        }
    };
    for (int k4 = 0; k4 < 4; ++k4) {
        const uint64_t here = uniform_u64(present[static_cast<int64_t>(l) * 4 + k4]);
        const int n = __popcll(here);
        const bool absent_last = k4 == 3 && here >> 63;
        uint64_t *out = planes + static_cast<int64_t>(__builtin_amdgcn_readfirstlane(wbase[static_cast<int64_t>(l) * 4 + k4])) * Wp +
                        kPad + w0;
        if (n > kBallots) {
            for (int i = lane; i < n * kRow; i += 64) tile[i] = 0;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < kPlaneWords; ++k)
                if (x[k] >> 6 == static_cast<uint32_t>(k4)) {
                    const int r = __popcll(here & ((1ull << (x[k] & 63)) - 1));
                    atomicOr(&tile[r * kRow + 2 * k + (lane >> 5)], 1u << (lane & 31));
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int v0 = 0; v0 < n; v0 += 4)
                put(out, v0, n, absent_last,
                    v0 + slot < n ? *reinterpret_cast<const uint64_t *>(tile + (v0 + slot) * kRow + 2 * col) : 0);
            __builtin_amdgcn_wave_barrier();
            continue;
        }
        uint64_t m = here;
        for (int v0 = 0; v0 < n; v0 += 4) {
            uint64_t word = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (m == 0) break;
                const uint32_t v = static_cast<uint32_t>(k4 * 64 + __builtin_ctzll(m));
                m &= m - 1;
#pragma unroll
                for (int k = 0; k < kPlaneWords; ++k) {
                    const uint64_t b = __ballot(x[k] == v);
                    word = lane == j * kPlaneWords + k ? b : word;
                }
            }
            put(out, v0, n, absent_last, word);
        }
    }
}

__device__ __forceinline__ bool pred_valid(uint32_t label, uint32_t op, uint32_t rsv0, uint32_t rsv1, uint64_t v3,
                                           int32_t L)
{
    return static_cast<int32_t>(label) < L && op <= 2 && rsv0 == 0 && rsv1 == 0 &&
           (op == PC_OP_EXISTS || (v3 >> 63) == 0);
}

// Small clusters: every row evaluated from the labels themselves in one
// launch, without planes or programs.  A workgroup holds the cluster's
// labels in LDS and takes a row per wavefront; lane j of a wavefront has node j of
// each 64-node word, so that a predicate test ends in a ballot, and a row's
// predicates come by scalar loads.  Labels are kept per label in quads of words:
// dword (w / 4) * 64 + j of a label's row holds node j of words w..w+3, a byte each.
// Bound by launch and latency: 64 rows over 16 nodes 35 us in seven launches, now
// 15 (most of it the caller's); later ones by the scalar loads and 64-bit shifts
// of a test, about 120 clocks per predicate and word.
constexpr int kSmallThreads = 1024;
constexpr size_t kSmallLds = 64 * 1024;      // labels of the cluster, at most: two workgroups per CU
constexpr int64_t kSmallW = 8;               // words of a row, at most
constexpr int64_t kSmallWork = 400000;       // predicates x (words + 2), at most
constexpr int64_t small_rows(int64_t W) { return W == 1 ? 1 << 20 : W <= 4 ? 1 << 18 : 1 << 15; }  // rows, at most

// bytes of a label's row: whole pairs of quads, and a dword against bank conflicts
__host__ __device__ inline int64_t small_pitch(int64_t W) { return (W + 7) / 8 * 8 * 64 + 4; }

template <int kWords>  // words tested together: 1, 4 or 8
__global__ __launch_bounds__(kSmallThreads) void k_sel_small(const uint8_t *__restrict__ labels, int32_t N, int32_t L,
                                                             const int32_t *__restrict__ pred_off,
                                                             const pc_pred *__restrict__ preds, int64_t n_preds,
                                                             int32_t I, int32_t W, uint64_t *__restrict__ feasible,
                                                             uint32_t *__restrict__ popcnt,
                                                             uint32_t *__restrict__ d_err)
{
    extern __shared__ uint32_t small_lab[];
    uint8_t *lab8 = reinterpret_cast<uint8_t *>(small_lab);
    const int32_t pitch = static_cast<int32_t>(small_pitch(W));
    auto put = [&](int32_t n, int32_t l, uint32_t x) {
        lab8[l * pitch + (n >> 8) * 256 + (n & 63) * 4 + ((n >> 6) & 3)] = static_cast<uint8_t>(x);
    };
    const int32_t n_bytes = N * L;
    const int32_t n_dwords = (reinterpret_cast<uintptr_t>(labels) & 3) == 0 ? n_bytes / 4 : 0;
    constexpr int kAhead = 8;  // loads in flight
    for (int32_t i0 = threadIdx.x; i0 < n_dwords; i0 += kAhead * kSmallThreads) {
        uint32_t x[kAhead];
#pragma unroll
        for (int c = 0; c < kAhead; ++c)
            x[c] = reinterpret_cast<const uint32_t *>(labels)[min(i0 + c * kSmallThreads, n_dwords - 1)];
#pragma unroll
        for (int c = 0; c < kAhead; ++c) {
            const int32_t i = i0 + c * kSmallThreads;
            if (i >= n_dwords) break;
            int32_t n = 4 * i / L, l = 4 * i - n * L;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                put(n, l, (x[c] >> (8 * k)) & 255);
                if (++l == L) {
                    l = 0;
                    ++n;
                }
            }
        }
    }
    for (int32_t i = 4 * n_dwords + threadIdx.x; i < n_bytes; i += kSmallThreads) put(i / L, i % L, labels[i]);
    __syncthreads();

    const int lane = threadIdx.x & 63;
    constexpr int kWaves = kSmallThreads / 64;
    uint32_t errs = 0;
    for (int32_t r = blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); r < I;
         r += gridDim.x * kWaves) {
        const int64_t b = pred_off[r], e = pred_off[r + 1];
        bool good = pc_range_ok(b, e, n_preds);
        if (!good) errs |= PC_DERR_OFFSETS;
        uint32_t cnt = 0;
        uint64_t mine = 0;  // lane j: word j of the current 64
        for (int32_t w0 = 0; w0 < W; w0 += kWords) {
            uint64_t hold[kWords];
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                const int32_t left = N - (w0 + k) * 64;
                hold[k] = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1 : 0ull;
            }
            pc_pred ahead;
            if (good && b < e) ahead = preds[b];
            for (int64_t p = b; good && p < e;) {
                const pc_pred q = ahead;
                if (++p < e) ahead = preds[p];
                if (!pred_valid(q.label, q.op, q.rsv0, q.rsv1, q.vals[3], L)) {
                    errs |= PC_DERR_PRED;
                    good = false;
                    break;
                }
                const uint32_t *at = small_lab + (q.label * pitch >> 2) + (w0 >> 2) * 64 + lane;
                uint32_t x4[(kWords + 3) / 4];
#pragma unroll
                for (int k = 0; k < (kWords + 3) / 4; ++k) x4[k] = at[64 * k];
                auto test = [&](auto admits) {
#pragma unroll
                    for (int k = 0; k < kWords; ++k) {
                        const uint32_t x = (x4[k / 4] >> (8 * (k & 3))) & 255;
                        hold[k] &= admits(x);
                    }
                };
                const uint64_t flip = q.op == PC_OP_NOTIN ? ~0ull : 0ull;
                if (q.op == PC_OP_EXISTS) {
                    test([&](uint32_t x) { return __ballot(x != PC_LABEL_ABSENT); });
                } else if ((q.vals[1] | q.vals[2] | q.vals[3]) == 0) {
                    test([&](uint32_t x) { return __ballot(x < 64 && ((q.vals[0] >> (x & 63)) & 1)) ^ flip; });
                } else {
                    test([&](uint32_t x) {
                        const uint64_t lo = x & 64 ? q.vals[1] : q.vals[0], hi = x & 64 ? q.vals[3] : q.vals[2];
                        return __ballot(((x & 128 ? hi : lo) >> (x & 63)) & 1) ^ flip;
                    });
                }
            }
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                const uint64_t h = good ? hold[k] : 0;
                cnt += __popcll(h);
                mine = lane == ((w0 + k) & 63) ? h : mine;
            }
            const int32_t base = w0 & ~63;
            if (feasible != nullptr && ((w0 & 63) == 64 - kWords || w0 + kWords >= W) && base + lane < W)
                feasible[static_cast<int64_t>(r) * W + base + lane] = mine;
        }
        if (lane == 0) popcnt[r] = cnt;
    }
    if (errs && lane == 0) atomicOr(d_err, errs);
}

// Program entries: plane id, plus flags on the last entry of a clause
// (kLast, kNeg) and, in affinity programs, on the last entry of a term.
constexpr uint32_t kTermEnd = 1u << 29;
constexpr uint32_t kLast = 1u << 30;
constexpr uint32_t kNeg = 1u << 31;
constexpr uint32_t kPidMask = kTermEnd - 1;
// Row record header (word 0); words 1..15 hold an inline program.
constexpr int32_t kRowFalse = -1;     // some clause admits no node (or a malformed predicate)
constexpr int32_t kRowIndirect = -2;  // program of more than 15 entries at prog[4 * word1], word2 entries
constexpr int32_t kRowLong = -3;      // program longer than 4 entries per predicate: decoded on the fly

__device__ __forceinline__ uint32_t plane_id(const uint64_t *pres, const uint32_t *wb, uint32_t v)
{
    const uint32_t k = v >> 6;
    return wb[k] + __popcll(pres[k] & ((1ull << (v & 63)) - 1));
}

// Values lo..hi (clipped to 0..254) as a 256-bit set.
__device__ __forceinline__ void value_range(int64_t lo, int64_t hi, uint64_t s[4])
{
    lo = lo < 0 ? 0 : lo;
    hi = hi > 254 ? 254 : hi;
    for (int k = 0; k < 4; ++k) {
        const int64_t a = lo > 64 * k ? lo : 64 * k;
        const int64_t b = hi < 64 * k + 63 ? hi : 64 * k + 63;
        if (a > b) {
            s[k] = 0;
        } else {
            const int n = static_cast<int>(b - a + 1);
            s[k] = (n == 64 ? ~0ull : ((1ull << n) - 1)) << (a - 64 * k);
        }
    }
}

// The value set a clause ORs over, and whether the OR is negated, for an
// expression with operator op.  Each label value of a node lies in exactly
// one present plane (the absent value 255 included), so In S = OR(S) =
// NOT OR(present \ S) and NotIn S = NOT OR(S) = OR(present \ S): the
// shorter form is taken.  Exists = NOT OR(plane of the absent value), an
// empty OR when every node carries the label; DoesNotExist = that OR.
// Gt t / Lt t are In of the values above / below t.
__device__ __forceinline__ uint32_t expr_clause(uint32_t op, const uint64_t vals[4], const uint64_t *pres,
                                                uint64_t sel[4], bool &neg)
{
    if (op == PC_OP_EXISTS || op == PC_OP_DOESNOTEXIST) {
        sel[0] = sel[1] = sel[2] = 0;
        sel[3] = pres[3] & (1ull << 63);
        neg = op == PC_OP_EXISTS;
        return static_cast<uint32_t>(sel[3] >> 63);
    }
    uint64_t set[4];
    bool is_in = op != PC_OP_NOTIN;
    if (op == PC_OP_GT || op == PC_OP_LT) {
        const int64_t t = static_cast<int64_t>(vals[0]);
        if (op == PC_OP_GT)
            value_range(t >= 254 ? 255 : t + 1, 254, set);
        else
            value_range(0, t <= 0 ? -1 : t - 1, set);
    } else {
        for (int k = 0; k < 4; ++k) set[k] = vals[k];
    }
    uint64_t in[4], out[4];
    uint32_t ms = 0, mc = 0;
    for (int k = 0; k < 4; ++k) {
        in[k] = set[k] & pres[k];
        out[k] = pres[k] & ~set[k];
        ms += __popcll(in[k]);
        mc += __popcll(out[k]);
    }
    const bool use_in = ms <= mc;
    for (int k = 0; k < 4; ++k) sel[k] = use_in ? in[k] : out[k];
    neg = is_in ? !use_in : use_in;
    return use_in ? ms : mc;
}

// The largest present value (0..254, the absent value 255 excluded) at or
// below x, or -1.
__device__ __forceinline__ int32_t pres_max_le(const uint64_t *pres, int64_t x)
{
    if (x < 0) return -1;
    if (x > 254) x = 254;
    const int kx = static_cast<int>(x >> 6);
    for (int k = kx; k >= 0; --k) {
        uint64_t m = pres[k];
        if (k == 3) m &= ~(1ull << 63);
        if (k == kx && (x & 63) != 63) m &= (1ull << ((x & 63) + 1)) - 1;
        if (m) return k * 64 + 63 - __builtin_clzll(m);
    }
    return -1;
}

// Gt / Lt over the label's prefix planes (plane pfx0 + plane_id(v) is the
// OR of the planes of the label's present values <= v, built by
// k_sel_planes): Lt t is the prefix of the largest present value below t,
// one entry; Gt t is NOT (the prefix of the largest present value <= t OR
// the absent-value plane), at most two entries.  The node sets are those
// expr_clause selects value by value.  Returns the entry count (ids in e)
// with neg as in expr_clause: 0 entries without neg is a clause no node
// satisfies, 0 entries with neg one every node does.
__device__ __forceinline__ uint32_t cmp_clause(uint32_t op, int64_t t, const uint64_t *pres, const uint32_t *wb,
                                               uint32_t pfx0, uint32_t (&e)[2], bool &neg)
{
    uint32_t n = 0;
    neg = false;
    if (op == PC_OP_LT) {
        const int32_t u = t <= 0 ? -1 : pres_max_le(pres, t - 1);
        if (u >= 0) e[n++] = pfx0 + plane_id(pres, wb, static_cast<uint32_t>(u));
        return n;
    }
    const int32_t top = pres_max_le(pres, 254);
    if (top < 0 || t >= top) return 0;  // no present value above t
    neg = true;
    const int32_t u = pres_max_le(pres, t);
    if (u >= 0) e[n++] = pfx0 + plane_id(pres, wb, static_cast<uint32_t>(u));
    if (pres[3] >> 63) e[n++] = plane_id(pres, wb, 255);
    return n;
}

// cmp_clause's entry count and neg, without the plane ids.
__device__ __forceinline__ uint32_t cmp_count(uint32_t op, int64_t t, const uint64_t *pres, bool &neg)
{
    neg = false;
    if (op == PC_OP_LT) return (t > 0 && pres_max_le(pres, t - 1) >= 0) ? 1u : 0u;
    const int32_t top = pres_max_le(pres, 254);
    if (top < 0 || t >= top) return 0;
    neg = true;
    return (pres_max_le(pres, t) >= 0 ? 1u : 0u) + static_cast<uint32_t>(pres[3] >> 63);
}

// The program entries of one affinity expression (label present table
// pres / plane bases wb): Gt / Lt through the prefix planes, the rest value
// by value.  emit(entry) receives each entry, the clause's last with kLast
// and, when the clause is negated, kNeg.  Returns the count and the
// clause's emptiness as expr_clause does (count 0 without neg: no node).
template <class Emit>
__device__ __forceinline__ uint32_t aff_entries(const pc_pred &q, const uint64_t *pres, const uint32_t *wb,
                                                uint32_t pfx0, bool &neg, const Emit &emit)
{
    if (q.op == PC_OP_GT || q.op == PC_OP_LT) {
        uint32_t e[2];
        const uint32_t n = cmp_clause(q.op, static_cast<int64_t>(q.vals[0]), pres, wb, pfx0, e, neg);
        for (uint32_t i = 0; i < n; ++i) emit(e[i] | (i + 1 == n ? kLast | (neg ? kNeg : 0u) : 0u));
        return n;
    }
    uint64_t sel[4];
    uint32_t cnt = expr_clause(q.op, q.vals, pres, sel, neg);
    const uint32_t n = cnt;
    for (int k = 0; k < 4; ++k) {
        uint64_t m = sel[k];
        while (m) {
            const uint32_t v = static_cast<uint32_t>(k * 64 + __builtin_ctzll(m));
            m &= m - 1;
            uint32_t ent = plane_id(pres, wb, v);
            if (--cnt == 0) ent |= kLast | (neg ? kNeg : 0u);
            emit(ent);
        }
    }
    return n;
}

__device__ __forceinline__ uint32_t pred_clause(const pc_pred &q, const uint64_t *pres, uint64_t sel[4], bool &neg)
{
    return expr_clause(q.op, q.vals, pres, sel, neg);
}

// Well-formed affinity expression: label < L, op <= 5, reserved fields 0,
// no value 255 in an In / NotIn set, vals[1..3] = 0 for Gt / Lt.
__device__ __forceinline__ bool aff_valid(const pc_pred &q, int32_t L)
{
    if (static_cast<int32_t>(q.label) >= L || q.op > PC_OP_LT || q.rsv0 != 0 || q.rsv1 != 0) return false;
    if (q.op <= PC_OP_NOTIN && (q.vals[3] >> 63)) return false;
    if ((q.op == PC_OP_GT || q.op == PC_OP_LT) && (q.vals[1] | q.vals[2] | q.vals[3])) return false;
    return true;
}

// A group of G lanes compiles one row: the lanes' own bits of a ballot, and
// the exclusive sum of x over the group's lower lanes with the group's total.
template <int G>
__device__ __forceinline__ uint32_t group_bits(bool x)
{
    return static_cast<uint32_t>(__ballot(x) >> ((threadIdx.x & 63) & ~(G - 1))) & ((1u << G) - 1);
}

template <int G>
__device__ __forceinline__ uint32_t group_scan(uint32_t x, uint32_t &total)
{
    uint32_t s = x;
#pragma unroll
    for (int off = 1; off < G; off <<= 1) {
        const uint32_t y = __shfl_up(s, off, G);
        if (static_cast<int>(threadIdx.x % G) >= off) s += y;
    }
    total = __shfl(s, G - 1, G);
    return s - x;
}

// The label tables that a row's expressions look up.
struct LabelTables {
    const uint64_t *present;  // [L][4]
    const uint32_t *wbase;    // [L][4]
};

// Up to this many labels the compiles hold them in LDS: a lane looks up each
// expression's presence words and then the base of each entry's plane, a chain of
// gathers from memory otherwise (233,017 rows of 64 labels: affinity 75 -> 61 us,
// preferred 89 -> 77).
constexpr int32_t kLdsLabels = 64;
__device__ __forceinline__ LabelTables stage_labels(const uint64_t *__restrict__ present,
                                                    const uint32_t *__restrict__ wbase, int32_t L, uint64_t *sp,
                                                    uint32_t *sw)
{
    for (int32_t x = threadIdx.x; x < L * 4; x += blockDim.x) {
        sp[x] = present[x];
        sw[x] = wbase[x];
    }
    __syncthreads();
    return {sp, sw};
}

// kSelLanes lanes per row, one predicate each: validate and size the
// predicates, then emit the program -- inline in the row record when it has
// at most 15 entries, else at prog[4 * pred_off[i] ...] (at most 4 entries
// per predicate; longer programs are decoded at evaluation time).  The record
// is built in LDS and written by the group.
// Bound by the chain offsets -> predicate -> presence words of a row, which
// the lanes walk together (a thread per row walked it once per predicate:
// 16,384 rows 22 us, now 7.5; 699,051 rows 113 us, 81 with the groups, now 57 with
// the label tables in LDS).
constexpr int kCompThreads = 256;
constexpr int kSelLanes = 8;
template <bool kLds>
__global__ __launch_bounds__(kCompThreads) void k_sel_compile(const int32_t *__restrict__ pred_off,
                                                              const pc_pred *__restrict__ preds, int64_t n_preds,
                                                              int32_t I, int32_t L,
                                                              const uint64_t *__restrict__ present_all,
                                                              const uint32_t *__restrict__ wbase_all,
                                                              uint32_t *__restrict__ prog, uint32_t *__restrict__ rec,
                                                              uint32_t *__restrict__ d_err)
{
    constexpr int G = kSelLanes;
    __shared__ uint32_t srec[kCompThreads / G][kRecWords + 2];  // each group's row record (padded)
    uint32_t *R = srec[threadIdx.x / G];
    const int gl = threadIdx.x % G;
    uint32_t errs = 0;
    const uint64_t *present = kLds ? nullptr : present_all;
    const uint32_t *wbase = kLds ? nullptr : wbase_all;
    __shared__ uint64_t sp[kLds ? kLdsLabels * 4 : 1];
    __shared__ uint32_t sw[kLds ? kLdsLabels * 4 : 1];
    if constexpr (kLds) {
        const LabelTables tab = stage_labels(present_all, wbase_all, L, sp, sw);
        present = tab.present;
        wbase = tab.wbase;
    }
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * (kCompThreads / G); i0 < I;
         i0 += static_cast<int64_t>(gridDim.x) * (kCompThreads / G)) {
        const int64_t i = i0 + threadIdx.x / G;
        int64_t b = 0, e = 0;
        bool good = false;
        if (i < I) {
            b = pred_off[i];
            e = pred_off[i + 1];
            good = pc_range_ok(b, e, n_preds);
            if (!good) errs |= PC_DERR_OFFSETS;
        }
        if (!good) b = e = 0;
        // the entries of the row's predicates in order; k0: the first one's place
        auto pass = [&](auto &&emit, bool &empty) {
            int64_t k0 = 0;
            empty = false;
            for (int64_t p0 = b; __ballot(p0 < e) != 0; p0 += G) {
                const int64_t p = p0 + gl;
                uint64_t sel[4] = {0, 0, 0, 0};
                const uint64_t *pres = nullptr;
                const uint32_t *wb = nullptr;
                uint32_t cnt = 0;
                bool neg = true;
                if (p < e) {
                    const pc_pred q = preds[p];
                    if (!pred_valid(q.label, q.op, q.rsv0, q.rsv1, q.vals[3], L)) {
                        errs |= PC_DERR_PRED;
                        neg = false;  // as an empty OR: no node
                    } else {
                        pres = present + static_cast<int64_t>(q.label) * 4;
                        wb = wbase + static_cast<int64_t>(q.label) * 4;
                        cnt = pred_clause(q, pres, sel, neg);
                    }
                }
                empty |= group_bits<G>(cnt == 0 && !neg) != 0;
                uint32_t total;
                int64_t k = k0 + group_scan<G>(cnt, total);
                k0 += total;
                for (int w = 0; w < 4; ++w) {
                    uint64_t m = sel[w];
                    while (m) {
                        const uint32_t v = static_cast<uint32_t>(w * 64 + __builtin_ctzll(m));
                        m &= m - 1;
                        emit(k++, plane_id(pres, wb, v) | (--cnt == 0 ? kLast | (neg ? kNeg : 0u) : 0u));
                    }
                }
            }
            return k0;
        };
        bool empty;
        const int64_t n = pass([&](int64_t k, uint32_t ent) {
            if (k < kInline) R[1 + k] = ent;
        }, empty);
        const bool fits = n <= 4 * (e - b);
        const bool indirect = good && !empty && n > kInline && fits;
        if (gl == 0) {
            // (the evaluator reads entries 1..n of an inline program only)
            if (!good || empty) R[0] = static_cast<uint32_t>(kRowFalse);
            else if (n <= kInline) R[0] = static_cast<uint32_t>(n);
            else if (!fits) R[0] = static_cast<uint32_t>(kRowLong);
            else {
                R[0] = static_cast<uint32_t>(kRowIndirect);
                R[1] = static_cast<uint32_t>(b);
                R[2] = static_cast<uint32_t>(n);
            }
        }
        if (__ballot(indirect)) {  // (rows of the wavefront that are not take part with no predicates)
            uint32_t *out = prog + 4 * b;
            const int64_t e_all = e;
            if (!indirect) e = b;
            pass([&](int64_t k, uint32_t ent) { out[k] = ent; }, empty);
            e = e_all;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (i < I) reinterpret_cast<uint2 *>(rec + i * kRecWords)[gl] = make_uint2(R[2 * gl], R[2 * gl + 1]);
        __builtin_amdgcn_wave_barrier();
    }
    if (errs) atomicOr(d_err, errs);
}

// Is every expression of [b, e) well-formed?  Bound by the latency of scattered
// 40-byte expressions, so four are requested together (233,017 affinity rows 31
// -> 16 us, 3.4 TB/s with the offsets; as many preferred ones 21 -> 15).
constexpr int kSweep = 4;
__device__ __forceinline__ bool exprs_valid(const pc_pred *__restrict__ preds, int64_t b, int64_t e, int32_t L)
{
    bool ok = true;
    for (int64_t p = b; p < e && ok; p += kSweep) {
        pc_pred q[kSweep];
#pragma unroll
        for (int k = 0; k < kSweep; ++k) q[k] = preds[min(p + k, e - 1)];
#pragma unroll
        for (int k = 0; k < kSweep; ++k) ok &= aff_valid(q[k], L);
    }
    return ok;
}

// Affinity input sweep: the data-error flags are properties of the whole
// input.  OFFSETS for any bad term or row offset pair, PRED for any
// malformed expression inside a term with a valid offset pair.
__global__ __launch_bounds__(256) void k_aff_validate(const int32_t *__restrict__ row_off, int32_t I,
                                                      const int32_t *__restrict__ term_off, int32_t n_terms,
                                                      const pc_pred *__restrict__ preds, int64_t n_preds, int32_t L,
                                                      uint32_t *__restrict__ d_err, Clears clears)
{
    clears.run();
    uint32_t errs = 0;
    const int64_t tot = I > n_terms ? I : n_terms;
    for (int64_t x = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; x < tot;
         x += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (x < n_terms) {
            const int64_t b = term_off[x], e = term_off[x + 1];
            if (!pc_range_ok(b, e, n_preds)) {
                errs |= PC_DERR_OFFSETS;
            } else {
                if (!exprs_valid(preds, b, e, L)) errs |= PC_DERR_PRED;
            }
        }
        if (x < I && !pc_range_ok(row_off[x], row_off[x + 1], n_terms)) errs |= PC_DERR_OFFSETS;
    }
    if (errs) atomicOr(d_err, errs);
}

// Inventory flags of one well-formed expression: its label carries no
// value on any node, or an In / NotIn value no node carries.
__device__ __forceinline__ uint32_t aff_unknown(const pc_pred &q, const uint64_t *pres)
{
    uint32_t u = 0;
    if ((pres[0] | pres[1] | pres[2] | (pres[3] & ~(1ull << 63))) == 0) u |= PC_UNKNOWN_KEY;
    if (q.op <= PC_OP_NOTIN &&
        ((q.vals[0] & ~pres[0]) | (q.vals[1] & ~pres[1]) | (q.vals[2] & ~pres[2]) | (q.vals[3] & ~pres[3])))
        u |= PC_UNKNOWN_VALUE;
    return u;
}

// Whether term [b, e) can hold for some node at all (valid offsets, at
// least one expression, every expression well-formed, no clause that is an
// empty OR), and its program length (Gt / Lt in the prefix form).
__device__ __forceinline__ bool aff_term(const pc_pred *__restrict__ preds, int64_t b, int64_t e, int64_t n_preds,
                                         int32_t L, const uint64_t *__restrict__ present, int64_t &len)
{
    len = 0;
    if (!pc_range_ok(b, e, n_preds) || b == e) return false;
    bool ok = true;
    for (int64_t p = b; p < e; ++p) {
        const pc_pred q = preds[p];
        if (!aff_valid(q, L)) return false;
        const uint64_t *pres = present + static_cast<int64_t>(q.label) * 4;
        bool neg;
        uint32_t cnt;
        if (q.op == PC_OP_GT || q.op == PC_OP_LT) {
            cnt = cmp_count(q.op, static_cast<int64_t>(q.vals[0]), pres, neg);
        } else {
            uint64_t sel[4];
            cnt = expr_clause(q.op, q.vals, pres, sel, neg);
        }
        if (cnt == 0 && !neg) ok = false;
        len += cnt;
    }
    return ok;
}

// Entries that a lane which compiles a row holds in LDS: programs past the inline
// words are copied from there, and only still longer ones, one row in hundreds
// of the generated ones, are formed again, which the whole wavefront waits for
// (233,017 affinity rows 55 -> 42 us).
constexpr int kHeldWords = 32;

// A row's expressions on one lane, each requested while the one before is looked at
// (adjacent terms' too) with kAhead (233,017 affinity rows 61 -> 55 us; not for a
// group's odd row, where the registers cost a wavefront per SIMD).
template <bool kAhead>
struct NextExpr {
    pc_pred q;
    int64_t at = -1;
    __device__ __forceinline__ pc_pred take(const pc_pred *__restrict__ preds, int64_t p, int64_t n_preds)
    {
        if constexpr (!kAhead) return preds[p];
        if (at != p) q = preds[p];
        const pc_pred now = q;
        at = p + 1;
        q = preds[min(at, n_preds - 1)];
        return now;
    }
};

// One affinity row, on one lane (rows that k_aff_compile's groups do not
// take): the record in rr, the inventory flags in unknown[i].
template <bool kAhead, int kHeld>
__device__ __forceinline__ void aff_compile_row(const int32_t *__restrict__ row_off, int32_t i, const int32_t *__restrict__ term_off,
                                int32_t n_terms, const pc_pred *__restrict__ preds, int64_t n_preds, int32_t L,
                                const uint64_t *__restrict__ present, const uint32_t *__restrict__ wbase,
                                uint32_t *__restrict__ prog, int64_t prog_cap,
                                unsigned long long *__restrict__ prog_used, uint32_t *rr,
                                uint8_t *__restrict__ unknown, uint32_t pfx0)
{
    const int64_t tb = row_off[i], te = row_off[i + 1];
    if (!pc_range_ok(tb, te, n_terms)) {
        rr[0] = static_cast<uint32_t>(kRowFalse);
        unknown[i] = 0;
        return;
    }
    // One pass over the row's expressions: the inventory flags (every
    // well-formed expression of every term with valid offsets), and
    // each term's entries emitted into the record's inline area as
    // they come (counted past its end) and taken back when the term
    // turns out to hold nowhere (a malformed expression, an empty
    // clause).  A live term with no entries holds everywhere, and so
    // does the row.
    uint32_t unk = 0;
    bool all = tb == te;
    int64_t n = 0, live = 0, k_out = 0;
    uint32_t *in_out = rr + 1;
    NextExpr<kAhead> ahead;
    for (int64_t t = tb; t < te; ++t) {
        const int64_t b = term_off[t], e = term_off[t + 1];
        if (!pc_range_ok(b, e, n_preds)) continue;
        bool ok = b != e;
        const int64_t start = k_out;
        int64_t len = 0;
        for (int64_t p = b; p < e; ++p) {
            const pc_pred q = ahead.take(preds, p, n_preds);
            if (!aff_valid(q, L)) {
                ok = false;
                continue;
            }
            const uint64_t *pres = present + static_cast<int64_t>(q.label) * 4;
            unk |= aff_unknown(q, pres);
            if (!ok || all) continue;
            bool neg;
            const uint32_t cnt = aff_entries(q, pres, wbase + static_cast<int64_t>(q.label) * 4, pfx0, neg,
                                             [&](uint32_t ent) {
                                                 if (k_out < kHeld) in_out[k_out] = ent;
                                                 ++k_out;
                                             });
            if (cnt == 0 && !neg) ok = false;
            len += cnt;
        }
        if (all) continue;
        if (!ok) {
            k_out = start;
            continue;
        }
        if (len == 0) {
            all = true;
            continue;
        }
        if (k_out <= kHeld) in_out[k_out - 1] |= kTermEnd;
        n += len;
        ++live;
    }
    unknown[i] = static_cast<uint8_t>(unk);
    if (all) {
        rr[0] = 0;
        return;
    }
    if (live == 0) {
        rr[0] = static_cast<uint32_t>(kRowFalse);
        return;
    }
    if (n <= kInline) {
        rr[0] = static_cast<uint32_t>(n);
        return;
    }
    // longer than the inline area: a slice of prog, copied from the entries
    // held or written by a second pass (slices are whole multiples of 4
    // entries: the record stores off / 4)
    const unsigned long long off = atomicAdd(prog_used, static_cast<unsigned long long>((n + 3) & ~int64_t(3)));
    if (static_cast<int64_t>(off) + n > prog_cap) {
        rr[0] = static_cast<uint32_t>(kRowLong);
        return;
    }
    uint32_t *out = prog + off;
    if (n <= kHeld)
        for (int32_t k = 0; k < static_cast<int32_t>(n); ++k) out[k] = in_out[k];
    rr[0] = static_cast<uint32_t>(kRowIndirect);
    rr[1] = static_cast<uint32_t>(off / 4);
    rr[2] = static_cast<uint32_t>(n);
    if (n <= kHeld) return;
    int64_t k2 = 0;
    for (int64_t t = tb; t < te; ++t) {
        const int64_t b = term_off[t], e = term_off[t + 1];
        int64_t len;
        if (!aff_term(preds, b, e, n_preds, L, present, len)) continue;
        for (int64_t p = b; p < e; ++p) {
            const pc_pred q = preds[p];
            bool neg;
            aff_entries(q, present + static_cast<int64_t>(q.label) * 4, wbase + static_cast<int64_t>(q.label) * 4,
                        pfx0, neg, [&](uint32_t ent) { out[k2++] = ent; });
        }
        out[k2 - 1] |= kTermEnd;
    }
}

// The expressions of a row whose terms a group of G lanes can take at once:
// at most G terms, all of valid offsets (which makes them adjacent), and at
// most G expressions.  Term t is lane t's: expressions [b, e).
struct GroupTerms {
    bool fits;       // (group-uniform)
    int32_t nt;      // terms
    int64_t first;   // the row's first expression
    int32_t n;       // expressions
    int32_t b, e;    // lane t: term t's expressions, from `first`
    uint32_t mask;   // lane t: them as lanes
};

template <int G>
__device__ __forceinline__ GroupTerms group_terms(int64_t tb, int64_t te, const int32_t *__restrict__ term_off,
                                                  int64_t n_preds, bool live)
{
    const int gl = threadIdx.x % G;
    GroupTerms g{false, 0, 0, 0, 0, 0, 0};
    const bool few = live && te - tb <= G;
    int64_t b = 0, e = 0;
    bool ok = true;
    if (few && tb + gl < te) {
        b = term_off[tb + gl];
        e = term_off[tb + gl + 1];
        ok = pc_range_ok(b, e, n_preds);
    }
    const bool all_ok = group_bits<G>(!ok) == 0;
    g.nt = few ? static_cast<int32_t>(te - tb) : 0;
    g.first = __shfl(b, 0, G);
    const int64_t end = __shfl(e, max(g.nt - 1, 0), G);
    g.fits = few && all_ok && end - g.first <= G;
    if (g.fits) {
        g.n = static_cast<int32_t>(end - g.first);
        if (gl < g.nt) {
            g.b = static_cast<int32_t>(b - g.first);
            g.e = static_cast<int32_t>(e - g.first);
            g.mask = ((1u << g.e) - 1) & ~((1u << g.b) - 1);
        }
    }
    return g;
}

// Lane j's term among the group's (the last one that begins at or before
// its expression; a term without expressions never is).
template <int G>
__device__ __forceinline__ int group_term_of(const GroupTerms &g)
{
    const int gl = threadIdx.x % G;
    int mine = 0;
    for (int t = 1; t < G; ++t) {
        if (!__ballot(t < g.nt)) break;
        const int32_t bt = __shfl(g.b, t, G);
        if (t < g.nt && bt <= gl) mine = t;
    }
    return mine;
}

// A group of kAffLanes lanes per affinity row, one expression each:
// inventory flags, then the program.  Terms that hold nowhere are dropped; a
// term with an empty program holds everywhere, and so does a row without
// terms (header 0); a row with no term left admits no node.  The last entry
// of each term carries kTermEnd.  Programs of at most 15 entries sit inline in
// the row record; longer ones take a slice of prog through a bump counter
// and, when it is exhausted, are decoded at evaluation time (kRowLong).  Rows
// that group_terms does not take are compiled by one lane.
// Bound by the chain offsets -> expression -> presence words, which a thread
// per row walked once per expression (3,001 rows 67 us, now 9); of many rows a
// thread each (G = 1) has the better throughput: bound there by the chains of its
// three or four wavefronts per SIMD (233,017 rows 75 us before the look-ahead, the tables in LDS
// and the held entries, now 42; expressions staged in LDS lost, 85).
constexpr int kAffLanes = 16;
// rows below which the groups win (a thread per row / groups, at 64 labels:
// affinity 45,000 rows 28 / 22 us, 60,000 rows 28 / 27, 100,000 rows 31 / 40;
// preferred 24,000 rows 26 / 22 us, 30,000 rows 26 / 24, 36,000 rows 26 / 28)
constexpr int32_t kAffGroupRows = 65536, kPrefGroupRows = 32768;
template <int G, bool kLds>
__global__ __launch_bounds__(256) void k_aff_compile(const int32_t *__restrict__ row_off, int32_t I,
                                                     const int32_t *__restrict__ term_off, int32_t n_terms,
                                                     const pc_pred *__restrict__ preds, int64_t n_preds, int32_t L,
                                                     const uint64_t *__restrict__ present_all,
                                                     const uint32_t *__restrict__ wbase_all,
                                                     uint32_t *__restrict__ prog, int64_t prog_cap,
                                                     unsigned long long *__restrict__ prog_used,
                                                     uint32_t *__restrict__ rec, uint8_t *__restrict__ unknown,
                                                     uint32_t pfx0)
{
    const uint64_t *present = kLds ? nullptr : present_all;
    const uint32_t *wbase = kLds ? nullptr : wbase_all;
    __shared__ uint32_t srec[256 / G][G == 1 ? kHeldWords + 1 : kRecWords + 1];
    uint32_t *rr = srec[threadIdx.x / G];
    __shared__ uint64_t sp[kLds ? kLdsLabels * 4 : 1];
    __shared__ uint32_t sw[kLds ? kLdsLabels * 4 : 1];
    if constexpr (kLds) {
        const LabelTables tab = stage_labels(present_all, wbase_all, L, sp, sw);
        present = tab.present;
        wbase = tab.wbase;
    }
    if constexpr (G == 1) {
        for (int32_t i = blockIdx.x * 256 + threadIdx.x; i < I; i += gridDim.x * 256) {
            aff_compile_row<true, kHeldWords>(row_off, i, term_off, n_terms, preds, n_preds, L, present, wbase, prog, prog_cap,
                            prog_used, rr, unknown, pfx0);
            uint4 *dst = reinterpret_cast<uint4 *>(rec + static_cast<int64_t>(i) * kRecWords);
#pragma unroll
            for (int k = 0; k < kRecWords / 4; ++k)
                dst[k] = make_uint4(rr[4 * k], rr[4 * k + 1], rr[4 * k + 2], rr[4 * k + 3]);
        }
        return;
    } else {
    const int gl = threadIdx.x % G;
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * (256 / G); i0 < I;
         i0 += static_cast<int64_t>(gridDim.x) * (256 / G)) {
        const int64_t i = i0 + threadIdx.x / G;
        int64_t tb = 0, te = 0;
        bool good = false;
        if (i < I) {
            tb = row_off[i];
            te = row_off[i + 1];
            good = pc_range_ok(tb, te, n_terms);
            if (!good && gl == 0) {
                rr[0] = static_cast<uint32_t>(kRowFalse);
                unknown[i] = 0;
            }
        }
        const GroupTerms g = group_terms<G>(tb, te, term_off, n_preds, good);
        if (good && !g.fits && gl == 0)
            aff_compile_row<false, kInline>(row_off, static_cast<int32_t>(i), term_off, n_terms, preds, n_preds, L, present, wbase,
                            prog, prog_cap, prog_used, rr, unknown, pfx0);
        // this lane's expression
        pc_pred q{};
        const uint64_t *pres = nullptr;
        const uint32_t *wb = nullptr;
        uint32_t cnt = 0, unk = 0;
        bool neg = true, valid = false;
        const bool mine = g.fits && gl < g.n;
        if (mine) {
            q = preds[g.first + gl];
            valid = aff_valid(q, L);
            if (valid) {
                pres = present + static_cast<int64_t>(q.label) * 4;
                wb = wbase + static_cast<int64_t>(q.label) * 4;
                unk = aff_unknown(q, pres);
                if (q.op == PC_OP_GT || q.op == PC_OP_LT) {
                    cnt = cmp_count(q.op, static_cast<int64_t>(q.vals[0]), pres, neg);
                } else {
                    uint64_t sel[4];
                    cnt = expr_clause(q.op, q.vals, pres, sel, neg);
                }
            }
        }
        const uint32_t bad = group_bits<G>(mine && (!valid || (cnt == 0 && !neg)));
        const uint32_t some = group_bits<G>(cnt != 0);
        const uint32_t u0 = group_bits<G>((unk & 1) != 0), u1 = group_bits<G>((unk & 2) != 0);
        // lane t: whether term t can hold, and whether it holds everywhere
        const bool term_ok = g.mask != 0 && !(bad & g.mask);
        const uint32_t live = group_bits<G>(term_ok);
        const bool all = group_bits<G>(term_ok && !(some & g.mask)) != 0 || (g.fits && g.nt == 0);
        const int term = group_term_of<G>(g);
        const bool keep = mine && ((live >> term) & 1u);
        uint32_t n;
        const uint32_t k0 = group_scan<G>(keep ? cnt : 0u, n);
        const bool write = g.fits && !all && live != 0;
        unsigned long long off = 0;
        if (write && n > kInline && gl == 0) off = atomicAdd(prog_used, static_cast<unsigned long long>((n + 3) & ~3u));
        off = __shfl(off, 0, G);
        const bool inl = n <= kInline;
        const bool room = static_cast<int64_t>(off) + n <= prog_cap;
        const uint32_t tmask = __shfl(g.mask, term, G);
        if (write && keep && cnt && (inl || room)) {
            uint32_t *out = inl ? rr + 1 : prog + off;
            uint32_t k = k0;
            // the term's last entry is in its last expression with any
            const bool closes = (some & tmask) >> (gl + 1) == 0;
            const uint32_t end = k0 + cnt - 1;
            aff_entries(q, pres, wb, pfx0, neg, [&](uint32_t ent) {
                out[k] = ent | (closes && k == end ? kTermEnd : 0u);
                ++k;
            });
        }
        if (g.fits && gl == 0) {
            unknown[i] = static_cast<uint8_t>((u0 ? 1u : 0u) | (u1 ? 2u : 0u));
            if (all) rr[0] = 0;
            else if (live == 0) rr[0] = static_cast<uint32_t>(kRowFalse);
            else if (inl) rr[0] = n;
            else if (!room) rr[0] = static_cast<uint32_t>(kRowLong);
            else {
                rr[0] = static_cast<uint32_t>(kRowIndirect);
                rr[1] = static_cast<uint32_t>(off / 4);
                rr[2] = n;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (i < I) rec[i * kRecWords + gl] = rr[gl];
        __builtin_amdgcn_wave_barrier();
    }
    }
}

struct Words {
    uint64_t a, b;
};
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ Words load_words(const uint64_t *p)
{
    const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(p);
    return {v.x, v.y};
}

// Fold one program entry's plane words into the running clause (c) and,
// at the end of a clause, into the row's conjunction (a).
// In affinity programs (kTerms) the end of a term ORs the term's
// conjunction into the row (r) and starts the next term.
template <bool kTerms>
__device__ __forceinline__ void fold(uint32_t ent, const Words &v, Words &c, Words &a, Words &r)
{
    c.a |= v.a;
    c.b |= v.b;
    if (ent & kLast) {
        if (ent & kNeg) {
            a.a &= ~c.a;
            a.b &= ~c.b;
        } else {
            a.a &= c.a;
            a.b &= c.b;
        }
        c.a = c.b = 0;
    }
    if constexpr (kTerms) {
        if (ent & kTermEnd) {
            r.a |= a.a;
            r.b |= a.b;
            a.a = a.b = ~0ull;
        }
    }
}

// This lane's two words of plane `pid`.  The buffer form (planes within
// 4 GiB) takes the plane offset as a scalar operand: one scalar multiply
// per load and no vector address arithmetic.
template <bool kBuf>
struct Planes {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t lane_off;  // bytes: this lane's first word within a plane row (set per row)
    uint32_t rowbytes;  // bytes per plane row
    const uint64_t *pcol;
    int64_t Wp;

    __device__ __forceinline__ Words operator()(uint32_t pid) const
    {
        if constexpr (kBuf) {
            const u32x4 v = __builtin_bit_cast(
                u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off, pid * rowbytes, 0));
            return {static_cast<uint64_t>(v.x) | static_cast<uint64_t>(v.y) << 32,
                    static_cast<uint64_t>(v.z) | static_cast<uint64_t>(v.w) << 32};
        } else {
            return load_words(pcol + static_cast<int64_t>(pid) * Wp);
        }
    }
};

// Rows whose program did not fit its slot: decode the predicates on the
// scalar unit.
template <bool kBuf>
__device__ Words eval_row_decoded(const pc_pred *__restrict__ preds, int64_t b, int64_t e,
                                  const uint64_t *__restrict__ present, const uint32_t *__restrict__ wbase,
                                  const Planes<kBuf> &pl)
{
    Words a{~0ull, ~0ull};
    for (int64_t p = b; p < e; ++p) {
        const pc_pred *q = preds + p;
        const uint32_t label = q->label, op = q->op;
        const uint64_t *pres = present + static_cast<int64_t>(label) * 4;
        const uint32_t *wb = wbase + static_cast<int64_t>(label) * 4;
        if (op == PC_OP_EXISTS) {
            if (pres[3] >> 63) {
                const Words v = pl(plane_id(pres, wb, 255));
                a.a &= ~v.a;
                a.b &= ~v.b;
            }
            continue;
        }
        Words c{0, 0};
        for (int k = 0; k < 4; ++k) {
            uint64_t m = q->vals[k] & pres[k];
            while (m) {
                const uint32_t v = static_cast<uint32_t>(k * 64 + __builtin_ctzll(m));
                m &= m - 1;
                const Words x = pl(plane_id(pres, wb, v));
                c.a |= x.a;
                c.b |= x.b;
            }
        }
        if (op == PC_OP_IN) {
            a.a &= c.a;
            a.b &= c.b;
        } else {
            a.a &= ~c.a;
            a.b &= ~c.b;
        }
    }
    return a;
}

// Affinity rows whose program found no slice: the terms decoded on the
// scalar unit (the same term rules as k_aff_compile).
template <bool kBuf>
__device__ Words eval_row_decoded_aff(const pc_pred *__restrict__ preds, int64_t n_preds,
                                      const int32_t *__restrict__ term_off, int64_t tb, int64_t te, int32_t L,
                                      const uint64_t *__restrict__ present, const uint32_t *__restrict__ wbase,
                                      const Planes<kBuf> &pl)
{
    Words r{0, 0};
    for (int64_t t = tb; t < te; ++t) {
        int64_t len;
        const int64_t b = term_off[t], e = term_off[t + 1];
        if (!aff_term(preds, b, e, n_preds, L, present, len)) continue;
        Words a{~0ull, ~0ull};
        for (int64_t p = b; p < e; ++p) {
            const pc_pred q = preds[p];
            const uint64_t *pres = present + static_cast<int64_t>(q.label) * 4;
            const uint32_t *wb = wbase + static_cast<int64_t>(q.label) * 4;
            uint64_t sel[4];
            bool neg;
            expr_clause(q.op, q.vals, pres, sel, neg);
            Words c{0, 0};
            for (int k = 0; k < 4; ++k) {
                uint64_t m = sel[k];
                while (m) {
                    const uint32_t v = static_cast<uint32_t>(k * 64 + __builtin_ctzll(m));
                    m &= m - 1;
                    const Words x = pl(plane_id(pres, wb, v));
                    c.a |= x.a;
                    c.b |= x.b;
                }
            }
            a.a &= neg ? ~c.a : c.a;
            a.b &= neg ? ~c.b : c.b;
        }
        r.a |= a.a;
        r.b |= a.b;
    }
    return r;
}

// Work item (tile, chunk): the wavefronts of a workgroup take turns on
// batches of brows (at most 64) consecutive rows of the chunk; lane l covers words
// tile * 128 + 2l and + 1.  A row's record is read with scalar loads (the
// next row's is requested while the current row's planes load), so the
// plane loads of a row are all in flight together.  Each lane leaves its
// popcount of row i as byte (i, lane) of an LDS table; at the end of a
// batch lane i sums row i's 64 bytes with dot4 and stores
// part[tile * I + r].  Lanes past the last word load in-bounds words and
// mask them.
// kTerms: affinity rows (pred_off holds the row -> term offsets, term_off
// the term -> expression offsets) whose programs OR their terms.  kStore
// false: popcounts only, no bitset written (verdict-only runs).
template <bool kBuf, bool kTerms, bool kStore = true>
__global__ __launch_bounds__(kEvalThreads) void k_sel_eval(
    const uint32_t *__restrict__ rec, const uint32_t *__restrict__ prog, const int32_t *__restrict__ pred_off,
    const pc_pred *__restrict__ preds, const uint64_t *__restrict__ present, const uint32_t *__restrict__ wbase,
    const uint64_t *__restrict__ planes, int64_t plane_bytes, int64_t Wp, int32_t I, int32_t W, int32_t N,
    uint64_t *__restrict__ feasible, uint32_t *__restrict__ part, int32_t ntiles, int32_t nchunks, int32_t rpc,
    int32_t brows, const int32_t *__restrict__ term_off, int64_t n_preds, int32_t L, int32_t shift)
{
    constexpr int kCntStride = 68;  // bytes per row of the count table (17 dwords: conflict-free column reads)
    __shared__ uint32_t cnt_lds[kEvalThreads / 64][64 * kCntStride / 4];
    const int64_t total = static_cast<int64_t>(ntiles) * nchunks;
    const int64_t item = pc_xcd_item(total);
    if (item >= total) return;
    const int32_t tile = static_cast<int32_t>(item / nchunks);
    const int32_t chunk = static_cast<int32_t>(item % nchunks);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t wt = tile * kTileW + lane * kWpl;  // this lane's first word of an unshifted row
    const uint64_t last = (N & 63) ? (1ull << (N & 63)) - 1 : ~0ull;
    // word index of the bitset's start within its 128-byte line
    const uint32_t base16 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(feasible) >> 3) & 15u;
    Planes<kBuf> pl;
    if constexpr (kBuf)
        pl.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(planes), static_cast<short>(0),
                                                    static_cast<int>(plane_bytes), 0x00020000);
    pl.rowbytes = static_cast<uint32_t>(Wp * 8);
    pl.Wp = Wp;
    // Per-row geometry.  With shift on, the tiles of row r start s(r) words
    // early, where s(r) is the row start's word offset within its 128-byte
    // line: every store then covers whole lines except at the row's two
    // ends, instead of splitting a line between two tiles at every tile
    // edge.  Lanes outside [0, W) load pad words of the plane rows and are
    // masked.
    int32_t w0 = 0;
    bool ok0 = false, ok1 = false, pair = false;
    uint64_t m0 = 0, m1 = 0;
    auto geom = [&](int32_t r) {
        const uint32_t rw = (static_cast<uint32_t>(r) & 15u) * (static_cast<uint32_t>(W) & 15u);  // r * W mod 16
        const int32_t sh = shift ? static_cast<int32_t>((base16 + rw) & 15u) : 0;
        w0 = wt - sh;
        ok0 = w0 >= 0 && w0 < W;
        ok1 = w0 + 1 >= 0 && w0 + 1 < W;
        m0 = ok0 ? (w0 == W - 1 ? last : ~0ull) : 0ull;
        m1 = ok1 ? (w0 + 1 == W - 1 ? last : ~0ull) : 0ull;
        pair = ok0 && ok1 && ((base16 + rw + static_cast<uint32_t>(w0)) & 1u) == 0;  // 16-byte aligned pair
        pl.lane_off = static_cast<uint32_t>(kPad + w0) * 8u;
        pl.pcol = planes + kPad + w0;
    };
    uint8_t *cb = reinterpret_cast<uint8_t *>(cnt_lds[wave]);
    uint32_t *prt = part + static_cast<int64_t>(tile) * I;
    const int32_t r0 = chunk * rpc;
    const int32_t r1 = min(I, r0 + rpc);
    // One row: its record R (uniform, in SGPRs) -> bitset store and count
    // byte.  kIn: an interior tile of a line-shifted row (every lane's two
    // words lie in [0, W - 1), so no masks, and every pair is 16-byte
    // aligned); its geometry is one subtraction per lane.
    const uint32_t lane_base = static_cast<uint32_t>(kPad + wt) * 8u;
    auto row_shift = [&](int32_t r) {
        const uint32_t rw = (static_cast<uint32_t>(r) & 15u) * (static_cast<uint32_t>(W) & 15u);  // r * W mod 16
        return shift ? static_cast<int32_t>((base16 + rw) & 15u) : 0;
    };
    auto row = [&](auto in_tag, int32_t r, int32_t i, const uint32_t (&R)[kRecWords]) {
        constexpr bool kIn = decltype(in_tag)::value;
        const int32_t hdr = static_cast<int32_t>(R[0]);
        if constexpr (kIn) {
            const int32_t sh = row_shift(r);
            w0 = wt - sh;
            pl.lane_off = lane_base - static_cast<uint32_t>(sh) * 8u;
            if constexpr (!kBuf) pl.pcol = planes + kPad + w0;
        } else {
            geom(r);
        }
        Words a{~0ull, ~0ull};
        Words rt{0, 0};  // affinity: OR of the finished terms
        if (hdr == kRowFalse) {
            a = Words{0, 0};
        } else if (hdr > 0) {
            // inline program of hdr entries: the length is uniform, so the
            // guards are scalar branches and only real entries are loaded
            Words c{0, 0};
            {
                Words V[kGroup];
#pragma unroll
                for (int k = 0; k < kGroup; ++k)
                    if (k < hdr) V[k] = pl(R[1 + k] & kPidMask);
#pragma unroll
                for (int k = 0; k < kGroup; ++k)
                    if (k < hdr) fold<kTerms>(R[1 + k], V[k], c, a, rt);
            }
            if (hdr > kGroup) {
                Words V[kInline - kGroup];
#pragma unroll
                for (int k = 0; k < kInline - kGroup; ++k)
                    if (kGroup + k < hdr) V[k] = pl(R[1 + kGroup + k] & kPidMask);
#pragma unroll
                for (int k = 0; k < kInline - kGroup; ++k)
                    if (kGroup + k < hdr) fold<kTerms>(R[1 + kGroup + k], V[k], c, a, rt);
            }
        } else if (hdr == kRowIndirect) {
            const uint32_t *pr = prog + 4 * static_cast<int64_t>(R[1]);
            const int32_t len = static_cast<int32_t>(R[2]);
            Words c{0, 0};
            for (int32_t e0 = 0; e0 < len; e0 += kGroup) {
                uint32_t E[kGroup];
                Words V[kGroup];
#pragma unroll
                for (int k = 0; k < kGroup; ++k) E[k] = (e0 + k < len) ? pr[e0 + k] : 0u;
#pragma unroll
                for (int k = 0; k < kGroup; ++k)
                    if (e0 + k < len) V[k] = pl(E[k] & kPidMask);
#pragma unroll
                for (int k = 0; k < kGroup; ++k)
                    if (e0 + k < len) fold<kTerms>(E[k], V[k], c, a, rt);
            }
        } else if (hdr == kRowLong) {
            if constexpr (kTerms)
                rt = eval_row_decoded_aff<kBuf>(preds, n_preds, term_off, pred_off[r], pred_off[r + 1], L, present,
                                                wbase, pl);
            else
                a = eval_row_decoded<kBuf>(preds, pred_off[r], pred_off[r + 1], present, wbase, pl);
        }
        if constexpr (kTerms) {
            if (hdr > 0 || hdr == kRowIndirect || hdr == kRowLong) a = rt;
        }
        if constexpr (!kIn) {
            a.a &= m0;
            a.b &= m1;
        }
        if constexpr (kStore) {
            const int64_t at = static_cast<int64_t>(r) * W + w0;
            if (kIn || pair) {
                __builtin_nontemporal_store(u64x2{a.a, a.b}, reinterpret_cast<u64x2 *>(feasible + at));
            } else {
                if (ok0) __builtin_nontemporal_store(a.a, feasible + at);
                if (ok1) __builtin_nontemporal_store(a.b, feasible + at + 1);
            }
        }
        cb[i * kCntStride + lane] = static_cast<uint8_t>(__popcll(a.a) + __popcll(a.b));
    };
    // (affinity programs measured slower with the interior path: it is
    // taken for selector rows only)
    auto row_any = [&](int32_t r, int32_t i, const uint32_t (&R)[kRecWords]) {
        const int32_t lo = tile * kTileW - row_shift(r);
        if (!kTerms && shift && lo >= 0 && lo + kTileW <= W - 1) row(std::true_type{}, r, i, R);
        else row(std::false_type{}, r, i, R);
    };
    auto load_rec = [&](int32_t r, uint32_t (&R)[kRecWords]) {
        const uint32_t *rp = rec + static_cast<int64_t>(r) * kRecWords;
#pragma unroll
        for (int k = 0; k < kRecWords; ++k) R[k] = rp[k];
    };
    for (int32_t bat = r0 + wave * brows; bat < r1; bat += kEvalWaves * brows) {
        const int32_t nb = min(brows, r1 - bat);
        // two record buffers: the next row's record loads while this row's
        // planes load (the last row reloads its own record)
        uint32_t RA[kRecWords], RB[kRecWords];
        load_rec(bat, RA);
        for (int32_t i = 0; i < nb; i += 2) {
            load_rec(bat + min(i + 1, nb - 1), RB);
            row_any(bat + i, i, RA);
            if (i + 1 < nb) {
                load_rec(bat + min(i + 2, nb - 1), RA);
                row_any(bat + i + 1, i + 1, RB);
            }
        }
        // the count table was written by every lane of this wavefront
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (lane < nb) {
            const uint32_t *row = cnt_lds[wave] + lane * (kCntStride / 4);
            uint32_t sum = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) sum = __builtin_amdgcn_udot4(row[k], 0x01010101u, sum, false);
            prt[bat + lane] = sum;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// popcnt[r] = sum over tiles of part[t * I + r].
__global__ __launch_bounds__(256) void k_sel_popsum(const uint32_t *__restrict__ part, int32_t I, int32_t ntiles,
                                                    uint32_t *__restrict__ popcnt)
{
    const int32_t r = blockIdx.x * 256 + threadIdx.x;
    if (r >= I) return;
    uint32_t s = 0;
    for (int32_t t = 0; t < ntiles; ++t) s += part[static_cast<int64_t>(t) * I + r];
    popcnt[r] = s;
}

// ---------------------------------------------------------------- preferred
// Preferred node affinity: per row, weighted terms (weight 1..100, terms as
// in required affinity); a node's score is the sum of the weights of the
// terms that hold for it; the best feasible node has the largest score, the
// lowest index among equal scores.  Scores are kept bit-sliced: bit b of
// every node's score of a 64-node word is one 64-bit word, so adding a
// term's weight to the nodes where it holds is a ripple add over the score
// bits, and the maximum over a word's nodes is found from the top bit down.
constexpr int kScoreBits = 16;         // 655 terms of weight <= 100 stay below 2^16
constexpr int32_t kPrefMaxTerms = 655;
constexpr uint32_t kPrefLenBits = 24;  // term header: weight << 24 | program entries
// row record, 16 words (one 64-byte line): word 0 = kind << 24 | score bits
// << 16 | live terms; word 1 = program offset in prog (kPrefIndirect);
// words 2..15 = the program itself when it has at most 14 words
enum : uint32_t { kPrefInline = 0, kPrefIndirect = 1, kPrefDecode = 2, kPrefNone = 3 };
constexpr int kPrefRec = 16;
constexpr int kPrefInlineWords = kPrefRec - 2;
constexpr uint32_t kPrefClasses = 4;  // row lists: scores within 8 bits, within 16 bits, decoded, <= 3 terms
constexpr uint32_t kPrefFewTerms = 3;  // rows with at most this many live terms: scores from term patterns

__device__ __forceinline__ bool pref_weight_ok(uint32_t w) { return w >= 1 && w <= 100; }

__device__ __forceinline__ bool pref_row_ok(const int32_t *__restrict__ row_off, int64_t i, int32_t n_terms)
{
    const int64_t b = row_off[i], e = row_off[i + 1];
    return pc_range_ok(b, e, n_terms) && e - b <= kPrefMaxTerms;
}

__device__ __forceinline__ uint32_t bit_length(uint32_t x) { return x ? 32u - __builtin_clz(x) : 0u; }

// Input sweep: the data-error flags are properties of the whole input.
// PRED for a weight outside 1..100 or a malformed expression inside a term
// with a valid offset pair; OFFSETS for a bad term or row offset pair or a
// row of more than kPrefMaxTerms terms.
__global__ __launch_bounds__(256) void k_pref_validate(const int32_t *__restrict__ row_off, int32_t I,
                                                       const int32_t *__restrict__ term_off, int32_t n_terms,
                                                       const uint32_t *__restrict__ weight,
                                                       const pc_pred *__restrict__ preds, int64_t n_preds, int32_t L,
                                                       uint32_t *__restrict__ d_err, Clears clears)
{
    clears.run();
    uint32_t errs = 0;
    const int64_t tot = I > n_terms ? I : n_terms;
    for (int64_t x = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; x < tot;
         x += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        if (x < n_terms) {
            if (!pref_weight_ok(weight[x])) errs |= PC_DERR_PRED;
            const int64_t b = term_off[x], e = term_off[x + 1];
            if (!pc_range_ok(b, e, n_preds)) {
                errs |= PC_DERR_OFFSETS;
            } else {
                if (!exprs_valid(preds, b, e, L)) errs |= PC_DERR_PRED;
            }
        }
        if (x < I && !pref_row_ok(row_off, x, n_terms)) errs |= PC_DERR_OFFSETS;
    }
    if (errs) atomicOr(d_err, errs);
}

// One row of k_pref_compile: its record, and its class (3: at most three
// live terms, including none; 0: scores fit 8 bits, 1: 16 bits; 2: decoded
// on the fly).
template <bool kAhead, int kHeld>
__device__ __forceinline__ uint32_t pref_compile_row(const int32_t *__restrict__ row_off, int32_t i,
                                     const int32_t *__restrict__ term_off, int32_t n_terms,
                                     const uint32_t *__restrict__ weight, const pc_pred *__restrict__ preds,
                                     int64_t n_preds, int32_t L, const uint64_t *__restrict__ present,
                                     const uint32_t *__restrict__ wbase, uint32_t *__restrict__ prog, int64_t prog_cap,
                                     unsigned long long *__restrict__ prog_used, uint32_t *rr, uint32_t pfx0)
{
    rr[0] = kPrefNone << 24;
    if (!pref_row_ok(row_off, i, n_terms)) return 3;
    int64_t tb = row_off[i];
    const int64_t te = row_off[i + 1];
    // One pass: each live term's header and entries go into the record's
    // inline words as they come (counted past their end); a term that turns
    // out dead (weight out of range, a malformed expression, an empty
    // clause) is taken back.  Programs past the inline words are written
    // again, into a slice of prog.
    int64_t n = 0, k_out = 0;
    uint32_t live = 0, sum = 0;
    bool decode = false;
    uint32_t *in_out = rr + 2;
    NextExpr<kAhead> ahead;
    auto put = [&](uint32_t word) {
        if (k_out < kHeld) in_out[k_out] = word;
        ++k_out;
    };
    for (int64_t t = tb; t < te; ++t) {
        const uint32_t w = weight[t];
        const int64_t b = term_off[t], e = term_off[t + 1];
        if (!pref_weight_ok(w) || !pc_range_ok(b, e, n_preds) || b == e) continue;
        const int64_t start = k_out;
        put(0u);  // the header, set below
        bool ok = true;
        int64_t len = 0;
        for (int64_t p = b; p < e && ok; ++p) {
            const pc_pred q = ahead.take(preds, p, n_preds);
            if (!aff_valid(q, L)) {
                ok = false;
                break;
            }
            bool neg;
            const uint32_t cnt = aff_entries(q, present + static_cast<int64_t>(q.label) * 4,
                                             wbase + static_cast<int64_t>(q.label) * 4, pfx0, neg, put);
            if (cnt == 0 && !neg) ok = false;
            len += cnt;
        }
        if (!ok) {
            k_out = start;
            continue;
        }
        if (len >= (int64_t(1) << kPrefLenBits)) decode = true;
        if (start < kHeld) in_out[start] = w << kPrefLenBits | static_cast<uint32_t>(len);
        n += 1 + len;
        sum += w;
        ++live;
    }
    if (live == 0) return 3;
    const uint32_t head = live | bit_length(sum) << 16;
    uint32_t kind = kPrefInline;
    if (!decode && n > kPrefInlineWords) {
        const unsigned long long off = atomicAdd(prog_used, static_cast<unsigned long long>(n));
        decode = static_cast<int64_t>(off) + n > prog_cap;
        if (!decode) {
            uint32_t *out = prog + off;
            rr[1] = static_cast<uint32_t>(off);
            kind = kPrefIndirect;
            int64_t k2 = 0;
            if (n <= kHeld) {
                for (; k2 < n; ++k2) out[k2] = in_out[k2];
                tb = te;
            }
            for (int64_t t = tb; t < te; ++t) {
                const int64_t b = term_off[t], e = term_off[t + 1];
                int64_t len;
                if (!pref_weight_ok(weight[t]) || !aff_term(preds, b, e, n_preds, L, present, len)) continue;
                out[k2++] = weight[t] << kPrefLenBits | static_cast<uint32_t>(len);
                for (int64_t p = b; p < e; ++p) {
                    const pc_pred q = preds[p];
                    bool neg;
                    aff_entries(q, present + static_cast<int64_t>(q.label) * 4,
                                wbase + static_cast<int64_t>(q.label) * 4, pfx0, neg,
                                [&](uint32_t ent) { out[k2++] = ent; });
                }
            }
        }
    }
    if (decode) {
        rr[0] = head | kPrefDecode << 24;
        return 2;
    }
    rr[0] = head | kind << 24;
    if (live <= kPrefFewTerms) return 3;
    return bit_length(sum) <= 8 ? 0u : 1u;
}

// A group of kAffLanes lanes per row, one expression each (rows that
// group_terms does not take: one lane): the row's live terms (weight in range, and able to
// hold somewhere) as a program of term headers, each followed by its clause
// entries (kLast / kNeg as in selector programs), inline in the row record
// when it has at most 14 words, else in a slice of prog taken through a
// bump counter.  When the slice does not fit, or a term has more than 2^24
// entries, the row is decoded at evaluation time.
// Each row is appended to the list of its class.
// Bound as k_aff_compile (3,001 rows 57 us, now 11).
template <int G, bool kLds>
__global__ __launch_bounds__(256) void k_pref_compile(const int32_t *__restrict__ row_off, int32_t I,
                                                      const int32_t *__restrict__ term_off, int32_t n_terms,
                                                      const uint32_t *__restrict__ weight,
                                                      const pc_pred *__restrict__ preds, int64_t n_preds, int32_t L,
                                                      const uint64_t *__restrict__ present_all,
                                                      const uint32_t *__restrict__ wbase_all, uint32_t *__restrict__ prog,
                                                      int64_t prog_cap, unsigned long long *__restrict__ prog_used,
                                                      uint32_t *__restrict__ rec, int32_t *__restrict__ list,
                                                      uint32_t *__restrict__ list_len, uint32_t pfx0, int32_t rpb)
{
    static_assert(G == 1 || G == kPrefRec, "a lane per record word");
    __shared__ uint32_t srec[256 / G][G == 1 ? kHeldWords + 1 : kPrefRec + 1];
    __shared__ uint8_t scls[256];  // the classes of the workgroup's rows
    uint32_t *rr = srec[threadIdx.x / G];
    const int gl = threadIdx.x % G;
    const int lane = threadIdx.x & 63;
    const int64_t block0 = static_cast<int64_t>(blockIdx.x) * rpb;
    const uint64_t *present = kLds ? nullptr : present_all;
    const uint32_t *wbase = kLds ? nullptr : wbase_all;
    __shared__ uint64_t sp[kLds ? kLdsLabels * 4 : 1];
    __shared__ uint32_t sw[kLds ? kLdsLabels * 4 : 1];
    if constexpr (kLds) {
        const LabelTables tab = stage_labels(present_all, wbase_all, L, sp, sw);
        present = tab.present;
        wbase = tab.wbase;
    }
    if constexpr (G == 1) {
        const int64_t i = block0 + threadIdx.x;
        if (i < I) {
            scls[threadIdx.x] = static_cast<uint8_t>(
                pref_compile_row<true, kHeldWords - 1>(row_off, static_cast<int32_t>(i), term_off, n_terms, weight, preds, n_preds, L,
                                 present, wbase, prog, prog_cap, prog_used, rr, pfx0));
            uint4 *dst = reinterpret_cast<uint4 *>(rec + i * kPrefRec);
#pragma unroll
            for (int k = 0; k < kPrefRec / 4; ++k)
                dst[k] = make_uint4(rr[4 * k], rr[4 * k + 1], rr[4 * k + 2], rr[4 * k + 3]);
        } else {
            scls[threadIdx.x] = kPrefClasses;
        }
    } else
    for (int32_t at = threadIdx.x / G; at < rpb; at += 256 / G) {
        const int64_t i = block0 + at;
        int64_t tb = 0, te = 0;
        bool good = false;
        if (i < I) {
            good = pref_row_ok(row_off, i, n_terms);
            tb = row_off[i];
            te = row_off[i + 1];
        }
        uint32_t cls = i < I ? 3u : kPrefClasses;  // (a bad row has no terms)
        const GroupTerms g = group_terms<G>(tb, te, term_off, n_preds, good);
        if (good && !g.fits && gl == 0)
            cls = pref_compile_row<false, kPrefInlineWords>(row_off, static_cast<int32_t>(i), term_off, n_terms, weight, preds, n_preds, L,
                                   present, wbase, prog, prog_cap, prog_used, rr, pfx0);
        // this lane's expression
        pc_pred q{};
        const uint64_t *pres = nullptr;
        const uint32_t *wb = nullptr;
        uint32_t cnt = 0;
        bool neg = true, valid = false;
        const bool mine = g.fits && gl < g.n;
        if (mine) {
            q = preds[g.first + gl];
            valid = aff_valid(q, L);
            if (valid) {
                pres = present + static_cast<int64_t>(q.label) * 4;
                wb = wbase + static_cast<int64_t>(q.label) * 4;
                if (q.op == PC_OP_GT || q.op == PC_OP_LT) {
                    cnt = cmp_count(q.op, static_cast<int64_t>(q.vals[0]), pres, neg);
                } else {
                    uint64_t sel[4];
                    cnt = expr_clause(q.op, q.vals, pres, sel, neg);
                }
            }
        }
        // this lane's term
        const uint32_t wt = g.fits && gl < g.nt ? weight[tb + gl] : 0u;
        const uint32_t bad = group_bits<G>(mine && (!valid || (cnt == 0 && !neg)));
        const bool term_ok = g.mask != 0 && !(bad & g.mask) && pref_weight_ok(wt);
        const uint32_t live = group_bits<G>(term_ok);
        const int term = group_term_of<G>(g);
        const bool keep = mine && ((live >> term) & 1u);
        uint32_t entries, sum;
        const uint32_t e0 = group_scan<G>(keep ? cnt : 0u, entries);
        group_scan<G>(term_ok ? wt : 0u, sum);
        const uint32_t n = entries + __popc(live);
        const uint32_t n_live = __popc(live);
        // entries ahead of term gl (its first expression's), and in it
        const uint32_t t0 = __shfl(e0, g.b & (G - 1), G);
        const uint32_t after = __shfl(e0 + (keep ? cnt : 0u), (g.e - 1) & (G - 1), G);
        const bool inl = n <= static_cast<uint32_t>(kPrefInlineWords);
        const bool write = g.fits && n_live != 0;
        unsigned long long off = 0;
        if (write && !inl && gl == 0) off = atomicAdd(prog_used, static_cast<unsigned long long>(n));
        off = __shfl(off, 0, G);
        const bool room = static_cast<int64_t>(off) + n <= prog_cap;
        uint32_t *out = inl ? rr + 2 : prog + off;
        if (write && (inl || room)) {
            if (term_ok) out[t0 + __popc(live & ((1u << gl) - 1))] = wt << kPrefLenBits | (after - t0);
            if (keep && cnt) {
                uint32_t k = e0 + __popc(live & ((2u << term) - 1));  // past its own term's header too
                aff_entries(q, pres, wb, pfx0, neg, [&](uint32_t ent) { out[k++] = ent; });
            }
        }
        if (gl == 0 && i < I && (g.fits || !good)) {
            rr[0] = kPrefNone << 24;
            if (write) {
                const uint32_t head = n_live | bit_length(sum) << 16;
                if (!inl && !room) {
                    rr[0] = head | kPrefDecode << 24;
                    cls = 2;
                } else {
                    rr[0] = head | (inl ? kPrefInline : kPrefIndirect) << 24;
                    if (!inl) rr[1] = static_cast<uint32_t>(off);
                    cls = n_live <= kPrefFewTerms ? 3u : (bit_length(sum) <= 8 ? 0u : 1u);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (i < I) rec[i * kPrefRec + gl] = rr[gl];
        __builtin_amdgcn_wave_barrier();
        if (gl == 0) scls[at] = static_cast<uint8_t>(cls);
    }
    __syncthreads();
    // append the rows to their class lists, one counter update per class and
    // workgroup: the counters share a line, and one per class and wavefront was
    // what bounded the launch (233,017 rows 71 -> 42 us)
    const uint32_t cls = static_cast<int>(threadIdx.x) < rpb ? scls[threadIdx.x] : kPrefClasses;
    const int wave = threadIdx.x >> 6;
    __shared__ uint32_t places[4][kPrefClasses];  // per wavefront and class: rows, then the first one's place
    uint32_t below = 0;
    for (uint32_t c = 0; c < kPrefClasses; ++c) {
        const uint64_t mask = __ballot(cls == c);
        if (lane == 0) places[wave][c] = static_cast<uint32_t>(__popcll(mask));
        if (cls == c)
            below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                              __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
    }
    __syncthreads();
    if (threadIdx.x < kPrefClasses) {
        uint32_t n = 0;
        for (int w = 0; w < 4; ++w) n += places[w][threadIdx.x];
        uint32_t at = n ? atomicAdd(list_len + threadIdx.x, n) : 0u;
        for (int w = 0; w < 4; ++w) {
            const uint32_t x = places[w][threadIdx.x];
            places[w][threadIdx.x] = at;
            at += x;
        }
    }
    __syncthreads();
    if (cls < kPrefClasses)
        list[static_cast<int64_t>(cls) * I + places[wave][cls] + below] = static_cast<int32_t>(block0 + threadIdx.x);
}


// Wavefront reductions of a 32-bit value with DPP: quad exchanges, then
// row rotations by 4 and 8 leave every lane with its 16-lane row's result;
// the four rows' results are combined on the scalar unit.
template <int kOp>
__device__ __forceinline__ uint32_t red_op(uint32_t a, uint32_t b)
{
    if constexpr (kOp == 0) return a > b ? a : b;
    else if constexpr (kOp == 1) return a < b ? a : b;
    else return a + b;
}

template <int kOp>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t x)
{
    int v = static_cast<int>(x);
    v = static_cast<int>(red_op<kOp>(static_cast<uint32_t>(v), static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false))));
    v = static_cast<int>(red_op<kOp>(static_cast<uint32_t>(v), static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false))));
    v = static_cast<int>(red_op<kOp>(static_cast<uint32_t>(v), static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0x124, 0xF, 0xF, false))));
    v = static_cast<int>(red_op<kOp>(static_cast<uint32_t>(v), static_cast<uint32_t>(__builtin_amdgcn_update_dpp(v, v, 0x128, 0xF, 0xF, false))));
    const uint32_t r0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 0));
    const uint32_t r1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 16));
    const uint32_t r2 = static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 32));
    const uint32_t r3 = static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 48));
    return red_op<kOp>(red_op<kOp>(r0, r1), red_op<kOp>(r2, r3));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) { return wave_reduce_u32<0>(x); }
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) { return wave_reduce_u32<1>(x); }
__device__ __forceinline__ uint32_t wave_add_u32(uint32_t x) { return wave_reduce_u32<2>(x); }

// acc += w * a, bit-sliced over kBits score bits (w <= 100 < 2^7): bits
// 0..6 are full adds of the weight's bit (masked by a) and the carry, above
// them only the carry moves.  The row's class guarantees that its weight
// sum fits kBits, so no carry leaves the top bit.  Branch-free, so the
// score words stay in place.
template <int kBits>
__device__ __forceinline__ void score_add(Words (&acc)[kBits], uint32_t w, const Words &a)
{
    Words carry{0, 0};
#pragma unroll
    for (int b = 0; b < 7; ++b) {
        const uint64_t wm = ((w >> b) & 1u) ? ~0ull : 0ull;
        const uint64_t xa = acc[b].a, xb = acc[b].b, ya = a.a & wm, yb = a.b & wm;
        acc[b].a = xa ^ ya ^ carry.a;
        acc[b].b = xb ^ yb ^ carry.b;
        carry.a = (xa & ya) | (carry.a & (xa ^ ya));
        carry.b = (xb & yb) | (carry.b & (xb ^ yb));
    }
#pragma unroll
    for (int b = 7; b < kBits; ++b) {
        const uint64_t xa = acc[b].a, xb = acc[b].b;
        acc[b].a = xa ^ carry.a;
        acc[b].b = xb ^ carry.b;
        carry.a &= xa;
        carry.b &= xb;
    }
}

// One term decoded from its expressions (rows whose program found no slice).
template <bool kBuf>
__device__ Words pref_term_decoded(const pc_pred *__restrict__ preds, int64_t b, int64_t e,
                                   const uint64_t *__restrict__ present, const uint32_t *__restrict__ wbase,
                                   const Planes<kBuf> &pl)
{
    Words a{~0ull, ~0ull};
    for (int64_t p = b; p < e; ++p) {
        const pc_pred q = preds[p];
        const uint64_t *pres = present + static_cast<int64_t>(q.label) * 4;
        const uint32_t *wb = wbase + static_cast<int64_t>(q.label) * 4;
        uint64_t sel[4];
        bool neg;
        expr_clause(q.op, q.vals, pres, sel, neg);
        Words c{0, 0};
        for (int k = 0; k < 4; ++k) {
            uint64_t m = sel[k];
            while (m) {
                const uint32_t v = static_cast<uint32_t>(k * 64 + __builtin_ctzll(m));
                m &= m - 1;
                const Words x = pl(plane_id(pres, wb, v));
                c.a |= x.a;
                c.b |= x.b;
            }
        }
        a.a &= neg ? ~c.a : c.a;
        a.b &= neg ? ~c.b : c.b;
    }
    return a;
}

// Work item (tile of 128 words, chunk of rows) as in k_sel_eval; one row at
// a time per wavefront.  Per row: the feasible words (every node when the
// bitset is absent), the bit-sliced scores of the live terms, the lane's
// best (score, lowest node) and tie count, reduced over the wavefront into
// part_key[tile * I + r] = (score + 1) << 32 | ~node (0: no feasible node)
// and part_cnt[tile * I + r].
// kCls: the rows of one class list (0: scores within 8 bits, 1: within 16
// bits, 2: decoded on the fly, 3: at most three live terms), so that each
// launch keeps only the score words it needs and the common one carries no
// decoding code.  Class 3 keeps the (at most) three term masks instead of
// score bits: a node's score is fixed by the set of terms that hold for it,
// so the lane's best score is the largest weight sum of a set of terms that
// hold together for some candidate.
// Bound by no unit alone: of 699,051 rows over 50,000 nodes in 1.54 ms, HBM moves
// 7.9 GB (0.64 of its peak: the feasible words, and plane words that miss L2), the
// scalar units issue at 59 % and the vector units at 37 % of their rates, and waves wait 55 %
// of their cycles.  Class 3 takes the term sets in one pass of
// positive intersections (two passes of exact patterns before: 1.6 times the vector
// instructions), one maximum for score and node, and skips the tiles without a feasible node;
// six waves per SIMD hide its plane loads better than five or seven.  233,017 rows
// x 50,000 nodes, a third of the rows without a feasible node: 1.35 -> 0.52
// ms; 100,000 three-term rows with every node feasible: the call 0.82 -> 0.48 ms.
template <bool kBuf, int kCls>
__global__ __launch_bounds__(kEvalThreads, kCls == 3 ? 6 : 1) void k_pref_eval(
    const uint32_t *__restrict__ rec, const uint32_t *__restrict__ prog, const int32_t *__restrict__ row_off,
    const int32_t *__restrict__ term_off, const uint32_t *__restrict__ weight, const pc_pred *__restrict__ preds,
    int64_t n_preds, int32_t L, const uint64_t *__restrict__ present, const uint32_t *__restrict__ wbase,
    const uint64_t *__restrict__ planes, int64_t plane_bytes, int64_t Wp, int32_t I, int32_t W, int32_t N,
    const uint64_t *__restrict__ feasible, uint64_t *__restrict__ part_key, uint32_t *__restrict__ part_cnt,
    int32_t ntiles, int32_t rpc, int32_t brows, const int32_t *__restrict__ list,
    const uint32_t *__restrict__ list_len, int64_t fstride)
{
    constexpr int kBits = kCls == 0 ? 8 : (kCls == 3 ? 1 : kScoreBits);
    constexpr bool kDecode = kCls == 2;
    constexpr uint32_t kTileNodes = kTileW * 64;
    // class 3: each wavefront stages its batch's records in LDS (one record
    // per lane), so a row's program words cost an LDS read instead of a
    // dependent memory load
    __shared__ uint4 lrec_all[kCls == 3 ? kEvalThreads * (kPrefRec / 4) : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t *lrec = reinterpret_cast<const uint32_t *>(lrec_all + (kCls == 3 ? wave * 64 * (kPrefRec / 4) : 0));
    const int32_t *rows = list + static_cast<int64_t>(kCls) * I;
    // The grid may hold fewer workgroups than the list has items (a class is
    // often empty): each takes every gridDim-th item, dealt to the XCDs in
    // contiguous ranges.
    const int32_t len = static_cast<int32_t>(list_len[kCls]);
    const int32_t nchunks = (len + rpc - 1) / rpc;
    const int64_t total = static_cast<int64_t>(ntiles) * nchunks;
    const int64_t per = (total + 7) / 8;
    const uint64_t last = (N & 63) ? (1ull << (N & 63)) - 1 : ~0ull;
    for (int64_t b = blockIdx.x; (b >> 3) < per; b += gridDim.x) {
    const int64_t item = (b & 7) * per + (b >> 3);
    if (item >= total) continue;
    const int32_t tile = static_cast<int32_t>(item / nchunks);
    const int32_t chunk = static_cast<int32_t>(item % nchunks);
    const int32_t w0 = tile * kTileW + lane * kWpl;
    const bool ok0 = w0 < W, ok1 = w0 + 1 < W;
    const uint64_t m0 = ok0 ? (w0 == W - 1 ? last : ~0ull) : 0ull;
    const uint64_t m1 = ok1 ? (w0 + 1 == W - 1 ? last : ~0ull) : 0ull;
    Planes<kBuf> pl;
    if constexpr (kBuf)
        pl.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(planes), static_cast<short>(0),
                                                    static_cast<int>(plane_bytes), 0x00020000);
    pl.lane_off = static_cast<uint32_t>(kPad + w0) * 8u;  // inside the plane row: kPad + w0 + 1 < Wp
    pl.rowbytes = static_cast<uint32_t>(Wp * 8);
    pl.pcol = planes + kPad + w0;
    pl.Wp = Wp;
    const int32_t r0 = chunk * rpc;
    const int32_t r1 = min(len, r0 + rpc);
    for (int32_t bat = r0 + wave * brows; bat < r1; bat += kEvalWaves * brows) {
        const int32_t nb_rows = min(brows, r1 - bat);
        // The batch's row ids, one per lane.  A row's record head and
        // feasible words (fstride 0: one all-ones row; lanes past the row's
        // end read its word 0 and mask it) are requested ahead: in class 3 by
        // two rows, so that their latency also hides behind a row that is
        // skipped, else by one (the second copy of the row's code would cost
        // the score words' classes 25 registers).
        constexpr int kAhead = kCls == 3 ? 2 : 1;
        const int32_t my_row = lane < nb_rows ? rows[bat + lane] : 0;
        if constexpr (kCls == 3) {
            // the previous batch's reads are done (LDS requests of one
            // wavefront complete in order; the fences keep the compiler's
            // order)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (lane < nb_rows) {
                const uint4 *src = reinterpret_cast<const uint4 *>(rec + static_cast<int64_t>(my_row) * kPrefRec);
                uint4 *dst = lrec_all + (wave * 64 + lane) * (kPrefRec / 4);
#pragma unroll
                for (int q = 0; q < kPrefRec / 4; ++q) dst[q] = src[q];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        struct Ahead {  // a row's head and feasible words, in flight
            int32_t r;
            uint32_t head;
            uint64_t a, b;
        };
        auto request = [&](int32_t i) {
            Ahead x;
            x.r = __builtin_amdgcn_readlane(my_row, i);
            x.head = kCls == 3 ? 0u : rec[static_cast<int64_t>(x.r) * kPrefRec];
            const uint64_t *fr = feasible + static_cast<int64_t>(x.r) * fstride;
            x.a = fr[ok0 ? w0 : 0];
            x.b = fr[ok1 ? w0 + 1 : 0];
            return x;
        };
        auto one_row = [&](int32_t i, Ahead &ahead) {
            const int32_t r = ahead.r;
            const uint32_t *R = rec + static_cast<int64_t>(r) * kPrefRec;
            const uint32_t head = kCls == 3 ? lrec[i * kPrefRec] : ahead.head;
            const uint32_t kind = head >> 24, live = head & 0xFFFFu;
            Words cand{m0 & ahead.a, m1 & ahead.b};
            uint64_t key = 0;
            uint32_t cnt = 0;
            uint32_t sc = 0;
            // a tile without a feasible node of the row has nothing to score
            const bool some = __ballot((cand.a | cand.b) != 0) != 0;
            if (some) {
            if constexpr (kCls == 3) {
                Words A[kPrefFewTerms];
                uint32_t wt[kPrefFewTerms];
                const uint32_t nt = __builtin_amdgcn_readfirstlane(kind == kPrefNone ? 0u : live);
#pragma unroll
                for (int t = 0; t < static_cast<int>(kPrefFewTerms); ++t) {
                    A[t] = Words{0, 0};
                    wt[t] = 0;
                }
                // the program: inline words from the LDS copy, or a slice of
                // prog; one walk for either source, inlined at each call
                auto walk = [&](const uint32_t *pr) {
#pragma unroll
                for (int t = 0; t < static_cast<int>(kPrefFewTerms); ++t) {
                    if (static_cast<uint32_t>(t) < nt) {
                        const uint32_t hdr = __builtin_amdgcn_readfirstlane(*pr++);
                        wt[t] = hdr >> kPrefLenBits;
                        const int32_t len = static_cast<int32_t>(hdr & ((1u << kPrefLenBits) - 1));
                        Words a{~0ull, ~0ull}, c{0, 0}, unused{0, 0};
                        for (int32_t e0 = 0; e0 < len; e0 += kGroup) {
                            uint32_t E[kGroup];
                            Words V[kGroup];
#pragma unroll
                            for (int k = 0; k < kGroup; ++k) E[k] = (e0 + k < len) ? pr[e0 + k] : 0u;
#pragma unroll
                            for (int k = 0; k < kGroup; ++k)
                                if (e0 + k < len) V[k] = pl(E[k] & kPidMask);
#pragma unroll
                            for (int k = 0; k < kGroup; ++k)
                                if (e0 + k < len) fold<false>(E[k], V[k], c, a, unused);
                        }
                        pr += len;
                        A[t] = a;
                    }
                }
                };
                if (kind == kPrefInline)
                    walk(lrec + i * kPrefRec + 2);
                else if (kind == kPrefIndirect)
                    walk(prog + lrec[i * kPrefRec + 1]);
                // The terms by falling weight (the weights are uniform).  Then
                // the sets of terms that may hold, by rising weight sum: a
                // lane's best nodes are its candidates in the last of them
                // that is not empty.  Nodes for which further terms hold are in
                // a later set, so a set needs only the terms that it names;
                // sets of equal sum are neighbours in this order and joined.
                auto order = [&](int x, int y) {
                    if (wt[x] < wt[y]) {
                        const uint32_t w = wt[x];
                        const Words m = A[x];
                        wt[x] = wt[y];
                        A[x] = A[y];
                        wt[y] = w;
                        A[y] = m;
                    }
                };
                static_assert(kPrefFewTerms == 3, "the order of the term sets below");
                Words best = cand, prev{0, 0};
                uint32_t prev_sum = 0;
                auto take = [&](const Words &m, uint32_t sum) {
                    Words t{cand.a & m.a, cand.b & m.b};
                    if (sum == prev_sum) {
                        t.a |= prev.a;
                        t.b |= prev.b;
                    }
                    const bool any = (t.a | t.b) != 0;
                    best.a = any ? t.a : best.a;
                    best.b = any ? t.b : best.b;
                    sc = any ? sum : sc;
                    prev = t;
                    prev_sum = sum;
                };
                auto both = [](const Words &x, const Words &y) { return Words{x.a & y.a, x.b & y.b}; };
                if (nt == 1) {
                    take(A[0], wt[0]);
                } else if (nt == 2) {
                    order(0, 1);
                    take(A[1], wt[1]);
                    take(A[0], wt[0]);
                    take(both(A[0], A[1]), wt[0] + wt[1]);
                } else if (nt == 3) {
                    order(0, 1);
                    order(1, 2);
                    order(0, 1);
                    const Words a12 = both(A[1], A[2]), a01 = both(A[0], A[1]);
                    take(A[2], wt[2]);
                    take(A[1], wt[1]);
                    if (wt[0] > wt[1] + wt[2]) {
                        take(a12, wt[1] + wt[2]);
                        take(A[0], wt[0]);
                    } else {
                        take(A[0], wt[0]);
                        take(a12, wt[1] + wt[2]);
                    }
                    take(both(A[0], A[2]), wt[0] + wt[2]);
                    take(a01, wt[0] + wt[1]);
                    take(both(a01, A[2]), wt[0] + wt[1] + wt[2]);
                }
                cand = best;
            } else {
                Words acc[kBits];
#pragma unroll
                for (int b = 0; b < kBits; ++b) acc[b] = Words{0, 0};
                // one loop over the row's terms, whatever their source, so the
                // score words have a single update site
                constexpr bool dec = kDecode;
                const int64_t tb = dec ? row_off[r] : 0;
                const uint32_t n_iter = dec ? static_cast<uint32_t>(row_off[r + 1] - tb)
                                            : (kind == kPrefNone ? 0u : live);
                const uint32_t *pr = kind == kPrefInline ? R + 2 : prog + R[1];
                for (uint32_t t = 0; t < n_iter; ++t) {
                    uint32_t w;
                    Words a{~0ull, ~0ull};
                    if constexpr (dec) {
                        w = weight[tb + t];
                        int64_t len;
                        if (!pref_weight_ok(w) ||
                            !aff_term(preds, term_off[tb + t], term_off[tb + t + 1], n_preds, L, present, len))
                            continue;
                        a = pref_term_decoded<kBuf>(preds, term_off[tb + t], term_off[tb + t + 1], present, wbase, pl);
                    } else {
                        const uint32_t hdr = *pr++;
                        w = hdr >> kPrefLenBits;
                        const int32_t len = static_cast<int32_t>(hdr & ((1u << kPrefLenBits) - 1));
                        Words c{0, 0}, unused{0, 0};
                        for (int32_t e0 = 0; e0 < len; e0 += kGroup) {
                            uint32_t E[kGroup];
                            Words V[kGroup];
#pragma unroll
                            for (int k = 0; k < kGroup; ++k) E[k] = (e0 + k < len) ? pr[e0 + k] : 0u;
#pragma unroll
                            for (int k = 0; k < kGroup; ++k)
                                if (e0 + k < len) V[k] = pl(E[k] & kPidMask);
#pragma unroll
                            for (int k = 0; k < kGroup; ++k)
                                if (e0 + k < len) fold<false>(E[k], V[k], c, a, unused);
                        }
                        pr += len;
                    }
                    score_add<kBits>(acc, w, a);
                }
                // best score among this lane's feasible nodes: keep the nodes
                // that have the highest remaining score bit set, top bit first
                auto narrow = [&](int b) {
                    const Words t{cand.a & acc[b].a, cand.b & acc[b].b};
                    const bool any = (t.a | t.b) != 0;
                    cand.a = any ? t.a : cand.a;
                    cand.b = any ? t.b : cand.b;
                    sc |= any ? (1u << b) : 0u;
                };
#pragma unroll
                for (int b = kBits - 1; b >= 0; --b) narrow(b);
            }
            }
            if (i + kAhead < nb_rows) ahead = request(i + kAhead);
            if (some) {
                // the wavefront's best (score + 1, lowest node) in one maximum
                // (scores fit 17 bits, a tile's nodes 13) and the tie count
                static_assert(kTileNodes == 8192, "13 bits of node");
                const bool has = (cand.a | cand.b) != 0;
                const uint32_t node = static_cast<uint32_t>(lane) * (64u * kWpl) +
                                      (cand.a ? static_cast<uint32_t>(__builtin_ctzll(cand.a))
                                              : 64u + static_cast<uint32_t>(__builtin_ctzll(cand.b | (1ull << 63))));
                const uint32_t top = wave_max_u32(has ? (sc + 1) << 13 | (kTileNodes - 1 - node) : 0u);
                cnt = wave_add_u32(has && sc + 1 == top >> 13
                                       ? static_cast<uint32_t>(__popcll(cand.a) + __popcll(cand.b))
                                       : 0u);
                const uint32_t nmin = static_cast<uint32_t>(tile) * kTileNodes + (kTileNodes - 1 - (top & (kTileNodes - 1)));
                key = (static_cast<uint64_t>(top >> 13) << 32) | (0xFFFFFFFFu - nmin);
            }
            if (lane == 0) {
                part_key[static_cast<int64_t>(tile) * I + r] = key;
                part_cnt[static_cast<int64_t>(tile) * I + r] = cnt;
            }
        };
        Ahead even = request(0);
        if constexpr (kAhead == 2) {
            Ahead odd = request(nb_rows > 1 ? 1 : 0);
            for (int32_t i = 0; i < nb_rows; i += 2) {
                one_row(i, even);
                if (i + 1 < nb_rows) one_row(i + 1, odd);
            }
        } else {
            for (int32_t i = 0; i < nb_rows; ++i) one_row(i, even);
        }
    }
    }
}

// Per row: the best key over the tiles and the tie count of that score.
__global__ __launch_bounds__(256) void k_pref_final(const uint64_t *__restrict__ part_key,
                                                    const uint32_t *__restrict__ part_cnt, int32_t I, int32_t ntiles,
                                                    int32_t *__restrict__ best, uint32_t *__restrict__ score,
                                                    uint32_t *__restrict__ count)
{
    const int32_t r = blockIdx.x * 256 + threadIdx.x;
    if (r >= I) return;
    uint64_t key = 0;
    for (int32_t t = 0; t < ntiles; ++t) {
        const uint64_t k = part_key[static_cast<int64_t>(t) * I + r];
        key = k > key ? k : key;
    }
    uint32_t cnt = 0;
    if (key != 0)
        for (int32_t t = 0; t < ntiles; ++t)
            if ((part_key[static_cast<int64_t>(t) * I + r] >> 32) == (key >> 32)) cnt += part_cnt[static_cast<int64_t>(t) * I + r];
    best[r] = key ? static_cast<int32_t>(0xFFFFFFFFu - static_cast<uint32_t>(key)) : -1;
    score[r] = key ? static_cast<uint32_t>(key >> 32) - 1u : 0u;
    count[r] = cnt;
}

}  // namespace

namespace {

// Evaluator geometry for N nodes: W bitset words per row, tiles of kTileW
// words, plane row pitch Wp.  Rows are shifted onto 128-byte lines when
// that costs no extra tile (W of at least one tile); every lane's word
// pair, shifted or not, lies inside [0, Wp - kPad) of a plane row.
struct EvalGeom {
    int64_t W, Wp, ntiles;
    int32_t shift;
};

EvalGeom eval_geom(int32_t N)
{
    EvalGeom g;
    g.W = (static_cast<int64_t>(N) + 63) / 64;
    g.ntiles = (g.W + kTileW - 1) / kTileW;
    g.shift = g.W >= kTileW && (g.W + 15 + kTileW - 1) / kTileW == g.ntiles;
    g.Wp = kPad + g.ntiles * kTileW;
    return g;
}

Clears clears(uint64_t *present, int32_t L, uint64_t *planes, int64_t pzero, int64_t Wp, uint64_t *ctl,
              uint64_t *ones = nullptr, int64_t n_ones = 0)
{
    return Clears{{present, planes + pzero * Wp, ctl, ones},
                  {static_cast<int64_t>(L) * 4, Wp, kCtlWords, n_ones},
                  {0, 0, 0, ~0ull}};
}

// Value planes of the node labels: presence, plane numbering, the planes
// themselves and, for a pfx0 other than 0, the prefix planes (present, the all-zero
// plane and ctl are cleared).
int build_planes(pc_ctx *ctx, const uint8_t *labels, int32_t N, int32_t L, int64_t W, int64_t Wp, uint32_t pfx0,
                 uint64_t *present, uint32_t *wbase, uint64_t *planes, uint64_t *ctl, hipStream_t stream)
{
    bool numbered = false;
    if (N > 0 && L > 0) {
        if (L <= kPresenceLdsL) {
            const int64_t n_bytes = static_cast<int64_t>(N) * L;
            const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((n_bytes + (4 << 10) - 1) / (4 << 10), 1024));
            // Few workgroups: the last one numbers the planes (one launch less, 3 us).
            // Many queue up for the count (1,024: 26 us, against 17 and 6 apart).
            numbered = blocks <= 256;
            PC_TIMED(ctx, "k_sel_presence", stream,
                     hipLaunchKernelGGL(k_sel_presence_flat, dim3(blocks), dim3(256), static_cast<size_t>(L) * 32,
                                        stream, labels, n_bytes, L, reinterpret_cast<uint32_t *>(present), wbase,
                                        numbered ? ctl + kCtlDone : nullptr));
            PC_LAUNCH_CHECK(ctx);
        } else {
            // about 2048 workgroups: a few hundred nodes each
            const int64_t ltiles = (L + 63) / 64;
            int64_t chunk = (static_cast<int64_t>(N) * ltiles + 2047) / 2048;
            chunk = chunk < 64 ? 64 : (chunk + 3) / 4 * 4;
            while ((N + chunk - 1) / chunk > 65535) chunk *= 2;
            dim3 gp((L + 63) / 64, static_cast<unsigned>((N + chunk - 1) / chunk));
            PC_TIMED(ctx, "k_sel_presence", stream,
                     hipLaunchKernelGGL(k_sel_presence, gp, dim3(256), 0, stream, labels, N, L, chunk,
                                        reinterpret_cast<uint32_t *>(present)));
            PC_LAUNCH_CHECK(ctx);
        }
    }
    if (L > 0 && !numbered) {
        PC_TIMED(ctx, "k_sel_label_scan", stream,
                 hipLaunchKernelGGL(k_sel_label_scan, dim3(1), dim3(1024), 0, stream, present, L, wbase));
        PC_LAUNCH_CHECK(ctx);
    }
    if (N > 0 && L > 0) {
        dim3 gb(static_cast<unsigned>((W + kPlaneWords - 1) / kPlaneWords), static_cast<unsigned>((L + 3) / 4));
        const bool wide = L % 4 == 0 && (reinterpret_cast<uintptr_t>(labels) & 3) == 0;
        const auto kern = pfx0 ? (wide ? k_sel_planes<true, true> : k_sel_planes<false, true>)
                               : (wide ? k_sel_planes<true, false> : k_sel_planes<false, false>);
        PC_TIMED(ctx, "k_sel_planes", stream,
                 hipLaunchKernelGGL(kern, gb, dim3(256), 0, stream, labels, N, L, present, wbase, planes, Wp, pfx0));
        PC_LAUNCH_CHECK(ctx);
    }
    return PC_OK;
}

// The evaluators' work items for I rows over ntiles tiles: nchunks chunks of
// rpc rows, taken by a workgroup's wavefronts in batches of brows rows.
struct RowSplit {
    int64_t rpc, nchunks, brows;
    unsigned blocks;
};

RowSplit row_split(int64_t I, int64_t ntiles)
{
    RowSplit s;
    // Batches of 64 rows while that leaves 32,768 of them, a few per wave
    // slot of the chip; fewer rows make smaller batches instead of idle
    // slots, and a chunk always has a batch for each of a workgroup's
    // wavefronts (whole 64-row batches at any size: 16,384 rows over 13 tiles
    // 98 us, now 55; affinity over 233,017 rows and 7 tiles 524 us, now 327; 6,001
    // rows over one tile 58 us, now 12).
    s.brows = 64;
    while (s.brows > 4 && I * ntiles < s.brows * 32768) s.brows /= 2;
    s.nchunks = std::max<int64_t>((32768 + ntiles - 1) / ntiles, 1);
    s.rpc = (I + s.nchunks - 1) / s.nchunks;
    const int64_t unit = kEvalWaves * s.brows;
    s.rpc = std::max<int64_t>((s.rpc + unit - 1) / unit, 1) * unit;
    s.nchunks = (I + s.rpc - 1) / s.rpc;
    s.blocks = static_cast<unsigned>(8 * ((ntiles * s.nchunks + 7) / 8));
    return s;
}

// The evaluator over every row (feasible nullptr: popcounts only), then
// the popcount partials' sum.
template <bool kTerms>
int launch_eval(pc_ctx *ctx, const uint32_t *rec, const uint32_t *prog, const int32_t *off,
                const pc_pred *preds, const uint64_t *present, const uint32_t *wbase, const uint64_t *planes,
                int64_t pmax, int64_t Wp, int32_t I, int64_t W, int32_t N, uint64_t *feasible, uint32_t *popcnt,
                uint32_t *part, int64_t ntiles, const int32_t *term_off, int64_t n_preds, int32_t L,
                int32_t shift, hipStream_t stream)
{
    const RowSplit sp = row_split(I, ntiles);
    uint32_t *cnt_out = ntiles > 1 ? part : popcnt;
    const int64_t pbytes = static_cast<int64_t>(pmax + 1) * Wp * 8;
    auto eval = [&](auto kern) {
        PC_TIMED(ctx, kTerms ? "k_aff_eval" : (feasible ? "k_sel_eval" : "k_sel_count"), stream,
                 hipLaunchKernelGGL(kern, dim3(sp.blocks), dim3(kEvalThreads), 0, stream, rec, prog, off, preds,
                                    present, wbase, planes, pbytes, Wp, I, static_cast<int32_t>(W), N, feasible,
                                    cnt_out, static_cast<int32_t>(ntiles), static_cast<int32_t>(sp.nchunks),
                                    static_cast<int32_t>(sp.rpc), static_cast<int32_t>(sp.brows), term_off, n_preds,
                                    L, shift));
    };
    if (!feasible) {
        if (pbytes < (int64_t(1) << 31)) eval(k_sel_eval<true, kTerms, false>);  // buffer offsets are 32-bit
        else eval(k_sel_eval<false, kTerms, false>);
    } else {
        if (pbytes < (int64_t(1) << 31)) eval(k_sel_eval<true, kTerms>);
        else eval(k_sel_eval<false, kTerms>);
    }
    PC_LAUNCH_CHECK(ctx);
    if (ntiles > 1) {
        PC_TIMED(ctx, kTerms ? "k_aff_popsum" : "k_sel_popsum", stream,
                 hipLaunchKernelGGL(k_sel_popsum, dim3(static_cast<unsigned>((I + 255) / 256)), dim3(256), 0, stream,
                                    part, I, static_cast<int32_t>(ntiles), popcnt));
        PC_LAUNCH_CHECK(ctx);
    }
    return PC_OK;
}

}  // namespace

int run_selectors(pc_ctx *ctx, const uint8_t *labels, int32_t N, int32_t L, const int32_t *pred_off,
                  const pc_pred *preds, int64_t n_preds, int32_t I, uint64_t *feasible, uint32_t *popcnt,
                  hipStream_t stream, char *fixed, size_t fixed_cap)
{
    const EvalGeom geo = eval_geom(N);
    const int64_t W = geo.W, Wp = geo.Wp, ntiles = geo.ntiles;
    const int64_t pmax = static_cast<int64_t>(L) * (N < 256 ? N : 256);
    const size_t plane_bytes = static_cast<size_t>(pmax + 1) * static_cast<size_t>(Wp) * 8;
    if (plane_bytes > (size_t(64) << 30))
        return pc_set_error(ctx, PC_ENOMEM, "pc_eval_selectors: value planes need %zu bytes (L=%d N=%d)", plane_bytes,
                            L, N);
    uint64_t *present, *planes, *ctl;
    uint32_t *wbase, *prog, *rec, *part;
    auto carve = [&](Carver &cv) {
        present = cv.take<uint64_t>(static_cast<size_t>(L) * 4 + 1);
        wbase = cv.take<uint32_t>(static_cast<size_t>(L) * 4 + 1);
        planes = cv.take<uint64_t>(static_cast<size_t>(pmax + 1) * Wp + 2);  // + the all-zero plane pmax
        prog = cv.take<uint32_t>(static_cast<size_t>(n_preds) * 4 + 4);
        rec = cv.take<uint32_t>(static_cast<size_t>(I) * kRecWords + kRecWords);
        part = ntiles > 1 ? cv.take<uint32_t>(static_cast<size_t>(ntiles) * I + 1) : nullptr;
        ctl = cv.take<uint64_t>(kCtlWords);
    };
    // Few words and predicates: the labels themselves, in one launch.  Planes
    // and programs / labels: 43 to 6,000 rows over 16 nodes 35 / 15 us, 20,000 rows
    // over 64 34 / 20, 6,000 over 300 34 / 18, 20,000 over 300 36 / 35; past the
    // limits 60,000 rows over 64 nodes 48 / 50, 6,000 over 1,500 35 / 50.  Rows
    // without predicates still take a wavefront each, so their number counts too:
    // 20,000 predicates in 25,000 rows over 500 nodes 27 / 26, in 50,000 32 / 34, in
    // 200,000 62 / 81; over 250 nodes 200,000 rows 60 / 56, 500,000 94 / 123; over
    // 64 500,000 rows 93 / 76, 1,000,000 146 / 151, 2,000,000 255 / 307.  (Where one row
    // has most of the predicates a wavefront tests them in turn, as the compile did: a row of
    // 5,000 over 64 nodes 2,330 / 1,790, over 300 2,340 / 2,880; of 300 163 / 113, 160 / 179.)
    const size_t small_lds = static_cast<size_t>(L) * static_cast<size_t>(small_pitch(W));
    const bool small = W > 0 && W <= kSmallW && small_lds <= kSmallLds && n_preds <= kSmallWork / (W + 2) &&
                       I <= small_rows(W);
    auto launch_small = [&]() -> int {
        const unsigned blocks = static_cast<unsigned>(std::min(I / (kSmallThreads / 64) + 1, 512));
        const auto kern = W == 1 ? k_sel_small<1> : W <= 4 ? k_sel_small<4> : k_sel_small<8>;
        if (small_lds > 48 * 1024)
            PC_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(small_lds)));
        PC_TIMED(ctx, "k_sel_small", stream,
                 hipLaunchKernelGGL(kern, dim3(blocks), dim3(kSmallThreads), small_lds, stream, labels, N, L,
                                    pred_off, preds, n_preds, I, static_cast<int32_t>(W), feasible, popcnt,
                                    ctx->d_err));
        PC_LAUNCH_CHECK(ctx);
        return PC_OK;
    };
    Carver dry{nullptr, 0};
    carve(dry);
    char *base = fixed;
    if (fixed != nullptr) {
        if (dry.off > fixed_cap)
            return pc_set_error(ctx, PC_EINVAL,
                                "pc_eval_selectors_noalloc: needs %zu bytes of scratch, above its maximum of %zu "
                                "(N=%d L=%d I=%d n_preds=%lld)",
                                dry.off, fixed_cap, N, L, I, static_cast<long long>(n_preds));
    } else {
        int rc = pc_ensure_arena(ctx, dry.off);
        if (rc) return rc;
        base = ctx->arena;
    }
    Carver real{base, 0};
    carve(real);
    if (small) return launch_small();
    int rc = PC_OK;

    if (W == 0) launch_fill_u32(popcnt, static_cast<size_t>(I), 0, stream);
    PC_TIMED(ctx, "k_sel_clear", stream,
             hipLaunchKernelGGL(k_sel_clear, dim3(static_cast<unsigned>(std::max<int64_t>(int64_t(4) * L, Wp) / 1024 + 1)),
                                dim3(256), 0, stream, clears(present, L, planes, pmax, Wp, ctl)));
    rc = build_planes(ctx, labels, N, L, W, Wp, 0, present, wbase, planes, ctl, stream);
    if (rc) return rc;
    constexpr int kRows = kCompThreads / kSelLanes;  // rows per workgroup
    // (a workgroup fills its label tables once: of 699,051 rows, 21,846 workgroups
    // 63.5 us, 8,192 56.7, 4,096 58.5, 2,048 62.6)
    const unsigned rgrid = static_cast<unsigned>(std::min<int64_t>((I + kRows - 1) / kRows, 8192));
    PC_TIMED(ctx, "k_sel_compile", stream,
             hipLaunchKernelGGL(L <= kLdsLabels ? k_sel_compile<true> : k_sel_compile<false>, dim3(rgrid), dim3(256), 0, stream, pred_off, preds, n_preds, I, L,
                                present, wbase, prog, rec, ctx->d_err));
    PC_LAUNCH_CHECK(ctx);
    if (W == 0) return PC_OK;
    return launch_eval<false>(ctx, rec, prog, pred_off, preds, present, wbase, planes, pmax, Wp, I, W, N, feasible,
                              popcnt, part, ntiles, nullptr, n_preds, L, geo.shift, stream);
}

int run_affinity(pc_ctx *ctx, const uint8_t *labels, int32_t N, int32_t L, const int32_t *row_off, int32_t I,
                 const int32_t *term_off, int32_t n_terms, const pc_pred *preds, int64_t n_preds, uint64_t *feasible,
                 uint32_t *popcnt, uint8_t *unknown, hipStream_t stream)
{
    const EvalGeom geo = eval_geom(N);
    const int64_t W = geo.W, Wp = geo.Wp, ntiles = geo.ntiles;
    const int64_t pmax = static_cast<int64_t>(L) * (N < 256 ? N : 256);
    // value planes [0, pmax), the all-zero plane pmax, prefix planes pmax + 1 + [0, pmax)
    const int64_t ptop = 2 * pmax;
    const size_t plane_bytes = static_cast<size_t>(ptop + 1) * static_cast<size_t>(Wp) * 8;
    if (plane_bytes > (size_t(64) << 30))
        return pc_set_error(ctx, PC_ENOMEM, "pc_eval_affinity: value planes need %zu bytes (L=%d N=%d)", plane_bytes,
                            L, N);
    // indirect programs take slices of prog: room for 4 entries per
    // expression on average, rounded per row; the rest decode on the fly
    const int64_t prog_cap = 4 * n_preds + 4 * static_cast<int64_t>(I) + 64;
    uint64_t *present, *planes, *ctl;
    uint32_t *wbase, *prog, *rec, *part;
    auto carve = [&](Carver &cv) {
        present = cv.take<uint64_t>(static_cast<size_t>(L) * 4 + 1);
        wbase = cv.take<uint32_t>(static_cast<size_t>(L) * 4 + 1);
        planes = cv.take<uint64_t>(static_cast<size_t>(ptop + 1) * Wp + 2);
        prog = cv.take<uint32_t>(static_cast<size_t>(prog_cap));
        rec = cv.take<uint32_t>(static_cast<size_t>(I) * kRecWords + kRecWords);
        part = ntiles > 1 ? cv.take<uint32_t>(static_cast<size_t>(ntiles) * I + 1) : nullptr;
        ctl = cv.take<uint64_t>(kCtlWords);
    };
    Carver dry{nullptr, 0};
    carve(dry);
    int rc = pc_ensure_arena(ctx, dry.off);
    if (rc) return rc;
    Carver real{ctx->arena, 0};
    carve(real);

    const int64_t nval = std::max<int64_t>(I, n_terms);
    if (nval > 0) {
        const unsigned vgrid = static_cast<unsigned>(std::min<int64_t>((nval + 255) / 256, 8192));
        PC_TIMED(ctx, "k_aff_validate", stream,
                 hipLaunchKernelGGL(k_aff_validate, dim3(vgrid), dim3(256), 0, stream, row_off, I, term_off, n_terms,
                                    preds, n_preds, L, ctx->d_err, clears(present, L, planes, pmax, Wp, ctl)));
        PC_LAUNCH_CHECK(ctx);
    }
    if (I == 0) return PC_OK;
    if (W == 0) launch_fill_u32(popcnt, static_cast<size_t>(I), 0, stream);
    rc = build_planes(ctx, labels, N, L, W, Wp, static_cast<uint32_t>(pmax + 1), present, wbase, planes, ctl, stream);
    if (rc) return rc;
    const bool groups = I < kAffGroupRows;
    const int64_t rows = groups ? 256 / kAffLanes : 256;  // per workgroup
    const unsigned rgrid = static_cast<unsigned>(std::min<int64_t>((I + rows - 1) / rows, 8192));
    const bool lds = L <= kLdsLabels;
    const auto kern = groups ? (lds ? k_aff_compile<kAffLanes, true> : k_aff_compile<kAffLanes, false>)
                             : (lds ? k_aff_compile<1, true> : k_aff_compile<1, false>);
    PC_TIMED(ctx, "k_aff_compile", stream,
             hipLaunchKernelGGL(kern, dim3(rgrid), dim3(256), 0, stream, row_off, I, term_off, n_terms,
                                preds, n_preds, L, present, wbase, prog, prog_cap,
                                reinterpret_cast<unsigned long long *>(ctl + kCtlProg), rec, unknown, static_cast<uint32_t>(pmax + 1)));
    PC_LAUNCH_CHECK(ctx);
    if (W == 0) return PC_OK;
    return launch_eval<true>(ctx, rec, prog, row_off, preds, present, wbase, planes, ptop, Wp, I, W, N, feasible,
                             popcnt, part, ntiles, term_off, n_preds, L, geo.shift, stream);
}

int run_preferred(pc_ctx *ctx, const uint8_t *labels, int32_t N, int32_t L, const uint64_t *feasible,
                  const int32_t *row_off, int32_t I, const int32_t *term_off, int32_t n_terms, const uint32_t *weight,
                  const pc_pred *preds, int64_t n_preds, int32_t *best, uint32_t *score, uint32_t *count,
                  hipStream_t stream)
{
    const int64_t W = (static_cast<int64_t>(N) + 63) / 64;
    const int64_t ntiles = (W + kTileW - 1) / kTileW;
    const int64_t Wp = kPad + ntiles * kTileW;  // unshifted tiles: every lane's pair lies inside a plane row
    const int64_t pmax = static_cast<int64_t>(L) * (N < 256 ? N : 256);
    const int64_t ptop = 2 * pmax;  // value planes, the all-zero plane pmax, prefix planes
    const size_t plane_bytes = static_cast<size_t>(ptop + 1) * static_cast<size_t>(Wp) * 8;
    if (plane_bytes > (size_t(64) << 30))
        return pc_set_error(ctx, PC_ENOMEM, "pc_score_preferred: value planes need %zu bytes (L=%d N=%d)",
                            plane_bytes, L, N);
    // room for a header per term and 4 entries per expression; rows beyond it decode on the fly
    const int64_t prog_cap = std::min<int64_t>(static_cast<int64_t>(n_terms) + 4 * n_preds + 64, int64_t(1) << 31);
    uint64_t *present, *planes, *part_key, *ones, *ctl;
    uint32_t *wbase, *prog, *rec, *part_cnt;
    int32_t *list;
    auto carve = [&](Carver &cv) {
        present = cv.take<uint64_t>(static_cast<size_t>(L) * 4 + 1);
        wbase = cv.take<uint32_t>(static_cast<size_t>(L) * 4 + 1);
        planes = cv.take<uint64_t>(static_cast<size_t>(ptop + 1) * Wp + 2);
        prog = cv.take<uint32_t>(static_cast<size_t>(prog_cap));
        rec = cv.take<uint32_t>(static_cast<size_t>(I) * kPrefRec + kPrefRec);
        list = cv.take<int32_t>(static_cast<size_t>(I) * kPrefClasses + 1);
        ones = cv.take<uint64_t>(feasible ? 1 : static_cast<size_t>(W) + 1);
        part_key = cv.take<uint64_t>(static_cast<size_t>(ntiles) * I + 1);
        part_cnt = cv.take<uint32_t>(static_cast<size_t>(ntiles) * I + 1);
        ctl = cv.take<uint64_t>(kCtlWords);
    };
    Carver dry{nullptr, 0};
    carve(dry);
    int rc = pc_ensure_arena(ctx, dry.off);
    if (rc) return rc;
    Carver real{ctx->arena, 0};
    carve(real);

    const int64_t nval = std::max<int64_t>(I, n_terms);
    if (nval > 0) {
        const unsigned vgrid = static_cast<unsigned>(std::min<int64_t>((nval + 255) / 256, 8192));
        PC_TIMED(ctx, "k_pref_validate", stream,
                 hipLaunchKernelGGL(k_pref_validate, dim3(vgrid), dim3(256), 0, stream, row_off, I, term_off, n_terms,
                                    weight, preds, n_preds, L, ctx->d_err,
                                    clears(present, L, planes, pmax, Wp, ctl, ones, feasible ? 0 : W)));
        PC_LAUNCH_CHECK(ctx);
    }
    if (I == 0) return PC_OK;
    rc = build_planes(ctx, labels, N, L, W, Wp, static_cast<uint32_t>(pmax + 1), present, wbase, planes, ctl, stream);
    if (rc) return rc;
    static_assert(kPrefClasses <= 2 * (kCtlWords - kCtlLists), "a length per class list");
    uint32_t *list_len = reinterpret_cast<uint32_t *>(ctl + kCtlLists);
    auto *prog_used = reinterpret_cast<unsigned long long *>(ctl + kCtlProg);
    // rows per workgroup: all 256 threads', or 16 at a time (up to 256, so that
    // the class lists' counters are not updated too often)
    const bool groups = I < kPrefGroupRows;
    const int32_t rpb =
        groups ? static_cast<int32_t>(std::min<int64_t>(256, std::max<int64_t>(16, I / 512 / 16 * 16))) : 256;
    const unsigned rgrid = static_cast<unsigned>((static_cast<int64_t>(I) + rpb - 1) / rpb);
    const bool lds = L <= kLdsLabels;
    const auto kern = groups ? (lds ? k_pref_compile<kAffLanes, true> : k_pref_compile<kAffLanes, false>)
                             : (lds ? k_pref_compile<1, true> : k_pref_compile<1, false>);
    PC_TIMED(ctx, "k_pref_compile", stream,
             hipLaunchKernelGGL(kern, dim3(rgrid), dim3(256), 0, stream, row_off, I, term_off, n_terms,
                                weight, preds, n_preds, L, present, wbase, prog, prog_cap, prog_used, rec, list,
                                list_len, static_cast<uint32_t>(pmax + 1), rpb));
    PC_LAUNCH_CHECK(ctx);
    if (W > 0) {
        const RowSplit sp = row_split(I, ntiles);
        const int64_t pbytes = static_cast<int64_t>(ptop + 1) * Wp * 8;
        auto eval = [&](auto kern, const char *name, unsigned blocks) {
            PC_TIMED(ctx, name, stream,
                     hipLaunchKernelGGL(kern, dim3(blocks), dim3(kEvalThreads), 0, stream, rec, prog, row_off, term_off,
                                        weight, preds, n_preds, L, present, wbase, planes, pbytes, Wp, I,
                                        static_cast<int32_t>(W), N, feasible ? feasible : ones, part_key, part_cnt,
                                        static_cast<int32_t>(ntiles), static_cast<int32_t>(sp.rpc),
                                        static_cast<int32_t>(sp.brows), list, list_len,
                                        feasible ? static_cast<int64_t>(W) : int64_t(0)));
        };
        // one launch per class list: the lists' lengths are known on the device
        // only.  The common class has a workgroup for every item of I rows, the
        // others, which are mostly empty, a grid that walks their items (a full
        // grid of 30,000 workgroups that exit at once took 11-17 us each).
        const unsigned few = std::min(sp.blocks, 4096u);
        if (pbytes < (int64_t(1) << 31)) {
            eval(k_pref_eval<true, 0>, "k_pref_eval", few);
            eval(k_pref_eval<true, 1>, "k_pref_eval16", few);
            eval(k_pref_eval<true, 2>, "k_pref_decode", few);
            eval(k_pref_eval<true, 3>, "k_pref_eval3", sp.blocks);
        } else {
            eval(k_pref_eval<false, 0>, "k_pref_eval", few);
            eval(k_pref_eval<false, 1>, "k_pref_eval16", few);
            eval(k_pref_eval<false, 2>, "k_pref_decode", few);
            eval(k_pref_eval<false, 3>, "k_pref_eval3", sp.blocks);
        }
        PC_LAUNCH_CHECK(ctx);
    }
    PC_TIMED(ctx, "k_pref_final", stream,
             hipLaunchKernelGGL(k_pref_final, dim3(static_cast<unsigned>((I + 255) / 256)), dim3(256), 0, stream,
                                part_key, part_cnt, I, static_cast<int32_t>(W > 0 ? ntiles : 0), best, score, count));
    PC_LAUNCH_CHECK(ctx);
    return PC_OK;
}

// ---------------------------------------------------------------- fixed scratch
// The allocation-free selector entry point carves its scratch from this
// array instead of the context's arena.  Each device holds its own copy (the
// code object's memory, from the first use on that device until the process
// ends).  In host code the name stands for no device address: only the
// pointer hipGetSymbolAddress returns for the current device is used.  A
// 64 KiB guard band follows the usable PC_NOALLOC_SCRATCH_BYTES.
static __device__ __align__(256) unsigned char scratch[PC_NOALLOC_SCRATCH_BYTES + 65536];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_ptr[kMaxDevices];  // this device's address of `scratch`, once looked up
}  // namespace

int pc_noalloc_setup(pc_ctx *ctx)
{
    if (ctx->device < 0 || ctx->device >= kMaxDevices)
        return pc_set_error(ctx, PC_EDEVICE, "device %d beyond the %d devices with fixed scratch", ctx->device,
                            kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[ctx->device] != nullptr) return PC_OK;
    void *p = nullptr;
    PC_HIP(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return pc_set_error(ctx, PC_EDEVICE, "no device address for the fixed scratch");
    g_scratch_ptr[ctx->device] = static_cast<char *>(p);
    return PC_OK;
}

int run_selectors_noalloc(pc_ctx *ctx, const uint8_t *labels, int32_t N, int32_t L, const int32_t *pred_off,
                          const pc_pred *preds, int64_t n_preds, int32_t I, uint64_t *feasible, uint32_t *popcnt,
                          hipStream_t stream)
{
    char *p = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (ctx->device >= 0 && ctx->device < kMaxDevices) p = g_scratch_ptr[ctx->device];
    }
    if (p == nullptr) return pc_set_error(ctx, PC_EDEVICE, "pc_eval_selectors_noalloc: fixed scratch not set up");
    return run_selectors(ctx, labels, N, L, pred_off, preds, n_preds, I, feasible, popcnt, stream, p,
                         PC_NOALLOC_SCRATCH_BYTES);
}
