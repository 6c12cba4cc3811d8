// Sampled shortest-path statistics: the average path length and the diameter
// estimate of the paper's Table 2 (Results), both taken over breadth-first
// searches from a sample of source vertices.
//
// Sources are searched 64 at a time, one bit per source in a 64-bit word per
// vertex (bit-parallel multi-source BFS).  Every level is one bottom-up sweep:
// a vertex ORs the frontier words of its neighbours, and the bits it had not
// seen yet are the sources that reach it at this level.  A vertex stops
// reading neighbours as soon as every source whose search still goes on has
// reached it, so late levels touch little memory.
//
// The sweep is bound by the L2 requests of the random reads of the
// neighbours' frontier words, so most of them are answered on the CU: a
// coarse bitmap of the vertices with a nonempty word (at most 2^18 bits, one
// per 2^k vertices) is held in LDS and looked up first, then an exact bitmap,
// then the word; in a level with a sparse frontier nearly every lookup ends
// in LDS.  The work is split by degree to keep the wavefronts busy: up to
// kSmallDeg edges two lanes take a vertex (16 edges in flight), up to kMidDeg
// eight, up to kHugeDeg a wavefront, and above that kSplit wavefronts share
// it (a hub's list of 10^5 edges on one wavefront took most of a level).  All but
// the smallest are taken from lists, since vertices of high degree stand
// together in generated graphs: 64 neighbours of 200 edges each were a chain of
// 64 round trips for one wavefront.  The bitmaps are written after the sweep, by
// plain stores from the new frontier's words, and only if the next level looks
// them up.  The
// levels are enqueued kBatch at a time and end themselves when the level
// before reached nothing, so the host waits once per batch and not once per
// level.  Measured against one lane per vertex up to 64 edges, one wavefront
// above, no bitmaps and a wait per level: 8.35 -> 0.96 ms for 64 sources over an
// R-MAT graph of 2 million vertices and 30 million entries, 332 -> 126 ms over a
// PBA graph of 2^27 vertices, whose words (1 GB) are read from memory.  Without
// the bitmaps the first took 2.9 ms; with the vertices up to kMidDeg swept where
// they stand and the bitmaps written by atomics 1.27 and 289 ms.
// Counts are integers and the OR is order-free, so the result does not depend
// on scheduling.
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace sfg {
namespace {

constexpr int kPathThreads = 512;
constexpr int kGroup = 64;           // sources per bit-parallel search
constexpr uint64_t kSmallDeg = 16;   // degree above which more than 2 lanes take the vertex
constexpr uint64_t kMidDeg = 256;    // degree above which a wavefront takes the vertex
constexpr uint64_t kHugeDeg = 4096;  // degree above which kSplit wavefronts share it
constexpr int kSplit = 64;
constexpr int kMoreLanes = 8;      // lanes of a vertex above kSmallDeg (8 edges each in flight)
constexpr int kBatch = 8;         // levels between two waits of the host
constexpr int kCountSlots = 4;    // words a level's count is spread over (workgroup b adds to word b mod 4)
constexpr int kListChunk = 16;    // vertices per thread of ps_init
constexpr int kCoarseWords = 8192;  // 32-bit words of the LDS bitmap
// The bitmaps are looked up while fewer than n / kDense vertices have a
// nonempty word; in a denser level most lookups would go on to the word.
constexpr uint64_t kDense = 8;

// Control words of a search (64-bit).
enum : int {
    kCtlMid = 0,     // vertices above kMidDeg in the list
    kCtlHuge = 1,    // those above kHugeDeg
    kCtlAlive = 2,   // sources that reached a vertex in the level before the batch (bits)
    kCtlFront = 3,   // vertices with a nonempty word in that level
    kCtlMore = 4,    // vertices above kSmallDeg in the list (BITS)
    kCtlLevel = 5,   // then the words kCtlAlive and kCtlFront for each level of the batch
    kCtlWords = kCtlLevel + 2 * kBatch,
};

struct PsPlan {
    size_t off_vis, off_f0, off_f1, off_list, off_ctl, off_cnt, total;
};

PsPlan ps_plan(uint64_t n) {
    PsPlan p;
    size_t o = 0;
    auto take = [&](size_t b) {
        size_t r = o;
        o += align256(b);
        return r;
    };
    p.off_vis = take(n * 8);
    p.off_f0 = take(n * 8);
    p.off_f1 = take(n * 8);
    p.off_list = take(n * 8);  // 32-bit lists and, behind them, the bitmap; or 64-bit lists
    p.off_ctl = take(kCtlWords * 8);
    p.off_cnt = take(kBatch * kCountSlots * 8);
    p.total = o;
    return p;
}

// The searches' device state.  BITS (n <= 2^32): list entries are 32-bit, and the
// second half of the list region holds the frontier's bitmap, the sweep tasks'
// idle counts and a list of the huge vertices, as many as fit (they are taken by one wavefront each beyond
// that: it takes a multigraph whose vertices nearly all have more than kHugeDeg
// edges).  Without BITS list entries are 64-bit, which leaves no room for either;
// vertices up to kMidDeg are then taken where they stand.
template <bool BITS> struct Search {
    using ListT = typename std::conditional<BITS, uint32_t, uint64_t>::type;
    uint64_t n;
    const uint64_t *rp;
    const void *col;
    uint64_t *vis, *front, *next;  // next is written for every vertex
    ListT *list;                   // BITS: above kSmallDeg from the start, above kMidDeg from the end
                                   // else: above kMidDeg from the start, huge ones from the end
    ListT *huge;                   // BITS: [huge_cap]
    uint64_t huge_cap;
    unsigned long long *ctl;
    const unsigned long long *before;  // alive sources and frontier size of the level before
    unsigned long long *now;           // the same of this level
    unsigned long long *cnt;           // [kCountSlots] pairs found by this level
    uint32_t *fine;                    // one bit per vertex of the frontier
    uint32_t *coarse;                  // one bit per 2^shift vertices; null when shift is 0 (fine fits the LDS words)
    uint8_t *idle;                     // BITS: sweeps that found nothing left to look for in 64 vertices, up to 2
    uint32_t shift;

    __device__ __forceinline__ uint64_t words() const { return (n + 31) / 32; }
    __device__ __forceinline__ uint64_t coarse_words() const { return ((n - 1) >> shift) / 32 + 1; }
    __device__ __forceinline__ void mark(uint64_t v) const {
        if (!BITS) return;
        atomicOr(&fine[v >> 5], 1u << (v & 31));
        if (shift) atomicOr(&coarse[v >> (shift + 5)], 1u << ((v >> shift) & 31));
    }
    // Whether a level whose frontier has `size` vertices looks the bitmap up.
    __device__ __forceinline__ bool sparse(uint64_t size) const { return BITS && (shift == 0 || size < n / kDense); }
    // Entries of the lists: above kMidDeg, and huge.
    __device__ __forceinline__ ListT &mid_at(uint64_t i) const { return BITS ? list[n - 1 - i] : list[i]; }
    __device__ __forceinline__ ListT &huge_at(uint64_t i) const { return BITS ? huge[i] : list[n - 1 - i]; }
};

// Per group of sources: no vertex reached, empty words and bitmap.  The first
// group also makes the lists (order irrelevant: every use is an OR or an integer
// sum per vertex), one reservation per list and workgroup chunk.
template <bool BITS>
__global__ __launch_bounds__(kPathThreads) void ps_init(Search<BITS> a, bool lists) {
    __shared__ uint32_t s_n[3];
    __shared__ unsigned long long s_base[3];
    constexpr uint64_t chunk = (uint64_t)kPathThreads * kListChunk;
    if (BITS) {
        const uint64_t stride = (uint64_t)gridDim.x * kPathThreads, words = a.words(), cw = a.coarse_words();
        const uint64_t i0 = (uint64_t)blockIdx.x * kPathThreads + threadIdx.x;
        for (uint64_t w = i0; w < words; w += stride) a.fine[w] = 0;
        for (uint64_t t = i0; t < (a.n + 63) / 64; t += stride) a.idle[t] = 0;
        if (a.shift)
            for (uint64_t w = i0; w < cw; w += stride) a.coarse[w] = 0;
    }
    for (uint64_t c0 = (uint64_t)blockIdx.x * chunk; c0 < a.n; c0 += (uint64_t)gridDim.x * chunk) {
        if (threadIdx.x < 3) s_n[threadIdx.x] = 0;
        __syncthreads();
        uint32_t more = 0, mid = 0, huge = 0;  // bit i: vertex c0 + i kPathThreads + threadIdx.x
#pragma unroll
        for (int i = 0; i < kListChunk; ++i) {
            const uint64_t v = c0 + (uint64_t)i * kPathThreads + threadIdx.x;
            if (v < a.n) {
                const uint64_t deg = a.rp[v + 1] - a.rp[v];
                more |= (uint32_t)(BITS && deg > kSmallDeg && deg <= kMidDeg) << i;
                mid |= (uint32_t)(deg > kMidDeg && deg <= kHugeDeg) << i;
                huge |= (uint32_t)(deg > kHugeDeg) << i;
            }
        }
#pragma unroll
        for (int i = 0; i < kListChunk; ++i) {
            const uint64_t v = c0 + (uint64_t)i * kPathThreads + threadIdx.x;
            if (v < a.n) {
                a.vis[v] = 0;
                a.front[v] = 0;
                if ((huge >> i) & 1u) a.next[v] = 0;  // (several wavefronts OR into it)
            }
        }
        if (lists) {
            uint32_t at[3] = {0, 0, 0};
            if (mid) at[kCtlMid] = atomicAdd(&s_n[kCtlMid], (uint32_t)__popc(mid));
            if (huge) at[kCtlHuge] = atomicAdd(&s_n[kCtlHuge], (uint32_t)__popc(huge));
            if (more) at[2] = atomicAdd(&s_n[2], (uint32_t)__popc(more));
            __syncthreads();
            if (threadIdx.x < 3 && s_n[threadIdx.x])
                s_base[threadIdx.x] = atomicAdd(&a.ctl[threadIdx.x == 2 ? (int)kCtlMore : (int)threadIdx.x],
                                                (unsigned long long)s_n[threadIdx.x]);
            __syncthreads();
            for (int i = 0; i < kListChunk; ++i) {
                const uint64_t v = c0 + (uint64_t)i * kPathThreads + threadIdx.x;
                using ListT = typename Search<BITS>::ListT;
                if ((more >> i) & 1u) a.list[s_base[2] + at[2]++] = (ListT)v;
                if ((mid >> i) & 1u) a.mid_at(s_base[kCtlMid] + at[kCtlMid]++) = (ListT)v;
                if ((huge >> i) & 1u) {
                    const uint64_t h = s_base[kCtlHuge] + at[kCtlHuge]++;
                    if (h < a.huge_cap)
                        a.huge_at(h) = (ListT)v;
                    else
                        a.mid_at(atomicAdd(&a.ctl[kCtlMid], 1ull)) = (ListT)v;
                }
            }
        }
        __syncthreads();
    }
}

struct Sources {
    int64_t v[kGroup];
    uint32_t count;
};

// One wavefront: sources may repeat, and their bits then share a word, which
// every one of them writes.  Every source's search starts alive: that its own
// row is empty does not say that no row lists it.
template <bool BITS> __global__ __launch_bounds__(64) void ps_seed(Search<BITS> a, Sources s) {
    const uint32_t i = threadIdx.x;
    const bool in = i < s.count;
    const int64_t v = in ? s.v[i] : 0;
    uint64_t word = 0;
    if (in) {
        for (uint32_t j = 0; j < s.count; ++j) word |= (uint64_t)(s.v[j] == v) << j;
        a.vis[v] = word;
        a.front[v] = word;
        a.mark((uint64_t)v);
    }
    const uint64_t alive = __ballot(in);
    if (i == 0) {
        a.ctl[kCtlAlive] = alive;
        a.ctl[kCtlFront] = s.count;
    }
}

__device__ __forceinline__ uint64_t or_lanes(uint64_t x, int lanes) {
    for (int off = 1; off < lanes; off <<= 1) x |= __shfl_xor(x, off, 64);
    return x;
}

// How a level looks its neighbours up.
struct Lookup {
    const uint32_t *lds;  // the coarse bitmap of the frontier
    uint32_t shift;
    bool bits;            // look the bitmaps up at all
};

// OR of the frontier words of the neighbours e, e + step, .. (N of them,
// those below end).  The loads of a stage go out together.
template <typename IdT, bool BITS, int N>
__device__ __forceinline__ uint64_t gather(const Search<BITS> &a, const Lookup &q, uint64_t e, uint64_t end,
                                           uint32_t step) {
    using U = typename std::conditional<sizeof(IdT) == 4, uint32_t, uint64_t>::type;
    const U *col = static_cast<const U *>(a.col);
    U x[N];
    uint32_t on = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) x[u] = e + (uint64_t)u * step < end ? col[e + (uint64_t)u * step] : (U)~(U)0;
#pragma unroll
    for (int u = 0; u < N; ++u)  // ids at or above n are not vertices
        on |= (uint32_t)(e + (uint64_t)u * step < end && (uint64_t)x[u] < a.n) << u;
    if (BITS && q.bits) {
        uint32_t b[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const uint32_t c = (uint32_t)x[u] >> q.shift;
            b[u] = (on >> u) & 1u ? q.lds[c >> 5] >> (c & 31) : 0u;
        }
#pragma unroll
        for (int u = 0; u < N; ++u) on &= ~((uint32_t)!(b[u] & 1u) << u);
        if (q.shift) {
#pragma unroll
            for (int u = 0; u < N; ++u) b[u] = (on >> u) & 1u ? a.fine[(uint32_t)x[u] >> 5] : 0u;
#pragma unroll
            for (int u = 0; u < N; ++u) on &= ~((uint32_t)!((b[u] >> ((uint32_t)x[u] & 31)) & 1u) << u);
        }
    }
    uint64_t w[N];
#pragma unroll
    for (int u = 0; u < N; ++u) w[u] = (on >> u) & 1u ? a.front[x[u]] : 0;
    uint64_t acc = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) acc |= w[u];
    return acc;
}

// OR over the neighbours [e0, e1) of one vertex, by a whole wavefront; the
// result is in every lane.  done: the sources that need not be looked for.
template <typename IdT, bool BITS>
__device__ __forceinline__ uint64_t gather_wave(const Search<BITS> &a, const Lookup &q, uint64_t e0, uint64_t e1,
                                                uint64_t done, uint32_t lane) {
    uint64_t acc = 0;
    for (uint64_t e = e0; e < e1; e += 512) {
        acc |= gather<IdT, BITS, 8>(a, q, e + lane, e1, 64);
        acc = or_lanes(acc, 64);
        if ((acc | done) == ~0ull) break;
    }
    return acc;
}

// The wavefront's vertices with `act`, 64 / LANES at a time, LANES lanes each,
// LANES N edges per step.  e0, e1 and done are those of the lane's own
// vertex, whose OR is returned (0 without act).  Called by whole wavefronts.
template <typename IdT, bool BITS, int LANES, int N>
__device__ __forceinline__ uint64_t sweep_class(const Search<BITS> &a, const Lookup &q, bool act, uint64_t e0,
                                                uint64_t e1, uint64_t done, uint32_t lane) {
    constexpr uint32_t kAtOnce = 64 / LANES;
    const uint64_t mask = __ballot(act);
    if (!mask) return 0;
    // Lane i learns the lane of the i-th vertex to sweep.
    const uint32_t nact = (uint32_t)__popcll(mask);
    const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
    const uint32_t rank = act ? before : nact + (lane - before);
    const int from = __builtin_amdgcn_ds_permute((int)rank * 4, (int)lane);
    uint64_t mine = 0;
    for (uint32_t base = 0; base < nact; base += kAtOnce) {
        const uint32_t gi = base + lane / LANES;
        const int sl = __shfl(from, (int)(gi & 63), 64);
        uint64_t e = __shfl(e0, sl, 64);
        const uint64_t e1s = __shfl(e1, sl, 64), dn = __shfl(done, sl, 64);
        const uint64_t end = gi < nact ? e1s : 0;
        uint64_t acc = 0;
        bool go = e < end;
        do {
            if (go) acc |= gather<IdT, BITS, N>(a, q, e + lane % LANES, end, LANES);
            acc = or_lanes(acc, LANES);
            e += LANES * N;
            go = e < end && (acc | dn) != ~0ull;
        } while (__any(go));
        const uint64_t got = __shfl(acc, (int)((rank - base) % kAtOnce) * LANES, 64);
        if (act && rank >= base && rank < base + kAtOnce) mine = got;
    }
    return mine;
}

// Adds a workgroup's (pairs found, vertices reached, sources that reached
// one) to the level's words.
template <bool BITS>
__device__ __forceinline__ void add_level(const Search<BITS> &a, uint64_t found, uint32_t reached, uint64_t alive) {
    __shared__ unsigned long long s_found, s_alive;
    __shared__ uint32_t s_reached;
    if (threadIdx.x == 0) {
        s_found = s_alive = 0;
        s_reached = 0;
    }
    __syncthreads();
    for (int off = 32; off > 0; off >>= 1) {
        found += __shfl_xor(found, off, 64);
        reached += __shfl_xor(reached, off, 64);
        alive |= __shfl_xor(alive, off, 64);
    }
    if ((threadIdx.x & 63) == 0 && found) {
        atomicAdd(&s_found, (unsigned long long)found);
        atomicAdd(&s_reached, reached);
        atomicOr(&s_alive, (unsigned long long)alive);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_found) {
        atomicAdd(&a.cnt[blockIdx.x % kCountSlots], s_found);
        atomicOr(&a.now[0], s_alive);
        atomicAdd(&a.now[1], (unsigned long long)s_reached);
    }
}

// One level.  The long lists come first, so that they do not end the sweep.
template <typename IdT, bool BITS>
__global__ __launch_bounds__(kPathThreads) void ps_sweep(Search<BITS> a) {
    __shared__ uint32_t s_bits[BITS ? kCoarseWords : 1];
    const uint64_t dead = ~a.before[0];  // sources whose search has ended
    if (dead == ~0ull) return;
    Lookup q{s_bits, a.shift, a.sparse(a.before[1])};
    if (BITS) {
        const uint32_t cw = (uint32_t)a.coarse_words();  // at most kCoarseWords
        const uint32_t *c = a.shift ? a.coarse : a.fine;
        if (q.bits)
            for (uint32_t i = threadIdx.x; i < cw; i += kPathThreads) s_bits[i] = c[i];
        __syncthreads();
    }
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t wave = ((uint64_t)blockIdx.x * kPathThreads + threadIdx.x) >> 6;
    const uint64_t waves = (uint64_t)gridDim.x * (kPathThreads / 64);
    const uint64_t nmid = a.ctl[kCtlMid], nhuge = min((uint64_t)a.ctl[kCtlHuge], a.huge_cap);
    uint64_t found = 0, alive = 0;
    uint32_t reached = 0;
    auto reach = [&](uint64_t v, uint64_t seen, uint64_t fresh) {
        a.vis[v] = seen | fresh;
        found += (uint64_t)__popcll(fresh);
        alive |= fresh;
        ++reached;
    };
    // The listed vertices, 64 items of the wavefront at a time: every lane reads
    // its item's vertex, and only those with sources left to look for are swept.
    struct Item {
        uint64_t v, e0, e1, seen;
        bool in, act;
    };
    auto item = [&](bool in, auto at, uint64_t i) {
        Item x{0, 0, 0, 0, in, false};
        if (in) {
            x.v = at(i);
            x.seen = a.vis[x.v];
            x.e0 = a.rp[x.v];
            x.e1 = a.rp[x.v + 1];
            x.act = (x.seen | dead) != ~0ull;
        }
        return x;
    };
    // Huge vertices: raw ORs into next (ps_commit takes them into vis).
    for (uint64_t i0 = wave; i0 < nhuge * kSplit; i0 += 64 * waves) {
        const uint64_t mine = i0 + lane * waves;
        const Item x = item(mine < nhuge * kSplit, [&](uint64_t i) { return a.huge_at(i); }, mine / kSplit);
        for (uint64_t todo = __ballot(x.act); todo; todo &= todo - 1) {
            const int sl = __builtin_ctzll(todo);
            const uint64_t r0 = __shfl(x.e0, sl, 64), r1 = __shfl(x.e1, sl, 64), seen = __shfl(x.seen, sl, 64);
            const uint64_t per = ((r1 - r0) / kSplit + 64) & ~63ull;  // (kSplit parts of at least deg / kSplit)
            const uint64_t e0 = r0 + ((i0 + sl * waves) % kSplit) * per;
            const uint64_t acc = gather_wave<IdT, BITS>(a, q, e0, min(r1, e0 + per), seen | dead, lane) & ~seen;
            if (lane == (uint32_t)sl && acc) atomicOr((unsigned long long *)&a.next[x.v], (unsigned long long)acc);
        }
    }
    for (uint64_t i0 = wave; i0 < nmid; i0 += 64 * waves) {
        const Item x = item(i0 + lane * waves < nmid, [&](uint64_t i) { return a.mid_at(i); }, i0 + lane * waves);
        uint64_t fresh = 0;
        for (uint64_t todo = __ballot(x.act); todo; todo &= todo - 1) {
            const int sl = __builtin_ctzll(todo);
            const uint64_t e0 = __shfl(x.e0, sl, 64), e1 = __shfl(x.e1, sl, 64), seen = __shfl(x.seen, sl, 64);
            const uint64_t acc = gather_wave<IdT, BITS>(a, q, e0, e1, seen | dead, lane) & ~seen;
            if (lane == (uint32_t)sl) fresh = acc;
        }
        if (x.in) a.next[x.v] = fresh;
        if (fresh) reach(x.v, x.seen, fresh);
    }
    if (BITS) {
        const uint64_t nmore = a.ctl[kCtlMore];
        constexpr uint32_t run = 64 / kMoreLanes;  // list entries that stand together in an item set
        for (uint64_t i0 = wave * run; i0 < nmore; i0 += 64 * waves) {
            const uint64_t mine = i0 + lane / run * run * waves + lane % run;
            const Item x = item(mine < nmore, [&](uint64_t i) { return a.list[i]; }, mine);
            const uint64_t fresh = sweep_class<IdT, BITS, kMoreLanes, 8>(a, q, x.act, x.e0, x.e1, x.seen | dead, lane) & ~x.seen;
            if (x.in) a.next[x.v] = fresh;
            if (fresh) reach(x.v, x.seen, fresh);
        }
    }
    // 64 consecutive vertices per wavefront: lane l reads the row and the word
    // of vertex l, then the vertices still to be swept are taken several at a
    // time.  A task whose vertices need no source any more never will: once it
    // has cleared its words of both frontier buffers it is left out (the flags
    // of 64 tasks are read together).
    const uint64_t tasks = (a.n + 63) / 64;
    for (uint64_t t0 = wave; t0 < tasks; t0 += 64 * waves) {
        const uint64_t mine = t0 + lane * waves;  // this lane's task
        const uint32_t idle = mine >= tasks ? 2u : BITS ? (uint32_t)a.idle[mine] : 0u;
        uint64_t todo = __ballot(idle < 2);
        uint64_t quiet = 0;  // tasks with nothing to look for
        while (todo) {
            const uint32_t which = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1;
            const uint64_t v = (t0 + which * waves) * 64 + lane;
            uint64_t e0 = 0, e1 = 0, seen = 0;
            if (v < a.n) {
                e0 = a.rp[v];
                e1 = a.rp[v + 1];
                seen = a.vis[v];
            }
            const uint64_t deg = e1 - e0, done = seen | dead;
            const bool here = v < a.n && deg <= (BITS ? kSmallDeg : kMidDeg), act = here && deg > 0 && done != ~0ull;
            uint64_t got = sweep_class<IdT, BITS, 2, 8>(a, q, act && deg <= kSmallDeg, e0, e1, done, lane);
            if (!BITS) got |= sweep_class<IdT, BITS, 16, 4>(a, q, act && deg > kSmallDeg, e0, e1, done, lane);
            const uint64_t fresh = got & ~seen;
            if (here) a.next[v] = fresh;
            if (fresh) reach(v, seen, fresh);
            if (BITS && !__any(act)) quiet |= 1ull << which;
        }
        if (BITS && ((quiet >> lane) & 1u)) a.idle[mine] = (uint8_t)(idle + 1);
    }
    add_level(a, found, reached, alive);
}

// After a level's sweep.  The huge vertices' new sources go into vis, and their
// words of the frontier just swept are cleared for the level after.  (What the
// sweep ORed into next had been filtered by vis: it is the new frontier's word.)
// The new frontier's bitmap, if the next level looks it up: a wavefront takes
// the vertices of a coarse word, or 64 where there is no coarse bitmap.
template <bool BITS> __global__ __launch_bounds__(kPathThreads) void ps_commit(Search<BITS> a) {
    if (a.before[0] == 0) return;
    const uint64_t nhuge = min((uint64_t)a.ctl[kCtlHuge], a.huge_cap);
    const bool bits = a.sparse(a.now[1]);  // (before the huge vertices are added: at most once too often)
    const uint64_t gtid = (uint64_t)blockIdx.x * kPathThreads + threadIdx.x, threads = (uint64_t)gridDim.x * kPathThreads;
    uint64_t found = 0, alive = 0;
    uint32_t reached = 0;
    for (uint64_t h = gtid; h < nhuge; h += threads) {
        const uint64_t v = a.huge_at(h);
        const uint64_t seen = a.vis[v], fresh = a.next[v];
        a.front[v] = 0;
        if (fresh) {
            a.vis[v] = seen | fresh;
            found += (uint64_t)__popcll(fresh);
            alive |= fresh;
            ++reached;
        }
    }
    if (BITS && bits) {
        const uint32_t lane = threadIdx.x & 63;
        const uint64_t per = a.shift ? 32ull << a.shift : 64, tasks = (a.n + per - 1) / per;
        for (uint64_t t = gtid >> 6; t < tasks; t += threads >> 6) {
            uint32_t m = 0;
            for (uint64_t v0 = t * per; v0 < min(a.n, (t + 1) * per); v0 += 256) {
                uint64_t w[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint64_t v = v0 + 64 * u + lane;
                    w[u] = 64 * u < per && v < a.n ? a.next[v] : 0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint64_t v = v0 + 64 * u + lane, on = __ballot(w[u] != 0);
                    if (lane < 2 && 64 * u < per && (v0 + 64 * u) / 32 + lane < a.words())
                        a.fine[(v0 + 64 * u) / 32 + lane] = (uint32_t)(on >> (32 * lane));
                    m |= w[u] ? 1u << ((v >> a.shift) & 31) : 0u;
                }
            }
            if (a.shift) {
                for (int off = 1; off < 64; off <<= 1) m |= __shfl_xor(m, off, 64);
                if (lane == 0) a.coarse[t] = m;
            }
        }
    }
    if (gtid - threadIdx.x < nhuge) add_level(a, found, reached, alive);  // (whole workgroups)
}

// A batch's counts into the totals; the last level's words go to the start of
// the next batch, whose own are cleared.
__global__ void ps_fold(unsigned long long *ctl, unsigned long long *cnt, uint64_t level0, uint64_t *out) {
    for (int i = 0; i < kBatch; ++i) {
        unsigned long long c = 0;
        for (int q = 0; q < kCountSlots; ++q) {
            c += cnt[i * kCountSlots + q];
            cnt[i * kCountSlots + q] = 0;
        }
        ctl[kCtlAlive] = ctl[kCtlLevel + 2 * i];
        ctl[kCtlFront] = ctl[kCtlLevel + 2 * i + 1];
        ctl[kCtlLevel + 2 * i] = ctl[kCtlLevel + 2 * i + 1] = 0;
        if (!c) break;  // (nor did any later level run)
        out[0] += (level0 + i) * (uint64_t)c;
        out[1] += (uint64_t)c;
        out[2] = out[2] > level0 + i ? out[2] : level0 + i;
    }
}

__global__ void ps_clear(uint64_t *out, unsigned long long *ctl, unsigned long long *cnt) {
    const uint32_t i = threadIdx.x;
    if (i < 3) out[i] = 0;
    if (i < kCtlWords) ctl[i] = 0;
    if (i < kBatch * kCountSlots) cnt[i] = 0;
}

int grid_of(uint64_t items) {
    return (int)std::max<uint64_t>(1, std::min<uint64_t>((items + kPathThreads - 1) / kPathThreads,
                                                         (uint64_t)device_cu_count() * 4));
}

template <typename IdT, bool BITS>
int run_paths(uint64_t n, const uint64_t *rp, const IdT *col, const int64_t *sources, uint32_t num_sources,
              uint64_t *out, char *ws, const PsPlan &P, hipStream_t s) {
    Search<BITS> a;
    memset(&a, 0, sizeof(a));
    a.n = n;
    a.rp = rp;
    a.col = col;
    a.vis = reinterpret_cast<uint64_t *>(ws + P.off_vis);
    a.front = reinterpret_cast<uint64_t *>(ws + P.off_f0);
    a.next = reinterpret_cast<uint64_t *>(ws + P.off_f1);
    a.list = reinterpret_cast<typename Search<BITS>::ListT *>(ws + P.off_list);
    a.ctl = reinterpret_cast<unsigned long long *>(ws + P.off_ctl);
    unsigned long long *cnt = reinterpret_cast<unsigned long long *>(ws + P.off_cnt);
    a.huge_cap = n;
    if (BITS) {
        // Behind the n list entries: ceil(n / 32) words, above 2^18 vertices
        // kCoarseWords more, a byte per 64 vertices, and the huge vertices' list
        // in what is left.
        const uint64_t words = (n + 31) / 32, region = align256(n * 8) / 4;
        while (((n - 1) >> a.shift) / 32 >= kCoarseWords) ++a.shift;
        uint32_t *b = reinterpret_cast<uint32_t *>(ws + P.off_list) + n;
        uint64_t used = n + words;
        a.fine = b;
        if (a.shift) {
            a.coarse = b + words;
            used += kCoarseWords;
        }
        a.idle = reinterpret_cast<uint8_t *>(ws + P.off_list) + used * 4;
        used += words / 2 / 4 + 1;  // (a byte per 64 vertices)
        a.huge = reinterpret_cast<typename Search<BITS>::ListT *>(ws + P.off_list) + used;
        a.huge_cap = region - used;
    }
    const int g = grid_of(n), gi = grid_of((n + kListChunk - 1) / kListChunk);
    ps_clear<<<1, 64, 0, s>>>(out, a.ctl, cnt);
    for (uint32_t g0 = 0; g0 < num_sources; g0 += kGroup) {
        Sources src;
        memset(&src, 0, sizeof(src));
        src.count = std::min<uint32_t>(kGroup, num_sources - g0);
        for (uint32_t i = 0; i < src.count; ++i) src.v[i] = sources[g0 + i];
        { ProfScope _ps("path_level", s); ps_init<BITS><<<gi, kPathThreads, 0, s>>>(a, g0 == 0); }
        ps_seed<BITS><<<1, 64, 0, s>>>(a, src);
        // A level reaches at least one new (source, vertex) pair or ends the
        // search, so at most n levels run.
        for (uint64_t level = 1;; level += kBatch) {
            a.before = a.ctl + kCtlAlive;
            for (int i = 0; i < kBatch; ++i) {
                a.cnt = cnt + i * kCountSlots;
                a.now = a.ctl + kCtlLevel + 2 * i;
                { ProfScope _ps("path_level", s); ps_sweep<IdT, BITS><<<g, kPathThreads, 0, s>>>(a); }
                { ProfScope _ps("path_level", s); ps_commit<BITS><<<BITS ? g : 8, kPathThreads, 0, s>>>(a); }
                a.before = a.now;
                std::swap(a.front, a.next);
            }
            ps_fold<<<1, 1, 0, s>>>(a.ctl, cnt, level, out);
            unsigned long long alive = 0;
            if (hipMemcpyAsync(&alive, a.ctl + kCtlAlive, sizeof(alive), hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess)
                return fail(SFG_EDEVICE, "path_stats: %s", hipGetErrorString(hipGetLastError()));
            if (alive == 0) break;
        }
    }
    return check_launch("path_stats");
}

template <typename IdT>
int run_paths_any(uint64_t n, const uint64_t *rp, const IdT *col, const int64_t *sources, uint32_t num_sources,
                  uint64_t *out, char *ws, const PsPlan &P, hipStream_t s) {
    if (n <= (1ull << 32)) return run_paths<IdT, true>(n, rp, col, sources, num_sources, out, ws, P, s);
    return run_paths<IdT, false>(n, rp, col, sources, num_sources, out, ws, P, s);
}

}  // namespace
}  // namespace sfg

using namespace sfg;

extern "C" size_t path_stats_workspace_bytes(uint64_t n) { return n ? ps_plan(n).total : 0; }

extern "C" int path_stats(uint64_t n, const uint64_t *row_ptr, const void *col, int id_bytes, const int64_t *sources,
                          uint32_t num_sources, uint64_t *out, void *workspace, size_t workspace_bytes, void *stream) {
    if (n == 0) return fail(SFG_EINVAL, "path_stats: n must be >= 1");
    if (id_bytes != 4 && id_bytes != 8) return fail(SFG_EINVAL, "path_stats: id_bytes must be 4 or 8");
    if (!row_ptr || !col || !out) return fail(SFG_EINVAL, "path_stats: NULL buffer");
    if (num_sources > 0 && !sources) return fail(SFG_EINVAL, "path_stats: NULL sources");
    for (uint32_t i = 0; i < num_sources; ++i)
        if (sources[i] < 0 || (uint64_t)sources[i] >= n)
            return fail(SFG_EINVAL, "path_stats: source %u = %lld is not a vertex", i, (long long)sources[i]);
    const PsPlan P = ps_plan(n);
    if (!workspace) return fail(SFG_EINVAL, "path_stats: workspace is NULL");
    if (workspace_bytes < P.total)
        return fail(SFG_ENOSPACE, "path_stats: workspace has %zu bytes, needs %zu", workspace_bytes, P.total);
    hipStream_t s = as_stream(stream);
    char *ws = static_cast<char *>(workspace);
    if (id_bytes == 4)
        return run_paths_any<int32_t>(n, row_ptr, static_cast<const int32_t *>(col), sources, num_sources, out, ws, P, s);
    return run_paths_any<int64_t>(n, row_ptr, static_cast<const int64_t *>(col), sources, num_sources, out, ws, P, s);
}
